"""What bench.py holds a kernel against: the larger of the two times its work takes, at the rates of what it runs on."""
import bench


def case(**kw):
    c = dict(in_dim=10000, hidden=1024, out_dim=10000, seq_len=256, batch=64, input_kind=0, loss_kind=0, act=0,
             _variant="xcd_mfma", _workgroups=256)
    c.update(kw)
    return c


def entry(name, us, c):
    return bench.roofline_entry(name, {name: dict(avg_us=us, total_ms=us, count=1)}, c)


LONG_DENSE = case(in_dim=128, hidden=256, out_dim=128, seq_len=4096, batch=128, input_kind=1, loss_kind=1, _variant="batch_mfma",
                  _workgroups=32)


def test_products_are_held_against_the_slower_of_memory_and_the_bf16_matrix_rate():
    big = entry("gemm_logits", 1600.0, case())
    assert big["bound"] == "mfma" and big["peak"] == bench.BF16_MFMA_PEAK_TFLOPS
    assert big["executed_flops"] == 6 * 2.0 * 16384 * 10000 * 1024
    two = entry("gemm_logits", 900.0, case(_bf16x3=True))
    assert two["executed_flops"] == 3 * 2.0 * 16384 * 10000 * 1024
    # 524288 x 256 x 128: 82 us of matrix instructions, 101 us of bytes
    thin = entry("gemm_U", 250.0, LONG_DENSE)
    assert thin["bound"] == "hbm" and thin["peak"] == bench.HBM_PEAK_GBS


def test_the_batched_loop_is_held_against_the_bf16_rate_of_its_units():
    r = entry("rec_fwd", 4200.0, LONG_DENSE)
    assert r["bound"] == "mfma" and r["peak"] == bench.BF16_MFMA_PEAK_TFLOPS
    on = r["on_chip"]
    assert on["n_cu"] == 32 and abs(on["peak"] - bench.BF16_MFMA_PEAK_TFLOPS * 32 / bench.N_CU) < 1e-9
    assert on["executed_flops"] == 9 * 2.0 * 4096 * 128 * 256 * 256 and 0.4 < on["frac_executed"] < 0.7
    wide = entry("rec_fwd", 540.0, case())["on_chip"]       # float32 instructions
    assert wide["peak"] == bench.FP32_MFMA_PEAK_TFLOPS


def test_launches_of_a_classifier_call():
    assert bench.mlp_launches(0, 400) == 1 and bench.mlp_launches(1, 400) == 2
    assert bench.mlp_launches(1, 1025) == 4 and bench.mlp_launches(3, 10) == 80


def test_the_line_stays_short():
    """A line of 20000 characters was not read.  Seven configurations with the kernels of the largest, their rooflines once."""
    names = ("gemm_logits", "gemm_dV", "gemm_G", "gemm_dWh", "gemm_dWx", "splitk_reduce", "rec_fwd", "rec_bwd", "ce_row_stats", "loss_reduce", "dz",
             "colsum_partial", "colsum_finish", "dwx_tokens", "misc", "mse_row_loss", "transpose")
    prof = {k: dict(launches=2, avg_us=1234.56789 / (i + 1), total_ms=2.46913578 / (i + 1)) for i, k in enumerate(names)}
    c = case(_name="C4")
    roofline = dict(bench.roofline_of(prof, c), peak_measured=2417.512345, frac_measured=0.533791234)
    r = dict(tokens_per_s=2641512.345, timesteps_per_s=41273.612, ms_per_step=6.2025123, entry_points="rnn_forward,rnn_loss,rnn_bptt",
             recurrence_variant="xcd_mfma", roofline=roofline, kernels=bench.kernel_times(prof))
    out = dict(kernels=r["kernels"], rooflines_all_kernels=bench.all_rooflines(prof, c),
               per_config={str(n): bench.per_config_entry(r) for n in range(7)})
    assert len(bench.line(out)) < 10000, len(bench.line(out))
