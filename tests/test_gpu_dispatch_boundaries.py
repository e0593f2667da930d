"""Parity at the sizes where the dispatcher changes kernel family: hidden sizes just below and
above 128, 256, 512 and 1024 against batch sizes just below and above 4 and 64 (one workgroup,
several workgroups, batched matrix-core loop, the one-launch wide loop, one launch per step), with
short windows, both activations, token and dense inputs, initial states and incoming gradients."""
import numpy as np
import pytest
import torch

import oracle
import paper_1211_5590_amd as rnn
import rnn_inputs as ri
from gpu_harness import Runner, compare

pytestmark = pytest.mark.gpu

HIDDEN = (128, 129, 256, 257, 512, 516, 1020, 1024, 1028)
BATCH = (1, 4, 5, 64, 65)


@pytest.mark.parametrize("H", HIDDEN)
def test_every_batch_size_at_this_hidden_size(H):
    rng = np.random.default_rng(H)
    seen = set()
    for n, B in enumerate(BATCH):
        T = int(rng.choice([1, 2, 3, 5, 9]))
        NV = int(rng.choice([64, 130, 200]))
        dense = n == 3
        kw = dict(in_dim=24 if dense else NV, hidden=H, out_dim=20 if dense else NV, seq_len=T, batch=B,
                  act=int(rng.integers(0, 2)), with_h0=bool(n % 2), with_dh_last=n % 3 == 0,
                  wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=1000 + 7 * H + n)
        if dense:
            kw.update(input_kind=ri.INPUT_DENSE, loss_kind=ri.LOSS_LINEAR_MSE)
        case = ri.make_case(**kw)
        r = Runner(case)
        variant = rnn.rnn_recurrence_variant(r.dims)
        seen.add(variant)
        print(f"H={H} B={B} T={T} NV={NV} dense={dense} variant={variant}", flush=True)
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))
    assert len(seen) >= 2, seen        # every hidden size crosses at least one family boundary over these batches


@pytest.mark.parametrize("H", (260, 512, 516, 1020, 1024))
def test_the_one_launch_wide_loop_at_its_edges(H):
    """Batch 5 and 64 (the smallest and the largest the one-launch wide loop takes), 10 steps (its
    shortest sequence) and 9 (one launch per step), batch 65 (beyond it)."""
    for n, (B, T, want) in enumerate(((5, 10, "xcd_mfma"), (64, 21, "xcd_mfma"), (64, 9, "step_mfma"),
                                      (65, 20, "step_mfma"))):
        case = ri.make_case(in_dim=90, hidden=H, out_dim=70, seq_len=T, batch=B, act=n % 2, with_h0=bool(n % 2),
                            with_dh_last=n >= 2, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=9000 + 11 * H + n)
        r = Runner(case)
        variant = rnn.rnn_recurrence_variant(r.dims)
        print(f"H={H} B={B} T={T} variant={variant}", flush=True)
        assert variant == want
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))


@pytest.mark.parametrize("H", (257, 258, 259, 511, 513, 650, 1021, 1023))
def test_the_one_launch_wide_loop_at_hidden_sizes_that_are_no_multiple_of_4(H):
    """Rows at 4-byte alignment and a ragged last piece of every row, in the first and in the second
    K half of a wavefront, with rows missing from the last batch group."""
    for n, (B, T) in enumerate(((5, 10), (63, 12), (18, 31))):
        case = ri.make_case(in_dim=90, hidden=H, out_dim=70, seq_len=T, batch=B, act=n % 2, with_h0=n != 1,
                            with_dh_last=n >= 1, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=9500 + 11 * H + n)
        r = Runner(case)
        print(f"H={H} B={B} T={T}", flush=True)
        assert rnn.rnn_recurrence_variant(r.dims) == "xcd_mfma"
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))


@pytest.mark.parametrize("H", (384, 385, 640, 641, 768, 769, 896, 897))
def test_the_one_launch_wide_loop_where_a_wavefronts_share_of_the_matrix_changes(H):
    """A wavefront takes an eighth of the hidden units in whole blocks of 16: the last and the first size of a
    share, and the second piece of the state that only some lanes hold."""
    for n, (B, T) in enumerate(((6, 10), (33, 17))):
        case = ri.make_case(in_dim=90, hidden=H, out_dim=70, seq_len=T, batch=B, act=n % 2, with_h0=n == 0,
                            with_dh_last=n == 1, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=9700 + 11 * H + n)
        r = Runner(case)
        print(f"H={H} B={B} T={T}", flush=True)
        assert rnn.rnn_recurrence_variant(r.dims) == "xcd_mfma"
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))


def test_the_one_launch_wide_loop_hands_on_a_nan_of_any_bits():
    """The loop marks words that are not there yet with one bit pattern of a NaN: a state that is that very
    NaN has to arrive as a NaN in the row it belongs to, and nowhere else, and no wait may expire for it."""
    case = ri.make_case(in_dim=90, hidden=300, out_dim=70, seq_len=12, batch=7, act=1, wdist=("normal", 0.03),
                        bias_std=0.1, seed=97)
    case["x"][:] = 1
    case["x"][4, 2] = 3
    bits = case["Wx"].view(np.uint32)
    bits[3, 17] = 0xFFFFFFFF
    r = Runner(case)
    r.forward()
    torch.cuda.synchronize()
    assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
    bad = torch.isnan(r.h_all).cpu().numpy()
    assert bad[5, 2, 17] and bad[5].sum() == 1
    assert bad[6:, 2].all() and not np.delete(bad, 2, axis=1).any()


@pytest.mark.parametrize("H,B,T,want", ((257, 1, 16, True), (500, 1, 15, False), (513, 2, 33, True), (640, 1, 40, True),
                                        (641, 1, 40, False), (641, 3, 17, True), (1024, 4, 16, True), (300, 1, 32, True)))
def test_the_wide_loop_for_the_smallest_batches(H, B, T, want):
    """Batch 1 to 4 on both sides of the rule that sends them to the one-launch wide loop, with token and with dense
    input, and the forward pass without the history, which that loop does not serve."""
    for kind in (0, 1):
        case = ri.make_case(in_dim=92, hidden=H, out_dim=72, seq_len=T, batch=B, act=kind, input_kind=kind, with_h0=True,
                            with_dh_last=kind == 0, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=9800 + 11 * H + kind)
        r = Runner(case)
        variant = rnn.rnn_recurrence_variant(r.dims)
        print(f"H={H} B={B} T={T} input={kind} variant={variant}", flush=True)
        assert (variant == "xcd_mfma") == want
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        ref = oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last"))
        compare(r.results(), ref)
        last = Runner(case, keep_history=False)
        last.forward()
        torch.cuda.synchronize()
        assert np.max(np.abs(last.h_last.cpu().numpy() - ref["h_all"][-1])) <= 2e-5


@pytest.mark.parametrize("H,T", ((1, 19), (3, 9), (8, 33), (9, 8), (16, 41), (17, 33), (32, 7), (33, 40), (64, 17), (65, 35),
                                 (80, 9), (81, 33), (96, 24), (97, 33), (113, 40), (128, 33), (129, 10), (160, 40), (161, 33),
                                 (192, 12), (193, 33), (255, 10), (256, 35)))
def test_the_loops_of_the_smallest_batches_at_their_edges(H, T):
    """Batch 1 to 4: every count of lanes and of pieces per lane of the one-workgroup loop, whole and ragged chunks of
    its eight steps, and the batched loop above 128 hidden units; the forward pass also without the history, whose two
    slots are then written in turn."""
    for n, B in enumerate((1, 3)):
        case = ri.make_case(in_dim=70, hidden=H, out_dim=68, seq_len=T, batch=B, act=n, with_h0=n == 0, with_dh_last=n == 1,
                            wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=9900 + 13 * H + n)
        r = Runner(case)
        print(f"H={H} B={B} T={T} variant={rnn.rnn_recurrence_variant(r.dims)}", flush=True)
        assert (rnn.rnn_recurrence_variant(r.dims) == "batch_mfma") == (H > 128)
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        ref = oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last"))
        compare(r.results(), ref)
        last = Runner(case, keep_history=False)
        last.forward()
        torch.cuda.synchronize()
        assert np.max(np.abs(last.h_last.cpu().numpy() - ref["h_all"][-1])) <= 2e-5


@pytest.mark.parametrize("H,B", ((512, 32), (512, 33), (513, 32), (513, 33), (1024, 32), (1024, 33), (300, 1), (384, 35)))
def test_the_one_launch_wide_loop_where_the_columns_of_a_workgroup_change(H, B):
    """16, 32 or 64 columns per workgroup: the last and the first size of each, with one and with two groups per die."""
    case = ri.make_case(in_dim=90, hidden=H, out_dim=70, seq_len=16, batch=B, act=H % 2, with_h0=True, with_dh_last=True,
                        wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=9900 + 11 * H + B)
    r = Runner(case)
    print(f"H={H} B={B}", flush=True)
    assert rnn.rnn_recurrence_variant(r.dims) == "xcd_mfma"
    r.step()
    assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
    compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))


@pytest.mark.parametrize("H", (192, 193, 200, 255, 256))
def test_the_one_launch_wide_loop_below_257_units(H):
    """Both sides of the rule that sends 193 to 256 units there, one to four groups per die, tokens and dense input, and the
    forward pass without the history, which that loop does not serve."""
    for n, (B, T, kind, want) in enumerate(((5, 33, 0, True), (33, 32, 0, False), (65, 64, 1, True), (97, 33, 0, True), (128, 63, 1, False),
                                            (128, 64, 1, True), (1, 64, 0, True), (4, 64, 1, True), (4, 63, 0, False), (129, 64, 0, False))):
        case = ri.make_case(in_dim=60, hidden=H, out_dim=40, seq_len=T, batch=B, act=n % 2, input_kind=kind, with_h0=n % 3 == 0,
                            with_dh_last=n % 2 == 0, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=9950 + 11 * H + n)
        r = Runner(case)
        print(f"H={H} B={B} T={T} input={kind}", flush=True)
        assert (rnn.rnn_recurrence_variant(r.dims) == "xcd_mfma") == (want and H > 192)
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        ref = oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last"))
        compare(r.results(), ref)
        last = Runner(case, keep_history=False)
        last.forward()
        torch.cuda.synchronize()
        assert np.max(np.abs(last.h_last.cpu().numpy() - ref["h_all"][-1])) <= 2e-5


@pytest.mark.parametrize("NV,H,T", ((4, 1, 17), (64, 2, 16), (64, 16, 32), (128, 17, 16), (128, 33, 17), (128, 128, 32), (132, 1, 32),
                                    (132, 64, 17), (260, 65, 31), (260, 128, 33)))
def test_the_column_strips_of_short_sequences_at_their_edges(NV, H, T):
    """One strip of 128 columns and more, one pass of 16 rows and two, hidden sizes at and beside powers of two; 33 rows are
    beyond the strips. Twice, the second time with the words of the first still in the exchange boxes."""
    case = ri.make_case(in_dim=NV, hidden=H, out_dim=NV, seq_len=T, batch=1, act=T % 2, with_h0=bool(T % 2),
                        wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=77000 + 100 * H + T)
    r = Runner(case)
    ref = oracle.fwd_bptt(case, h0=case.get("h0"))
    for _ in range(2):
        print(f"NV={NV} H={H} T={T}", flush=True)
        r.step()
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), ref)
