"""Gradient of the token-indexed input matrix at the row widths where its four-columns-per-lane kernels
change form (fewer than four columns, ragged ends, more than one 256-column chunk), with a vocabulary
smaller and larger than the hidden size, overwriting and accumulating, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1211_5590_amd as rnn
import rnn_inputs as ri
from gpu_harness import Runner, grad_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,NV", [(1, 50), (2, 9), (3, 300), (4, 70), (5, 40), (255, 60), (257, 30), (261, 900), (514, 20)])
def test_token_gradient_at_this_row_width(H, NV):
    case = ri.make_case(NV, H, NV, 21, 29, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=40 + H)
    ref = oracle.fwd_bptt(case)
    r = Runner(case)
    r.step()
    once = r.results()
    grad_close("dWx", once["dWx"], ref["dWx"])
    unseen = np.setdiff1d(np.arange(NV), np.unique(case["x"]))
    assert not once["dWx"][unseen].any()
    r.set_flags(rnn.FLAG_ACCUMULATE | rnn.FLAG_BPTT_RECOMPUTE)
    r.bptt()
    grad_close("2x dWx", r.results()["dWx"], 2.0 * ref["dWx"])


@pytest.mark.parametrize("T,B,H", [(5, 7, 63), (16, 16, 64), (257, 1, 65), (771, 5, 129), (1024, 64, 9), (1025, 64, 9), (2049, 64, 9),
                                   (250, 256, 192), (191, 256, 193), (3, 16299, 193), (95, 256, 257), (11, 2211, 257), (1, 65537, 257),
                                   (3, 43691, 257)])
def test_token_gradient_of_this_many_ids(T, B, H):
    """One and several ranges of ids, a range that is full and one of a single id, ranges of 256, 512 and 1024 ids, and slices of
    64 columns and, from 192 ranges by 256 columns on, of 256; one token makes up most of the ids."""
    case = ri.make_case(40, H, 8, T, B, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=60 + T)
    x = case["x"].reshape(-1)
    x[np.arange(x.size) % 3 > 0] = 17
    case["y"][:] %= 8
    ref = oracle.fwd_bptt(case)
    r = Runner(case)
    r.step()
    got = r.results()["dWx"]
    grad_close("dWx", got, ref["dWx"])
    # every token's own row: the tolerance above is one for the whole matrix
    scale = np.abs(ref["dWx"]).max(axis=1, keepdims=True)
    assert (np.abs(got - ref["dWx"]) <= 1e-3 * scale + 1e-12).all()


@pytest.mark.parametrize("T,B,H,NV,O", ((4097, 4096, 2, 20, 3), (3, 5, 1, 67_108_900, 4), (11, 4, 1, 67_108_900, 4)))
def test_more_rows_and_more_tokens_than_one_dimension_of_a_grid_holds(T, B, H, NV, O):
    """A grid holds 2^32 threads per dimension: 16.8 million workgroups of 256 threads, one per row or one per four tokens."""
    case = ri.make_case(NV, H, O, T, B, wdist=("normal", 0.5), bias_std=0.1, seed=80, with_h0=True)
    case["x"].reshape(-1)[-1] = NV - 1                    # the last token occurs
    ref = oracle.fwd_bptt(case, h0=case["h0"])
    r = Runner(case)
    r.step()
    got = r.results()
    assert abs(got["loss"] - ref["loss"]) <= 1e-4 * abs(ref["loss"])
    for k in ("dWx", "dWh", "db", "dV", "dc", "dh0"):
        grad_close(k, got[k], ref[k])


def test_token_gradient_beside_the_column_sums_of_very_many_outputs():
    """Workgroups of the same launch finish the column sums of dc: with one range of ids and 2.2 million outputs more of them than a
    grid's second dimension holds."""
    case = ri.make_case(30, 4, 2_200_004, 33, 1, wdist=("normal", 0.5), bias_std=0.1, seed=78)
    ref = oracle.fwd_bptt(case)
    r = Runner(case)
    r.step()
    got = r.results()
    for k in ("dWx", "dc", "db", "dV"):
        grad_close(k, got[k], ref[k])
