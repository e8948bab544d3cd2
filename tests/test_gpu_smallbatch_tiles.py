"""Edges of the small-batch kernel's tiling (fp32 outputs, so that only fp32
sums separate it from the oracle): chunks of groups, waves without a group,
partial row and column tiles, records in every pass, and rows of X that are
not finite."""

import numpy as np
import pytest
import torch

from gpu_helpers import Case, log
from oracle import packed
from paper_2609_09240_amd import synth, tq

pytestmark = pytest.mark.gpu


def sum_bound(case, X):
    """Each product is exact in fp32 and every term passes through at most
    K + 4 G roundings of 2^-24 (its group's sum, the scale, the other groups'
    and waves' sums), so the error is below that times sum |w x|, which the
    acceptance bound holds 2e-3 times.  (At the longest rows that covers a
    group: what is left out or taken twice there shows in
    test_smallbatch_exact.py, whose sums are exact.)"""
    K = case.inp.n_in
    return case.bound(X) / 2e-3 * (K + 4 * (K // 128)) * 2.0 ** -24


@pytest.mark.parametrize("n_out,n_in,B,f2,offset0,host", [
    (16, 128, 5, 1.0, False, True),        # one group: seven waves idle
    (17, 1024, 8, 0.0, True, True),        # offsets without records, a second workgroup of one row
    (40, 12288, 9, 0.1, False, True),      # 96 groups: the longest single chunk of one row tile
    (40, 12416, 16, 0.1, True, False),     # 97: two chunks
    (20, 32768, 6, 0.3, False, False),     # 256 groups, the longest row: three chunks
    (33, 24576, 64, 1.0, False, True),     # every group two-plane over two chunks
    (4100, 6272, 17, 0.1, False, True),    # two row tiles, 49 groups: two chunks; four rows in the last workgroup
    (8200, 4224, 33, 0.3, True, True),     # three row tiles, 33 groups: two chunks, up to three passes of plane 1
    (8200, 640, 64, 1.0, False, True),     # three row tiles, three passes everywhere
    (12300, 3200, 12, 1.0, True, False),   # four row tiles, 25 groups: two chunks, four passes
    (12300, 384, 48, 0.5, False, True),    # past three row tiles with several column tiles: several rounds
    (12300, 384, 17, 0.5, False, True),    # four row tiles and two column tiles
    (16384, 3200, 32, 0.3, True, False),   # the same, 25 groups in two chunks, every row tile full
    (16400, 256, 16, 0.3, False, True),    # one row past a round of four row tiles: three
    (16385, 128, 40, 1.0, False, True),    # and with three column tiles
])
def test_tile_edges(n_out, n_in, B, f2, offset0, host):
    case = Case(synth.linear(n_out, n_in, f2, (41, n_out, n_in, B), offset0=offset0), host_rowptr=host)
    X = synth.activations(n_in, (41, n_out, n_in, 90), batch=B, outlier_frac=0.01)
    Y = tq.tq_gemm_smallbatch(case.gpu, torch.from_numpy(X).cuda(), out_f32=True)
    got = Y.cpu().numpy().astype(np.float64)
    worst = float((np.abs(got - case.oracle_gemm(X)) / sum_bound(case, X)).max())
    log(f"tiles {n_out}x{n_in} B={B}: max err/bound {worst:.3g}")
    assert worst <= 1.0


@pytest.mark.parametrize("B,f2", [(5, 0.3), (20, 0.3), (40, 0.0)])
def test_rows_that_are_not_finite(B, f2):
    """An infinity or NaN in one row of X stays in that row of Y, and +-inf
    there stays +-inf for the outputs whose weight is not zero (records of
    other rows, which share a tile row, do not turn it into NaN)."""
    n_out, n_in = 300, 1024
    inp = synth.linear(n_out, n_in, f2, (43, n_out, n_in, B))
    case = Case(inp)
    X = synth.activations(n_in, (43, n_out, n_in, 90), batch=B)
    clean = tq.tq_gemm_smallbatch(case.gpu, torch.from_numpy(X).cuda(), out_f32=True).cpu().numpy()
    X[1, 700] = np.inf
    X[B - 1, 3] = np.nan
    got = tq.tq_gemm_smallbatch(case.gpu, torch.from_numpy(X).cuda(), out_f32=True).cpu().numpy()
    rows = [b for b in range(B) if b not in (1, B - 1)]
    assert np.array_equal(got[rows].view(np.uint32), clean[rows].view(np.uint32))
    assert np.isnan(got[B - 1]).all()
    # One-plane rows of the infinity's group: trit times infinity.
    g = 700 // 128
    one = np.ones(n_out, bool)
    for r in range(n_out):
        one[r] = g not in inp.gidx1[inp.rowptr1[r]:inp.rowptr1[r + 1]]
    t = inp.t0[:, 700]
    assert np.array_equal(got[1][one & (t == 1)], np.full((one & (t == 1)).sum(), np.inf, np.float32))
    assert np.array_equal(got[1][one & (t == -1)], np.full((one & (t == -1)).sum(), -np.inf, np.float32))


def kinds(y):
    """0 finite, 1 +inf, 2 -inf, 3 NaN."""
    return np.select([np.isnan(y), np.isposinf(y), np.isneginf(y)], [3, 1, 2], 0)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("n_out,n_in,B,f2,offset0,mu,host", [
    (300, 1024, 5, 0.3, True, None, True),
    (300, 1024, 9, 0.3, False, None, False),
    (300, 640, 20, 0.3, True, 0.0, True),     # records' offsets 0, as a matrix quantised with group offsets has
    (4100, 256, 40, 0.1, False, None, True),  # two row tiles
    (100, 512, 64, 0.0, True, None, True),
    (100, 12800, 16, 0.1, True, None, True),  # two chunks of groups
    (100, 512, 6, 0.0, False, None, True),    # one plane: 0 times infinity is NaN by the definition
])
def test_infinities_under_offsets(n_out, n_in, B, f2, offset0, mu, host, f32):
    """An infinite input gives what the weights give one by one: +-inf also
    where both trits are 0 and an offset is the weight, NaN where the weight is
    0 or infinities cancel; and so do scales and offsets that are not finite."""
    inp = synth.linear(n_out, n_in, f2, (47, n_out, n_in, B), offset0=offset0)
    if mu is not None:
        inp.mu1[:] = mu
    inp.s0[7, 0], inp.s0[8, 1], inp.s0[9, 0] = np.inf, np.nan, 0.0
    if offset0:
        inp.mu0[10, 1], inp.mu0[11, 0] = -np.inf, 0.0
    if inp.nnz1:
        inp.s1[3], inp.s1[inp.nnz1 // 2] = -np.inf, np.nan
    case = Case(inp, host_rowptr=host)
    X = synth.activations(n_in, (47, n_out, n_in, 90), batch=B)
    X[0, 100] = np.inf
    X[1, n_in - 1] = -np.inf
    X[2, 3], X[2, 200] = np.inf, np.inf
    X[3, 127], X[3, n_in - 2] = np.inf, -np.inf
    X[B - 1, 5], X[B - 1, 6] = np.inf, np.nan
    got = tq.tq_gemm_smallbatch(case.gpu, torch.from_numpy(X).cuda(), out_f32=f32).cpu().numpy()
    with np.errstate(invalid="ignore"):
        w = packed.dequantize(*case.oracle_args(), offset0=inp.mu0)
        want = np.stack([(w * x.astype(np.float64)).sum(axis=1) for x in X])
    np.testing.assert_array_equal(kinds(got), kinds(want))
    assert (kinds(want)[0] == (3 if f2 == 0 and not offset0 else 1)).any()
