"""The small-batch kernel on inputs whose sums are exact in fp32, in any order,
so that every output has one value and a group, a record or a chunk of groups
that is left out or taken twice shows, however long the row is.  (A bound on
the error of a long sum grows until it covers a whole group.)

Activations are whole numbers up to 4, scales 2^-6 to 2^-4, offsets multiples
of 2^-6 up to 2^-5: every product and partial sum is a multiple of 2^-6, and at
most 32768 inputs * 4 * (4 + 4 + 2 + 2) of them, below 2^24."""

import numpy as np
import pytest
import torch

from gpu_helpers import Case, log
from oracle import codec, packed
from paper_2609_09240_amd import synth, tq

UNIT = 2.0 ** -6

# n_out, n_in, B, f2, offset0, host row pointers
EDGES = [
    (16, 128, 5, 1.0, False, True),        # one group: seven waves idle
    (17, 1024, 8, 0.0, True, True),
    (40, 12288, 9, 0.1, False, True),      # 96 groups: the longest single chunk of one row tile
    (40, 12416, 16, 0.1, True, False),     # 97: two chunks
    (20, 32768, 6, 0.3, False, False),     # 256 groups, the longest row: three chunks
    (20, 32768, 4, 0.3, True, False),      # the same, one quad of rows
    (33, 24576, 64, 1.0, False, True),     # every group two-plane over two chunks
    (4100, 6272, 17, 0.1, False, True),    # two row tiles, 49 groups: two chunks
    (8200, 4224, 33, 0.3, True, True),     # three row tiles, 33 groups: two chunks
    (12300, 3200, 12, 1.0, True, False),   # four row tiles, 25 groups: two chunks
    (12300, 3200, 24, 0.3, False, True),   # with two column tiles
]


def exact_inputs(n_out, n_in, B, f2, offset0):
    key = (53, n_out, n_in, B)
    inp = synth.linear(n_out, n_in, f2, key, offset0=offset0)
    r = np.random.default_rng(key)
    scales = lambda shape: (UNIT * 2.0 ** r.integers(0, 3, shape)).astype(np.float16)
    offsets = lambda shape: (UNIT * r.integers(-2, 3, shape)).astype(np.float16)
    inp.s0 = scales(inp.s0.shape)
    inp.s1, inp.mu1 = scales(inp.s1.shape), offsets(inp.mu1.shape)
    if offset0:
        inp.mu0 = offsets(inp.mu0.shape)
    X = r.integers(-4, 5, (B, n_in)).astype(np.float16)
    return inp, X


@pytest.mark.gpu
@pytest.mark.parametrize("n_out,n_in,B,f2,offset0,host", EDGES)
def test_exact_sums(n_out, n_in, B, f2, offset0, host):
    inp, X = exact_inputs(n_out, n_in, B, f2, offset0)
    case = Case(inp, host_rowptr=host)
    got = tq.tq_gemm_smallbatch(case.gpu, torch.from_numpy(X).cuda(), out_f32=True).cpu().numpy()
    want = case.oracle_gemm(X)
    assert np.abs(want).max() < 2.0 ** 24 * UNIT
    wrong = got.astype(np.float64) != want
    log(f"exact {n_out}x{n_in} B={B}: {int(wrong.sum())} of {wrong.size} differ")
    assert not wrong.any()


@pytest.mark.parametrize("n_out,n_in,B,f2,offset0,host", [e for e in EDGES if e[0] <= 40])
def test_every_group_and_record_shows(n_out, n_in, B, f2, offset0, host):
    """Leaving out plane 0, the offsets or the records of any one group changes
    outputs; so does any one record, and any one row's group."""
    inp, X = exact_inputs(n_out, n_in, B, f2, offset0)
    ng = n_in // 128
    x = X.astype(np.float64).reshape(B, ng, 128)
    # What plane 0 of a group adds to the outputs: [B, n_out, ng].
    t0 = inp.t0.reshape(n_out, ng, 128).astype(np.float64) * inp.s0.astype(np.float64)[:, :, None]
    plane0 = np.einsum("bgk,rgk->brg", x, t0)
    assert plane0.any(axis=0).mean() > 0.99          # a group of one row
    assert plane0.any(axis=(0, 1)).all()             # a group of all rows
    xs = x.sum(axis=2)
    if offset0:
        assert (xs[:, None, :] * inp.mu0.astype(np.float64)[None]).any(axis=(0, 1)).all()
    if inp.nnz1:
        t1 = inp.t1.astype(np.float64) * inp.s1.astype(np.float64)[:, None] + inp.mu1.astype(np.float64)[:, None]
        add = np.einsum("bjk,jk->jb", x[:, inp.gidx1.astype(int)], t1)
        assert add.any(axis=1).mean() > 0.99         # one record
        for g in np.unique(inp.gidx1):
            assert add[inp.gidx1 == g].any()         # a group's records
    # The parts are the whole.
    c0, _ = codec.pack(inp.t0.reshape(-1, 128))
    c1 = codec.pack(inp.t1.reshape(-1, 128))[0] if inp.nnz1 else np.zeros(0, np.uint8)
    want = packed.gemm(n_out, n_in, c0, inp.s0, inp.rowptr1, inp.gidx1, c1, inp.mu1, inp.s1, X, offset0=inp.mu0)
    total = plane0.sum(axis=2)
    if offset0:
        total += xs @ inp.mu0.astype(np.float64).T
    if inp.nnz1:
        rows = np.repeat(np.arange(n_out), np.diff(inp.rowptr1))
        for b in range(B):
            total[b] += np.bincount(rows, weights=add[:, b], minlength=n_out)
    np.testing.assert_array_equal(total, want)
