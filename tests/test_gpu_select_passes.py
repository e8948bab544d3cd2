"""The selection's passes: one workgroup up to 32768 groups; above, digits
until at most 256 keys are left, which the next pass collects and ranks.  The
cut falls among unique keys, among ties that are few enough to be collected,
among ties that are not, and where every key left is taken; above 32768 groups
also among NaNs, zeros of both signs, infinities and subnormals, among long
runs of ties, and with workspaces that hold anything."""

import numpy as np
import pytest
import torch

from paper_2609_09240_amd import tq
from test_gpu_select import check, expected

pytestmark = pytest.mark.gpu


def energies(n, kind):
    r = np.random.default_rng(n)
    e = r.exponential(1.0, n)
    order = np.argsort(-e, kind="stable")
    nnz = n // 10
    ties = {"unique": 0, "few": 100, "collected": 256, "one more": 257, "many": n // 3}[kind]
    if ties:   # the cut in the middle of the ties
        lo = max(0, nnz - ties // 2)
        e[order[lo:lo + ties]] = e[order[lo]]
    return e, nnz


@pytest.mark.parametrize("kind", ["unique", "few", "collected", "one more", "many"])
@pytest.mark.parametrize("n_out,G", [(1024, 32), (32767, 1), (32769, 1), (3000, 37)])
def test_cut(n_out, G, kind):
    e, nnz = energies(n_out * G, kind)
    check(e, n_out, G, nnz, f"{kind} of {n_out * G}")


@pytest.mark.parametrize("n_out,G", [(5, 3), (40000, 1)])
@pytest.mark.parametrize("nnz", [1, 2, None])
def test_first_and_last(n_out, G, nnz):
    """One group, two groups, all groups."""
    n = n_out * G
    check(np.random.default_rng(3).exponential(1.0, n), n_out, G, n if nnz is None else nnz, f"{nnz} of {n}")


@pytest.mark.parametrize("n_out,G", [(1, 1), (255, 1), (256, 1), (1, 256), (300, 17), (40000, 1), (33000, 128)])
def test_nothing_to_select(n_out, G):
    """No records: -1 for every group, zero row pointers, nothing behind them."""
    n = n_out * G
    e = torch.zeros(n, dtype=torch.float64, device="cuda")
    rec = torch.full((n + 1,), 7, dtype=torch.int32, device="cuda")
    rowptr = torch.full((n_out + 2,), 7, dtype=torch.int32, device="cuda")
    tq.tq_select_two_plane(e, n_out, G, 0, rec_index=rec, rowptr1=rowptr)
    assert (rec[:n] == -1).all() and rec[n].item() == 7
    assert (rowptr[:n_out + 1] == 0).all() and rowptr[n_out + 1].item() == 7


LARGE = (2500, 17)   # 42500 groups: eleven tiles, the last ragged


@pytest.mark.parametrize("count", [40, 300])
def test_special_values_above_one_workgroup(count):
    """`count` of each value: 40 are collected and ranked, 300 are not."""
    n_out, G = LARGE
    n = n_out * G
    r = np.random.default_rng(17)
    e = r.exponential(1.0, n)
    idx = r.permutation(n)
    for i, v in enumerate([np.nan, 0.0, -0.0, np.inf, 5e-324, 1e300, -np.inf]):
        e[idx[i * count:(i + 1) * count]] = v
    assert np.isfinite(e[e > 0]).sum() > count
    above = int((e > 0).sum())                     # inf, 1e300, the numbers, the subnormals
    cuts = {
        "one infinity": 1, "among the infinities": count // 2, "all infinities": count,
        "among 1e300": count + 1, "among the subnormals": above - 1, "all above zero": above,
        "among the zeros": above + count // 2, "all zeros": above + 2 * count,
        "among -inf": above + 2 * count + 3, "among the NaNs": n - count // 2, "all but one NaN": n - 1, "all": n,
    }
    for what, nnz in cuts.items():
        check(e, n_out, G, nnz, f"{count} specials, {what}")


@pytest.mark.parametrize("levels,f2", [(3, 0.1), (5, 0.37), (1, 0.25), (2, 0.5)])
def test_ties_above_one_workgroup(levels, f2):
    n_out, G = LARGE
    e = np.random.default_rng(levels).integers(0, levels, n_out * G).astype(np.float64) * 0.5
    check(e, n_out, G, int(f2 * n_out * G), f"ties levels={levels} f2={f2}")


def same(got, want):
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a.cpu().numpy().view(b.dtype), b)


@pytest.mark.parametrize("fill", [0x00, 0xAB, 0xFF])
def test_workspace_contents_do_not_matter(fill):
    n_out, G = LARGE
    n = n_out * G
    ws = torch.full((tq.tq_select_workspace_bytes(n),), fill, dtype=torch.uint8, device="cuda")
    for seed, nnz in ((1, n // 10), (2, n // 3), (3, 1)):   # and what the call before left there
        e = np.random.default_rng(seed).exponential(1.0, n)
        if seed == 2:
            e = np.round(e)
        same(tq.tq_select_two_plane(torch.from_numpy(e).cuda(), n_out, G, nnz, workspace=ws),
             expected(e, n_out, G, nnz))


def test_library_scratch_above_one_workgroup():
    """The call that allocates nothing, twice with other energies and a smaller
    matrix last: each finds what the one before left in the library's scratch."""
    for seed, n_out, G in ((4, 2500, 17), (5, 2500, 17), (6, 1200, 28)):
        n, nnz = n_out * G, n_out * G // 7
        e = np.random.default_rng(seed).exponential(1.0, n)
        rec = torch.full((n,), 7, dtype=torch.int32, device="cuda")
        rowptr = torch.full((n_out + 1,), 7, dtype=torch.int32, device="cuda")
        gidx = torch.full((nnz,), 7, dtype=torch.int16, device="cuda")
        same(tq.tq_select_two_plane_noalloc(torch.from_numpy(e).cuda(), n_out, G, nnz, rec, rowptr, gidx),
             expected(e, n_out, G, nnz))
