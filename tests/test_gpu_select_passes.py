"""The selection's passes: one workgroup up to 32768 groups; above, digits
until at most 256 keys are left, which the next pass collects and ranks.  The
cut falls among unique keys, among ties that are few enough to be collected,
among ties that are not, and where every key left is taken."""

import numpy as np
import pytest
import torch

from paper_2609_09240_amd import tq
from test_gpu_select import check

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
