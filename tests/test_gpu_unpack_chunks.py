"""GPU parity of tq_unpack at the edges of its launch: one group, a workgroup's
128 groups and one to either side, more groups than one round of workgroups
takes, every code byte at every position of a group, and the count of bad
bytes, each of which lies in the codes of one or two threads."""

import numpy as np
import pytest
import torch

from oracle import codec
from paper_2609_09240_amd import tq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 1000, 2048 * 128 + 3])
def test_unpack_matches_the_trits(n):
    rng = np.random.default_rng(n)
    trits = rng.integers(-1, 2, (n, 128), dtype=np.int8)
    codes, _ = codec.pack(trits)
    guard = torch.full((n + 1, 128), 7, dtype=torch.int8, device="cuda")
    tq.tq_unpack(torch.from_numpy(codes).cuda(), n, trits=guard[:n])
    out = guard.cpu().numpy()
    np.testing.assert_array_equal(out[:n], trits)
    assert (out[n] == 7).all()


def test_every_code_byte_at_every_position():
    """Group f holds code (f + 7 j) mod 256 at byte j, so that every code meets
    every position; codes above 242 are bad and give zeros."""
    n = 256
    j = np.arange(26)
    by_group = ((np.arange(n)[:, None] + 7 * j[None, :]) % 256).astype(np.uint8)
    codes = np.concatenate([by_group[:, :24].reshape(-1), by_group[:, 24:].reshape(-1)])
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = tq.tq_unpack(torch.from_numpy(codes).cuda(), n, d_err=err).cpu().numpy()
    c = np.where(by_group > 242, 121, by_group).astype(np.int64)
    digits = np.stack([c // 3**k % 3 - 1 for k in range(5)], axis=-1).reshape(n, 130)
    np.testing.assert_array_equal(got, digits[:, :128].astype(np.int8))
    assert err.item() == int((by_group > 242).sum())


def test_past_one_round_of_workgroups():
    """The launch has at most 2^14 workgroups, of 128 groups each: three more
    groups than that, with bad bytes in both rounds.  Group f is group f % 4999
    of a small buffer."""
    n, period = (1 << 14) * 128 + 3, 4999
    rng = np.random.default_rng(4999)
    trits = rng.integers(-1, 2, (period, 128), dtype=np.int8)
    codes, _ = codec.pack(trits)
    f = torch.arange(n, device="cuda") % period
    stored = torch.cat([torch.from_numpy(part).cuda().view(period, -1)[f].view(-1)
                        for part in (codes[:24 * period], codes[24 * period:])])
    want = torch.full((n + 1, 128), 7, dtype=torch.int8, device="cuda")
    want[:n] = torch.from_numpy(trits).cuda()[f]
    bad = [(0, 0), (1, 12), (127, 25), (n // 2, 24), (n - 4, 7), (n - 3, 3), (n - 2, 25), (n - 1, 16), (n - 1, 24)]
    for g, j in bad:
        stored[24 * g + j if j < 24 else 24 * n + 2 * g + j - 24] = 243 + (g + j) % 13
        want[g, 5 * j:5 * j + 5] = 0
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = torch.full((n + 1, 128), 7, dtype=torch.int8, device="cuda")
    tq.tq_unpack(stored, n, trits=got[:n], d_err=err)
    assert torch.equal(got, want)
    assert err.item() == len(bad)
