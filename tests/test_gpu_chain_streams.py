"""Chains that share the device: two chains launched at once on two streams,
each holding CUs that the other waits for, both end with the bits of
tq_gemv_grouped and no wait given up, as does a call whose workgroups take
every item by ticket; and a captured chain repeats them on every replay,
between eager work."""

import pytest
import torch

from gpu_helpers import Case
from paper_2609_09240_amd import synth, tq

pytestmark = pytest.mark.gpu


def build(seed, shapes):
    """A chain of dependent stages; its matrices, x, outputs and the outputs of
    the same stages launched one after another."""
    cases = [Case(synth.linear(n, k, f2, (seed, n, k, i))) for i, (n, k, f2) in enumerate(shapes)]
    x0 = torch.from_numpy(synth.activations(shapes[0][1], (seed, 0, 0, 9))).cuda()
    ys = [torch.empty(n, dtype=torch.float16, device="cuda") for n, _, _ in shapes]
    xs = [x0] + ys[:-1]
    want, x = [], x0
    for c in cases:
        x = tq.tq_gemv_grouped([c.gpu], x, out_f32=False)[0]
        want.append(x)
    return cases, tq.Chain([([c.gpu], x, [y]) for c, x, y in zip(cases, xs, ys)]), ys, want


def same(ys, want):
    return all(torch.equal(y.view(torch.int16), w.view(torch.int16)) for y, w in zip(ys, want))


# Stages of fewer rows than workgroups leave idle items; the first stage of the
# last chain has one item with a row.
SHAPES = [[(512, 256, 0.1), (640, 512, 0.2), (256, 640, 0.1), (384, 256, 0.0)],
          [(1024, 4096, 0.1), (4096, 1024, 0.0), (256, 4096, 0.2)],
          [(1, 128, 0.0), (256, 128, 0.5)]]


@pytest.mark.parametrize("a, b", [(0, 1), (1, 1), (2, 0)])
def test_two_chains_on_two_streams(a, b):
    chains = [build(60 + i, SHAPES[k]) for i, k in enumerate((a, b))]
    streams = [torch.cuda.Stream() for _ in chains]
    for call in range(4):
        for _, _, ys, _ in chains:
            for y in ys:
                y.fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(8):
            for (_, chain, _, _), s in zip(chains, streams):
                chain.run(stream=s)
        torch.cuda.synchronize()
        for _, chain, ys, want in chains:
            assert chain.error_flag() == 0
            assert same(ys, want), f"call {call}"


@pytest.mark.parametrize("k", range(3))
def test_items_by_ticket(k):
    """Word 16 of the sync block is the call's mode; 2, every item by ticket,
    is what a call takes where its workgroups do not all start."""
    _, chain, ys, want = build(66 + k, SHAPES[k])
    mode = chain.sync[64:68].view(torch.int32)
    for call in range(3):
        for y in ys:
            y.fill_(float("nan"))
        mode.fill_(2 if call != 1 else 0)   # a call in the other mode between
        chain.run()
        torch.cuda.synchronize()
        assert mode.item() == 0 and chain.error_flag() == 0
        assert same(ys, want), f"call {call}"


def test_captured_chain_replays():
    _, chain, ys, want = build(63, SHAPES[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        chain.run()
    for replay in range(4):
        for y in ys:
            y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert same(ys, want), f"replay {replay}"
        assert chain.error_flag() == 0
