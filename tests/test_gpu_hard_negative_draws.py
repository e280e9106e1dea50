"""Hard negatives counted on chip: draws over the whole ranking (pins visited once and
more often, many draws per query) with the CU to itself (at most 256 queries) and
shared, at every slot width; a star graph where one pin takes half the landings and
one where every landing is a pin of its own. Bit for bit against the oracle."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _check(orc, off, col, P, B, q, k, walks, hops, lo, hi):
    import paper_1806_01973_amd as ps
    g = ps.DeviceGraph(off, col, P, B)
    out, _ = ps.hard_negatives(g, torch.as_tensor(q).cuda(), k, 5, walks, hops, lo, hi)
    ref = orc.hard_negatives(off, col, P, 5, walks, hops, q, lo, hi, k)
    np.testing.assert_array_equal(out.cpu().numpy(), ref)
    return ref


@pytest.fixture(scope="module")
def graph():
    wl = synth.WORKLOADS["medium"].scaled(30_000, 6_000)
    off, col, _ = synth.make_graph(wl)
    return wl.num_pins, wl.num_boards, off, col


@pytest.mark.parametrize("nq", [40, 257])
@pytest.mark.parametrize("walks,hops", [(512, 2), (1000, 2), (1024, 4), (2048, 4), (4096, 4)])
def test_draws_over_the_whole_ranking(orc, graph, nq, walks, hops):
    P, B, off, col = graph
    print(f"[case] draws nq={nq} W={walks} H={hops}", flush=True)
    q = np.random.default_rng(nq + walks).integers(0, P, nq).astype(np.int32)
    ref = _check(orc, off, col, P, B, q, 130, walks, hops, 0, 40_000)
    assert len(np.unique(ref[0])) > 10


@pytest.mark.parametrize("walks,hops", [(1024, 1), (4096, 2), (4096, 4)])
def test_few_and_many_distinct_pins(orc, walks, hops):
    print(f"[case] few and many distinct pins W={walks} H={hops}", flush=True)
    # Two pins on one board: every landing is one of them.
    off, col = synth.csr_from_edges(3, 2, [(0, 0), (1, 0), (2, 1)])
    _check(orc, off, col, 3, 2, np.array([0, 1, 2, 3], np.int32), 9, walks, hops, 0, 5)
    # One board of 200,000 pins: nearly every landing is a pin of its own.
    P = 200_000
    off, col = synth.csr_from_edges(P, 1, np.stack([np.arange(P), np.zeros(P, np.int64)], 1))
    q = np.array([0, 7, P - 1, P], np.int32)
    _check(orc, off, col, P, 1, q, 70, walks, hops, 100, 20_000)


@pytest.mark.parametrize("nq", [7, 300])
@pytest.mark.parametrize("lo,hi", [(0, 40_000), (0, 300), (6_000, 40_000)])
def test_many_draws_per_query(orc, graph, nq, lo, hi):
    """More draws than threads, over the whole ranking, over pins visited more than once
    alone, and over pins visited once alone."""
    P, B, off, col = graph
    print(f"[case] many draws nq={nq} lo={lo} hi={hi}", flush=True)
    q = np.random.default_rng(nq).integers(0, P, nq).astype(np.int32)
    for k, walks, hops in ((1025, 500, 2), (2100, 4096, 4)):
        _check(orc, off, col, P, B, q, k, walks, hops, lo, hi)
