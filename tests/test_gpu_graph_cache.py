"""Chunks of several replayed graphs, and the cache of graphs past its bound of 64."""
import pytest
import torch

import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu


def _run(b, k, flags=0):
    J, g, res = wri.objective_grad(b, max_iter=k, flags=flags)
    assert [r["iters"] for r in res] == [k] * 3 and {r["status"] for r in res} == {"max_iter"}
    return J, g[0].cpu()


def _problem():
    return wri_synth.custom_problem((22, 19, 17), nb=4, n_src=3, n_rec=8, seed=23, freqs=(9.0,), rtol=0.0)


@pytest.mark.parametrize("k", [79, 95, 111, 112, 127, 160])
def test_chunks_of_several_graphs(k):
    """The third chunk of k + 1 iterations is one graph, two in a row without a look at
    the statuses (32 and 16), one of 64, and one with launches after it: the bits of
    eager launches each time, captured and replayed."""
    print(f"limit {k}", flush=True)
    b = wri.Batch(_problem(), device="cuda:0")
    want = _run(b, k, wri.FLAG_NO_GRAPH)
    for _ in range(3):
        J, g = _run(b, k)
        assert J == want[0] and torch.equal(g, want[1])


def test_cache_emptied_between_two_graphs_of_a_chunk():
    """Every workspace adds three graphs (16, 32 and 16 later iterations), the last one
    while the one before it replays: over 64 of them the cache is emptied there."""
    p = _problem()
    batches = [wri.Batch(p, device="cuda:0") for _ in range(48)]   # held: workspaces of their own
    want = _run(batches[0], 95, wri.FLAG_NO_GRAPH)
    for rep in range(2):
        for i, b in enumerate(batches):
            J, g = _run(b, 95)
            assert J == want[0] and torch.equal(g, want[1]), (rep, i)
