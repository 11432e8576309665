"""Where a call's host path branches: limits on the iterations around the lengths
of a chunk, and receiver lists shared, alternating or empty between systems."""
import dataclasses

import numpy as np
import pytest
import torch

import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu


def _problem(n_src=3):
    return wri_synth.custom_problem((22, 19, 17), nb=4, n_src=n_src, n_rec=8, seed=23, freqs=(9.0,), rtol=0.0)


@pytest.mark.parametrize("k", [0, 1, 15, 16, 17, 31, 32, 33, 47, 48, 49])
def test_iteration_limits(k):
    """rtol 0: every system makes exactly k iterations, the same in one launch after
    another, from replayed graphs and with a status check after every chunk (timed
    launches); the off-grid solver at the cells' own positions and the
    preconditioned one stop there as well."""
    print(f"limit {k}", flush=True)
    p = _problem()
    b = wri.Batch(p, device="cuda:0")
    runs = []
    for flags in (0, 0, wri.FLAG_NO_GRAPH, wri.FLAG_TIMING):
        J, g, res = wri.objective_grad(b, max_iter=k, flags=flags)
        assert [r["iters"] for r in res] == [k] * 3 and {r["status"] for r in res} == {"max_iter"}
        runs.append((J, g[0].cpu()))
    for J, g in runs[1:]:
        assert J == runs[0][0] and torch.equal(g, runs[0][1])
    g = p.grids[0]
    xyz = lambda c: np.stack([c % g.nx, c // g.nx % g.ny, c // (g.nx * g.ny)], axis=-1) * g.h
    for _, _, res in (wri.objective_grad_offgrid(b, [xyz(np.int64(s.src)) for s in p.systems],
                                                 [xyz(np.asarray(s.rec, np.int64)) for s in p.systems], max_iter=k),
                      wri.objective_grad_precond(b, max_iter=k)):
        assert [r["iters"] for r in res] == [k] * 3 and {r["status"] for r in res} == {"max_iter"}


def test_receiver_lists():
    """Five systems with lists A A B A and none give the bits of five calls."""
    p = _problem(5)
    lists = [p.systems[0].rec, p.systems[0].rec, p.systems[0].rec[::-1][:5].copy(), p.systems[0].rec, np.zeros(0, np.int32)]
    systems = [dataclasses.replace(s, rec=r, d=s.d[:len(r)]) for s, r in zip(p.systems, lists)]
    g = p.grids[0]
    rng = np.random.default_rng(1)
    at = {len(r): rng.uniform(1.0, g.h * 15, (len(r), 3)) for r in lists}
    src = [rng.uniform(1.0, g.h * 15, 3) for _ in lists]

    def run(idx):
        b = wri.Batch(dataclasses.replace(p, systems=[systems[i] for i in idx]), device="cuda:0")
        u, off, pre = (wri.alloc_wavefields(b) for _ in range(3))
        wri.solve(b, max_iter=9, u_out=u)
        wri.objective_grad_offgrid(b, [src[i] for i in idx], [at[len(lists[i])] for i in idx], max_iter=9, u_out=off)
        wri.objective_grad_precond(b, max_iter=3, u_out=pre)
        return [[t.cpu() for t in v] for v in (u, off, pre)]

    together = run(range(5))
    for i in range(5):
        for name, all_, one in zip(("solve", "off-grid", "preconditioned"), together, run([i])):
            assert torch.equal(all_[i], one[0]), (name, i)
