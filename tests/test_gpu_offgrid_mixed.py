"""Off-grid systems give the same bits alone and in any batch: their passes depend on
their own grid only.  Grids of the column march (rows over 512 cells), of one and of two
cells a thread, and more grids of a kind than ride in the launch arguments."""
import dataclasses

import numpy as np
import pytest
import torch

import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu

MARCH = [(513, 4, 5), (600, 3, 4)]
ONE = [(22, 19, 17), (40, 5, 9), (16, 16, 4), (127, 129, 5), (9, 30, 8)]
TWO = [(128, 128, 6), (200, 90, 5)]


def _parts(shapes):
    return [wri_synth.custom_problem(s, nb=2, n_src=2, n_rec=5, seed=i, freqs=(12.0,), rtol=0.0)
            for i, s in enumerate(shapes)]


def _run(parts, max_iter=20):
    systems = [dataclasses.replace(s, grid=i) for i, q in enumerate(parts) for s in q.systems]
    systems = systems[::2] + systems[1::2]   # the systems of a grid apart
    p = wri_synth.Problem("mixed", [q.grids[0] for q in parts], [q.m[0] for q in parts],
                          [q.m_true[0] for q in parts], systems)

    def xyz(s, cells):
        g = p.grids[s.grid]
        c = np.asarray(cells, np.int64)
        return (np.stack([c % g.nx, c // g.nx % g.ny, c // (g.nx * g.ny)], axis=-1) + 0.31) * g.h

    b = wri.Batch(p, device="cuda:0")
    u = wri.alloc_wavefields(b)
    J, g, res = wri.objective_grad_offgrid(b, [xyz(s, s.src) for s in systems], [xyz(s, s.rec) for s in systems],
                                           max_iter=max_iter, u_out=u)
    assert {r["iters"] for r in res} == {max_iter}
    return [x.cpu() for x in g], [x.cpu() for x in u], [(r["relres"], r["J"], r["alpha_ls"]) for r in res]


@pytest.mark.parametrize("shapes", [[ONE[0], TWO[0]], [TWO[0], ONE[0]], [MARCH[0], ONE[0]], [MARCH[1]] + ONE + TWO,
                                    MARCH, ONE])
def test_alone_and_in_a_mixed_batch(shapes):
    print(f"mixed {shapes}", flush=True)
    parts = _parts(shapes)
    n = len(parts)
    g, u, scal = _run(parts)
    for i, q in enumerate(parts):
        g1, u1, s1 = _run([q])
        assert [scal[i], scal[n + i]] == s1, shapes[i]
        assert torch.equal(u[i], u1[0]) and torch.equal(u[n + i], u1[1]), shapes[i]
        assert torch.equal(g[i], g1[0]), shapes[i]
