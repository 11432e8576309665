"""Edges of the tiled stencil passes of the off-grid solver: wavefield, source
unknown and residual after k iterations against CGLS with the oracle's A, e and
P in float64, at the tolerance of the other short iterates (float32 storage:
1e-4)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu


def _cgls(A, e, P, s, c, mode, k):
    """k iterations on [[A, -c e], [lam P, 0]] [u; a] = [0; lam d] (KNOWN: no source
    column, right-hand side alpha e)."""
    est = mode == "estimate"
    d = np.asarray(s.d).astype(np.complex64).astype(np.complex128)
    AH, PT = A.conj().T.tocsr(), P.T.tocsr()
    S = lambda x: (A @ x[0] - (c * x[1] * e if est else 0.0), s.lam * (P @ x[0]))
    SH = lambda r: (AH @ r[0] + s.lam * (PT @ r[1]), -c * np.vdot(e, r[0]) if est else 0j)
    dot = lambda v: float(np.vdot(v[0], v[0]).real + np.vdot(v[1], v[1]).real)
    add = lambda y, a, x: (y[0] + a * x[0], y[1] + a * x[1])
    x = (np.zeros(A.shape[0], complex), 0j)
    r = (np.zeros(A.shape[0], complex) if est else complex(s.alpha) * e, s.lam * d)
    z = SH(r)
    p, g0 = z, dot(z)
    gamma = g0
    for _ in range(k):
        t = S(p)
        a = gamma / dot(t)
        x, r = add(x, a, p), add(r, -a, t)
        z = SH(r)
        new = dot(z)
        p, gamma = add(z, new / gamma, p), new
    return x[0], c * x[1], np.sqrt(gamma / g0)


def _problem(*shapes):
    ps = [wri_synth.custom_problem(s, nb=min(4, min(s) // 2), n_src=2, n_rec=7, seed=5 + i, freqs=(9.0,), rtol=0.0)
          for i, s in enumerate(shapes)]
    return dataclasses.replace(ps[0], grids=[p.grids[0] for p in ps], m=[p.m[0] for p in ps],
                               systems=[dataclasses.replace(s, grid=i) for i, p in enumerate(ps) for s in p.systems])


# two cells a thread with a ragged last tile; the widest tiled row; one wider (column
# march); a single plane; rows wider than a tile; grids of different tile counts
CASES = [[(131, 129, 5)], [(512, 33, 3)], [(513, 5, 4)], [(24, 22, 1)], [(300, 3, 6)],
         [(21, 19, 13), (40, 33, 17), (9, 8, 7)]]


@pytest.mark.parametrize("mode,k", [("estimate", 2), ("known", 1)])
@pytest.mark.parametrize("shapes", CASES)
def test_tile_edges_match_cgls(shapes, mode, k):
    print(f"off-grid tiles {shapes} {mode}", flush=True)
    p = _problem(*shapes)
    rng = np.random.default_rng(3)
    xyz = lambda g, c: np.array([c % g.nx, c // g.nx % g.ny, c // (g.nx * g.ny)]) * g.h + rng.uniform(-.5, .5, 3) * g.h
    src = [xyz(p.grids[s.grid], int(s.src)) for s in p.systems]
    rec = [np.array([xyz(p.grids[s.grid], int(c)) for c in s.rec]) for s in p.systems]
    b = wri.Batch(p, device="cuda:0", mode=mode)
    u = wri.alloc_wavefields(b)
    _, _, res = wri.objective_grad_offgrid(b, src, rec, max_iter=k, u_out=u, with_grad=False)
    for i, s in enumerate(p.systems):
        g = p.grids[s.grid]
        m32 = np.asarray(p.m[s.grid], dtype=np.float32).astype(np.float64).reshape(-1)
        e, P = oracle.offgrid_operators(g, src[i], rec[i])
        ref, alpha, relres = _cgls(oracle.helmholtz(g, m32, s.omega).tocsr(), e, P, s, np.sqrt(42.0) / g.h ** 2, mode, k)
        err = np.linalg.norm(u[i].cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  sys {i}: u err {err:.2e} relres {res[i]['relres']:.6e} reference {relres:.6e}", flush=True)
        assert res[i]["iters"] == k and err < 1e-4
        assert abs(res[i]["relres"] - relres) <= 1e-4 * relres
        if mode == "estimate":
            assert abs(res[i]["alpha"] - alpha) <= 1e-4 * abs(alpha)
