"""Edges of the tiled V-cycle passes: the preconditioned iterates after k steps
against the oracle's preconditioned CGLS at the tolerance of the other
preconditioner tests (float32 storage: 1e-4)."""
import numpy as np
import pytest
import torch

import oracle
import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu

# odd axes with a level beside the one-workgroup cycle's largest; two cells a thread
# with a ragged last tile and one row of coarse planes; the widest tiled row; one
# wider (per-cell passes); a level of exactly 4096 cells as the coarse cycle's first
SHAPES = [(41, 47, 29), (131, 129, 5), (512, 33, 4), (513, 7, 5), (32, 32, 32)]


@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_tile_edges_match_oracle(shape, k):
    print(f"precond tiles {shape} k={k}", flush=True)
    p = wri_synth.custom_problem(shape, nb=min(4, min(shape) // 2), n_src=2, n_rec=7, seed=17, freqs=(9.0,), rtol=0.0)
    b = wri.Batch(p, device="cuda:0")
    u = wri.alloc_wavefields(b)
    _, _, res = wri.objective_grad_precond(b, max_iter=k, u_out=u, with_grad=False)
    for i, s in enumerate(p.systems):
        g = p.grids[s.grid]
        m32 = np.asarray(p.m[s.grid], dtype=np.float32).astype(np.float64).reshape(-1)
        A, P, _ = oracle.system_operators(p, i, m=m32)
        lev = oracle.csl_levels(g, m32)
        d = np.asarray(s.d).astype(np.complex64).astype(np.complex128)
        ref = oracle.pcgls(A, P, s.lam, s.src, "estimate", s.alpha, d, 0.0, k,
                           lambda v: oracle.csl_vcycle(lev, s.omega, v),
                           lambda v: oracle.csl_vcycle(lev, s.omega, v, adjoint=True))
        got = u[i].cpu().numpy().astype(np.complex128)
        err = np.linalg.norm(got - ref["u"]) / np.linalg.norm(ref["u"])
        print(f"  sys {i}: u err {err:.2e} relres {res[i]['relres']:.6e} oracle {ref['relres']:.6e}", flush=True)
        assert res[i]["iters"] == k and err < 1e-4
        assert abs(res[i]["relres"] - ref["relres"]) <= 1e-4 * ref["relres"]
