"""Arrays that the tiled V-cycle passes share (r and p by parity, the level-0 residual in
t, partial sums in level 1): iterates through both parities against the oracle's
preconditioned CGLS, with the tolerance of the tiles' other tests, where level 1 is the
coarsest and fits a workgroup, and for systems that stop at different iterations."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(64, 16, 5), (41, 47, 29), (131, 129, 5)])
def test_iterates_match_oracle(shape):
    print(f"precond shared {shape}", flush=True)
    p = wri_synth.custom_problem(shape, nb=2, n_src=1, n_rec=5, seed=17, freqs=(9.0,), rtol=0.0)
    m32 = np.asarray(p.m[0], dtype=np.float32).astype(np.float64).reshape(-1)
    A, P, _ = oracle.system_operators(p, 0, m=m32)
    lev, s = oracle.csl_levels(p.grids[0], m32), p.systems[0]
    d = np.asarray(s.d).astype(np.complex64).astype(np.complex128)
    b = wri.Batch(p, device="cuda:0")
    for k in (1, 2, 3, 4):
        u = wri.alloc_wavefields(b)
        _, _, res = wri.objective_grad_precond(b, max_iter=k, u_out=u, with_grad=False)
        ref = oracle.pcgls(A, P, s.lam, s.src, "estimate", s.alpha, d, 0.0, k,
                           lambda v: oracle.csl_vcycle(lev, s.omega, v),
                           lambda v: oracle.csl_vcycle(lev, s.omega, v, adjoint=True))
        got = u[0].cpu().numpy().astype(np.complex128)
        err = np.linalg.norm(got - ref["u"]) / np.linalg.norm(ref["u"])
        print(f"  k {k}: u err {err:.2e} relres {res[0]['relres']:.6e} oracle {ref['relres']:.6e}", flush=True)
        assert res[0]["iters"] == k and err < 1e-4
        assert abs(res[0]["relres"] - ref["relres"]) <= 1e-4 * ref["relres"]


def test_systems_that_stop_apart():
    """Tolerances that stop two systems at iterations of both parities: J and the gradient
    of the batch are those of the systems alone (a finished system's buffers are left)."""
    p = wri_synth.custom_problem((41, 47, 29), nb=2, n_src=2, n_rec=5, seed=17, freqs=(9.0, 11.0), rtol=1e-2)
    p = dataclasses.replace(p, systems=[dataclasses.replace(s, rtol=r)
                                        for s, r in zip(p.systems, (3e-1, 1e-1, 3e-2, 1e-2))])
    b = wri.Batch(p, device="cuda:0")
    u = wri.alloc_wavefields(b)
    J, g, res = wri.objective_grad_precond(b, u_out=u)
    print("iterations", [r["iters"] for r in res], flush=True)
    assert len({r["iters"] for r in res}) > 1
    gsum = torch.zeros_like(g[0], dtype=torch.float64)
    for i, s in enumerate(p.systems):
        b1 = wri.Batch(dataclasses.replace(p, systems=[s]), device="cuda:0")
        u1 = wri.alloc_wavefields(b1)
        J1, g1, r1 = wri.objective_grad_precond(b1, u_out=u1)
        assert r1[0]["iters"] == res[i]["iters"] and r1[0]["J"] == res[i]["J"] and torch.equal(u1[0], u[i])
        gsum += g1[0].double()
    assert float((gsum - g[0].double()).abs().max()) <= 1e-6 * float(gsum.abs().max())   # four float32 roundings
