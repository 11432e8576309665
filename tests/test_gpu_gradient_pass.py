"""The gradient pass over many systems and the transposed resampling, at the
edges of their tilings."""
import numpy as np
import pytest
import torch

import oracle
import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 256 cells per workgroup (one short, exactly, one over) and 1, 7, 8, 9, 64 and 70
# systems: full and ragged rounds of 8, one table of 64 and a second
@pytest.mark.parametrize("shape,n_src,n_freq", [((17, 5, 3), 1, 1), ((16, 16, 1), 7, 1), ((257, 1, 1), 8, 1),
                                                ((16, 8, 4), 3, 3), ((32, 8, 2), 32, 2), ((14, 9, 5), 14, 5)])
def test_gradient_is_the_sum_over_systems(shape, n_src, n_freq):
    """One call over all systems against the float64 sum of one call per system
    (same tile, so the same iterates): float32 gradients, one rounding each."""
    print(f"gradient {shape} {n_src}x{n_freq}", flush=True)
    p = wri_synth.custom_problem(shape, nb=1, n_src=n_src, n_rec=min(4, shape[2]), seed=9,
                                 freqs=tuple(12.0 + k for k in range(n_freq)), rtol=0.0)
    flags = wri.FLAG_NO_AUTOTUNE
    J, g, res = wri.objective_grad(wri.Batch(p, device=DEV), max_iter=3, flags=flags)
    total, scale, Js = 0.0, 0.0, 0.0
    for k in range(len(p.systems)):
        Jk, gk, _ = wri.objective_grad(wri.Batch(p.subset([k]), device=DEV), max_iter=3, flags=flags)
        gk = gk[0].cpu().numpy().astype(np.float64)
        total, scale, Js = total + gk, scale + np.abs(gk), Js + Jk
        assert res[k]["J"] == pytest.approx(Jk, rel=1e-12)
    assert J == pytest.approx(Js, rel=1e-12)
    assert np.all(np.abs(g[0].cpu().numpy() - total) <= 2e-7 * scale + 1e-30)


# cell-size ratios at the edges of the candidate counts (3 up to ratio 1, 5 up to 2,
# 14 up to 6.5), one-cell axes, and a model of more than 1024 tiles of 64 x 16 x 4
@pytest.mark.parametrize("model,ratio", [((9, 7, 5), 1.0), ((30, 11, 8), 0.37), ((30, 11, 8), 1.03),
                                         ((67, 18, 9), 2.0), ((40, 5, 6), 2.01), ((12, 6, 4), 6.4), ((65, 1, 1), 1.0),
                                         ((260, 130, 70), 0.8)])
def test_transposed_resampling(model, ratio):
    print(f"resample {model} h_m / h_g {ratio}", flush=True)
    gm = wri_synth.Grid(*model, 10.0 * ratio, 0, 1500.0)
    n = [1 if k == 1 else max(2, int((k - 1) * ratio) + 1) for k in model]
    gg = wri_synth.Grid(*n, 10.0, 0, 1500.0)
    rng = np.random.default_rng(4)
    v = rng.standard_normal(gg.n).astype(np.float32)
    R = oracle.resample_matrix(gm, gg)
    want = R.T @ v.astype(np.float64)
    out = torch.full((gm.n,), 0.5, dtype=torch.float32, device=DEV)
    wri.grid_to_model_adjoint(gm, gg, torch.as_tensor(v, device=DEV), out)
    bound = 1e-6 * (np.abs(R).T @ np.abs(v.astype(np.float64))).max()
    assert np.abs(out.cpu().numpy() - want).max() <= bound
    wri.grid_to_model_adjoint(gm, gg, torch.as_tensor(v, device=DEV), out, accumulate=True)
    assert np.abs(out.cpu().numpy() - 2.0 * want).max() <= 2.0 * bound
