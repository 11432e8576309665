"""Solves in workspaces without room for the window passes' sums and tables give the
general passes' results, before and after calls with room for them."""

import pytest
import torch

import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu


def _close(a, b, tol):
    return float((a - b).abs().max()) <= tol * float(b.abs().max())


@pytest.mark.parametrize("shape,was", [((70, 37, 19), 11054336), ((64, 64, 64), None)])
def test_solver(monkeypatch, shape, was):
    """(64^3: large enough to be tuned, once with and once without the window tiles.)"""
    p = wri_synth.custom_problem(shape, nb=2, n_src=2, n_rec=19, seed=3, freqs=(9.0, 12.0), rtol=0.0)
    b = wri.Batch(p, device="cuda:0")
    full = b.workspace(b.mode, 0).numel()
    short = full - 256 if was is None else was
    assert short < full
    run = lambda: wri.objective_grad(b, max_iter=9)
    J, g, res = run()
    with monkeypatch.context() as mp:
        mp.setattr(b, "workspace", lambda mode, flags: torch.empty(short, dtype=torch.uint8, device="cuda:0"))
        small = [run() for _ in range(2)]
        mp.setenv("WRI_TILE", "4,1,2,4,0")   # a window tile does not fit there: the slabs run
        small.append(run())
        mp.delenv("WRI_TILE")
        if was is not None:
            mp.setattr(b, "workspace", lambda mode, flags: torch.empty(was - 1, dtype=torch.uint8, device="cuda:0"))
            with pytest.raises(wri.WriError):
                run()
    J2, g2, _ = run()
    assert J2 == J and torch.equal(g2[0], g[0])
    for Js, gs, rs in small:   # the order of the float64 sums differs, over 9 iterations
        assert [r["iters"] for r in rs] == [r["iters"] for r in res]
        assert abs(Js - J) <= 1e-6 * abs(J) and _close(gs[0], g[0], 1e-4)


def test_fwi(monkeypatch):
    p = wri_synth.custom_problem((70, 37, 19), nb=2, n_src=2, n_rec=19, seed=3, freqs=(9.0, 12.0), rtol=1e-3)
    b = wri.Batch(p, device="cuda:0")
    full = b.fwi_workspace(b.mode, 0).numel()
    f, g, _ = wri.fwi_objective_grad(b, max_iter=400)
    monkeypatch.setattr(b, "fwi_workspace", lambda mode, flags: torch.empty(14206976, dtype=torch.uint8, device="cuda:0"))
    assert full > 14206976
    fs, gs, _ = wri.fwi_objective_grad(b, max_iter=400)
    assert abs(fs - f) <= 1e-4 * abs(f) and _close(gs[0], g[0], 1e-2)
