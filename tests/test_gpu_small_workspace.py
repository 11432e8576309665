"""Solves in workspaces without room for the window passes' sums and tables give the
general passes' results, before and after calls with room for them."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

import oracle
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


@pytest.mark.parametrize("n,count", [(1000, 5), (6400, 5), (6657, 5), (200000, 3), (200000, 8)])
def test_direction(n, count):
    """The former 8704 bytes hold the partials of all inner products on small vectors
    only (5 pairs: up to 25 workgroups of 256 cells); past that the recursion runs.  Both
    against the oracle, with the tolerance of the direction's own test."""
    rng = np.random.default_rng(7)
    g, S = rng.standard_normal(n).astype(np.float32), rng.standard_normal((count, n)).astype(np.float32)
    Y = (S * (1.0 + 9.0 * rng.random(n)).astype(np.float32)).astype(np.float32)
    pairs = [(S[i].astype(np.float64), Y[i].astype(np.float64)) for i in range(count)]
    s, y = pairs[-1]
    want = -oracle.lbfgs_two_loop(g.astype(np.float64), pairs, np.dot(s, y) / np.dot(y, y))
    dev = [torch.as_tensor(a, device="cuda:0") for a in (g, S, Y)]
    for size in (8704, wri.lib().wri_lbfgs_workspace_bytes(count)):
        ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda:0")
        d = torch.empty_like(dev[0])
        p = [ctypes.c_void_p(t.data_ptr()) for t in dev]
        code = wri.lib().wri_lbfgs_direction(n, *p, count, count, count - 1, 0.0, ctypes.c_void_p(d.data_ptr()),
                                             ctypes.c_void_p(ws.data_ptr()), size, None)
        torch.cuda.synchronize()
        assert code == wri.OK
        assert np.linalg.norm(d.cpu().numpy() - want) < 1e-5 * np.linalg.norm(want), size


def test_outer_loop_with_many_systems():
    """600 systems: the window march's sums no longer fit beside the TV pass, and the query
    grows; the former size runs the slab marches.  One update of each agrees to the
    difference of the solves."""
    p = wri_synth.custom_problem((22, 19, 17), nb=2, n_src=12, n_rec=8, seed=3, freqs=tuple(9.0 + 0.1 * i for i in range(50)),
                                 rtol=1e-3, data="none")
    rng = np.random.default_rng(2)
    p = p.with_data([1e-3 * (rng.standard_normal(len(s.rec)) + 1j * rng.standard_normal(len(s.rec))) for s in p.systems])
    out = []
    for was in (False, True):
        b = wri.Batch(p, device="cuda:0")
        L = wri.lib()
        query = L.wri_awri_workspace_bytes(b.cgrids, b.csys, b.nsys, b.mode, 0, 2)
        size = query - 4096 if was else query
        o = wri.WriAwriOptions(0.0, 1e-9, 1e-3, 1e-6, 0.02, 0.0, 0.0, 0.0, 1, 2, 2000, 0, 1, 0)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        rec = ctypes.c_int32(0)
        hist = (wri.WriAwriRecord * 8)()
        code = L.wri_awri(b.cgrids, ctypes.c_void_p(b.m[0].data_ptr()), b.csys, b.nsys, b.mode, ctypes.byref(o), hist, 8,
                          ctypes.byref(rec), ctypes.c_void_p(ws.data_ptr()), size, None)
        assert code == wri.OK and rec.value == 2
        out.append((b.m[0].clone(), hist[1].F))
    assert abs(out[0][1] - out[1][1]) <= 1e-4 * abs(out[0][1])
    m0 = torch.as_tensor(p.m[0].reshape(-1), dtype=torch.float32, device="cuda:0")
    assert _close(out[1][0] - m0, out[0][0] - m0, 1e-2)


def test_offgrid(monkeypatch):
    """One system of 64^3, large enough for more sums than the march has, beside a small one."""
    parts = [wri_synth.custom_problem(s, nb=4, n_src=1, n_rec=9, seed=3, freqs=(9.0,), rtol=0.0)
             for s in ((64, 64, 64), (22, 19, 17))]
    systems = [dataclasses.replace(q.systems[0], grid=i) for i, q in enumerate(parts)]
    p = wri_synth.Problem("two", [q.grids[0] for q in parts], [q.m[0] for q in parts], [q.m[0] for q in parts], systems)
    b = wri.Batch(p, device="cuda:0")
    rng = np.random.default_rng(1)
    src, rec = rng.uniform(40.0, 120.0, (2, 3)), rng.uniform(40.0, 120.0, (2, 9, 3))
    run = lambda: wri.objective_grad_offgrid(b, list(src), list(rec), max_iter=9)
    J, g, _ = run()
    full = b._ws[("offgrid",)].numel()
    monkeypatch.setattr(wri.lib(), "wri_offgrid_workspace_bytes", lambda *a: full - 512)
    del b._ws[("offgrid",)]
    Js, gs, _ = run()
    assert b._ws[("offgrid",)].numel() == full - 512
    assert abs(Js - J) <= 1e-6 * abs(J) and _close(gs[0], g[0], 1e-4) and _close(gs[1], g[1], 1e-4)
    monkeypatch.setattr(wri.lib(), "wri_offgrid_workspace_bytes", lambda *a: full - 2048)
    del b._ws[("offgrid",)]
    with pytest.raises(wri.WriError):
        run()


@pytest.mark.parametrize("shape,n_src,n_freq", [((33, 31, 1), 13, 5), ((32, 32, 1), 16, 4), ((41, 25, 1), 14, 5),
                                                ((41, 25, 4), 13, 1)])
def test_gradient_with_four_cells_a_thread(monkeypatch, shape, n_src, n_freq):
    """One workgroup's 1024 cells less one, exactly and one more, and 13 to 70 systems (a
    table of 64 and a second): on the same iterates (a forced slab tile) the gradient has
    the bits of the pass with one cell a thread, and J differs in the order of its sums."""
    print(f"gradient {shape} {n_src}x{n_freq}", flush=True)
    p = wri_synth.custom_problem(shape, nb=1, n_src=n_src, n_rec=min(4, shape[2]), seed=9,
                                 freqs=tuple(12.0 + k for k in range(n_freq)), rtol=0.0)
    b = wri.Batch(p, device="cuda:0")
    full = b.workspace(b.mode, 0).numel()
    monkeypatch.setenv("WRI_TILE", "4,4,32,0,0")
    J, g, res = wri.objective_grad(b, max_iter=3)
    monkeypatch.setattr(b, "workspace", lambda mode, flags: torch.empty(full - 256, dtype=torch.uint8, device="cuda:0"))
    Js, gs, rs = wri.objective_grad(b, max_iter=3)
    assert torch.equal(gs[0], g[0])
    for x, y in zip(rs, res):   # some 4000 terms in float64
        assert x["relres"] == y["relres"] and abs(x["J"] - y["J"]) <= 1e-12 * y["J"]
    assert abs(Js - J) <= 1e-12 * abs(J)
