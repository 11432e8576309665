"""The window march (tile pf = 4) against the slab march 4,4,32,0,0: the same
stencil arithmetic on another tiling, so the iterates of a few steps agree to
the effect of the summation order of the float64 partials, and the oracle's
complex128 CGLS within complex64 storage.  Sizes sit where the tiling can go
wrong: planes of one tile less, exactly and more than one tile's cells, rows
wider than a workgroup (a second round of halo cells), one to five planes
around the two- and four-plane tiles, receivers on every cell of a tile (more
than a workgroup's threads) and sources in the first and last cell."""
import sys

import numpy as np
import pytest
import torch

import oracle
import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu

WINDOWS = ("4,1,2,4,0", "4,1,4,4,0", "4,2,4,4,0", "8,2,4,4,0")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def _solve(p, mode, monkeypatch, tile, k, **kw):
    monkeypatch.setenv("WRI_TILE", tile)
    out = wri.solve(wri.Batch(p, device="cuda:0", mode=mode), max_iter=k, **kw)
    monkeypatch.delenv("WRI_TILE")
    return out


@pytest.mark.parametrize("mode", ["estimate", "known"])
@pytest.mark.parametrize("shape", [(16, 16, 4), (15, 17, 5), (257, 1, 2), (1, 513, 3), (32, 32, 1), (70, 37, 9),
                                   (380, 3, 6), (300, 2, 4)])
def test_window_march_gives_the_slab_iterates(monkeypatch, shape, mode):
    print(f"window {shape} {mode}", flush=True)
    sys.stdout.flush()
    p = wri_synth.custom_problem(shape, nb=1, n_src=1, n_rec=min(shape[2], 8), seed=3, freqs=(14.0, 19.0), rtol=0.0)
    g = p.grids[0]
    p.systems[0].src, p.systems[1].src = 0, g.n - 1
    # the second system: a receiver on every cell of the top plane (at most 600)
    n = min(600, g.nx * g.ny)
    p.systems[1].rec = np.arange(n, dtype=np.int32)
    p.systems[1].d = np.exp(0.1j * np.arange(n)) * 1e-3
    k = 6
    ref_u, ref = _solve(p, mode, monkeypatch, "4,4,32,0,0", k)
    for tile in WINDOWS:
        u, res = _solve(p, mode, monkeypatch, tile, k)
        for i in range(2):
            scale = float(ref_u[i].abs().max())
            assert float((u[i] - ref_u[i]).abs().max()) <= 1e-5 * scale, (tile, i)
            assert abs(res[i]["J"] - ref[i]["J"]) <= 1e-6 * abs(ref[i]["J"]), (tile, i)
            assert res[i]["iters"] == ref[i]["iters"] and res[i]["status"] == ref[i]["status"], (tile, i)


@pytest.mark.parametrize("tile", WINDOWS)
def test_window_march_warm_start_and_many_grids(monkeypatch, tile):
    """Five grids in one call (more groups than ride in the launch arguments),
    cold and warm started, against the slab march."""
    print(f"window, five grids, {tile}", flush=True)
    parts = [wri_synth.custom_problem(s, nb=2, n_src=2, n_rec=6, seed=i, freqs=(12.0,), rtol=0.0)
             for i, s in enumerate(((20, 9, 7), (16, 16, 4), (33, 5, 12), (9, 30, 8), (12, 11, 13)))]
    for i, q in enumerate(parts):
        for s in q.systems:
            s.grid = i
    p = wri_synth.Problem("five", [q.grids[0] for q in parts], [q.m[0] for q in parts], [q.m_true[0] for q in parts],
                          [s for q in parts for s in q.systems])
    ref_u, ref = _solve(p, "estimate", monkeypatch, "4,4,32,0,0", 6)
    u, res = _solve(p, "estimate", monkeypatch, tile, 6)
    warm = [[0.5 * x for x in ref_u] for _ in range(2)]
    _solve(p, "estimate", monkeypatch, "4,4,32,0,0", 4, flags=wri.FLAG_WARM_START, u_out=warm[0])
    _solve(p, "estimate", monkeypatch, tile, 4, flags=wri.FLAG_WARM_START, u_out=warm[1])
    for i in range(len(p.systems)):
        for a, b in ((u[i], ref_u[i]), (warm[1][i], warm[0][i])):
            assert float((a - b).abs().max()) <= 1e-5 * float(b.abs().max()), (tile, i)
        assert abs(res[i]["J"] - ref[i]["J"]) <= 1e-6 * abs(ref[i]["J"]), (tile, i)


@pytest.mark.parametrize("mode", ["estimate", "known"])
@pytest.mark.parametrize("shape", [(16, 16, 4), (15, 17, 5), (257, 1, 2), (1, 513, 3), (32, 32, 1), (70, 37, 9),
                                   (380, 3, 6), (300, 2, 4)])
def test_window_march_gives_the_oracle_iterates(monkeypatch, shape, mode):
    """Two steps against the oracle's complex128 CGLS (float32 storage: 1e-4, as in the other
    solvers' tile tests), receivers on the top plane, sources in the first and last cell."""
    print(f"window oracle {shape} {mode}", flush=True)
    p = wri_synth.custom_problem(shape, nb=1, n_src=1, n_rec=min(shape[2], 8), seed=3, freqs=(14.0, 19.0), rtol=0.0)
    g = p.grids[0]
    p.systems[0].src, p.systems[1].src = 0, g.n - 1
    n = min(600, g.nx * g.ny)
    p.systems[1].rec = np.arange(n, dtype=np.int32)
    p.systems[1].d = np.exp(0.1j * np.arange(n)) * 1e-3
    k = 2
    m32 = np.asarray(p.m[0], dtype=np.float32).astype(np.float64).reshape(-1)
    refs = []
    for i, s in enumerate(p.systems):
        A, P, _ = oracle.system_operators(p, i, m=m32)
        d = np.asarray(s.d).astype(np.complex64).astype(np.complex128)
        refs.append(oracle.cgls(A, P, s.lam, s.src, mode, s.alpha, d, 0.0, k, alpha_scale=np.sqrt(42.0) / g.h ** 2))
    for tile in WINDOWS:
        u, res = _solve(p, mode, monkeypatch, tile, k)
        for i, ref in enumerate(refs):
            err = np.linalg.norm(u[i].cpu().numpy() - ref["u"]) / np.linalg.norm(ref["u"])
            print(f"  {tile} sys {i}: u err {err:.2e} relres {res[i]['relres']:.6e} oracle {ref['relres']:.6e}", flush=True)
            assert res[i]["iters"] == k and err < 1e-4
            assert abs(res[i]["relres"] - ref["relres"]) <= 1e-4 * ref["relres"]
