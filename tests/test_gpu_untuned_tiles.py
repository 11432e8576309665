"""Without tuning a system gives the same bits alone and in any batch: each grid has a
tile of its own, also where the batch mixes grids that the window march fits with grids
of too many tiles or too wide rows for it."""
import dataclasses

import pytest
import torch

import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu

FIT = [(22, 19, 17), (70, 3, 5), (16, 16, 4)]
WIDE = [(1200, 3, 4), (1153, 2, 6)]       # rows past the march's LDS
MANY = [(128, 128, 66)]                   # 33 x 64 = 2112 tiles


def _parts(shapes):
    return [wri_synth.custom_problem(s, nb=2, n_src=2, n_rec=4, seed=i, freqs=(12.0,), rtol=0.0)
            for i, s in enumerate(shapes)]


def _join(parts):
    systems = [dataclasses.replace(s, grid=i) for i, q in enumerate(parts) for s in q.systems]
    return wri_synth.Problem("mixed", [q.grids[0] for q in parts], [q.m[0] for q in parts],
                             [q.m_true[0] for q in parts], systems)


def _run(p, flags, warm=None):
    b = wri.Batch(p, device="cuda:0")
    if flags == "noalloc":
        u, res = wri.solve_noalloc(b, max_iter=21)
        return None, [x.cpu() for x in u], [r["relres"] for r in res]
    u = wri.alloc_wavefields(b) if warm is None else [x.cuda() for x in warm]
    J, g, res = wri.objective_grad(b, max_iter=21, flags=flags, u_out=u)
    return [x.cpu() for x in g], [x.cpu() for x in u], [(r["relres"], r["J"]) for r in res]


@pytest.mark.parametrize("shapes,flags", [
    (FIT + WIDE, 0),                                    # below the size that is tuned
    ([FIT[0], WIDE[0], FIT[1], WIDE[1], FIT[2]], wri.FLAG_NO_AUTOTUNE),
    (MANY + FIT, wri.FLAG_NO_AUTOTUNE),
    (MANY + FIT, wri.FLAG_NO_AUTOTUNE | wri.FLAG_NO_GRAPH),
    (FIT + WIDE, wri.FLAG_NO_AUTOTUNE | wri.FLAG_TIMING),
    (WIDE, wri.FLAG_NO_AUTOTUNE),
    ([WIDE[0]] + FIT, "noalloc"),
])
def test_alone_and_in_a_mixed_batch(shapes, flags):
    print(f"mixed {shapes} flags {flags}", flush=True)
    parts = _parts(shapes)
    g, u, scal = _run(_join(parts), flags)
    for i, q in enumerate(parts):
        g1, u1, s1 = _run(q, flags)
        assert scal[2 * i:2 * i + 2] == s1, shapes[i]
        assert all(torch.equal(a, b) for a, b in zip(u[2 * i:2 * i + 2], u1)), shapes[i]
        assert g is None or torch.equal(g[i], g1[0]), shapes[i]


def test_mixed_batch_warm_started():
    parts = _parts([FIT[0], WIDE[0], FIT[2]])
    _, u, _ = _run(_join(parts), wri.FLAG_NO_AUTOTUNE)
    warm = [0.5 * x for x in u]
    flags = wri.FLAG_NO_AUTOTUNE | wri.FLAG_WARM_START
    _, w, _ = _run(_join(parts), flags, warm)
    for i, q in enumerate(parts):
        _, w1, _ = _run(q, flags, warm[2 * i:2 * i + 2])
        assert all(torch.equal(a, b) for a, b in zip(w[2 * i:2 * i + 2], w1)), i


def test_scratch_holds_the_largest_share_of_sums():
    """Many systems on planes of one cell, where a tile has the fewest cells, and with a
    receiver on every cell, up to the limit of the fixed scratch."""
    q = wri_synth.custom_problem((1, 1, 2048), nb=0, n_src=1, n_rec=2048, seed=1, freqs=(9.0,), rtol=0.0)
    q = dataclasses.replace(q, systems=[dataclasses.replace(q.systems[0], rec=q.systems[0].rec[i:].copy(),
                                                            d=q.systems[0].d[i:]) for i in range(250)])
    u, res = wri.solve_noalloc(wri.Batch(q, device="cuda:0"), max_iter=3)
    v, _ = wri.solve(wri.Batch(dataclasses.replace(q, systems=q.systems[100:101]), device="cuda:0"), max_iter=3,
                     flags=wri.FLAG_NO_AUTOTUNE)
    assert {r["iters"] for r in res} == {3} and torch.equal(u[100], v[0])
