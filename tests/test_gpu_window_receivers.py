"""Long receiver lists in the window march (tile pf = 4), found through buckets of 64
cells, against the slab march 4,4,32,0,0: list lengths around the longest list that is
scanned (1024) and a receiver on every cell, scattered and unsorted, on planes and grids
that are no multiple of a bucket, beside a system with a short list and one with none.
The iterates of a few steps differ by the summation order of the float64 partials only."""
import dataclasses

import numpy as np
import pytest

import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu

WINDOWS = ("4,1,2,4,0", "4,1,4,4,0", "4,2,4,4,0", "8,2,4,4,0")


@pytest.mark.parametrize("shape,n_rec", [((22, 19, 17), 600), ((22, 19, 17), 1024), ((22, 19, 17), 1025),
                                         ((22, 19, 17), 22 * 19 * 17), ((64, 16, 5), 64 * 16 * 5), ((257, 3, 4), 1537),
                                         ((1, 163, 9), 1467), ((41, 25, 6), 3000)])
def test_long_lists_give_the_slab_iterates(monkeypatch, shape, n_rec):
    print(f"receivers {shape} {n_rec}", flush=True)
    p = wri_synth.custom_problem(shape, nb=1, n_src=1, n_rec=min(shape[2], 6), seed=3, freqs=(14.0, 17.0, 19.0, 21.0),
                                 rtol=0.0)
    rng = np.random.default_rng(5)
    for k, n in ((0, n_rec), (1, n_rec), (2, 0)):   # the fourth keeps its short list
        rec = rng.permutation(p.grids[0].n)[:n].astype(np.int32)
        d = (np.exp(0.1j * np.arange(n)) * 1e-3).astype(np.complex64)
        p.systems[k] = dataclasses.replace(p.systems[k], rec=rec, d=d)

    def run(tile):
        monkeypatch.setenv("WRI_TILE", tile)
        b = wri.Batch(p, device="cuda:0")
        u, res = wri.solve(b, max_iter=6)
        assert [r["iters"] for r in res] == [6, 6, 0, 6]   # no receivers: the right side is zero
        return u, res

    ref_u, ref = run("4,4,32,0,0")
    for tile in WINDOWS:
        u, res = run(tile)
        for i in range(4):
            assert float((u[i] - ref_u[i]).abs().max()) <= 1e-5 * float(ref_u[i].abs().max()), (tile, i)
            assert abs(res[i]["J"] - ref[i]["J"]) <= 1e-6 * abs(ref[i]["J"]), (tile, i)
