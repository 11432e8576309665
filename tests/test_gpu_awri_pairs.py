"""The outer loop's ring of curvature pairs on a grid whose vectors are padded in the
ring (1320 cells): every update is the two-loop recursion on the pairs of the updates
before it."""
import numpy as np
import pytest
import torch

import oracle
import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu

OPTS = dict(gamma=3e5, eps_tv=1e-9, eps0=1e-6, eps_min=1e-7, step0=0.02, max_step=0.05, mask_sponge=False)


def _problem():
    return wri_synth.custom_problem((12, 11, 10), nb=3, n_src=3, n_rec=12, seed=43, freqs=(6.0, 9.0)).with_rtol(1e-6)


@pytest.mark.parametrize("memory", [2, 3])
def test_updates_are_the_recursion_on_the_stored_pairs(memory):
    """Models after 0 .. 5 updates (separate runs of the same deterministic loop), their
    gradients from the public calls that the loop makes; with memory 2 the ring wraps.
    Tolerance: m is stored in float32 (6e-8 of m) and an update is at least 1e-4 of m
    here, so a difference of two models holds it to 1e-3."""
    p = _problem()
    models, grads, n_acc = [], [], 0
    for k in range(6):
        b = wri.Batch(p, device="cuda:0")
        if k > 0:
            code, recs = wri.awri(b, max_outer=k, memory=memory, **OPTS)
            kinds = [r["kind"] for r in recs]
            if code != wri.OK or kinds != ["eval"] + ["accepted"] * k:
                break
            n_acc = k
        _, g, _ = wri.objective_grad(b)
        wri.tv(p.grids[0], b.m[0], OPTS["eps_tv"], OPTS["gamma"], g[0])
        models.append(b.m[0].cpu().numpy().astype(np.float64))
        grads.append(g[0].cpu().numpy().astype(np.float64))
    print(f"memory {memory}: {n_acc} updates in a row accepted", flush=True)
    assert n_acc >= 4   # the fourth update uses the pairs of slots 0 to 2 (memory 2: 1 and 0)
    pairs = []
    for k in range(n_acc):
        m, g, dm = models[k], grads[k], models[k + 1] - models[k]
        if pairs:
            s, y = pairs[-1]
            h0 = np.dot(s, y) / np.dot(y, y)
        else:
            h0 = OPTS["step0"] * np.abs(m).max() / np.abs(g).max()
        want = -oracle.lbfgs_two_loop(g, pairs[-memory:], h0)
        cap = OPTS["max_step"] * np.abs(m).max()
        want *= min(1.0, cap / np.abs(want).max())
        err = np.linalg.norm(dm - want) / np.linalg.norm(want)
        step = np.linalg.norm(dm) / np.linalg.norm(m)
        print(f"  update {k + 1}: {step:.2e} of m, rel difference {err:.2e}", flush=True)
        assert step > 1e-4 and err < 1e-3
        s, y = models[k + 1] - m, grads[k + 1] - g
        if np.dot(s, y) > 0.0:
            pairs.append((s, y))
