"""The single-operator kernel by window tiles, the one-pass total variation and
the l-BFGS direction from inner products, at the edges of their tilings and
rules, against the oracle.

Tolerances: one float32 rounding of a float64 result is 6e-8 of the largest
value (operator: 1e-6); TV values are float64 sums of the same terms (1e-12),
the TV gradient one rounding (1e-6); the direction is one rounding of a float64
combination of float32 inputs (2e-7 of its norm; the two-loop recursion of the
longer memories rounds after every update, so a few times that)."""
import numpy as np
import pytest
import torch

import oracle
import wri_synth
from paper_2410_18429_amd import wri

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / max(np.linalg.norm(np.asarray(b)), 1e-300))


# small grids (one cell a thread); the largest of them and the first larger grids:
# planes of whole and ragged tiles (1024 cells), narrow rows, one row, the widest row of
# the tiled kernel (512) and wider, slabs of one to four planes at the end
@pytest.mark.parametrize("shape", [(1, 1, 1), (31, 33, 4), (32, 32, 5), (41, 25, 3), (300, 4, 9), (512, 3, 2),
                                   (513, 3, 2), (1, 1500, 1), (64, 64, 64), (64, 64, 65), (67, 61, 65), (512, 129, 4),
                                   (513, 128, 4), (1, 70001, 4), (300, 4, 222), (511, 523, 1)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_operator_tiles(shape, adjoint):
    print(f"operator {shape} adjoint={adjoint}", flush=True)
    g = wri_synth.Grid(*shape, 10.0, 2, 1500.0)
    rng = np.random.default_rng(5)
    m = (2.5e-7 * (1.0 + 0.2 * rng.random(g.n))).astype(np.float32)
    x = (rng.standard_normal(g.n) + 1j * rng.standard_normal(g.n)).astype(np.complex64)
    y = wri.apply_helmholtz(g, torch.as_tensor(m, device=DEV), 60.0, torch.as_tensor(x, device=DEV), adjoint)
    A = oracle.helmholtz(g, m.astype(np.float64).reshape(g.shape), 60.0)
    want = (A.conj().T if adjoint else A) @ x.astype(np.complex128)
    assert np.abs(y.cpu().numpy() - want).max() <= 1e-6 * np.abs(want).max()


# planes around one tile (1024 cells), rows up to the widest with rows in LDS
# (1024) and wider, slabs of 2 to 16 planes and a remainder
@pytest.mark.parametrize("shape", [(1, 1, 1), (33, 31, 4), (32, 32, 3), (1024, 3, 3), (1025, 3, 3), (2100, 2, 2),
                                   (64, 48, 37), (200, 130, 33)])
def test_tv_one_pass(shape):
    print(f"tv {shape}", flush=True)
    g = wri_synth.Grid(*shape, 10.0, 0, 1500.0)
    rng = np.random.default_rng(6)
    m = (3e-7 * (1.0 + 0.1 * rng.standard_normal(g.n))).astype(np.float32)
    grad = torch.full((g.n,), -0.5, dtype=torch.float32, device=DEV)
    mt = torch.as_tensor(m, device=DEV)
    v = wri.tv(g, mt, 1e-10, gamma=3.0, grad=grad)
    assert v == pytest.approx(oracle.tv(g, m.astype(np.float64), 1e-10), rel=1e-12)
    assert rel(grad.cpu().numpy(), -0.5 + 3.0 * oracle.tv_grad(g, m.astype(np.float64), 1e-10)) < 1e-6
    before = grad.clone()
    assert wri.tv(g, mt, 1e-10, gamma=0.0, grad=grad) == v and torch.equal(grad, before)


@pytest.mark.parametrize("n", [1, 255, 131073])
@pytest.mark.parametrize("count", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_lbfgs_from_inner_products(n, count):
    print(f"lbfgs n={n} count={count}", flush=True)
    rng = np.random.default_rng(100 * count + n % 7)
    cap, newest = count + 1, 0      # the ring wraps
    count = min(count, n)           # at most n independent pairs
    g = rng.standard_normal(n).astype(np.float32)
    S = rng.standard_normal((cap, n)).astype(np.float32)
    Y = (S * (1.0 + 4.0 * rng.random(n)).astype(np.float32)[None, :]).astype(np.float32)
    order = [((newest - (count - 1) + j) % cap) for j in range(count)]
    pairs = [(S[i].astype(np.float64), Y[i].astype(np.float64)) for i in order]
    for h0 in (0.0, 0.3):
        hh = h0 if h0 > 0.0 else float(np.dot(*pairs[-1]) / np.dot(pairs[-1][1], pairs[-1][1]))
        want = -oracle.lbfgs_two_loop(g.astype(np.float64), pairs, hh)
        d = wri.lbfgs_direction(torch.as_tensor(g, device=DEV), torch.as_tensor(S, device=DEV),
                                torch.as_tensor(Y, device=DEV), count, newest, h0)
        assert rel(d.cpu().numpy(), want) < (2e-7 if count <= 8 else 5e-6), h0
