"""Workspaces of the sizes that the queries gave before the window passes needed more:
accepted (the calls get past the workspace check, and fail without a device), refused
one byte short, and never more than the queries ask for."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2410_18429_amd import wri

FAKE = ctypes.c_void_p(0x3000)   # not dereferenced by the host
no_device = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up pointers: only where no launch can follow")

CASES = {   # name: grids, systems per grid, receivers
    "tiny": ([(10, 9, 8)], [1], 4),
    "ragged": ([(70, 37, 19)], [4], 19),
    "medium": ([(64, 64, 64)], [8], 64),
    "receivers": ([(64, 64, 64)], [8], 2000),
    "three": ([(48, 48, 48), (64, 64, 64), (96, 96, 96)], [8, 8, 8], 40),
    "none": ([(128, 128, 128)], [2], 0),
    "wide": ([(24, 20, 18), (600, 30, 20)], [30, 1], 9),
}


def _case(name):
    shapes, counts, n_rec = CASES[name]
    g = (wri.WriGrid * len(shapes))(*[wri.WriGrid(*s, 2, 10.0, 1500.0) for s in shapes])
    keep, sy = [], []
    for i, (s, c) in enumerate(zip(shapes, counts)):
        keep.append(np.arange(n_rec, dtype=np.int32) * ((s[0] * s[1] * s[2]) // max(n_rec, 1)))
        sy += [wri.WriSystem(i, 5, 30.0, 0.1, 1e-6, wri.WriC64(1.0, 0.0), n_rec, 0,
                             keep[-1].ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), FAKE) for _ in range(c)]
    return shapes, g, (wri.WriSystem * len(sy))(*sy), len(sy), keep


def _check(call, query, was):
    assert query >= was
    assert call(was - 1) == wri.ENOWS
    for size in (was, (was + query) // 2, query):
        assert call(size) == wri.EHIP, size


SOLVER = {"tiny": (45312, 58112, 51712), "ragged": (11054336, 14206976, 11448320),
          "medium": (117509376, 151071232, 119606784), "receivers": (117782784, 151533056, 119880192),
          "three": (563709184, 724687104, 573769216), "none": (235072512, 302182912, 251849984),
          "wide": (34949376, 44876288, 37898752)}


@no_device
@pytest.mark.parametrize("name", CASES)
def test_solver_fwi_and_model_grid(name):
    L = wri.lib()
    shapes, g, s, n, keep = _case(name)
    ng = len(shapes)
    ptr = (ctypes.c_void_p * ng)(*[0x2000] * ng)
    res = (wri.WriResult * n)()
    J = ctypes.c_double(0.0)
    _check(lambda b: L.wri_solve(g, ng, ptr, s, n, wri.ESTIMATE, 10, 0, None, res, FAKE, b, None),
           L.wri_workspace_bytes(g, ng, s, n, wri.ESTIMATE, 0), SOLVER[name][0])
    fres = (wri.WriFwiResult * n)()
    _check(lambda b: L.wri_fwi_objective_grad(g, ng, ptr, s, n, wri.ESTIMATE, 10, 0, J, None, None, fres, FAKE, b, None),
           L.wri_fwi_workspace_bytes(g, ng, s, n, wri.ESTIMATE, 0), SOLVER[name][1])
    model = wri.WriGrid(*[max(x[i] for x in shapes) for i in range(3)], 0, 10.0, 1500.0)
    _check(lambda b: L.wri_objective_grad_model(ctypes.byref(model), FAKE, g, ng, s, n, wri.ESTIMATE, 10, 0, J, None,
                                                None, res, FAKE, b, None),
           L.wri_model_workspace_bytes(ctypes.byref(model), g, ng, s, n, wri.ESTIMATE, 0), SOLVER[name][2])


AWRI = {"tiny": (138496, 137984), "ragged": (15217920, 17580288), "medium": (139558912, 168919040),
        "receivers": (139832320, 169192448), "none": (411262720, 444817152)}


@no_device
@pytest.mark.parametrize("name", AWRI)
def test_outer_loop(name):
    """Memory 5 cold and memory 3 warm started: no more than before for these."""
    L = wri.lib()
    _, g, s, n, keep = _case(name)
    for (memory, warm), was in zip(((5, 0), (3, 1)), AWRI[name]):
        o = wri.WriAwriOptions(0.0, 1e-9, 1e-2, 1e-6, 0.01, 0.0, 0.0, 0.0, 3, memory, 100, 0, 1, warm)
        rec = ctypes.c_int32(0)
        query = L.wri_awri_workspace_bytes(g, s, n, wri.ESTIMATE, wri.FLAG_WARM_START if warm else 0, memory)
        assert query == was
        _check(lambda b: L.wri_awri(g, FAKE, s, n, wri.ESTIMATE, ctypes.byref(o), None, 0, ctypes.byref(rec), FAKE, b, None),
               query, was)


@no_device
@pytest.mark.parametrize("capacity,was", [(1, 8704), (5, 8704), (8, 8704), (9, 8704), (40, 9216)])
def test_direction(capacity, was):
    L = wri.lib()
    _check(lambda b: L.wri_lbfgs_direction(100000, FAKE, FAKE, FAKE, capacity, capacity, 0, 0.0, FAKE, FAKE, b, None),
           L.wri_lbfgs_workspace_bytes(capacity), was)


OFFGRID = {"tiny": 46336, "ragged": 11058432, "medium": 117591808, "receivers": 120901376, "three": 563667200,
           "none": 234887168, "wide": 34871296}


@no_device
@pytest.mark.parametrize("name", OFFGRID)
def test_offgrid(name):
    L = wri.lib()
    shapes, g, s, n, keep = _case(name)
    n_rec = CASES[name][2]
    rng = np.random.default_rng(0)
    xyz = [rng.uniform(0, 80, (n_rec, 3)) for _ in shapes]
    pos = (wri.WriPositions * n)(*[wri.WriPositions(
        (ctypes.c_double * 3)(41.0, 33.0, 21.0),
        xyz[s[i].grid].ctypes.data_as(ctypes.POINTER(ctypes.c_double)) if n_rec else None) for i in range(n)])
    ptr = (ctypes.c_void_p * len(shapes))(*[0x2000] * len(shapes))
    res = (wri.WriResult * n)()
    J = ctypes.c_double(0.0)
    _check(lambda b: L.wri_objective_grad_offgrid(g, len(shapes), ptr, s, n, pos, wri.ESTIMATE, 10, 0, J, None, None, res,
                                                  FAKE, b, None),
           L.wri_offgrid_workspace_bytes(g, len(shapes), s, n, pos), OFFGRID[name])


PRECOND = {"tiny": 74752, "ragged": 15900416, "medium": 165393152, "receivers": 165706496, "three": 793365248,
           "none": 359514368, "wide": 54234624}


@no_device
@pytest.mark.parametrize("name", PRECOND)
def test_precond(name):
    """The query is the former size: the tiled passes share what they need more."""
    L = wri.lib()
    shapes, g, s, n, keep = _case(name)
    ptr = (ctypes.c_void_p * len(shapes))(*[0x2000] * len(shapes))
    res = (wri.WriResult * n)()
    J = ctypes.c_double(0.0)
    query = L.wri_precond_workspace_bytes(g, len(shapes), s, n, wri.ESTIMATE)
    assert query == PRECOND[name]
    _check(lambda b: L.wri_objective_grad_precond(g, len(shapes), ptr, s, n, wri.ESTIMATE, 10, 0, J, None, None, res, FAKE,
                                                  b, None), query, query)
