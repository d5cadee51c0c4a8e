"""Spreading on the matrix cores, in plans whose blocks do spread.

With dft_max given, every asymptotic block has a spread grid (at tight
tolerances the library's own choice applies most of them through Chebyshev
expansions, which spread nothing), so the matrix-core kernels take most items.
nuht_plan_spreading says how many: dense items at every channel count up to
32, medium ones up to 16, none at 36 channels, at an ES width of 17, in FP32
or with vector_spread.

Workload: n = 30000 points r ~ U[0, 1), m = 2000 frequencies omega ~ U[0, 2000)
(about a thousand points a block on grids of the smallest size, and one
top-level block of tens of points a cell), and the random transforms of
workloads.random_case.

Bars: matrix against vector spreading, 5e-15 of the largest output up to 16
channels (each cell adds about a thousand terms in another order; rounding
moves a sum by about 1e-16 of its terms), above, where the channels' terms
grow beyond the result before they cancel, a twentieth of the vector path's
own error; and the method's own eps |c|_1 against the direct sum.
"""
import ctypes

import numpy as np
import pytest
import torch

import workloads
from oracle import direct

CASES = [  # nu, eps, channels (2M padded)
    (0, 1e-6, 4), (0, 1e-9, 6), (0, 1e-12, 8), (6, 1e-12, 10), (10, 1e-12, 12), (16, 1e-12, 14), (20, 1e-12, 16),
    (30, 1e-12, 20), (40, 1e-12, 24), (50, 1e-12, 28), (60, 1e-12, 32), (0, 1e-13, 8), (1.5, 1e-12, 2),
    (2.5, 1e-10, 4),
]
VECTOR_ONLY = [(0, 1e-14, {}), (70, 1e-12, {}), (0, 1e-12, {"vector_spread": True}), (0, 1e-6, {"precision": 1})]


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


@pytest.fixture(scope="module")
def data():
    r, w, c = workloads.uniform(30000, 2000, 1.0, 2000.0, seed=120)
    return r, w, c, {}


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


def run(nuht, nu, eps, r, w, c, **kw):
    p = nuht.Plan(dev(r), dev(w), nu, eps, **kw)
    g = p.execute(dev(c)).cpu().numpy()
    info, counts = p.info(), p.spreading()
    p.close()
    assert sum(counts.values()) == info["spread_items"]
    assert counts["dense"] + counts["medium"] <= info["dense_items"]
    return g, info, counts


def test_null_arguments():
    import paper_2411_09583_amd as lib
    assert lib.load_library().nuht_plan_spreading(None, (ctypes.c_int32 * 4)()) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("nu,eps,nch", CASES)
def test_matrix_against_vector(nuht, data, nu, eps, nch):
    r, w, c, cache = data
    g, info, counts = run(nuht, nu, eps, r, w, c, dft_max=48)
    gv, _, counts_v = run(nuht, nu, eps, r, w, c, dft_max=48, vector_spread=True)
    print(nu, eps, "M", info["M"], "w", info["es_width"], counts, counts_v, flush=True)
    assert 2 * info["M"] == nch
    assert counts["dense"] > info["spread_items"] // 2 and counts["not_spread"] == 0
    assert counts["medium"] > 0 if nch <= 16 else counts["medium"] == 0
    assert counts_v["dense"] == counts_v["medium"] == 0 and counts_v["vector"] == info["spread_items"]
    if nu not in cache:
        cache[nu] = direct.dht(nu, r, c, w)
    ref, top = cache[nu], np.max(np.abs(cache[nu]))
    diff, err_v = np.max(np.abs(g - gv)) / top, np.max(np.abs(gv - ref)) / top
    print("  matrix vs vector", diff, "vector vs direct sum", err_v, "matrix", np.max(np.abs(g - ref)) / top, flush=True)
    assert diff <= (5e-15 if nch <= 16 else max(5e-15, err_v / 20))
    assert np.max(np.abs(g - ref)) <= eps * np.sum(np.abs(c))


@pytest.mark.gpu
@pytest.mark.parametrize("nu,eps,kw", VECTOR_ONLY)
def test_vector_units_alone(nuht, data, nu, eps, kw):
    r, w, c, cache = data
    g, info, counts = run(nuht, nu, eps, r, w, c, dft_max=48, **kw)
    print(nu, eps, kw, counts, flush=True)
    assert counts["vector"] == info["spread_items"] > 0
    if nu not in cache:
        cache[nu] = direct.dht(nu, r, c, w)
    assert np.max(np.abs(g - cache[nu])) <= eps * np.sum(np.abs(c))


@pytest.mark.gpu
def test_own_choice_spreads_little(nuht, data):
    r, w, c, _ = data
    _, info, counts = run(nuht, 0, 1e-12, r, w, c)
    print(counts, info["dense_items"], flush=True)
    assert counts["not_spread"] > info["spread_items"] // 2
    assert counts["dense"] + counts["medium"] < info["dense_items"]


@pytest.mark.gpu
@pytest.mark.parametrize("seed", range(40))
def test_random_case(nuht, seed):
    nu, eps, r, w, c, kind = workloads.random_case(seed)
    g, _, counts = run(nuht, nu, eps, r, w, c, dft_max=48)
    ref = direct.dht(nu, r, c, w)
    print(seed, kind, "nu", nu, "eps", eps, counts, flush=True)
    assert np.all(np.abs(g - ref) <= 2.0 * eps * np.sum(np.abs(c)))
    if counts["dense"] + counts["medium"] > 0:
        gv, _, _ = run(nuht, nu, eps, r, w, c, dft_max=48, vector_spread=True)
        assert np.max(np.abs(g - gv)) <= 5e-15 * max(np.max(np.abs(gv)), 1e-300)
