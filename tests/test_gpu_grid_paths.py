"""GPU: dft_max says how the asymptotic blocks are applied.

Positive: every block has a grid, summed directly up to that many cells and
transformed above; negative: every grid is transformed; 0: the library's own
choice (in FP64 at tight tolerances Chebyshev expansions for most blocks).  The
plan's statistics say which path ran: cells times rows of the direct sums
(at least the smallest grid, w + 2 cells, for every row of every block), FFT
blocks, grid cells.  Orders and tolerances over the channel counts, FP32
spreading too.

Bar: the method's own eps |c|_1 against the direct sum.

Tuning: dft_max is tuned in plans where it decides something, and a plan with
expansions keeps its 0, also when the cache holds another plan's value.
"""
import json

import numpy as np
import pytest
import torch

import workloads
from oracle import direct

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


@pytest.mark.parametrize("nu,eps", [(0, 1e-4), (0, 1e-6), (0, 1e-9), (0, 1e-12), (0, 1e-14), (1, 1e-12), (7, 1e-7),
                                    (12, 1e-12), (25, 1e-10), (45, 1e-12), (63, 1e-12), (0.5, 1e-12), (3.5, 1e-9)])
def test_dft_max_selects_the_path(nuht, nu, eps):
    r, w, c = workloads.uniform(2500, 2300, 1.0, 1200.0, seed=8)
    ref = direct.dht(nu, r, c, w)
    for fp32 in (False, True):
        if fp32 and eps < 1e-7:
            continue
        for dft_max in (100000, 48, 1, -1):
            p = nuht.Plan(dev(r), dev(w), nu, eps, dft_max=dft_max,
                         precision=nuht.NUHT_FP32_SPREAD if fp32 else nuht.NUHT_FP64)
            info = p.info()
            err = np.max(np.abs(p.execute(dev(c)).cpu().numpy() - ref)) / np.sum(np.abs(c))
            p.close()
            print(nu, eps, "fp32" if fp32 else "fp64", dft_max, "err", err, "blocks", info["n_asy"],
                  "by FFT", info["n_fft_blocks"], "row cells", info["dft_row_cells"], flush=True)
            assert err <= eps
            assert info["n_asy"] > 1
            if dft_max == 100000:
                assert info["n_fft_blocks"] == 0 and info["fft_points"] == 0
                assert info["dft_row_cells"] >= info["asy_row_members"] * (info["es_width"] + 2)
            elif dft_max == 48:
                assert 0 < info["n_fft_blocks"] < info["n_asy"]
                assert info["fft_row_members"] < info["asy_row_members"] and info["dft_row_cells"] > 0
            else:
                assert info["n_fft_blocks"] == info["n_asy"] and info["dft_row_cells"] == 0
                assert info["fft_row_members"] == info["asy_row_members"]


def test_tuning_keeps_the_path(nuht, tmp_path):
    r, w, c = workloads.uniform(12000, 9000, 1.0, 1e4, seed=16)
    path = str(tmp_path / "tune.json")

    def tuned(**kw):
        p = nuht.Plan(dev(r), dev(w), 3, 1e-12, tune_cache=path, **kw)
        best, info = p.tune(dev(c)), p.info()
        p.close()
        return best, info

    own, info_own = tuned()
    assert own["dft_max"] == 0
    (entry,) = json.load(open(path))["entries"]
    assert entry["dft_max"] == 0
    # an entry without a value for it leaves a caller's own
    kept, info = tuned(dft_max=48)
    assert kept["dft_max"] == 48 and kept["ms"] == entry["ms"]
    assert info["dft_row_cells"] > 10 * info_own["dft_row_cells"]   # expansions in place of small grids
    # and one with a value leaves the plan with expansions alone
    text = open(path).read().replace('"dft_max": 0', '"dft_max": 24')
    open(path, "w").write(text)
    again, info = tuned()
    assert again["dft_max"] == 0 and again["ms"] == entry["ms"]
    assert info["dft_row_cells"] == info_own["dft_row_cells"]
    kept, _ = tuned(dft_max=48)
    assert kept["dft_max"] == 24
    # timed: one of the candidates
    path = str(tmp_path / "other.json")
    best, _ = tuned(dft_max=48)
    assert best["dft_max"] in (24, 48, 96)
