"""GPU: items of the column-side kernels at their edges.

Sparse spreading: few points over many grid cells, so that an item's cells
take several turns of the workgroup and every turn reaches only some of the
item's sub-chunks of 256 points; evenly spread points, and clusters with wide
gaps (turns that no point reaches).  Item sizes below, at and above a
sub-chunk.  Local moments: point counts around the item sizes and around the
counts at which the item size changes, with as many items as blocks allow.

Bar: the method's own eps |c|_1 against the direct sum.
"""
import numpy as np
import pytest
import torch

from oracle import direct
from oracle import params as oparams

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


@pytest.mark.parametrize("n", [65, 256, 257, 700, 1500])
@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("precision", ["NUHT_FP64", "NUHT_FP32_SPREAD"])
def test_sparse_spreading(nuht, n, clustered, precision):
    rng = np.random.default_rng(n + clustered)
    r = rng.uniform(0.05, 1.0, n)
    if clustered:
        r = rng.choice([0.1, 0.35, 0.36, 0.8, 1.0], n) + 1e-3 * rng.uniform(-1.0, 1.0, n)
    m = 400
    w = rng.uniform(0.0, 6.0 * n + 3000.0, m)
    c = rng.standard_normal(n)
    for nu, eps in ((0, 1e-12), (4, 1e-9), (1.5, 1e-7)):
        if precision != "NUHT_FP64":
            eps = 1e-5
        ref = direct.dht(nu, r, c, w)
        for chunk in (0, 64, 300, 4096):
            p = nuht.Plan(dev(r), dev(w), nu, eps, precision=getattr(nuht, precision),
                         dft_max=-1, min_size=16, spread_chunk=chunk)
            assert p.info()["grid_cells"] > n
            err = np.max(np.abs(p.execute(dev(c)).cpu().numpy() - ref)) / np.sum(np.abs(c))
            print(n, clustered, precision, nu, eps, chunk, "err", err, flush=True)
            assert err <= eps
            p.close()


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1 << 17, (1 << 17) + 1, (1 << 19) + 700])
def test_local_items(nuht, n):
    for nu in (0, 33, 2.5):
        eps = 1e-12
        z = oparams.any_parameters(nu, eps)[1]
        rng = np.random.default_rng(n)
        r = rng.uniform(0.0, 1.0, n)
        w = rng.uniform(0.0, 0.999 * z, 30)
        c = rng.standard_normal(n)
        p = nuht.Plan(dev(r), dev(w), nu, eps)
        assert p.info()["n_local"] == 1
        err = np.max(np.abs(p.execute(dev(c)).cpu().numpy() - direct.dht(nu, r, c, w))) / np.sum(np.abs(c))
        print(n, nu, "err", err, flush=True)
        assert err <= eps
        p.close()
