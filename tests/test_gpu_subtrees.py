"""GPU: the subdivision with its subtrees side by side (large transforms).

Bar: the blocks are the oracle's (Alg. 1 over the same staircase): the same
counts of local, asymptotic and direct blocks, the same levels, rows, columns
and entries.  Sizes around the one from which subtrees are apart, the sizes of
one side far from the other's, inputs whose subtrees are uneven (one of them
outgrows its share of the tables, and the subdivision is done again by one
workgroup), a single local or asymptotic block (no subtrees at all), and every
row a candidate of the splits.
"""
import numpy as np
import pytest
import torch

from oracle import direct
from oracle import params as oparams
from oracle import partition

pytestmark = pytest.mark.gpu

APART = 1 << 19


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


def check(nuht, r, w, nu, eps, min_size, ncand=0):
    r, w = np.sort(r), np.sort(w)
    z = oparams.any_parameters(nu, eps)[1]
    K = direct.staircase(r, w, z)
    blocks = partition.subdivide(K, w.size, r.size, min_size, ncand if ncand else 16)
    p = nuht.Plan(dev(r), dev(w), nu, eps, min_size=min_size, split_candidates=ncand)
    info = p.info()
    for kind, name in (("L", "n_local"), ("A", "n_asy"), ("D", "n_direct")):
        assert info[name] == sum(b.kind == kind for b in blocks), (name, r.size, w.size)
    assert info["direct_entries"] == sum(b.rows * b.cols for b in blocks if b.kind == "D")
    c = np.zeros(r.size)
    c[:: max(1, r.size // 97)] = 1.0
    k = np.nonzero(c)[0]
    rows = np.unique(np.linspace(0, w.size - 1, 300).astype(int))
    g = p.execute(dev(c)).cpu().numpy()[rows]
    p.close()
    ref = direct.dht(nu, r[k], c[k], w[rows])
    err = np.max(np.abs(g - ref)) / np.sum(np.abs(c))
    print(r.size, w.size, "err", err, flush=True)
    assert err <= eps


@pytest.mark.parametrize("n,m", [(APART // 2, APART // 2), (APART // 2 + 1, APART // 2), (APART + 3, 2000), (900, APART),
                                 (300000, 400000)])
@pytest.mark.parametrize("kind", ["uniform", "decades"])
def test_subtrees(nuht, n, m, kind):
    rng = np.random.default_rng(n + m)
    if kind == "uniform":
        r, w = rng.uniform(0.0, 1.0, n), rng.uniform(0.0, 0.2 * m, m)
    else:
        r, w = 10.0 ** rng.uniform(-3.0, 3.0, n), 10.0 ** rng.uniform(-3.0, 2.0, m)
    check(nuht, r, w, 2, 1e-9, 1024)


def test_uneven_subtrees(nuht):
    # all products but a few near the crossover: small blocks crowd one place
    rng = np.random.default_rng(5)
    n = m = 300000
    z = oparams.any_parameters(0, 1e-9)[1]
    r = np.concatenate([rng.uniform(0.0, 100.0, 2000), 1.0 + 1e-3 * rng.uniform(-1.0, 1.0, n - 2000)])
    w = np.concatenate([rng.uniform(0.0, 100.0 * z, 2000), z * (1.0 + 1e-3 * rng.uniform(-1.0, 1.0, m - 2000))])
    check(nuht, r, w, 0, 1e-9, 64)


def test_no_subtrees(nuht):
    rng = np.random.default_rng(6)
    n = APART
    check(nuht, rng.uniform(0.0, 1.0, n), rng.uniform(0.0, 1.0, 1000), 0, 1e-9, 1024)
    check(nuht, rng.uniform(1.0, 1.01, n), rng.uniform(500.0, 510.0, 1000), 0, 1e-9, 1024)


def test_every_row_a_candidate(nuht):
    rng = np.random.default_rng(7)
    check(nuht, rng.uniform(0.0, 1.0, APART), rng.uniform(0.0, 900.0, 3000), 1, 1e-9, 512, ncand=64)
