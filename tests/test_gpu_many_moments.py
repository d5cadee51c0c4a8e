"""GPU: more local moments than 32 bits count in lanes.

A partition's moments, blocks times (L + 1), are added up eight lanes each, so
2^28 of them are already 2^31 lanes.  Log-spaced points and frequencies with a
small min_size give that many blocks; a local rank of 2000 gives each 2001
moments.  Small counts around a workgroup's 32 moments, and the largest that
one pass over the moments takes, run the same kernel.

Bar: the method's own eps |c|_1 against the direct sum, at sampled rows of
sparse weights (every block's moments still enter the rows).
"""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("n,min_size,rank,least", [(3000, 0, 31, 0), (60000, 64, 200, 1 << 20), (200000, 4, 900, 1 << 25),
                                                   (500000, 4, 2000, 1 << 28)])
def test_moment_counts(nuht, n, min_size, rank, least):
    print("moments", n, min_size, rank, flush=True)
    rng = np.random.default_rng(n)
    half = 0.5 * np.log10(n)
    r, w = 10.0 ** rng.uniform(-half, half, n), 10.0 ** rng.uniform(-half, half, n)
    c = np.zeros(n)
    c[:: n // 211] = 1.0 + rng.uniform(size=c[:: n // 211].size)
    k = np.nonzero(c)[0]
    rows = rng.choice(n, 300, replace=False)
    p = nuht.Plan(dev(r), dev(w), 0, 1e-8, min_size=min_size, local_rank=rank)
    info = p.info()
    assert info["n_local"] * (info["L"] + 1) > least
    g = p.execute(dev(c)).cpu().numpy()[rows]
    p.close()
    err = np.max(np.abs(g - direct.dht(0, r[k], c[k], w[rows]))) / np.sum(np.abs(c))
    print("  blocks", info["n_local"], "L", info["L"], "err", err, flush=True)
    assert err <= 1e-8
