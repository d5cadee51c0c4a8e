"""GPU: the planning tables follow the blocks.

Crowded points and frequencies near the crossover give a geometry's subtrees
more blocks than an even share of the first tables, or more than the tables.
Three plans of one geometry with falling min_size, alive at once in a process
of their own (memory of released plans is reused, and would hide the sizes):
where the first tables hold every block, the plan's memory grows with its
blocks alone, so the third lies on the line through the first two (10% for what
does not follow the number of blocks; tables of twice the size add 18%).

Overflows of every kind give the oracle's blocks: one subtree beyond its share,
all of them, tables that have to grow once and several times over, at sizes
where the subtrees go side by side and below.
"""
import json
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import direct
from oracle import params as oparams
from oracle import partition

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


def crowded(n, far, seed):
    rng = np.random.default_rng(seed)
    z = oparams.any_parameters(0, 1e-9)[1]
    r = np.concatenate([rng.uniform(0.0, 100.0, far), 1.0 + 1e-3 * rng.uniform(-1.0, 1.0, n - far)])
    w = np.concatenate([rng.uniform(0.0, 100.0 * z, far), z * (1.0 + 1e-3 * rng.uniform(-1.0, 1.0, n - far))])
    return np.sort(r), np.sort(w), z


MEASURE = """
import json, sys
import numpy as np, torch
import paper_2411_09583_amd as nuht
sys.path.insert(0, "tests")
from test_gpu_plan_tables import crowded
r, w, _ = crowded(300000, 2000, 5)
r, w = (torch.as_tensor(x, device="cuda") for x in (r, w))
plans = [nuht.Plan(r, w, 0, 1e-9, min_size=s) for s in (32768, 4096, 1024)]
print(json.dumps([(p.info()["n_nodes"], p.info()["workspace_bytes"]) for p in plans]))
"""


def test_memory_follows_the_blocks():
    out = subprocess.run([sys.executable, "-c", MEASURE], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr[-2000:]
    (n0, b0), (n1, b1), (n2, b2) = json.loads(out.stdout.strip().split("\n")[-1])
    print(n0, b0, n1, b1, n2, b2, flush=True)
    assert n0 < n1 < n2 < 600000 // 32 + 4096
    line = b1 + (b1 - b0) * (n2 - n1) / (n1 - n0)
    assert b2 <= 1.1 * line


@pytest.mark.parametrize("n,far,min_size", [(300000, 2000, 1024), (300000, 2000, 256), (300000, 2000, 4), (300000, 299000, 16),
                                            (270000, 150000, 64), (100000, 2000, 4)])
def test_blocks_after_overflows(nuht, n, far, min_size):
    print("tables", n, far, min_size, flush=True)
    r, w, z = crowded(n, far, n + far)
    blocks = partition.subdivide(direct.staircase(r, w, z), n, n, min_size)
    p = nuht.Plan(dev(r), dev(w), 0, 1e-9, min_size=min_size)
    info = p.info()
    for kind, name in (("L", "n_local"), ("A", "n_asy"), ("D", "n_direct")):
        assert info[name] == sum(b.kind == kind for b in blocks), name
    c = np.zeros(n)
    c[:: n // 97] = 1.0
    k = np.nonzero(c)[0]
    rows = np.unique(np.linspace(0, n - 1, 300).astype(int))
    g = p.execute(dev(c)).cpu().numpy()[rows]
    p.close()
    err = np.max(np.abs(g - direct.dht(0, r[k], c[k], w[rows]))) / np.sum(np.abs(c))
    print("  nodes", info["n_nodes"], "first tables", 2 * n // 32 + 4096, "err", err, flush=True)
    assert err <= 1e-9
