"""GPU: the plan's sort where workgroups place keys by bins (nuht_plan_order).

Bar: bit-exact, as for every path of the sort: the sorted values are numpy's
and the permutations numpy's stable argsort.  Inputs that bins take (evenly
spread, over decades, with gaps), that they leave to the radix sorts (clusters,
repeats), and around the limit between the two (a bin of 96 keys), at sizes
around a workgroup's capacity and the limits of the sort's paths.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


def inputs(n, kind, rng):
    if kind == "uniform":
        return rng.uniform(0.0, 1.0, n)
    if kind == "decades":
        return 10.0 ** rng.uniform(-300.0, 300.0, n)
    if kind == "ends":
        return 0.5 * (1.0 - np.cos(np.pi * rng.uniform(0.0, 1.0, n)))
    if kind == "subnormal":
        return 5e-324 * rng.integers(0, 2 * n, n)
    if kind == "largest":
        return 1.7976931348623157e308 * rng.uniform(0.0, 1.0, n)
    if kind == "clusters":
        return np.concatenate([[0.0, 1e6], 3.0 + 1e-9 * rng.uniform(0.0, 1.0, n)])[-n:]
    if kind == "repeats":
        return rng.integers(0, max(1, n // 40), n).astype(float)
    if kind == "equal":
        return np.full(n, 2.5)
    k = int(kind[4:])                  # "fullK": K keys within one bin, the others evenly spread
    x = np.arange(n) / n
    x[:min(k, n)] = 0.5 + 1e-9 * rng.permutation(min(k, n)) / n
    return rng.permutation(x)


KINDS = ["uniform", "decades", "ends", "subnormal", "largest", "clusters", "repeats", "equal", "full94", "full95",
         "full96", "full97", "full300"]


def check(nuht, r, w):
    p = nuht.Plan(dev(r), dev(w), 0, 1e-8)
    rs, pr, ws, pw = (t.cpu().numpy() for t in p.order())
    p.close()
    for x, xs, perm in ((r, rs, pr), (w, ws, pw)):
        order = np.argsort(x, kind="stable")
        assert np.array_equal(perm, order)
        assert np.array_equal(xs, x[order])


@pytest.mark.parametrize("kind", KINDS)
def test_orders(nuht, kind):
    rng = np.random.default_rng(KINDS.index(kind))
    for n, m in ((1, 2), (96, 97), (255, 1025), (2048, 4095), (4096, 4096), (4097, 3000), (65536, 70000), (300001, 5)):
        print(kind, n, m, flush=True)
        # zeros on the other side: every product is 0, so any values plan
        check(nuht, inputs(n, kind, rng), np.zeros(m))
        check(nuht, np.zeros(n), inputs(m, kind, rng))


@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1])
def test_largest_splitter_sort(nuht, n):
    rng = np.random.default_rng(n)
    print(n, flush=True)
    check(nuht, rng.uniform(0.0, 1.0, n), 10.0 ** rng.uniform(-3.0, 2.0, n - 5))
