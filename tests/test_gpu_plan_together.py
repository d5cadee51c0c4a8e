"""GPU: partitions planned together equal partitions planned one by one.

A plan's first full gradient builds its five partitions (orders nu - 1 and
nu + 1 forward and transposed, order nu transposed) in one set of launches; a
plan that has met them one at a time (adjoint, set_order, single derivatives)
built each on its own.  The planning kernels are the same, so the derivatives
must agree bit for bit.  Cases: uniform points; log-spaced ones with min_size
4, whose block tables outgrow their first guess, so that some partitions of
the set are planned again; and one frequency, where most blocks are empty.
"""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


def case(kind):
    if kind == "uniform":
        return workloads.uniform(5001, 3003, 1.0, 1500.0, seed=210), 2, {}
    if kind == "tables_grow":
        return workloads.exponential(20000, seed=211), 1, dict(min_size=4)
    return workloads.uniform(700, 1, 1.0, 900.0, seed=212), 3, {}


@pytest.mark.parametrize("kind", ["uniform", "tables_grow", "one_frequency"])
def test_gradient_partitions(nuht, kind):
    print("plan together", kind, flush=True)
    (r, w, c), nu, opts = case(kind)
    r, w, c = (torch.as_tensor(np.ascontiguousarray(a), device="cuda") for a in (r, w, c))
    y = torch.as_tensor(np.random.default_rng(213).standard_normal(w.numel()), device="cuda")
    together = nuht.Plan(r, w, nu, 1e-10, **opts)
    if kind == "tables_grow":
        i = together.info()
        guess = (r.numel() + w.numel()) // 32 + 4096      # blocks the tables first hold
        assert max(i["n_nodes"], i["n_local"], i["n_asy"]) > guess
    a = together.gradient(c, y)
    single = nuht.Plan(r, w, nu, 1e-10, **opts)
    single.adjoint(y)
    for order in (nu - 1, nu + 1):
        single.set_order(order)
        single.adjoint(y)
    single.set_order(nu)
    b = single.gradient(c, y)
    again = together.gradient(c, y)
    torch.cuda.synchronize()
    together.close()
    single.close()
    for u, v, x in zip(a, b, again):
        assert torch.equal(u, v) and torch.equal(u, x)
