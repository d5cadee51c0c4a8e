"""GPU: every way an execution uses its side stream gives the one-stream result.

Sizes just below and above the counts of points and frequencies from which an
execution forks (2^11 at half-integer orders, 2^13 at the others), from which
its rank blocks go aside beside grids (2^14), and from which rows do not wait
for the direct blocks (1024 rows and fewer from 2^14 or 2^17 on; any sizes with
long direct blocks: half-integer and high orders).  Plans with grids and
without, FP32 spreading included.

Bar: bit for bit.  Each kernel adds in a fixed order, and a row's direct part is
the last term of its sum wherever it is added.  Several executions in a row
with other weights, on the plan's streams alone, must not disturb each other,
nor the transposed transforms on the same plan, nor a second plan on another
stream.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


def inputs(n, m, top, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    f64 = dict(dtype=torch.float64, device="cuda", generator=g)
    return torch.rand(n, **f64), torch.rand(m, **f64) * top, torch.randn(n, **f64), torch.randn(m, **f64)


def both_ways(p, c, y):
    return [p.execute(c), p.adjoint(y)]


FORMS = [  # nu, eps, n, m, largest omega, options
    (1.5, 1e-12, 1500, 547, 400.0, {}), (1.5, 1e-12, 1500, 549, 400.0, {}),
    (0.5, 1e-10, 2000, 300, 2000.0, {}),
    (0, 1e-12, 8000, 192, 2000.0, {}), (0, 1e-12, 8000, 193, 2000.0, {}), (2, 1e-6, 5000, 3193, 900.0, {}),
    (0, 1e-10, 10000, 6384, 9000.0, {}), (0, 1e-10, 10000, 6385, 9000.0, {}),
    (3, 1e-5, 15900, 484, 100.0, {}), (3, 1e-5, 15900, 485, 100.0, {}), (3, 1e-5, 15900, 485, 100.0, {"precision": 1}),
    (0, 1e-6, 20000, 1024, 90.0, {}), (0, 1e-6, 20000, 1025, 90.0, {}), (0, 1e-6, 300, 30000, 5000.0, {}),
    (0, 1e-12, 131000, 72, 100.0, {}), (0, 1e-12, 131000, 73, 100.0, {}), (1, 1e-9, 140000, 1024, 100.0, {}),
    (1.5, 1e-12, 30000, 500, 100.0, {}), (2.5, 1e-8, 30000, 30000, 7500.0, {}), (5.5, 1e-12, 20000, 9000, 20000.0, {}),
    (40, 1e-12, 30000, 500, 7500.0, {}), (63, 1e-10, 5000, 20000, 8000.0, {}), (2.5, 1e-9, 30000, 3000, 7500.0, {"dft_max": 48}),
]


@pytest.mark.parametrize("nu,eps,n,m,top,opts", FORMS)
def test_forked_equals_serial(nuht, nu, eps, n, m, top, opts):
    print("fork form", nu, eps, n, m, top, opts, flush=True)
    r, w, c, y = inputs(n, m, top, n + m)
    p = nuht.Plan(r, w, nu, eps, **opts)
    q = nuht.Plan(r, w, 2, 1e-7)
    both_ways(p, c, y)
    ref_q = both_ways(q, c, y)
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    outs, beside = [], []
    for k in range(5):
        outs.append(both_ways(p, c * (1.0 + k), y * (2.0 - k)))
        with torch.cuda.stream(other):
            beside.append(both_ways(q, c, y))
    torch.cuda.synchronize()
    p.profile(True, stages=["local_moments"])                 # keeps an execution on one stream
    serial = [both_ways(p, c * (1.0 + k), y * (2.0 - k)) for k in range(5)]
    torch.cuda.synchronize()
    p.profile(False)
    p.profile(True, stages=["rows_asymptotic", "rows_local"])  # timed, but forked
    timed = both_ways(p, c, y)
    p.profile(False)
    torch.cuda.synchronize()
    for a, b in zip(outs, serial):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    for a in beside:
        assert torch.equal(a[0], ref_q[0]) and torch.equal(a[1], ref_q[1])
    assert torch.equal(timed[0], serial[0][0])
    p.close()
    q.close()


@pytest.mark.parametrize("nu,n,m,top", [(2.5, 30000, 500, 7500.0), (40, 9000, 900, 9000.0), (1, 140000, 900, 100.0)])
def test_gradient_forms(nuht, nu, n, m, top):
    print("gradient form", nu, n, m, flush=True)
    r, w, c, y = inputs(n, m, top, 77)
    p = nuht.Plan(r, w, nu, 1e-10)
    p.gradient(c, y)
    a = p.gradient(c, y)
    p.profile(True, stages=["local_moments"])
    b = p.gradient(c, y)
    torch.cuda.synchronize()
    p.close()
    for u, v in zip(a, b):
        assert torch.equal(u, v)
