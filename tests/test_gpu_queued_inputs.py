"""GPU: a plan reads its points and frequencies after the work that is queued
on the caller's stream, the default stream included.

Each case queues some tens of milliseconds of matrix products, then writes
the inputs (valid other values until then) and plans at once, with nothing
waiting in between.  Sizes take every sort path; the one-shot call, the
autograd function and the batch plan the same way.

Bar: the outputs equal, bit for bit, those of the same call on finished copies
of the same inputs, and the default stream behaves as a stream of its own does.
"""
import contextlib

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nuht():
    import paper_2411_09583_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.load_library()
    return lib


@pytest.fixture(scope="module")
def busy():
    x = torch.eye(4096, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)

    def queue():
        for _ in range(12):
            torch.matmul(x, x, out=y)
    queue()
    torch.cuda.synchronize()
    return queue


def inputs(n, m, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    f64 = dict(dtype=torch.float64, device="cuda")
    r = torch.rand(n, generator=g, **f64)
    w = torch.rand(m, generator=g, **f64) * max(100.0, 0.2 * n)
    c = torch.randn(n, generator=g, **f64)
    torch.cuda.synchronize()
    return r, w, c


def on(stream):
    return torch.cuda.stream(stream) if stream is not None else contextlib.nullcontext()


CALLS = ["plan", "oneshot", "autograd", "batch"]


def call(nuht, kind, r, w, c):
    if kind == "plan":
        p = nuht.Plan(r, w, 1, 1e-10)
        return [p.execute(c), p]
    if kind == "oneshot":
        return [nuht.nuht(c, r, w, 1, 1e-10)]
    if kind == "autograd":
        r, w, c = (x.detach().requires_grad_(True) for x in (r, w, c))
        g = nuht.NuhtFunction.apply(c, r, w, 1, 1e-10)
        return [g.detach()] + list(torch.autograd.grad(g.square().sum(), (c, r, w)))
    b = nuht.Batch([r, r], [w, w], [0, 3], 1e-10)
    return b.execute([c, c]) + [b]


@pytest.mark.parametrize("kind", CALLS)
@pytest.mark.parametrize("n,m", [(300, 400), (3000, 9000), (70000, 30000), (600000, 500000)])
@pytest.mark.parametrize("own_stream", [False, True])
def test_inputs_still_queued(nuht, busy, kind, n, m, own_stream):
    print(kind, n, m, own_stream, flush=True)
    r, w, c = inputs(n, m, n + m)
    old = [torch.linspace(0.0, 1.0, n, dtype=torch.float64, device="cuda"),
           torch.linspace(0.0, 50.0, m, dtype=torch.float64, device="cuda"), torch.ones_like(c)]
    stream = torch.cuda.Stream() if own_stream else None
    torch.cuda.synchronize()
    with on(stream):
        busy()
        for a, b in zip(old, (r, w, c)):
            a.copy_(b)
        out = call(nuht, kind, *old)
        torch.cuda.synchronize()
        ref = call(nuht, kind, r, w, c)
        torch.cuda.synchronize()
    for a, b in zip(out, ref):
        if isinstance(a, torch.Tensor):
            assert torch.equal(a, b)
        else:
            a.close()
            b.close()
