"""GPU: rank blocks (asymptotic blocks applied through Chebyshev expansions).

Wholly asymptotic matrices, r in [1, 1.2], omega in [w0, w0 + dw] with w0 three
times the crossover, make one asymptotic block whose product of half-ranges xi
= 0.1 dw / 2 decides its form: one expansion (xi of at most a few), several
panels (up to 40), beyond them the type-3 transform.  n runs over the edges of
the moment kernel's waves and items (64 columns a step, 256 columns for one
wave, 1024 an item, several items; 16 items for one wave's translation) and m
over single rows and wave edges.

Bar, per entry of g: the expansions are made for eps / 1000 in each variable,
a Lebesgue constant of about 3 multiplies one of them, and Hankel's terms at
omega r >= 3 z are off by at most eps 3^-(2M + 1/2) <= eps / 100 from M = 2 on;
with the floor that rounding leaves on n terms of magnitude at most |c| the
sum is within (0.02 eps + 2e-14) |c|_1.  The type-3 form of the same plan
(dft_max = -1) is held to its own eps / 10 on top.
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


def inputs(n, m, xi, nu, eps, seed):
    M, z, L = oparams.any_parameters(nu, eps)
    rng = np.random.default_rng(seed)
    r = np.concatenate([[1.0, 1.2], rng.uniform(1.0, 1.2, max(n - 2, 0))])[:n]
    w0, dw = 3.0 * z, xi / 0.05
    w = np.concatenate([[w0, w0 + dw], rng.uniform(w0, w0 + dw, max(m - 2, 0))])[:m]
    return rng.permutation(r), rng.permutation(w), rng.standard_normal(n), rng.standard_normal(m)


def check(nuht, n, m, xi, nu, eps, seed):
    r, w, c, y = inputs(n, m, xi, nu, eps, seed)
    p = nuht.Plan(dev(r), dev(w), nu, eps)
    info = p.info()
    g, cb = p.execute(dev(c)), p.adjoint(dev(y))
    q = nuht.Plan(dev(r), dev(w), nu, eps, dft_max=-1)
    h = q.execute(dev(c))
    torch.cuda.synchronize()
    assert info["n_local"] == 0 and info["n_direct"] == 0 and info["n_asy"] == 1
    bar = 0.02 * eps + 2e-14
    ref, refa = direct.dht(nu, r, c, w), direct.dht(nu, w, y, r)
    err = np.max(np.abs(g.cpu().numpy() - ref)) / np.sum(np.abs(c))
    erra = np.max(np.abs(cb.cpu().numpy() - refa)) / np.sum(np.abs(y))
    errh = np.max(np.abs(h.cpu().numpy() - ref)) / np.sum(np.abs(c))
    print("n", n, "m", m, "xi", xi, "nu", nu, "eps", eps, "err", err, "adjoint", erra, "type-3", errh, flush=True)
    p.close()
    q.close()
    assert err <= bar and erra <= bar
    assert errh <= bar + 0.1 * eps
    return info


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 16384, 16385])
def test_rank_sizes(nuht, n):
    for m, xi in ((1, 1.0), (2, 0.5), (64, 3.0), (65, 9.0)):
        info = check(nuht, n, m, xi, 0, 1e-12, 1000 + n + m)
        assert info["n_fft_blocks"] == 0 and info["grid_cells"] == 0


@pytest.mark.parametrize("xi", [0.0, 1e-9, 0.3, 1.0, 2.5, 4.0, 5.0, 12.0, 60.0, 130.0, 400.0])
def test_rank_widths(nuht, xi):
    for nu, eps in ((0, 1e-8), (1, 1e-10), (10, 1e-12), (0, 1e-14), (0.5, 1e-10), (3.5, 1e-9), (30, 1e-8)):
        info = check(nuht, 700, 300, xi, nu, eps, int(2000 + xi))
        if xi <= 12.0:      # ten panels or fewer at every tolerance
            assert info["n_fft_blocks"] == 0
        elif xi >= 400.0:   # over 40 panels at every tolerance
            assert info["n_fft_blocks"] == 1


@pytest.mark.parametrize("n", [5, 64, 255, 256])
def test_rank_few_points_many_panels(nuht, n):
    # items of one wave's columns over more panels than one wave takes, and
    # about as many as it takes
    for xi in (3.0, 12.0, 25.0, 130.0):
        check(nuht, n, 300, xi, 1.5, 1e-12, 3000 + n + int(xi))
        check(nuht, n, 300, xi, 2, 1e-10, 3500 + n + int(xi))
