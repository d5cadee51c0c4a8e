"""GPU: the times of the execution's stages are those of their own kernels.

An execution runs local moments, direct blocks and (beside grids) the blocks
applied through expansions on a second stream.  Two geometries where that shows
in the times: one wholly below the crossover, whose execution is almost all
local moments (millions of points, few frequencies), and one of many blocks
through expansions beside a grid.  Against the times with every stage profiled
(one stream):
* the rows timed alone do not contain the wait for the second stream: they
  stay far below the local moments' time, which such a wait would add;
* the spreading and the grid assembly timed alone contain the expansions'
  kernels.
The margins are factors of two where a wait or a missing kernel makes one of
five and more.
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


def stage_ms(p, c, stages=None, calls=12):
    for _ in range(3):
        p.execute(c)
    torch.cuda.synchronize()
    p.profile(True, stages=stages)
    for _ in range(calls):
        p.execute(c)
    ms, n = p.profile_read()
    p.profile(False)
    assert n == calls
    return {k: v / calls for k, v in ms.items()}


def uniform(n, m, top, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    f64 = dict(dtype=torch.float64, device="cuda", generator=g)
    return torch.rand(n, **f64), torch.rand(m, **f64) * top, torch.randn(n, **f64)


def test_rows_without_the_wait(nuht):
    r, w, c = uniform(8_000_000, 40, 9.0, 1)
    p = nuht.Plan(r, w, 0, 1e-12)
    assert p.info()["n_local"] == 1 and p.info()["n_asy"] == 0
    every, rows = stage_ms(p, c), stage_ms(p, c, ["rows_asymptotic"])
    p.close()
    print("all stages", every, "rows alone", rows["rows_asymptotic"], flush=True)
    assert every["local_moments"] > 5.0 * every["rows_asymptotic"]
    assert rows["rows_asymptotic"] < 0.5 * every["local_moments"]
    assert sum(v for k, v in rows.items() if k != "rows_asymptotic") == 0.0


def test_spreading_with_the_expansions(nuht):
    # log-spaced: hundreds of blocks through expansions, few points on grids
    n = 300_000
    g = torch.Generator(device="cuda").manual_seed(2)
    f64 = dict(dtype=torch.float64, device="cuda", generator=g)
    r, w = 10.0 ** (5.0 * torch.rand(n, **f64) - 2.5), 10.0 ** (3.0 * torch.rand(n, **f64) - 2.0)
    c = torch.randn(n, **f64)
    p = nuht.Plan(r, w, 0, 1e-10)
    how = p.spreading()
    assert p.info()["grid_cells"] > 0 and how["not_spread"] > 0
    every = stage_ms(p, c)
    alone = {s: stage_ms(p, c, [s])[s] for s in ("spread", "grid_assembly")}
    p.close()
    print("items", how, "all stages", every, "alone", alone, flush=True)
    for s, ms in alone.items():
        assert 0.5 * every[s] < ms < 2.0 * every[s], s
