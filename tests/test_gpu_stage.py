"""Stage inputs formed by the x forward pass (every row of both tableaus, the
last Dormand-Prince one with its error sum) on rows of odd and even length,
shorter and longer than a thread's share, with both spectrum layouts: three
adaptive steps against the oracle's.  In double the step path is the oracle's
(state to 1e-9, the bar of the same path elsewhere); in single precision the
state is compared at equal time at 1e-4."""
import numpy as np
import pytest

from gpu_util import banner, to_np

pytestmark = pytest.mark.gpu

# (grid): spectrum with y fastest (ny >= 5) and x fastest (ny 4)
GRIDS = [(2, 5, 2), (3, 6, 1), (8, 9, 2), (33, 7, 3), (130, 5, 2), (261, 5, 2), (5, 4, 3),
         (64, 4, 2), (129, 4, 1)]


@pytest.fixture(scope="module")
def mm():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2302_08843_amd import mm as _mm

    _mm.lib()
    return _mm


@pytest.mark.parametrize("method", ["dp45", "rkf45"])
@pytest.mark.parametrize("cells", [False, True])
@pytest.mark.parametrize("grid", GRIDS)
def test_three_steps(mm, orc, grid, cells, method):
    banner("stages %s cells %s %s" % (grid, cells, method))
    nx, ny, nz = grid
    g = np.random.Generator(np.random.PCG64(nx + 100 * ny + 10000 * nz + cells))
    m0 = g.standard_normal((3, nz, ny, nx))
    m0 = (m0 / np.linalg.norm(m0, axis=0)).astype(np.float32).astype(float)
    Ms = 8e5
    if cells:
        Ms = g.uniform(4e5, 1.2e6, (nz, ny, nx)).astype(np.float32).astype(float)
        Ms[0, 0, 0] = 0.0
        m0[:, Ms == 0.0] = 0.0
    d, H = (3e-9, 3e-9, 3e-9), np.array([1e4, -5e3, 2e4])
    o = orc.Oracle(grid, d, Ms=Ms, A=1.3e-11, Ku=2e4, alpha=0.3)
    o.set_field(H)
    step = o.dp45 if method == "dp45" else o.rkf45
    kind = mm.MM_DP45 if method == "dp45" else mm.MM_RKF45
    ref = step(m0, rtol=1e-6, max_steps=3)
    for prec in ("fp64", "fp32"):
        plan = mm.Plan(grid, d, Ms=1.0 if cells else Ms, A=1.3e-11, Ku=2e4, alpha=0.3, prec=prec)
        if cells:
            plan.set_ms(Ms)
        m = plan._v(m0).clone()
        _, t, _, st = plan.llg_step(m, H, mm.MM_ALL, rtol=1e-6, max_steps=3, method=kind)
        if prec == "fp64":
            want, bar = ref[0], 1e-9
            assert st["rejected"] == ref[3]["rejected"] and abs(t - ref[1]) <= 1e-9 * ref[1]
        else:
            want, bar = step(m0, rtol=1e-8, t_end=t)[0], 1e-4
        assert np.abs(to_np(m) - want).max() <= bar, prec
