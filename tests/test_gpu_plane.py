"""The one-kernel y/z passes (csrc/plane.h) against the oracle at the edges of
their shapes: the smallest grids, extents just below and above the powers of
two, one and many lanes per z pencil, both halves of the y transform at once
and one after the other, and the narrowest and widest x extents, each next to
a grid that the three separate passes take.

Tolerances (relative L2): a transform of length L carries a relative rounding
error of about eps log2 L, so the field one of eps (log2 Px Py Pz + a few)
times a small factor: below 1e-12 in double and 2e-6 in single precision."""
import numpy as np
import pytest

from gpu_util import banner, rel_l2, to_np

pytestmark = pytest.mark.gpu

BAR = {"fp64": 1e-12, "fp32": 2e-6}
# smallest; LZ 1, 2, 4, 8; ny at YP and YP/2 + 1; packed columns with nx = 2;
# NQ = 1 shapes; single layers (256, 5, 1: too large for the spectrum's place);
# just outside (ny 4, nz 33, one cell along x, Px too small for a large plane)
GRIDS = [(2, 5, 2), (3, 8, 2), (2, 9, 4), (5, 16, 3), (9, 17, 8), (33, 31, 5), (17, 24, 9),
         (12, 32, 16), (6, 33, 17), (10, 12, 31), (64, 65, 2), (40, 100, 7), (130, 129, 3),
         (32, 257, 2), (35, 300, 4), (257, 130, 9), (300, 260, 2), (512, 9, 2),
         (2, 5, 1), (31, 64, 1), (65, 33, 1), (130, 257, 1), (300, 20, 1), (1, 9, 3), (256, 5, 1),
         (8, 4, 3), (12, 20, 33), (8, 300, 7)]


@pytest.fixture(scope="module")
def mm():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2302_08843_amd import mm as _mm

    _mm.lib()
    return _mm


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", GRIDS)
def test_field_and_transpose(mm, orc, grid, prec):
    banner("plane %s %s" % (grid, prec))
    nx, ny, nz = grid
    g = np.random.Generator(np.random.PCG64(nx + 1000 * ny + 7 * nz))
    d = (3e-9, 2e-9, 4e-9)
    m = g.standard_normal((3, nz, ny, nx))
    w = g.standard_normal((3, nz, ny, nx))
    if prec == "fp32":  # the oracle sees the values the plan sees
        m, w = m.astype(np.float32).astype(float), w.astype(np.float32).astype(float)
    Ms = g.uniform(4e5, 1.2e6, (nz, ny, nx))
    Ms[g.random((nz, ny, nx)) < 0.1] = 0.0
    Ms = Ms.astype(np.float32).astype(float)
    o = orc.Oracle(grid, d, Ms=Ms, A=0.0)
    plan = mm.Plan(grid, d, Ms=1.0, prec=prec)
    plan.set_ms(Ms)
    h = to_np(plan.heff(m, None, mm.MM_DEMAG))
    assert rel_l2(h, o.heff(m, terms=orc.DEMAG)) <= BAR[prec]
    gm, gms = plan.heff_vjp(m, w, mm.MM_DEMAG)
    ref, ref_ms = o.heff_vjp(m, w, terms=orc.DEMAG)
    assert rel_l2(to_np(gm), ref) <= BAR[prec]
    assert rel_l2(to_np(gms), ref_ms) <= BAR[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", [(7, 12, 65), (3, 9, 70), (20, 33, 130), (33, 12, 34),
                                  (120, 6, 65), (260, 5, 66)])
def test_narrow_rows_through_three_passes(mm, orc, grid, prec):
    """The z pass over the columns of the spectrum alone (few cells along x) and
    over whole lines; a batchless field twice, so that columns between them
    that the first one left behind cannot enter."""
    banner("columns %s %s" % (grid, prec))
    nx, ny, nz = grid
    g = np.random.Generator(np.random.PCG64(nx + 31 * ny + nz))
    m = g.standard_normal((2, 3, nz, ny, nx)).astype(np.float32).astype(float)
    d = (3e-9, 2e-9, 4e-9)
    o = orc.Oracle(grid, d, Ms=8e5, A=0.0)
    plan = mm.Plan(grid, d, Ms=8e5, prec=prec)
    for v in m:
        h = to_np(plan.heff(v, None, mm.MM_DEMAG))
        assert rel_l2(h, o.heff(v, terms=orc.DEMAG)) <= BAR[prec]
