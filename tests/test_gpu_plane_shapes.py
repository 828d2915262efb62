"""Every shape of the one-kernel y/z passes (the tables of csrc/plane.h), each
at a ragged grid inside it: that the dispatch sends the grid there (on the CPU
by its rule, on the GPU by the passes that ran) and that the field and its
transpose agree with the oracle.  Then batches of requests on grids with odd
ny, where the rows of the transposed spectrum are one longer than the grid's.

Tolerances (relative L2): those of a transform chain, eps (log2 Px Py Pz + a
few) times a small factor: 1e-12 in double and 2e-6 in single precision."""
import ctypes as C
import os
import re
import time

import numpy as np
import pytest
import torch  # its HIP runtime is the one that the library shares: loaded first

from conftest import ROOT
from gpu_util import banner, rel_l2, to_np
from paper_2302_08843_amd import mm, workloads as W

BAR = {"fp64": 1e-12, "fp32": 2e-6}


def _shapes():
    """(prec, YP, PZ, NQ) of every entry of MMX_PLANE_F32 and MMX_PLANE_F64."""
    with open(os.path.join(ROOT, "paper_2302_08843_amd", "csrc", "plane.h")) as f:
        text = f.read()
    out = []
    for prec, name in (("fp32", "MMX_PLANE_F32"), ("fp64", "MMX_PLANE_F64")):
        body = re.search(r"#define %s\(X\)((?:.*\\\n)*.*)" % name, text).group(1)
        for e in re.findall(r"X\(([^)]*)\)", body):
            yp, _, pz, _, nq, _ = (int(v) for v in e.split(","))
            out.append((prec, yp, pz, nq))
    return out


def _padded(n):
    p = 1
    while p < 2 * n - 1:
        p *= 2
    return p


def _is_plane(prec, grid):
    """The rule of plan set-up: plane_shape, and for one layer a spectrum that
    fits its place."""
    rule = mm.lib()["_ZN3mmx11plane_shapeEiPKiS1_"]
    rule.restype = C.c_bool
    P = [_padded(v) for v in grid]
    ok = rule(mm.MM_FP32 if prec == "fp32" else mm.MM_FP64, (C.c_int * 3)(*grid), (C.c_int * 3)(*P))
    align = 32 if prec == "fp32" else 16
    hxp = -(-(P[0] // 2 + 1) // align) * align
    return bool(ok) and (P[2] > 1 or P[0] // 2 * ((grid[1] + 1) & ~1) <= grid[1] * hxp)


def _grid(prec, yp, pz):
    """An odd ny and a ragged nz inside the shape, and the fewest cells along x
    of four sizes that the dispatch takes there (None: it takes none)."""
    ny, nz = (yp - yp // 4) | 1, 1 if pz == 1 else 2 if pz == 4 else pz // 2 - pz // 16 - 1
    assert _padded(ny) == 2 * yp and _padded(nz) == pz
    for nx in (3, 17, 33, 129):
        if _is_plane(prec, (nx, ny, nz)):
            return nx, ny, nz
    return None


SHAPES = _shapes()


def test_every_shape_is_reached():
    assert len(SHAPES) == len(set(SHAPES)) and {s[3] for s in SHAPES} == {1, 2}
    assert {s[0] for s in SHAPES} == {"fp32", "fp64"}
    for prec, yp, pz, nq in SHAPES:
        assert _grid(prec, yp, pz) is not None, (prec, yp, pz, nq)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,yp,pz,nq", SHAPES)
def test_shape_against_oracle(orc, prec, yp, pz, nq):
    grid = _grid(prec, yp, pz)
    banner("plane shape %s %d %d nq %d: %s" % (prec, yp, pz, nq, grid))
    nx, ny, nz = grid
    g = np.random.Generator(np.random.PCG64(yp + 1000 * pz))
    d = (3e-9, 2e-9, 4e-9)
    m, w = (g.standard_normal((3, nz, ny, nx)).astype(np.float32).astype(float) for _ in range(2))
    Ms = g.uniform(4e5, 1.2e6, (nz, ny, nx))
    Ms[g.random((nz, ny, nx)) < 0.1] = 0.0
    Ms = Ms.astype(np.float32).astype(float)
    o = orc.Oracle(grid, d, Ms=Ms, A=0.0)
    plan = mm.Plan(grid, d, Ms=1.0, prec=prec)
    plan.set_ms(Ms)
    plan.profile(True)
    h = to_np(plan.heff(m, None, mm.MM_DEMAG))
    ran = {k: v[1] for k, v in plan.profile_read().items()}
    plan.profile(False)
    assert [ran[k] for k in ("x_fwd", "y_fwd", "mid", "y_inv", "x_inv_local")] == [1, 0, 1, 0, 1]
    assert rel_l2(h, o.heff(m, terms=orc.DEMAG)) <= BAR[prec]
    gm, gms = plan.heff_vjp(m, w, mm.MM_DEMAG)
    ref, ref_ms = o.heff_vjp(m, w, terms=orc.DEMAG)
    assert rel_l2(to_np(gm), ref) <= BAR[prec]
    assert rel_l2(to_np(gms), ref_ms) <= BAR[prec]


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("grid", [(12, 9, 2), (20, 15, 2), (31, 33, 1), (66, 49, 7)])
def test_batch_with_odd_rows(grid, prec):
    """Three requests in shared launches and each on a plan of its own: the
    same arithmetic on other strides, so the same bits.  (The shapes that hold
    one half of the y transform at a time have more cells than a batch takes.)"""
    assert _is_plane(prec, grid)
    banner("batch %s %s" % (grid, prec))
    dt = torch.float32 if prec == "fp32" else torch.float64
    res = {}
    for batch in (1, 3):
        srv = mm.Server(max_active=2, steps_per_launch=4, prec=prec, batch=batch)
        ms = []
        for i in range(3):
            m = torch.tensor(W.smooth_random(grid, 4.0, seed=60 + i), dtype=dt, device="cuda")
            ms.append(m.contiguous())
            srv.submit(ms[i], grid, ((3.0 + 0.5 * i) * 1e-9,) * 3, 6e5 + 1e5 * i, 1e-11, 1e4 * i,
                       alpha=0.1 + 0.2 * i, h_ext=(2e4, 1e4 * i, -1e4), kind=mm.MM_SERVE_INTEGRATE,
                       rtol=1e-6, t_end=4e-12, tag=i)
        done, start = [], time.time()
        while len(done) < 3:
            done += srv.poll()
            assert time.time() - start < 60.0, "server did not finish"
        assert all(c["status"] == mm.MM_OK for c in done), done
        assert srv.stats()["max_batch"] == batch
        srv.close()
        res[batch] = [to_np(m) for m in ms]
    for one, three in zip(res[1], res[3]):
        assert np.isfinite(one).all() and np.array_equal(one, three)
