"""The one-launch RK4 step of a micromagnetic region at every compiled tile width
and precision, bit for bit against the stage kernels (a spot that "moves" at zero
speed takes them) and, in FP64, against the oracle.  Which width a mesh takes is
checked on the CPU (test_mm_tiles_cpu.py) from the lists here."""
import numpy as np
import pytest

import workloads as W
from paper_2502_02236_amd import asd as A
from paper_2502_02236_amd import bridge
from test_gpu_mm import SPOT, gpu, make_pair, random_m  # noqa: F401 (gpu: the module's fixture)

pytestmark = pytest.mark.gpu

FP64, FP32 = A.ASD_FP64, A.ASD_FP32
# (cells, periodic axes, precision, tile width; 0: the stage kernels): no width
# divides its mesh; the last planes that a precision takes and one more; a tall
# mesh of many rounds
CASES = [
    ((30, 21, 14), (0, 1, 0), FP64, 5), ((30, 21, 15), (1, 0, 1), FP64, 0),
    ((161, 71, 7), (1, 0, 1), FP64, 6), ((301, 59, 8), (0, 0, 0), FP64, 8),
    ((211, 97, 3), (0, 1, 1), FP64, 10), ((301, 203, 1), (1, 1, 0), FP64, 16),
    ((401, 203, 2), (0, 0, 1), FP64, 16), ((201, 61, 12), (0, 0, 0), FP64, 0),
    ((97, 61, 8), (0, 1, 1), FP32, 5), ((31, 21, 16), (1, 0, 0), FP32, 5),
    ((31, 21, 17), (0, 0, 1), FP32, 0), ((161, 71, 7), (0, 1, 0), FP32, 6),
    ((131, 71, 10), (1, 0, 1), FP32, 8), ((211, 97, 4), (0, 0, 0), FP32, 10),
    ((333, 287, 3), (0, 1, 0), FP32, 16), ((307, 299, 1), (1, 0, 1), FP32, 26),
    ((601, 301, 2), (0, 1, 0), FP32, 26), ((301, 151, 16), (0, 0, 0), FP32, 0),
]
# regions of a window (columns of each, rows, planes) stepped together
PAIRS = [((131, 97), 71, 4, FP64, 10), ((131, 97), 71, 4, FP32, 10), ((167, 75), 41, 7, FP64, 6),
         ((301, 307), 61, 2, FP64, 16), ((67, 65), 71, 9, FP32, 8), ((141, 139), 71, 8, FP64, 8),
         ((307, 301), 151, 1, FP32, 26)]


def ids(v):
    return str(v).replace(" ", "") if isinstance(v, tuple) else {FP64: "fp64", FP32: "fp32"}.get(v)


@pytest.mark.parametrize("n,per,prec,width", CASES, ids=ids)
def test_every_width_equals_the_stage_kernels(n, per, prec, width):
    h, steps = (1e-9, 1.1e-9, 2e-9), 3
    spot = dict(B=(0.1, 0.0, -0.8), x0=0.4e-9 * n[0], y0=0.6e-9 * n[1], **SPOT)
    m = random_m(n[0] * n[1] * n[2], 11)
    out = []
    for mode in (A.ASD_SPOT_LOCKED, A.ASD_SPOT_MOVING):
        g, o = make_pair(n, h, per, prec, dict(spot=mode, v=0.0, **spot), graph_steps=2)
        torch = g.torch
        g.set_m(m)
        if not per[0]:  # neighbours across the x faces, some of the cells empty
            for face in (0, 1):
                d = random_m(n[1] * n[2], 7 + face).T.copy()
                d[face::4] = 0.0
                vec = torch.as_tensor(d, device="cuda").contiguous()
                torch.cuda.synchronize()
                A._mm_check(A.lib().asd_mm_set_face(g.h, face, vec.data_ptr(), 3), g.h)
                g.stream.synchronize()
                r = np.sqrt((d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2])
                o.set_ghost(face, np.where(r[:, None] > 0, d / np.where(r > 0, r, 1.0)[:, None], 0.0))
        g.step(steps)
        out.append(g.get_m())
        g.close()
    np.testing.assert_array_equal(out[0], out[1])
    if prec == FP64:
        np.testing.assert_array_equal(out[0], o.rk4(m, 0, steps))


def window(columns, ny, nz, prec, spot):
    cell = (2, 1, 1)
    w = W.c2_granular_slab().scaled(nx=12, ny=ny, nz=nz, track_nx=20, bc=(2, 0, 0), spot_mode=0,
                                    grains=False, ku_spread=0.0, bits=None, steps_per_bit=0)
    h = bridge.make_handle(w, prec, kernel=A.ASD_KERNEL_AUTO)
    h.shift_window(cell[0] + 1)
    h.set_spins(W.initial_spins(len(h.labels()), 5))
    regions = []
    for k, nx in enumerate(columns):
        p = A.asd_mm_params()
        p.precision = prec
        p.nx, p.ny, p.nz = nx, ny, nz
        for d in range(3):
            p.h[d] = cell[d] * w.a
        p.Ms0, p.A0, p.K0 = w.mu_s / w.a ** 3, w.J[0] / (2 * w.a), w.ku / w.a ** 3
        p.lambda_, p.gamma, p.Tc, p.mu_s, p.dt = w.alpha, w.gamma, 710.0, w.mu_s, w.dt
        g = A.MMHandle(p, stream=h.stream)
        dr = A.asd_drive()
        dr.B[2], dr.T_amb, dr.spot_mode = -0.8, 300.0, spot
        dr.T_peak, dr.fwhm = 300.0, 5e-9  # no warmer than the rest
        g.set_drive(dr)
        g.set_m(W.random_spins(g.n, 20 + k))
        regions.append(g)
    return h, regions, cell


@pytest.mark.parametrize("columns,ny,nz,prec,width", PAIRS, ids=ids)
def test_paired_regions_equal_the_stage_kernels(columns, ny, nz, prec, width):
    out = []
    for spot in (A.ASD_SPOT_LOCKED, A.ASD_SPOT_MOVING):
        h, (L, R), cell = window(columns, ny, nz, prec, spot)
        A.multiscale_step(h, 0, L, R, cell, 3)
        out.append([h.get_spins(), L.get_m(), R.get_m()])
        for o in (L, R, h):
            o.close()
    for a, b in zip(*out, strict=True):
        np.testing.assert_array_equal(a, b)
