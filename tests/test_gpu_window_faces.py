"""Coupled steps of the multiscale window (all face work of both sides in one
launch) against the same sequence through the single calls."""
import numpy as np
import pytest

import workloads as W
from paper_2502_02236_amd import asd as A
from paper_2502_02236_amd import bridge

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    A.lib()
    return torch


def window(base, n, cell, prec):
    nx, ny, nz = n
    w = base.scaled(nx=nx, ny=ny, nz=nz, track_nx=nx + 2 * cell[0] + 3, bc=(2, 0, 0), spot_mode=0,
                    grains=True, grain_pitch=3.0e-9, ku_spread=0.0, bits=None, steps_per_bit=0)
    h = bridge.make_handle(w, prec, kernel=A.ASD_KERNEL_AUTO)
    h.shift_window(cell[0] + 1)
    lab = h.labels()
    S = W.initial_spins(len(lab), 5)
    S[:, lab < 0] = 0
    h.set_spins(S)
    edge = (cell[0] * w.a, cell[1] * w.a, cell[2] * (w.a if w.kind == W.SC else w.c))
    regions = []
    for k, m in enumerate((4, 7)):
        p = A.asd_mm_params()
        p.precision = prec
        p.nx, p.ny, p.nz = m, -(-ny // cell[1]), -(-nz // cell[2])
        for d in range(3):
            p.h[d] = edge[d]
        p.Ms0, p.A0, p.K0 = w.mu_s / w.a ** 3, w.J[0] / (2 * w.a), w.ku / w.a ** 3
        p.lambda_, p.gamma, p.Tc, p.mu_s, p.dt = w.alpha, w.gamma, 710.0, w.mu_s, w.dt
        g = A.MMHandle(p, stream=h.stream)
        dr = A.asd_drive()
        dr.B[2], dr.T_amb = -0.8, 300.0
        g.set_drive(dr)
        g.set_m(W.random_spins(g.n, 20 + k))
        regions.append(g)
    return h, regions


# whole and ragged cells; fewer and more boundary cells than a workgroup holds;
# both lattices
@pytest.mark.parametrize("lattice,n,cell", [
    ("sc", (24, 12, 4), (2, 2, 2)), ("sc", (31, 71, 9), (3, 2, 2)), ("sc", (25, 17, 7), (5, 4, 3)),
    ("l10", (14, 11, 6), (2, 3, 2)), ("l10", (17, 13, 5), (4, 4, 5)),
], ids=lambda v: str(v).replace(" ", ""))
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_window_faces_equal_the_single_calls(gpu, lattice, n, cell, prec):
    torch = gpu
    base = W.c2_granular_slab() if lattice == "sc" else W.c3_l10_window()
    steps = 3
    h, (L, R) = window(base, n, cell, prec)
    A.multiscale_step(h, 0, L, R, cell, steps)
    got = [h.get_spins(), L.get_m(), R.get_m()]
    h2, (L2, R2) = window(base, n, cell, prec)
    org = h2.state()[1]
    lib = A.lib()
    for _ in range(steps):
        dirs = []
        for g, face, x in ((L2, 1, org), (R2, 0, org + n[0] - cell[0])):
            sums = h2.coarse_grain(0, x, cell[0], *cell)
            A._mm_check(lib.asd_mm_set_face(g.h, face, sums.data_ptr(), 4), g.h)
            d = torch.empty((g.params.ny * g.params.nz, 3), dtype=torch.float64, device="cuda")
            A._mm_check(lib.asd_mm_get_face(g.h, face, d.data_ptr()), g.h)
            h2.synchronize()
            dirs.append(d)
        for d, x in zip(dirs, (org - cell[0], org + n[0])):
            A._check(lib.asd_set_columns(h2.h, 0, x, cell[0], *cell, d.data_ptr()), h2.h)
        h2.step(1)
        L2.step(1)
        R2.step(1)
        h2.synchronize()
    for a, b in zip(got, [h2.get_spins(), L2.get_m(), R2.get_m()]):
        np.testing.assert_array_equal(a, b)
    assert h.state()[0] == h2.state()[0] and L.step_count() == L2.step_count() == steps
    for o in (L, R, L2, R2, h, h2):
        o.close()
