"""The step's tiles: whatever tile and z-chunk a step runs with, the same spins."""
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


def run(prec, dims, zper, rounds, variant, base=W.c2_granular_slab):
    nx, ny, nz = dims
    w = base().scaled(nx=nx, ny=ny, nz=nz, x0=2e-9, y0=2e-9, grain_pitch=3e-9)
    if zper:
        w = w.scaled(bc=w.bc[:2] + (W.BC_PERIODIC,))
    kernel = A.ASD_KERNEL_PLAIN if variant == "two-pass" else A.ASD_KERNEL_FUSED
    sys = bridge.SystemInputs(w)
    h = A.Handle(bridge.params_for(w, prec, kernel, rounds=rounds), [sys.desc])
    drive, _ = bridge.drive_for(w)
    h.set_drive(drive)
    if isinstance(variant, int):
        h.set_variant(kernel, variant)
    lab = h.labels()
    S = W.initial_spins(len(lab), 9)
    S[:, lab < 0] = 0
    h.set_spins(S)
    h.step(3)
    out = h.get_spins()
    h.close()
    return out


# one plane, fewer than, as many as and one more than the chunks of 1, 2, 3 and 6;
# interiors of 30 and 62 columns and of 6 and 14 rows reached, passed and missed by one
DIMS = [(5, 3, 1), (30, 6, 2), (31, 7, 3), (62, 14, 4), (63, 15, 7), (29, 13, 12)]


@pytest.mark.parametrize("dims,zper", [(d, z) for d in DIMS for z in (False, True) if d[2] > 2 or not z])
def test_fp64_tiles_equal_the_two_pass_step(dims, zper):
    """FP64 rounds every operation of the definition: no tolerance."""
    ref = run(A.ASD_FP64, dims, zper, 10, "two-pass")
    for v in ["auto", 0, 9, 10, 11, 12]:
        np.testing.assert_array_equal(run(A.ASD_FP64, dims, zper, 10, v), ref, err_msg=str(v))


@pytest.mark.parametrize("dims,rounds,zper", [(d, r, z) for d in DIMS for r, z in
                                              ((10, False), (7, False), (10, True)) if d[2] > 2 or not z])
def test_fp32_tiles_agree(dims, rounds, zper):
    """FP32 names its fused multiply-adds, so every tile rounds alike: no tolerance
    between tiles; against the two-pass step, which leaves them to the compiler, three
    steps of at most 2^-22 each on unit spins, 8 times that for the fields' sums."""
    ref = run(A.ASD_FP32, dims, zper, rounds, 0)
    for v in ["auto", 1, 4, 14, 18, 19, 20, 21, 22, 23, 24, 25]:
        np.testing.assert_array_equal(run(A.ASD_FP32, dims, zper, rounds, v), ref, err_msg=str(v))
    two = run(A.ASD_FP32, dims, zper, rounds, "two-pass")
    assert np.abs(ref - two).max() <= 3 * 8 * 2.0 ** -22


# chunks of 1, 2, 3, 5 and 9 planes against one, two and more than nine; interiors of
# 30 columns and 6 rows reached, passed and missed by one
@pytest.mark.parametrize("dims,zper", [((30, 6, 2), False), ((31, 7, 4), False), ((31, 7, 4), True),
                                       ((29, 5, 6), False), ((12, 13, 10), False), ((12, 13, 10), True)])
def test_fp64_l10_tiles_equal_the_two_pass_step(dims, zper):
    """FP64 rounds every operation of the definition: no tolerance."""
    ref = run(A.ASD_FP64, dims, zper, 10, "two-pass", W.c3_l10_window)
    for v in ["auto", 0, 1, 3, 4, 5, 6]:
        np.testing.assert_array_equal(run(A.ASD_FP64, dims, zper, 10, v, W.c3_l10_window), ref,
                                      err_msg=str(v))
