"""The y-z pass of the demagnetising field: a column in three workgroups (few columns)
and in one (many systems) give the same field."""
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


def spins(prec, dims, cell, n_sys):
    nx, ny, nz = dims
    w = W.c2_granular_slab().scaled(nx=nx, ny=ny, nz=nz, x0=2e-9, y0=2e-9, grain_pitch=3e-9)
    h = bridge.make_handle(w, prec, kernel=A.ASD_KERNEL_FUSED, n_systems=n_sys, demag_cell=cell)
    lab = h.labels()
    S = W.initial_spins(len(lab), 9)
    S[:, lab < 0] = 0
    for k in range(n_sys):
        h.set_spins(S, k)
    h.step(2)
    out = h.get_spins(0)
    h.close()
    return out


# one cell along y; no padding rows; one plane; more planes than the four lane groups
@pytest.mark.parametrize("dims,cell", [((20, 3, 6), (2, 3, 2)), ((33, 16, 3), (1, 2, 3)),
                                       ((40, 10, 11), (1, 2, 1))])
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32])
def test_split_columns_give_the_same_steps(prec, dims, cell):
    """Same sums in the same order; the compiler may fuse other products, so a few
    units in the last place of a field that turns the spin by at most 1e-2 a step."""
    few = spins(prec, dims, cell, 1)
    many = spins(prec, dims, cell, 24)
    atol = 64 * np.finfo(np.float64 if prec == A.ASD_FP64 else np.float32).eps
    np.testing.assert_allclose(many, few, rtol=0, atol=atol)
