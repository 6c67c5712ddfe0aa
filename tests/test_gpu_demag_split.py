"""The demagnetising field with a column's y-z pass in three workgroups (few
columns) and in one (many systems): the fields themselves, component by component."""
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


def field(prec, dims, cell, n_sys):
    nx, ny, nz = dims
    w = W.c2_granular_slab().scaled(nx=nx, ny=ny, nz=nz, x0=2e-9, y0=2e-9, grain_pitch=3e-9)
    h = bridge.make_handle(w, prec, kernel=A.ASD_KERNEL_FUSED, n_systems=n_sys, demag_cell=cell)
    lab = h.labels()
    rng = np.random.default_rng(17)
    S = rng.normal(size=(3, len(lab)))
    S /= np.linalg.norm(S, axis=0)
    S[:, lab < 0] = 0
    for k in range(n_sys):
        h.set_spins(S, k)
    B, _ = h.demag_field()
    h.close()
    return B


# one cell along y (the only mesh without padding rows); one plane; as many planes as
# two workgroups a CU take, and more; planes that the four lane groups share unevenly
@pytest.mark.parametrize("dims,cell", [((20, 3, 6), (2, 3, 2)), ((33, 16, 3), (1, 2, 3)),
                                       ((40, 10, 11), (1, 2, 1)), ((24, 20, 16), (2, 2, 1)),
                                       ((50, 40, 13), (2, 3, 2))])
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_split_columns_give_the_same_field(prec, dims, cell):
    """The same sums in the same order, but other products fused: a rounding each of
    the 3 ncz terms of a sum and of the about six operations of each of the FFT stages,
    forward and back, on values of up to four times the field."""
    few = field(prec, dims, cell, 1)[0]
    many = field(prec, dims, cell, 24)
    n = [-(-d // c) for d, c in zip(dims, cell)]
    stages = sum(max(2 * v - 1, 1).bit_length() for v in n[:2])
    eps = np.finfo(np.float64 if prec == A.ASD_FP64 else np.float32).eps
    top = np.abs(few).max()
    assert all(np.abs(few[c]).max() > 0.1 * top for c in range(3))
    for k in (0, 11, 23):
        np.testing.assert_allclose(many[k], few, rtol=0, atol=4 * (3 * n[2] + 12 * stages) * eps * top)
