"""FP32 steps of every compiled tile and z-chunk: the same spins, so that a system's
trajectory does not depend on what the default picks for the batch it is in."""
import numpy as np
import pytest

import workloads as W
from paper_2502_02236_amd import asd as A
from test_gpu_step_tiles import DIMS, gpu, run  # noqa: F401 (gpu: the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,zper", [(d, z) for d in DIMS for z in (False, True) if d[2] > 2 or not z])
def test_fp32_sc_tiles_agree(dims, zper):
    ref = run(A.ASD_FP32, dims, zper, 10, 0)
    for v in range(1, 26):
        np.testing.assert_array_equal(run(A.ASD_FP32, dims, zper, 10, v), ref, err_msg=str(v))


# chunks of 1, 2, 3, 5 and 9 planes against one, two and more than nine; interiors of
# 30 columns and 6 rows reached, passed and missed by one
@pytest.mark.parametrize("dims,zper", [((30, 6, 2), False), ((31, 7, 4), False), ((31, 7, 4), True),
                                       ((29, 5, 6), False), ((12, 13, 10), False), ((12, 13, 10), True)])
@pytest.mark.parametrize("rounds", [10, 7])
def test_fp32_l10_tiles_agree(dims, zper, rounds):
    ref = run(A.ASD_FP32, dims, zper, rounds, 0, W.c3_l10_window)
    for v in ["auto", 1, 2, 3, 4, 5, 6, 7, 8]:
        np.testing.assert_array_equal(run(A.ASD_FP32, dims, zper, rounds, v, W.c3_l10_window), ref,
                                      err_msg=str(v))
