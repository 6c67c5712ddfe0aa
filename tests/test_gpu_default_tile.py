"""The tile an FP64 handle starts with: eight wavefronts only where they were measured
ahead of four."""
import pytest

import workloads as W
from paper_2502_02236_amd import asd as A
from paper_2502_02236_amd import bridge
from test_gpu_split_sums import gpu  # noqa: F401 (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,systems,waves", [((304, 92, 44), 2, 4), ((32, 32, 32), 16, 4),
                                             ((134, 137, 14), 7, 4), ((162, 188, 14), 3, 8),
                                             ((96, 293, 23), 1, 8)], ids=str)
def test_eight_wavefronts_where_they_are_ahead(n, systems, waves):
    nx, ny, nz = n
    w = W.c1_plain_sc().scaled(nx=nx, ny=ny, nz=nz, bc=(1, 0, 0))
    h = bridge.make_handle(w, A.ASD_FP64, kernel=A.ASD_KERNEL_AUTO, n_systems=systems)
    assert h.variant_name().startswith("k_fused_sc<double, 32, %d, 1," % waves)
    h.close()
