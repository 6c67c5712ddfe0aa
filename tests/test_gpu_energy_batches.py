"""Energies of batches whose largest system has as many tiles as one thread, one
wavefront or a workgroup adds."""
import numpy as np
import pytest

import workloads as W
from oracle_build import oracle_system
from paper_2502_02236_amd import asd as A
from paper_2502_02236_amd import bridge
from test_gpu_split_sums import gpu  # noqa: F401 (the module's fixture)

pytestmark = pytest.mark.gpu


# tiles of 256 sites; the last system's last tile holds 16 sites
@pytest.mark.parametrize("tiles", [(8, 1, 3), (9, 2), (64, 5), (65, 1)], ids=str)
@pytest.mark.parametrize("n", [3, 66])
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_energies_of_a_batch(prec, n, tiles):
    w = W.c1_plain_sc().scaled(bc=(0, 0, 0))
    kinds = [w.scaled(nx=16 * t, ny=16, nz=1) for t in tiles] + [w.scaled(nx=16 * tiles[-1] - 15, ny=16, nz=1)]
    ws = [kinds[k % len(kinds)] for k in range(n)]
    h = A.Handle(bridge.params_for(w, prec), [bridge.SystemInputs(q).desc for q in ws])
    dr, bits = bridge.drive_for(w)
    h.set_drive(dr)
    ref = []
    for k, q in enumerate(ws):
        h.set_spins(W.random_spins(q.nx * 16, 3 + k % 5), k)
        ref.append(np.asarray(oracle_system(q).energy(h.get_spins(k).astype(np.float64), 0)))
    # N terms of up to 6 J each added through at most 64 levels of chain and tree, four sums
    tol = 4 * 64 * 1.2e-16 * 256 * max(tiles) * 6 * w.J[0]
    np.testing.assert_allclose(h.energy(), ref, rtol=0, atol=tol)
    h.close()
