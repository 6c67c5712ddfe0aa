"""Sums of a batch whose systems have as many grains as one wavefront covers, one
more, and few: by one wavefront per system or by a whole workgroup."""
import numpy as np
import pytest

import workloads as W
from paper_2502_02236_amd import asd as A
from paper_2502_02236_amd import bridge
from test_gpu_split_sums import gpu, slabs  # noqa: F401 (gpu: the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grains", [(64, 1, 63), (65, 1, 64), (1,), (2, 130)], ids=str)
@pytest.mark.parametrize("cross", [(3, 2), (60, 50)], ids=["small", "many-parts"])
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_sums_of_few_and_many_grains(prec, cross, grains):
    nx, (ny, nz) = 2 * max(max(grains), 10) + 1, cross
    w = W.c1_plain_sc().scaled(nx=nx, ny=ny, nz=nz, bc=(0, 0, 0))
    labs = [slabs(nx, ny, nz, g) for g in grains]
    h = A.Handle(bridge.params_for(w, prec), [bridge.SystemInputs(w, labels=q).desc for q in labs])
    ref = []
    for k, lab in enumerate(labs):
        S = W.random_spins(len(lab), 3 + k)
        S[:, lab < 0] = 0
        h.set_spins(S, k)
        S = h.get_spins(k).astype(np.float64)
        ref.append(np.array([[*S[:, lab == g].sum(1), (lab == g).sum()] for g in range(grains[k])]))
    pg, ps = h.magnetization()
    # N terms of size <= 1 added through at most 64 levels of chain and tree
    tol = 64 * 1.2e-16 * len(labs[0])
    np.testing.assert_allclose(pg, np.concatenate(ref), rtol=0, atol=tol)
    np.testing.assert_allclose(ps, [r.sum(0) for r in ref], rtol=0, atol=tol)
    h.accumulate_moments(reset=True)
    m = np.array([np.linalg.norm(r.sum(0)[:3]) / r.sum(0)[3] for r in ref])
    np.testing.assert_allclose(h.moment_stats()[:, :4], np.stack([m ** 0, m, m ** 2, m ** 4], 1), rtol=0,
                               atol=4 * 64 * 1.2e-16)
    h.close()
