"""Sums of batches of isolated grains, one grain or none per system, in one part and in
several."""
import numpy as np
import pytest

import workloads as W
from paper_2502_02236_amd import asd as A
from paper_2502_02236_amd import bridge
from test_gpu_split_sums import gpu  # noqa: F401 (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cell", [(12, 12, 8), (31, 17, 19)], ids=["one-part", "five-parts"])
@pytest.mark.parametrize("n", [1, 64, 65])
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_sums_of_isolated_grains(prec, n, cell):
    nx, ny, nz = cell
    w = W.c1_plain_sc().scaled(nx=nx, ny=ny, nz=nz, bc=(0, 0, 0))
    rng = np.random.default_rng(4)
    labs = []
    for k in range(n):  # uneven grains; every seventh system but the first has none
        lab = np.where(rng.random(nx * ny * nz) < 0.5 + 0.5 * k / n, 0, -1).astype(np.int32)
        labs.append(np.full_like(lab, -1) if k % 7 == 6 else lab)
    h = A.Handle(bridge.params_for(w, prec), [bridge.SystemInputs(w, labels=q).desc for q in labs])
    ref = np.zeros((n, 4))
    for k, lab in enumerate(labs):
        S = W.random_spins(len(lab), 3 + k % 5)
        S[:, lab < 0] = 0
        h.set_spins(S, k)
        S = h.get_spins(k).astype(np.float64)
        ref[k] = [*S.sum(1), (lab == 0).sum()]
    some = np.array([h.grain_count(k) for k in range(n)]) > 0
    pg, ps = h.magnetization()
    # N terms of size <= 1 added through at most 64 levels of chain and tree
    tol = 64 * 1.2e-16 * nx * ny * nz
    np.testing.assert_allclose(pg, ref[some], rtol=0, atol=tol)
    np.testing.assert_allclose(ps, ref, rtol=0, atol=tol)
    h.accumulate_moments(reset=True)
    h.accumulate_moments()
    m = np.linalg.norm(ref[:, :3], axis=1) / np.maximum(ref[:, 3], 1)
    np.testing.assert_allclose(h.moment_stats()[:, :4], 2 * np.stack([m ** 0, m, m ** 2, m ** 4], 1), rtol=0,
                               atol=2 * 4 * 64 * 1.2e-16)
    h.close()
