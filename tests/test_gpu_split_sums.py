"""GPU sums whose work is split over workgroups: the grain sums in parts and the
energy's tiles, at the sizes where the split changes."""
import numpy as np
import pytest

import workloads as W
from oracle_build import oracle_system
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


def slabs(nx, ny, nz, n_grains):
    """Grains as layers along x separated by one non-magnetic column, uneven."""
    lab = np.full((nz, ny, nx), -1, np.int32)
    edges = np.linspace(0, nx, n_grains + 1).astype(int)
    for g in range(n_grains):
        lab[:, :, edges[g]:edges[g + 1] - (1 if g + 1 < n_grains else 0)] = g
    return lab.reshape(-1)


# one part per grain; several (a thread per grain adds them); more than sixteen
# (a wavefront per grain); a single site; more tiles than threads of a workgroup
@pytest.mark.parametrize("n,n_grains", [((1, 1, 1), 1), ((17, 11, 5), 3), ((40, 30, 20), 1),
                                        ((40, 30, 20), 4), ((61, 53, 31), 1), ((97, 64, 44), 7)],
                         ids=lambda v: str(v).replace(" ", ""))
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_split_sums_match_host_sums(n, n_grains, prec):
    nx, ny, nz = n
    w = W.c1_plain_sc().scaled(nx=nx, ny=ny, nz=nz, bc=(0, 0, 0))
    lab = slabs(nx, ny, nz, n_grains)
    h = bridge.make_handle(w, prec, labels=lab)
    S = W.random_spins(len(lab), 3)
    S[:, lab < 0] = 0
    h.set_spins(S)
    S = h.get_spins().astype(np.float64)
    pg, ps = h.magnetization()
    ref = np.array([[*S[:, lab == g].sum(1), (lab == g).sum()] for g in range(n_grains)])
    # N terms of size <= 1 added through at most 64 levels of chain and tree
    tol = 64 * 1.2e-16 * len(lab)
    np.testing.assert_allclose(pg, ref, rtol=0, atol=tol)
    np.testing.assert_allclose(ps[0], ref.sum(0), rtol=0, atol=tol)
    h.accumulate_moments(reset=True)
    m = np.linalg.norm(ref.sum(0)[:3]) / ref.sum(0)[3]
    np.testing.assert_allclose(h.moment_stats()[0, :4], [1, m, m * m, m ** 4], rtol=0,
                               atol=4 * 64 * 1.2e-16)
    e = oracle_system(w, labels=lab).energy(S, 0)
    np.testing.assert_allclose(h.energy()[0], np.asarray(e), rtol=0, atol=4 * tol * 6 * w.J[0])
    h.close()


# rows of 16-byte chunks, of 4-byte words, and a destination no chunk fits
@pytest.mark.parametrize("nx", [3, 4, 13, 64])
@pytest.mark.parametrize("shift", [0, 4, 8, 1], ids=lambda v: f"dst+{v}")
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_device_copy_of_the_spins(gpu, nx, shift, prec):
    torch = gpu
    w = W.c1_plain_sc().scaled(nx=nx, ny=3, nz=5, bc=(0, 0, 0))
    ins = [bridge.SystemInputs(w) for _ in range(2)]
    h = A.Handle(bridge.params_for(w, prec), [i.desc for i in ins])
    for k in range(2):
        h.set_spins(W.random_spins(nx * 15, k), k)
        ref = h.get_spins(k)
        nb = ref.nbytes
        buf = torch.zeros(nb + 64, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        A.asd_get_spins(h.h, k, buf.data_ptr() + shift, True)
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert got[shift:shift + nb].tobytes() == ref.tobytes()
        assert not got[:shift].any() and not got[shift + nb:].any()
    h.close()
