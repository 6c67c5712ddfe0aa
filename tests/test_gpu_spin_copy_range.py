"""asd_get_spins to device memory: an allocation that ends before the three rows do is
refused and nothing is written past what the refused copy left out."""
import ctypes

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


@pytest.fixture
def clear_error():
    yield
    ctypes.CDLL("libamdhip64.so.7").hipGetLastError()  # the refused copy's, not the next test's


# rows that fit before the end of the allocation: none, two, all three (accepted)
@pytest.mark.parametrize("fit", [0, 2, 3])
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_short_device_buffer_is_refused(gpu, clear_error, prec, fit):
    torch = gpu
    w = W.c1_plain_sc().scaled(nx=16, ny=13, nz=5, bc=(0, 0, 0))
    h = bridge.make_handle(w, prec)
    h.set_spins(W.random_spins(16 * 13 * 5, 2))
    ref = h.get_spins()
    nb = ref.nbytes // 3
    buf = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    seg = [s for s in torch.cuda.memory_snapshot()
           if s["address"] <= buf.data_ptr() < s["address"] + s["total_size"]][0]
    end = seg["address"] + seg["total_size"]
    # the last bytes of the allocation are this buffer's own
    assert buf.data_ptr() + buf.numel() == end
    start = buf.numel() - fit * nb - (16 if fit < 3 else 0)
    if fit == 3:
        A.asd_get_spins(h.h, 0, buf.data_ptr() + start, True)
    else:
        with pytest.raises(A.AsdError) as e:
            A.asd_get_spins(h.h, 0, buf.data_ptr() + start, True)
        assert e.value.code == A.ASD_EHIP
    h.synchronize()
    got = buf.cpu().numpy()
    assert not got[:start].any()
    assert got[start:start + fit * nb].tobytes() == ref.tobytes()[:fit * nb]
    assert not got[start + fit * nb:].any()
    np.testing.assert_array_equal(h.get_spins(), ref)
    h.close()
