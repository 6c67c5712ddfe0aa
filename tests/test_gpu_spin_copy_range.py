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
def buffer(gpu):
    """64 MiB of device memory in an allocation of its own (a cached one of torch's may
    go on behind it), zeroed: its address, its size and its bytes read back."""
    hip, size, p = A.lib(), 64 << 20, ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(size)) == 0
    zero = gpu.zeros(size, dtype=gpu.uint8, device="cuda")

    def copy(dst, src):
        gpu.cuda.synchronize()
        assert hip.hipMemcpy(ctypes.c_void_p(dst), ctypes.c_void_p(src), ctypes.c_size_t(size), 4) == 0

    def read():
        out = np.empty(size, dtype=np.uint8)
        copy(out.ctypes.data, p.value)
        return out

    copy(p.value, zero.data_ptr())
    gpu.cuda.synchronize()
    yield p.value, size, read
    hip.hipGetLastError()  # the refused copy's, not the next test's
    assert hip.hipFree(p) == 0


# rows that fit before the end of the allocation: none, two, all three (accepted)
@pytest.mark.parametrize("fit", [0, 2, 3])
@pytest.mark.parametrize("prec", [A.ASD_FP64, A.ASD_FP32], ids=["fp64", "fp32"])
def test_short_device_buffer_is_refused(buffer, prec, fit):
    base, size, read = buffer
    w = W.c1_plain_sc().scaled(nx=16, ny=13, nz=5, bc=(0, 0, 0))
    h = bridge.make_handle(w, prec)
    h.set_spins(W.random_spins(16 * 13 * 5, 2))
    ref = h.get_spins()
    nb = ref.nbytes // 3
    start = size - fit * nb - (16 if fit < 3 else 0)
    if fit == 3:
        A.asd_get_spins(h.h, 0, base + start, True)
    else:
        with pytest.raises(A.AsdError) as e:
            A.asd_get_spins(h.h, 0, base + start, True)
        assert e.value.code == A.ASD_EHIP
    h.synchronize()
    A.lib().hipGetLastError()
    got = read()
    assert not got[:start].any()
    assert got[start:start + fit * nb].tobytes() == ref.tobytes()[:fit * nb]
    assert not got[start + fit * nb:].any()
    np.testing.assert_array_equal(h.get_spins(), ref)
    h.close()
