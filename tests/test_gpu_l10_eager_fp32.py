"""FP32 L1_0 steps: eager launches, the handle's graphs and the caller's own graph run
the same steps, bit for bit, in every compiled tile."""
import numpy as np
import pytest

import workloads as W
from paper_2502_02236_amd import asd as A
from paper_2502_02236_amd import bridge
from test_gpu_split_sums import gpu  # noqa: F401 (the module's fixture)

pytestmark = pytest.mark.gpu


def handle(tile, dims, graph):
    nx, ny, nz = dims
    w = W.c3_l10_window().scaled(nx=nx, ny=ny, nz=nz, x0=2e-9, y0=2e-9, grain_pitch=3e-9,
                                 bc=(1, 0, nz % 2))
    h = bridge.make_handle(w, A.ASD_FP32, kernel=A.ASD_KERNEL_FUSED, graph_steps=graph)
    h.set_variant(A.ASD_KERNEL_FUSED, tile)
    lab = h.labels()
    S = W.initial_spins(len(lab), 9)
    S[:, lab < 0] = 0
    h.set_spins(S)
    h.set_step(5)
    return h


@pytest.mark.parametrize("dims", [(37, 29, 11), (64, 18, 4)], ids=str)
@pytest.mark.parametrize("tile", range(9))
def test_eager_and_captured_steps_are_the_same(gpu, tile, dims):  # noqa: F811
    torch = gpu
    ref, mixed, own = handle(tile, dims, 0), handle(tile, dims, 4), handle(tile, dims, 0)
    for n in (1, 4, 3):
        ref.step(n)
    for n in (1, 4, 3):  # eager, a graph, eager
        mixed.step(n)
    assert mixed.state()[0] == ref.state()[0] == 13
    np.testing.assert_array_equal(mixed.get_spins(), ref.get_spins())
    own.step(2)
    own.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=own.stream):
        own.step(2)
    with torch.cuda.stream(own.stream):
        for _ in range(2):
            g.replay()
            own.synchronize()
    own.step(2)
    np.testing.assert_array_equal(own.get_spins(), ref.get_spins())
    for h in (ref, mixed, own):
        h.close()
