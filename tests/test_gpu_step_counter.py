"""The step counter of eager, captured and replayed steps: every way to run the
same steps gives the same spins."""
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


def handle(lattice="sc", kernel=A.ASD_KERNEL_FUSED, graph=0, demag=False, start=0):
    base = W.c2_granular_slab() if lattice == "sc" else W.c3_l10_window()
    w = base.scaled(nx=18, ny=14, nz=6, x0=2e-9, y0=2e-9, grain_pitch=3e-9)
    h = bridge.make_handle(w, A.ASD_FP64, kernel=kernel, graph_steps=graph,
                           demag_cell=(3, 3, 2) if demag else (0, 0, 0))
    lab = h.labels()
    S = W.initial_spins(len(lab), 9)
    S[:, lab < 0] = 0
    h.set_spins(S)
    h.set_step(start)
    return h


KINDS = [("sc", A.ASD_KERNEL_FUSED, False), ("sc", A.ASD_KERNEL_PLAIN, False),
         ("l10", A.ASD_KERNEL_FUSED, False), ("sc", A.ASD_KERNEL_FUSED, True),
         ("sc", A.ASD_KERNEL_PLAIN, True)]


@pytest.mark.parametrize("lattice,kernel,demag", KINDS)
def test_eager_and_graph_steps_share_the_counter(lattice, kernel, demag):
    ref = handle(lattice, kernel, demag=demag, start=5)
    for n in (1, 4, 2, 4, 1):  # the demagnetising field sums the spins anew in every call
        ref.step(n)
    mixed = handle(lattice, kernel, graph=4, demag=demag, start=5)
    for n in (1, 4, 2, 5):  # eager, graph, eager, graph + eager
        mixed.step(n)
    assert mixed.state()[0] == ref.state()[0] == 17
    np.testing.assert_array_equal(mixed.get_spins(), ref.get_spins())
    np.testing.assert_array_equal(mixed.energy(), ref.energy())
    ref.close()
    mixed.close()


@pytest.mark.parametrize("lattice,kernel,demag", KINDS[:4])
def test_steps_captured_by_the_caller_advance(gpu, lattice, kernel, demag):
    """Eager steps captured into the caller's own graph: each replay is the next
    steps, and eager steps after the replays go on from there."""
    torch = gpu
    ref = handle(lattice, kernel, demag=demag)
    for n in (2, 2, 2, 2, 1, 1):
        ref.step(n)
    h = handle(lattice, kernel, demag=demag)
    h.step(2)
    h.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=h.stream):
        h.step(2)
    with torch.cuda.stream(h.stream):
        for _ in range(3):
            g.replay()
            h.synchronize()
    h.step(1)
    h.step(1)
    np.testing.assert_array_equal(h.get_spins(), ref.get_spins())
    ref.close()
    h.close()


def test_sweeps_and_steps_share_the_counter():
    a, b = handle(), handle()
    a.mc_sweep(3)
    a.step(2)
    a.mc_sweep(1)
    for n in (1, 1, 1):
        b.mc_sweep(n)
    b.step(1)
    b.step(1)
    b.mc_sweep(1)
    assert a.state()[0] == b.state()[0] == 6
    np.testing.assert_array_equal(a.get_spins(), b.get_spins())
    a.close()
    b.close()
