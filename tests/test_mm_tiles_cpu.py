"""The rule that picks the tile width of a micromagnetic step, on the CPU: the
widths that the GPU tests rely on, the tiles' limits, and the meshes that the
stage kernels step faster."""
import os
import shutil
import subprocess

import pytest

from test_gpu_mm_widths import CASES, FP64, PAIRS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    exe = str(tmp_path_factory.mktemp("mm") / "mm_tiles")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2502_02236_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", "mm_tiles.cpp"), "-o", exe], check=True)

    def run(meshes):
        """(nx0, nx1, ny, nz, bytes per value) -> (width, LDS bytes)"""
        text = "".join("%d %d %d %d %d\n" % m for m in meshes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, ln.split())) for ln in out.splitlines()]

    return run


def elem(prec):
    return 8 if prec == FP64 else 4


def test_the_gpu_tests_run_every_width(pick):
    got = pick([(n[0], 0, n[1], n[2], elem(p)) for n, _, p, _ in CASES])
    assert [w for w, _ in got] == [w for *_, w in CASES]
    got = pick([(c[0], c[1], ny, nz, elem(p)) for c, ny, nz, p, _ in PAIRS])
    assert [w for w, _ in got] == [w for *_, w in PAIRS]
    # each region of a pair takes tiles on its own, too (else the pair does not)
    assert all(w for w, _ in pick([(c, 0, ny, nz, elem(p)) for cs, ny, nz, p, _ in PAIRS for c in cs]))
    assert {w for *_, p, w in CASES if p == FP64} == {0, 5, 6, 8, 10, 16}
    assert {w for *_, p, w in CASES if p != FP64} == {0, 5, 6, 8, 10, 16, 26}


def test_tiles_fit_the_threads_and_the_lds(pick):
    meshes = [(nx, 0, ny, nz, e) for nx in (1, 30, 300, 2000) for ny in (1, 47, 900)
              for nz in list(range(1, 20)) + [1 << 20] for e in (4, 8) if nx * ny * nz <= 1 << 28]
    for (nx, _, ny, nz, e), (w, lds) in zip(meshes, pick(meshes)):
        assert w in (0, 5, 6, 8, 10, 16, 26) and lds <= 128 * 1024
        assert (w + 6) ** 2 * nz <= 2048 or w == 0
        assert nz <= (14 if e == 8 else 16) or w == 0
        assert w > 0 or nz > 4  # low meshes are tiled at any size


def test_tall_meshes_of_many_rounds_keep_the_stage_kernels(pick):
    """Measured on MI355X (us a step): in tiles slower than in the stage kernels
    by 20 to 100 %."""
    slower = [(300, 60, 12, 8), (300, 60, 14, 8), (300, 60, 16, 4), (600, 300, 10, 8), (600, 300, 10, 4),
              (600, 300, 12, 4), (1500, 600, 12, 8), (1500, 600, 16, 4), (420, 200, 10, 4),
              (420, 200, 14, 8), (300, 150, 12, 4)]
    assert [w for w, _ in pick([(nx, 0, ny, nz, e) for nx, ny, nz, e in slower])] == [0] * len(slower)
    faster = [(30, 20, 14, 8), (100, 60, 12, 8), (300, 60, 8, 4), (300, 150, 6, 8), (600, 300, 4, 4),
              (1500, 600, 6, 8), (1500, 600, 2, 4), (150, 60, 14, 4)]
    assert all(w for w, _ in pick([(nx, 0, ny, nz, e) for nx, ny, nz, e in faster]))
    # the regions on both sides of a window count together
    assert pick([(150, 0, 150, 12, 4), (150, 150, 150, 12, 4)])[1][0] == 0
