"""The autotuner's choice among timed candidates, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    exe = str(tmp_path_factory.mktemp("tune") / "tune_pick")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2502_02236_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", "tune_pick.cpp"), "-o", exe], check=True)

    def run(rounds, incumbent):
        text = "%d %d %d\n" % (len(rounds), len(rounds[0]), incumbent)
        text += " ".join("%r" % t for v in rounds for t in v)
        return int(subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout)

    return run


A, B = [18.4, 18.5, 18.3, 18.6, 18.4], [19.5, 19.4, 19.6, 19.5, 19.4]


@pytest.mark.parametrize("rounds,incumbent,want", [
    ([A, B], 0, 0), ([A, B], 1, 0),                              # a clear gain either way
    ([B, [19.2, 19.5, 19.3, 19.6, 19.4]], 0, 0),                 # ahead by less than the rounds differ
    ([B, [19.2, 19.5, 19.3, 19.6, 19.4]], 1, 1),
    ([A, [18.3, 18.2, 18.3, 18.2, 18.3], B], 2, 1),              # the least median of several
    ([B, [18.4, 18.5, 40.0, 18.6, 18.4]], 0, 1),                 # one disturbed round does not count
    ([[19.5, 60.0, 19.6, 19.5, 19.4], A], 0, 1),
    ([[18.4, 25.0, 26.0, 18.5, 18.4], [19.5, 19.4, 19.6, 19.5, 19.4]], 0, 0),
    ([A], 0, 0),
], ids=str)
def test_near_ties_stay_with_the_incumbent(pick, rounds, incumbent, want):
    assert pick(rounds, incumbent) == want
