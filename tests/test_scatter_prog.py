"""The scatter programs of the FP32 one-block sigma_3 kernel (csrc/scatter_prog.h)
on the host: for every space of up to 16 orbitals the packed words of every tile
reproduce the plain per-target sums exactly (integers), write each target once and
stay inside their arrays; some program holds every tile of each space."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("scatter_prog") / "driver")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(ROOT, "tests", "scatter_prog_driver.cpp")])
    return exe


@pytest.mark.parametrize("n", range(2, 17))
def test_programs_hold_every_tile(driver, n):
    inp = "".join(f"{n} {e}\n" for e in range(1, n))
    out = subprocess.run([driver], input=inp, capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    lines = [tuple(int(x) for x in l.split()) for l in out.stdout.split("\n") if l]
    assert [(a, b) for a, b, _ in lines] == [(n, e) for e in range(1, n)]
    assert all(p >= 0 for _, _, p in lines), lines
