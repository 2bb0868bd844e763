"""The search for the antennas behind a list of baselines (csrc/ant_layout.h) is part
of creating an observation: its cost stays near linear in the rows also where rows
share coordinates, baselines repeat or there is nothing to find."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def cost(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("cost") / "ant_layout_cost_test")
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "ant_layout_cost_test.cpp"),
                    os.path.join(ROOT, "paper_2005_09316_amd", "csrc", "ant_layout.cpp"), "-o", exe], check=True)

    def run(n, keep, kind):
        out = subprocess.run([exe, str(n), str(keep), kind], check=True, capture_output=True, text=True, timeout=110)
        return dict(zip(("rows", "n", "bad", "seconds"), map(float, out.stdout.split())))
    return run


@pytest.mark.parametrize("kind", ["general", "plane", "line", "lattice", "rail", "one-place", "random"])
@pytest.mark.parametrize("n,keep", [(256, 1.0), (512, 0.85), (900, 0.85)])
def test_cost_of_the_search(cost, n, keep, kind):
    """5 microseconds a row, some ten times what a list in general position with
    gaps takes here (a table that degenerates into a list takes 70 and more)."""
    r = cost(n, keep, kind)
    print(n, keep, kind, r, flush=True)
    assert r["bad"] == 0
    assert r["seconds"] <= 5e-6 * r["rows"]
    if kind in ("general", "plane", "line"):
        assert r["n"] == n
