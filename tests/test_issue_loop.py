"""Host logic of a solve's issue loop (IssueLoop, in
paper_2206_14780_amd/csrc/issue_plan.hpp): tests/issue_loop_sim.cpp runs it
against synthetic residual histories with a host that looks at every outcome or
only now and then.  No GPU."""
import os
import shutil
import subprocess
from collections import namedtuple

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
Run = namedtuple("Run", "name poll_every period H issued most idle")


@pytest.fixture(scope="module")
def runs(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("issue_loop") / "sim")
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2206_14780_amd", "csrc"),
                    os.path.join(HERE, "issue_loop_sim.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return [Run(f[0], *map(int, f[1:])) for f in map(str.split, out.splitlines())]


def test_the_halt_is_always_issued_and_the_limit_kept(runs):
    assert len(runs) > 200
    for r in runs:
        assert r.issued >= r.H, r
        assert r.most <= (r.poll_every or 2), r


def test_few_iterations_are_issued_past_the_halt(runs):
    # the run-ahead without a forecast, or none; a caller who asks for more can
    # lose at most that, and only where the history misleads the forecast: a
    # collapse, or noise whose peaks look like many iterations more
    for r in runs:
        most = r.poll_every if r.name in ("collapse", "noisy") and r.poll_every > 2 else 1
        assert r.issued - r.H <= most, r
        assert r.issued - r.H <= r.H // 2 + 1, r


def test_a_host_that_is_kept_away_can_let_the_device_run_ahead(runs):
    # a look every 12 iterations: with two ahead the device waits for most of
    # the solve, with 16 hardly ever; asking for more than that many is honoured
    by = {(r.name, r.poll_every, r.period): r for r in runs}
    two, many = by["slow", 2, 12], by["slow", 16, 12]
    assert two.idle > 0.7 * 12 / 2 * two.H
    assert many.most == 16 and many.idle < 0.1 * two.idle
    assert by["slow", 1000, 12].most > 100
    assert by["slow", 0, 12].idle == two.idle


def test_one_iteration_per_look_leaves_no_gap(runs):
    # the default never lets the device wait when the host sees every outcome
    # (but where it waits for the forecast halt, and at the start)
    for r in runs:
        if r.period == 1 and r.poll_every != 1 and r.name in ("geometric", "slow", "noisy", "plateau"):
            assert r.idle <= 3, r
