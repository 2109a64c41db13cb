"""The library's rules on how particles fill cells (occupancy.hpp), compiled for
the host, for tests that mean to be on one side of one of them."""
import functools
import os
import shutil
import subprocess
import tempfile
from collections import namedtuple

import numpy as np
import pytest

from paper_2206_14780_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIST_CAP = {W.KERNEL_WENDLAND: 96, W.KERNEL_GAUSSIAN: 288}
Rules = namedtuple("Rules", "cap sums_by_cells delta scan_by_rows no_lists caller_order")


@functools.lru_cache(maxsize=None)
def _exe():
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = os.path.join(tempfile.mkdtemp(prefix="occupancy"), "rules")
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2206_14780_amd", "csrc"), os.path.join(HERE, "occupancy_rules.cpp"),
                    "-o", exe], check=True)
    return exe


def rules(n, ncell, gauss=False, fullest=0, support=4.19, cap=None):
    cap = (288 if gauss else 96) if cap is None else cap
    out = subprocess.run([_exe()], input=f"{n} {ncell} {int(gauss)} {fullest} {support!r} {cap}\n", text=True,
                         capture_output=True, check=True).stdout.split()
    return Rules(int(out[0]), *(x == "1" for x in out[1:]))


def cells_of(w):
    """Particles per cell of a workload, as the neighbour build bins them, and
    the cells' sides."""
    r = (3.0 if w.kernel == W.KERNEL_GAUSSIAN else 2.0) * w.h
    side = np.asarray(w.hi, float) - np.asarray(w.lo, float)
    nc = np.maximum(np.floor(side / (r * (1 + 1e-9))).astype(int), 1)
    cs = np.where(side > 0, side / nc, 1.0)
    cs = np.where((nc == 1) & (np.asarray(w.periodic) == 0), np.where(side > 0, 2 * side, 1.0), cs)
    c = np.floor((w.pos - w.lo) / cs).astype(int)
    c = np.where(np.asarray(w.periodic) != 0, c % nc, np.clip(c, 0, nc - 1))
    return np.bincount((c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0], minlength=int(nc.prod())), cs


def rules_of(w):
    count, cs = cells_of(w)
    gauss = w.kernel == W.KERNEL_GAUSSIAN
    r = (3.0 if gauss else 2.0) * w.h
    return rules(w.n, count.size, gauss, int(count.max()), float(4.19 * r ** 3 / cs.prod()))
