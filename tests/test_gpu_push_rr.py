"""The round-robin push's workgroups of their own for electrons and for ions, against the
oracle's binary32 mode.  The rule that chooses them is evaluated here too, so that each
case is known to take the way it names.

Bars: counts exact, both populations bit-equal as multisets, gap voltage and surface
charge within 1e-5.
"""
import ctypes
import os
import re
import subprocess
import tempfile

import numpy as np
import pytest

import oracle
from paper_2603_24010_amd import workloads as W
from test_gpu_parity import run_pair
from test_gpu_push_split import _check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILE = 2048


def electrons(te, ti, nwg):
    """Workgroups that take the te electron tiles alone, 0 when all take both (k_push's
    rr_electrons)."""
    up = lambda a, b: -(-a // b)  # noqa: E731
    m = up(te + ti, nwg)
    if te == 0 or 4 * te > ti or m < 2:
        return 0
    best, most = 0, m if m < 8 else m + 1
    for ne in (up(te, m), up(te, m) - 1):
        if 0 < ne < nwg:
            c = max(up(te, ne), up(ti, nwg - ne))
            if c <= most:
                best, most = ne, c - 1
    return best


def test_rule_is_the_kernels():
    """electrons() is the kernel's function, compiled for the host; and whatever it says,
    the workgroups' first tiles and strides (as in k_push) take every tile once."""
    src = open(os.path.join(ROOT, "paper_2603_24010_amd", "csrc", "gs_kernels.hip")).read()
    text = re.search(r"^__device__ inline (int rr_electrons\(.*?^\})", src, re.S | re.M).group(1)
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "rr.cpp"), "w") as f:
            f.write("#include <algorithm>\nusing std::max;\nextern \"C\" " + text)
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", f"{d}/rr.so", f"{d}/rr.cpp"], check=True)
        lib = ctypes.CDLL(f"{d}/rr.so")
        for nwg in list(range(1, 24)) + [256]:
            for te in list(range(0, 24)) + [100, 700]:
                for ti in list(range(0, 120)) + [400, 1999, 2800]:
                    if te + ti < nwg:
                        continue
                    ne = electrons(te, ti, nwg)
                    assert lib.rr_electrons(te, ti, nwg) == ne, (te, ti, nwg)
                    if ne:
                        took = [t for b in range(ne) for t in range(b, te, ne)]
                        took += [t for b in range(ne, nwg) for t in range(te + b - ne, te + ti, nwg - ne)]
                        assert sorted(took) == list(range(te + ti)), (te, ti, nwg)


# tiles of electrons and ions, workgroups, those the electrons get, beam ions a step
@pytest.mark.gpu
@pytest.mark.parametrize("te,ti,grid,own,beam", [
    (1, 8, 5, 1, 301),        # two tiles each, one workgroup for the one electron tile
    (4, 17, 20, 2, 301),      # 18 workgroups for 17 ion tiles: one has nothing
    (10, 50, 12, 2, 0),       # five tiles each, no beam
    (12, 60, 9, 2, 7),        # eight and more tiles each: one more than the mean is taken
    (20, 81, 10, 2, 5000),
    (3, 100, 40, 1, 13),      # a partial round of the ions
    (1, 9, 5, 0, 301),        # the split would give some a third tile: shared
    (9, 30, 13, 0, 301),      # too many electrons
    (30, 9, 13, 0, 301),
    (1, 4, 5, 0, 301),        # a tile each
])
def test_own_workgroups(te, ti, grid, own, beam):
    from paper_2603_24010_amd import gapsim as gs
    ne, ni = (te - 1) * TILE + 77, (ti - 1) * TILE + 1003
    cfg = W.config2(n_cells=90, beam_per_step=beam, weight=1e3)
    rng = np.random.default_rng(1000 * te + ti)
    # (few electrons come and go, so that the tiles stay these)
    loads = {0: (rng.uniform(0, cfg.d, ne), rng.normal(0, 4e6, ne)),
             1: (rng.uniform(0, cfg.d, ni), rng.uniform(4e5, 3e6, ni))}
    sim, orc, recs = run_pair(cfg, loads, oracle.WEAK, 3, True, (ne + 60_000, ni + 20_000),
                              {gs.OPT_STREAM: 1, gs.OPT_GRID: grid})
    assert sim.launch()["tile"] == TILE
    slots = [(ne, ni)] + [tuple(int(v) for v in dg["n_slots"]) for dg, _ in recs[:-1]]
    took = [electrons(-(-e // TILE), -(-i // TILE), grid) for e, i in slots]
    assert took[0] == own and (own > 0) == all(took), took
    _check(sim, orc, recs)
