"""The push's split of small and uneven work, and its emission of many electrons per
ion, against the oracle's binary32 mode.

Bars: counts exact, both populations bit-equal as multisets, gap voltage and surface
charge within 1e-5.
"""
import numpy as np
import pytest

import oracle
from paper_2603_24010_amd import workloads as W
from test_gpu_parity import _series_rel, assert_counts_equal, run_pair, sorted_state

pytestmark = pytest.mark.gpu


def _check(sim, orc, recs):
    for dg, do in recs:
        assert_counts_equal(dg, do)
    for key in ("phi0", "sigma"):
        assert _series_rel([d[key] for d, _ in recs], [o[key] for _, o in recs]) <= 1e-5, key
    for s in (0, 1):
        xg, ug, _ = sim.particles(0, s)
        xo, uo, _ = orc.particles_f32(s)
        for a, b in zip(sorted_state(xg, ug), sorted_state(xo, uo)):
            np.testing.assert_array_equal(a, b)
    sim.close()


@pytest.mark.parametrize("law", [W.SEE_FIXED, W.SEE_EXP, W.SEE_LOGNORMAL])
@pytest.mark.parametrize("ions,amp", [(40, 30.0), (3000, 30.0), (3000, 0.7), (60_000, 6.0)])
def test_many_electrons_per_ion(ions, amp, law):
    # ions that reach the grounded electrode in the first steps: from a few of them
    # in one workgroup's wave to several rounds of one workgroup (its grid is one) and
    # the gap's list (room for an eighth of the ion slots)
    cfg = W.config2(n_cells=200, beam_per_step=7, weight=1.0).replace(
        see_amp=amp, see_max=70, see_law=law, see_ln_mu=1.2, see_ln_sigma=0.8)
    rng = np.random.default_rng(ions)
    v = 3e6
    x = cfg.d - rng.uniform(0.0, 3.0, ions) * v * cfg.dt
    from paper_2603_24010_amd import gapsim as gs
    sim, orc, recs = run_pair(cfg, {1: (x, np.full(ions, v))}, oracle.WEAK, 4, True,
                              (80 * ions + 1000, 10 * ions + 1000), {gs.OPT_GRID: 1} if ions > 3000 else None)
    assert recs[-1][0]["emit_cum"].sum() > 0.3 * min(amp, 60.0) * ions
    _check(sim, orc, recs)


@pytest.mark.parametrize("cells,n,beam", [
    (64, 0, 0), (64, 0, 5), (64, 1, 3), (64, 2048, 1), (64, 2049, 3000),
    (64, 120_000, 40), (700, 600_001, 90), (4096, 600_001, 1000), (16384, 40_000, 17),
])
@pytest.mark.parametrize("opts", [{}, {"OPT_STREAM": 1}, {"OPT_STEAL": 4}, {"OPT_GRID": 3}, {"OPT_BLOCK": 1024}])
def test_split_of_small_work(cells, n, beam, opts):
    from paper_2603_24010_amd import gapsim as gs
    cfg = W.config2(n_cells=cells, beam_per_step=beam, weight=1e3)
    loads = {}
    if n:
        rng = np.random.default_rng(n + cells)
        loads = {0: (rng.uniform(0, cfg.d, n // 3 + 1), rng.normal(0, 4e6, n // 3 + 1)),
                 1: (rng.uniform(0, cfg.d, n), rng.uniform(4e5, 3e6, n))}
    sim, orc, recs = run_pair(cfg, loads, oracle.STRICT, 3, True, (n + 20_000, n + 20_000),
                              {getattr(gs, k): v for k, v in opts.items()})
    _check(sim, orc, recs)


@pytest.mark.parametrize("ne,ni,grid", [
    (30_000, 30_000, 2), (2100, 150_000, 5), (150_000, 2100, 5), (70_000, 80_001, 7), (5, 200_000, 256),
    (200_000, 5, 11), (2048 * 9, 2048 * 7, 4),
])
def test_round_robin_split(ne, ni, grid):
    # round-robin workgroups of their own for electrons and ions, and shared ones where
    # that would give some a tile too many
    from paper_2603_24010_amd import gapsim as gs
    cfg = W.config2(n_cells=90, beam_per_step=301, weight=1e3)
    rng = np.random.default_rng(ne + ni)
    loads = {0: (rng.uniform(0, cfg.d, ne), rng.normal(0, 4e6, ne)), 1: (rng.uniform(0, cfg.d, ni), rng.uniform(4e5, 3e6, ni))}
    sim, orc, recs = run_pair(cfg, loads, oracle.WEAK, 3, True, (ne + 60_000, ni + 20_000),
                              {gs.OPT_STREAM: 1, gs.OPT_GRID: grid})
    _check(sim, orc, recs)


@pytest.mark.parametrize("opts", [{}, {"OPT_STEAL": 3, "OPT_GRID": 20}, {"OPT_STREAM": 1}, {"OPT_SORT_BIN": 16}])
def test_many_gaps_with_empty_ones_as_each_alone(opts):
    # the lookup of a tile's region among those of many gaps, runs of empty ones between
    # them, through two compactions: bit for bit what each gap does by itself
    from paper_2603_24010_amd import gapsim as gs
    rng = np.random.default_rng(5)
    cfgs, loads, caps = [], [], []
    for g in range(90):
        ne, ni = (0, 0) if g % 7 in (2, 3, 4) else (int(rng.integers(0, 5000)), int(rng.integers(0, 9000)))
        cfg = W.config2(n_cells=20 + g, beam_per_step=g % 3, weight=1e3, seed=g)
        cfgs.append(cfg)
        loads.append([(rng.uniform(0, cfg.d, n), rng.normal(0, 3e6, n)) for n in (ne, ni)])
        caps.append((ne + 9000, ni + 500))

    def run(which):
        sim = gs.GapSim([cfgs[g] for g in which], particle_fp=32, capacity=[caps[g] for g in which])
        for k, v in opts.items():
            sim.set_option(getattr(gs, k), v)
        for i, g in enumerate(which):
            for s in (0, 1):
                if loads[g][s][0].size:
                    sim.inject(i, s, *loads[g][s])
        sim.step_weak(70)
        out = []
        for i in range(len(which)):
            d = sim.diag(i)
            out.append([np.asarray(d[k]) for k in ("phi0", "sigma", "n_live", "abs_cum", "emit_cum", "inj_cum", "pushed_cum")])
        sim.close()
        return out

    for g, a in enumerate(run(range(90))):
        for x, y in zip(a, run([g])[0]):
            np.testing.assert_array_equal(x, y)
