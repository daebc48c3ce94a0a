"""Node sums kept in rows (small grids of contexts with many slots) against the one
row of a context with fewer slots: the sums are of integers, so that every output is
the same bit for bit, whichever workgroup added where.
"""
import numpy as np
import pytest

from paper_2603_24010_amd import workloads as W

pytestmark = pytest.mark.gpu

SLOTS = 1 << 19  # from here on, of one gap's two regions together


def _run(cells, gaps, slots, weak, guess, opts):
    from paper_2603_24010_amd import gapsim as gs
    cfgs, caps = [], []
    for g in range(gaps):
        n = max(2, cells - 5 * g)
        cfgs.append(W.config2(n_cells=n, beam_per_step=40 + g, weight=1e3, seed=g).replace(
            see_amp=2.0, **W.circuit_coupled_lc(1e-6, 1e-6, 1e-2, 50e-12, 0.5, 3e3, 50.0)))
        caps.append((slots - 60_000, 60_000) if g == gaps - 1 else (30_000, 60_000))
    sim = gs.GapSim(cfgs, particle_fp=32, capacity=caps)
    for k, v in opts.items():
        sim.set_option(getattr(gs, k), v)
    if guess == gs.GUESS_MLP:
        rng = np.random.default_rng(7)
        sim.mlp_set_weights(rng.normal(0, 0.1, gs.MLP_NPARAM).astype(np.float32),
                            np.concatenate([np.zeros(48), np.ones(48), np.zeros(3), np.full(3, 1e-3)]))
    rng = np.random.default_rng(cells)
    for g, cfg in enumerate(cfgs):
        m = 50_000 // gaps + 100
        sim.inject(g, 0, rng.uniform(0, cfg.d, m // 3), rng.normal(0, 4e6, m // 3))
        sim.inject(g, 1, rng.uniform(0, cfg.d, m), rng.uniform(-3e6, 3e6, m))
    out = []
    for _ in range(3):
        if weak:
            sim.step_weak(12)
        else:
            sim.step_strict(12, guess)
        for g in range(gaps):
            d = sim.diag(g)
            out += [np.asarray(d[k], dtype=np.float64) for k in
                    ("phi0", "sigma", "qconv", "q", "I", "n_live", "abs_step", "abs_cum", "emit_cum", "inj_cum",
                     "pushed_cum", "q_space")]
            out += list(sim.fields(g))
    sim.close()
    return out


@pytest.mark.parametrize("cells,gaps,opts", [
    (2, 1, {}), (30, 1, {}), (31, 1, {}), (32, 1, {}), (767, 1, {}), (768, 2, {}), (1535, 1, {"OPT_GRID": 700}),
    (1536, 3, {}), (2558, 1, {"OPT_STREAM": 1}), (2559, 1, {}), (300, 16, {}), (512, 1, {"OPT_GRAPH": 1}),
])
def test_rows_change_nothing(cells, gaps, opts):
    from paper_2603_24010_amd import gapsim as gs
    for weak, guess in ((True, gs.GUESS_DIRECT), (False, gs.GUESS_DIRECT), (False, gs.GUESS_MLP)):
        a = _run(cells, gaps, SLOTS, weak, guess, opts)
        b = _run(cells, gaps, SLOTS - 64, weak, guess, opts)
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
