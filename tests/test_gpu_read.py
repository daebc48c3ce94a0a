"""Read-backs at the edges of their kernels' tiles: the time-step check against the
particles read back (largest speeds and the fullest cell exactly), the potential
against the field it is summed from (1e-13 of its largest value, the rounding of a
sum of up to 16384 terms), for gaps of different sizes in one context.
"""
import numpy as np
import pytest

from paper_2603_24010_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp", [32, 64])
@pytest.mark.parametrize("cells,ne,ni", [(2, 0, 5), (2, 9, 0), (63, 251, 1001), (64, 257, 2048), (1000, 70_003, 90_001),
                                         (8192, 100_000, 33)])
def test_dt_check_matches_particles(cells, ne, ni, fp):
    from paper_2603_24010_amd import gapsim as gs
    cfg = W.config2(n_cells=cells, beam_per_step=0, weight=1e3)
    rng = np.random.default_rng(cells + ne)
    sim = gs.GapSim(cfg, particle_fp=fp, capacity=(ne + 40_000, ni + 64))
    for s, n, v in ((0, ne, 5e6), (1, ni, 2e6)):
        if n:
            sim.inject(0, s, rng.uniform(0, cfg.d, n), rng.normal(0, v, n))
    sim.step_weak(3)
    for _ in range(2):  # (the second finds the counters cleared)
        r = sim.dt_check(0)
        dx = cfg.d / cells
        for s in (0, 1):
            _, u, _ = sim.particles(0, s)
            top = float(np.abs(u).max()) if u.size else 0.0
            assert r["beta"][s] == top and r["v_max"][s] == top * dx / cfg.dt
        x, _, _ = sim.particles(0, 0)
        full = np.bincount(np.minimum(x.astype(np.int64), cells - 1), minlength=cells).max() if x.size else 0
        assert r["n_e_max"] == float(full) * cfg.weight / dx
    sim.close()


def test_fields_of_gaps_of_different_sizes():
    from paper_2603_24010_amd import gapsim as gs
    cells = [2, 1023, 1024, 1025, 4097, 16384, 5]
    cfgs = [W.config2(n_cells=c, beam_per_step=0, weight=1e3) for c in cells]
    sim = gs.GapSim(cfgs, particle_fp=32, capacity=(64, 60_000))
    rng = np.random.default_rng(1)
    for g, cfg in enumerate(cfgs):
        sim.inject(g, 1, rng.uniform(0, cfg.d, 50_000), np.full(50_000, 1e5))
    sim.step_strict(2)
    for g, cfg in enumerate(cfgs):
        phi, E, rho = sim.fields(g)
        dx = cfg.d / cfg.n_cells
        want = np.append(np.cumsum(dx * E[::-1])[::-1], 0.0)
        assert np.abs(phi - want).max() <= 1e-13 * np.abs(want).max()
        # Gauss' law on every interior node
        np.testing.assert_allclose(np.diff(E), dx * rho[1:-1] / cfg.eps0, rtol=0, atol=1e-12 * np.abs(E).max())
        assert abs(sim.diag(g)["phi0"] - phi[0]) <= 1e-11 * abs(phi[0])
    sim.close()
