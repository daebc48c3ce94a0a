"""Infinities where a quantity overflows its type are what plain division gives.

Bars: counts exact, both populations bit-equal to the oracle's as multisets; fields and
the network's answers equal.
"""
import numpy as np
import pytest

import oracle
from paper_2603_24010_amd import workloads as W
from test_gpu_parity import assert_counts_equal, run_pair, sorted_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp", [32, 64])
@pytest.mark.parametrize("mu,sigma", [(800.0, 0.5), (660.0, 40.0)])
def test_electrons_of_infinite_energy_cross_in_one_step(fp, mu, sigma):
    # lognormal energies past the largest binary64 number, all of them or some (and
    # some whose speed alone is): absorbed at the other electrode in the step after
    cfg = W.config2(n_cells=50, beam_per_step=0, weight=1.0).replace(
        see_amp=5.0, see_max=8, see_law=W.SEE_LOGNORMAL, see_ln_mu=mu, see_ln_sigma=sigma)
    n = 900
    rng = np.random.default_rng(fp)
    v = np.full(n, 3e6)
    x = cfg.d - rng.uniform(0.0, 3.0, n) * v * cfg.dt
    sim, orc, recs = run_pair(cfg, {1: (x, v)}, oracle.WEAK, 5, fp == 32, (20_000, 2000))
    assert recs[-1][0]["emit_cum"].sum() > n
    for dg, do in recs:
        assert_counts_equal(dg, do)
    assert recs[-1][0]["abs_cum"][0].sum() > n
    for s in (0, 1):
        xg, ug, _ = sim.particles(0, s)
        assert len(xg) == recs[-1][0]["n_live"][s]
        if fp == 32:
            xo, uo, _ = orc.particles_f32(s)
            for a, b in zip(sorted_state(xg, ug), sorted_state(xo, uo)):
                np.testing.assert_array_equal(a, b)
    sim.close()


@pytest.mark.parametrize("cells", [64, 9000])  # the one-kernel solve and the three-kernel one
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_field_past_the_largest_number(cells, sign):
    # a surface charge that binary64 holds and whose field it does not
    from paper_2603_24010_amd import gapsim as gs
    cfg = W.config2(n_cells=cells, beam_per_step=0)
    q0 = np.zeros(cfg.n_mesh)
    q0[cfg.gap_mesh] = sign * 1e307 * (cfg.eps0 * cfg.area / cfg.d + cfg.c_par)  # 1e307 V over d < 1 / 20
    sim = gs.GapSim(cfg.replace(q0=q0), particle_fp=32, capacity=(64, 64))
    sim.step_weak(1)
    d, E = sim.diag(0), sim.fields(0)[1]
    assert cfg.d < 0.05 and np.isfinite(d["sigma"]) and np.abs(d["phi0"] - sign * 1e307) < 1e303
    np.testing.assert_array_equal(E, np.full(cells, sign * np.inf))
    assert d["e_ground"] == sign * np.inf
    sim.close()


@pytest.mark.parametrize("n", [769, 5000])
def test_network_with_a_weight_that_rounds_to_infinity(n):
    """A finite weight may round to an infinite bfloat16: many rows then answer as few do,
    which the matrix cores' split activations cannot (zero times infinity)."""
    import torch
    from paper_2603_24010_amd import gapsim as gs
    rng = np.random.default_rng(n)
    theta = rng.normal(0.0, 0.12, oracle.MLP_NPARAM).astype(np.float32)
    theta[oracle.MLP_NPARAM - 3 - 3 * 128 + 5] = 3.4e38  # of the first output
    sim = gs.GapSim(W.config2(64), particle_fp=32, capacity=(64, 64))
    norm = np.concatenate([np.zeros(48), np.ones(48), np.zeros(3), np.ones(3)])
    sim.mlp_set_weights(theta, norm)
    x = torch.from_numpy(rng.normal(0, 1.5, (n, 48)).astype(np.float32)).cuda()
    y = sim.mlp_forward(x).cpu().numpy()
    few = np.concatenate([sim.mlp_forward(x[b:b + 700]).cpu().numpy() for b in range(0, n, 700)])
    np.testing.assert_array_equal(y, few)
    assert np.isinf(y[:, 0]).all() and np.isfinite(y[:, 1:]).all()
    # finite weights again: the matrix cores again, equal to binary32's rounding
    theta[oracle.MLP_NPARAM - 3 - 3 * 128 + 5] = 0.1
    sim.mlp_set_weights(theta, norm)
    y = sim.mlp_forward(x).cpu().numpy()
    yo = oracle.mlp_forward(oracle.round_bf16(theta).astype(np.float64), x.cpu().numpy().astype(np.float64))
    assert np.abs(y - yo).max() <= 1e-5 * np.abs(yo).max()
    sim.close()
