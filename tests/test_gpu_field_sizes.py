"""The field solve at the grid sizes where its workgroup changes (threads and nodes
per thread), against the oracle.

Bars: counts exact; fields, gap voltage, surface and space charge within 1e-12
(binary64 particles) as for the usual sizes (the circuit's own charges do not depend
on the workgroup; at these first levels of a sinusoid they pass through zero); the
guess network's
in-step proposal within 1e-5 of the one a 256-cell context gives the same gap (its
binary32 inputs are normalised histories that may round differently).
"""
import numpy as np
import pytest

import oracle
from paper_2603_24010_amd import workloads as W
from test_gpu_parity import _series_rel, assert_counts_equal, check_fields, run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [oracle.STRICT, oracle.WEAK])
@pytest.mark.parametrize("cells", [2, 63, 191, 192, 193, 255, 767, 768, 1535, 1536, 2559, 2560, 4607, 4608, 8192])
def test_field_at_workgroup_edges(cells, mode):
    cfg = W.config1(n_cells=cells).replace(beam_per_step=20, beam_Emin_eV=1e3, beam_Emax_eV=2e4)
    loads = {s: (x, v * 30.0) for s, (x, v) in W.load_config1(n_per_species=3000, seed=cells).items()}
    sim, orc, recs = run_pair(cfg, loads, mode, 6, False, (20_000, 20_000))
    for dg, do in recs:
        assert_counts_equal(dg, do)
    for key in ("phi0", "sigma", "q_space"):
        assert _series_rel([d[key] for d, _ in recs], [o[key] for _, o in recs]) <= 1e-12, key
    check_fields(sim, orc, 1e-12)
    sim.close()


@pytest.mark.parametrize("other", [700, 1000, 2000, 4000, 8000, 12000])
def test_network_proposal_at_workgroup_edges(other):
    from paper_2603_24010_amd import gapsim as gs
    rng = np.random.default_rng(9)
    theta = rng.normal(0.0, 0.1, oracle.MLP_NPARAM).astype(np.float32)
    norm = np.concatenate([np.zeros(48), np.tile([300.0, 1.0, 1e-2, 1e-6, 1e-9, 1e-9], 8), np.zeros(3),
                           [1e-3, 1e-6, 1e-6]])
    got = []
    for cells in (256, other):
        # (the largest grid of a context sets the workgroup of all)
        cfgs = [W.config2(n_cells=256, beam_per_step=200), W.config2(n_cells=cells, beam_per_step=50)]
        sim = gs.GapSim(cfgs, particle_fp=32, capacity=(100_000, 100_000))
        for g in (0, 1):
            for s, (x, v) in W.load_config2(n=20_000, seed=3).items():
                sim.inject(g, s, x, v)
        sim.mlp_set_weights(theta, norm)
        sim.step_strict(12, gs.GUESS_MLP)
        d = sim.diag(0)
        got.append((d["mlp_proposal"], d["phi0"], d["I"]))
        assert d["newton_converged"]
        sim.close()
    for a, b in zip(got[0], got[1]):
        np.testing.assert_allclose(a, b, rtol=1e-5)
