"""A step's absorbed ions have the same room however the push splits its work: with few
workgroups of a single gap (their number limited by its nodes), and with workgroups that
take ions alone.

Bars: no capacity error, counts exact, both populations bit-equal to the oracle's
binary32 mode as multisets.
"""
import numpy as np
import pytest

import oracle
from paper_2603_24010_amd import workloads as W
from test_gpu_parity import assert_counts_equal, run_pair, sorted_state

pytestmark = pytest.mark.gpu

EVQ, OVQ = 128, 1024  # events in a workgroup's LDS queue and in its overflow region


@pytest.mark.parametrize("cells,ne,ni,hits,opts,wgs,before", [
    # 2.3e6 slots on 4097 nodes: 256 workgroups where 768 fit
    (4096, 100, 2_300_000, 950_000, {}, 256, 768),
    # round robin over 256: 47 workgroups for the electrons' 235 tiles, 209 for the ions' 977
    (256, 480_000, 2_000_000, 535_000, {"OPT_STREAM": 1, "OPT_GRID": 256}, 209, 256),
])
def test_room_for_a_steps_absorbed_ions(cells, ne, ni, hits, opts, wgs, before):
    from paper_2603_24010_amd import gapsim as gs
    # more than the regions of wgs workgroups and the gap's list (an eighth of the ion
    # slots and 4096) hold, less than those of `before` do
    cap = (ne + 200_000, ni + 5000)
    listed = cap[1] // 8 + 4096
    assert wgs * (EVQ + OVQ) + listed < hits < before * (EVQ + OVQ) + listed
    cfg = W.config2(n_cells=cells, beam_per_step=0, weight=1.0).replace(see_amp=0.1, see_max=4)
    rng = np.random.default_rng(cells)
    x, v = rng.uniform(0.3 * cfg.d, 0.6 * cfg.d, ni), np.zeros(ni)
    out = rng.permutation(ni)[:hits]
    x[out], v[out] = cfg.d - rng.uniform(0.0, 1.0, hits) * 1e-6, 2e6
    loads = {0: (rng.uniform(0, cfg.d, ne), rng.normal(0, 1e5, ne)), 1: (x, v)}
    sim, orc, recs = run_pair(cfg, loads, oracle.WEAK, 2, True, cap, {getattr(gs, k): q for k, q in opts.items()})
    assert recs[0][0]["abs_cum"][1].sum() == hits and recs[0][0]["emit_cum"].sum() > 0.02 * hits
    for dg, do in recs:
        assert_counts_equal(dg, do)
    for s in (0, 1):
        xg, ug, _ = sim.particles(0, s)
        xo, uo, _ = orc.particles_f32(s)
        for a, b in zip(sorted_state(xg, ug), sorted_state(xo, uo)):
            np.testing.assert_array_equal(a, b)
    sim.close()
