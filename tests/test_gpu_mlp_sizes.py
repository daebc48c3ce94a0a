"""The guess network's training and evaluation at the edges of their row tiles,
from arrays aligned to their element only.

Bars: 1e-5 of the largest value of the oracle's binary64 gradient, loss and output
(binary32 sums of up to 128 terms, and over the batch in slices: errors of a few
1e-7), as for the usual sizes.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _view(a, shift):
    """The array on the GPU, `shift` elements past an aligned address."""
    import torch
    t = torch.zeros(a.size + shift, dtype=torch.from_numpy(a).dtype, device="cuda")
    t[shift:] = torch.from_numpy(a.reshape(-1)).cuda()
    return t[shift:].view(a.shape)


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 64, 129, 1000, 4096, 4097, 4129])
def test_training_step_at_tile_edges(B):
    from paper_2603_24010_amd import gapsim as gs
    rng = np.random.default_rng(B)
    n, shift = 5000, B % 4
    x = rng.normal(0, 1, (n, 48)).astype(np.float32)
    t = rng.normal(0, 1, (n, 3)).astype(np.float32)
    order = rng.integers(0, n, 2 * B + B // 2).astype(np.int32)  # two steps and a remainder
    theta0 = rng.normal(0.0, 0.1, oracle.MLP_NPARAM).astype(np.float32)
    m0 = rng.normal(0.0, 1e-3, theta0.size).astype(np.float32)
    v0 = rng.uniform(1e-5, 2e-5, theta0.size).astype(np.float32)
    th, m, v = (_view(a, shift) for a in (theta0, m0, v0))
    loss, grad = gs.mlp_train(_view(x, shift), _view(t, shift), _view(order, shift), B, th, m, v, step0=40, lr=1e-3,
                              want_grad=True)
    tho, mo, vo = (a.astype(np.float64) for a in (theta0, m0, v0))
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))  # the rates as the library rounds them
    lo = []
    for k in range(2):
        i = order[k * B:(k + 1) * B]
        l, go = oracle.mlp_loss_grad(tho, x[i].astype(np.float64), t[i].astype(np.float64))
        lo.append(l)
        oracle.adam_step(tho, mo, vo, 41 + k, go, 1e-3, b1, b2)
    np.testing.assert_allclose(loss.cpu().numpy(), lo, rtol=1e-5)
    assert np.abs(grad.cpu().numpy() - go).max() <= 1e-5 * np.abs(go).max()
    for a, b in ((th, tho), (m, mo), (v, vo)):
        assert np.abs(a.cpu().numpy() - b).max() <= 1e-5 * np.abs(b).max()


def test_bad_sample_indices_are_reported():
    import torch
    from paper_2603_24010_amd import gapsim as gs
    x, t = torch.randn(64, 48, device="cuda"), torch.randn(64, 3, device="cuda")
    for bad in (-1, 64):
        th = torch.zeros(oracle.MLP_NPARAM, device="cuda")
        order = torch.zeros(20, dtype=torch.int32, device="cuda")
        order[19] = bad
        with pytest.raises(gs.GapsimError):
            gs.mlp_train(x, t, order, 20, th, torch.zeros_like(th), torch.zeros_like(th))


@pytest.mark.parametrize("n", [1, 31, 33, 768, 769, 1024, 1025, 1055, 1057, 16385, 50_001])
def test_forward_at_tile_edges(n):
    from paper_2603_24010_amd import gapsim as gs
    from paper_2603_24010_amd import workloads as W
    rng = np.random.default_rng(n)
    theta = rng.normal(0.0, 0.12, oracle.MLP_NPARAM).astype(np.float32)
    sim = gs.GapSim(W.config2(64), particle_fp=32, capacity=(64, 64))
    sim.mlp_set_weights(theta, np.concatenate([np.zeros(48), np.ones(48), np.zeros(3), np.ones(3)]))
    x = rng.normal(0, 1.5, (n, 48)).astype(np.float32)
    # (outside the caller's rows nothing is read or written)
    y = sim.mlp_forward(_view(x, n % 4)).cpu().numpy()
    yo = oracle.mlp_forward(oracle.round_bf16(theta).astype(np.float64), x.astype(np.float64))
    assert np.abs(y - yo).max() <= 1e-5 * np.abs(yo).max()
    sim.close()


def test_forward_rows_stay_apart():
    """A row of infinities, NaN or the largest values touches no other row, and gives
    no finite answer where the row kernel gives none."""
    from paper_2603_24010_amd import gapsim as gs
    from paper_2603_24010_amd import workloads as W
    rng = np.random.default_rng(3)
    theta = rng.normal(0.0, 0.12, oracle.MLP_NPARAM).astype(np.float32)
    sim = gs.GapSim(W.config2(64), particle_fp=32, capacity=(64, 64))
    sim.mlp_set_weights(theta, np.concatenate([np.zeros(48), np.ones(48), np.zeros(3), np.ones(3)]))
    x = rng.normal(0, 1.5, (4000, 48)).astype(np.float32)
    clean = sim.mlp_forward(_view(x, 0)).cpu().numpy()
    odd = {5: np.inf, 70: -np.inf, 133: np.nan, 1000: np.finfo(np.float32).max, 3999: 1e-42}
    z = x.copy()
    for r, v in odd.items():
        z[r, r % 48] = v
    y = sim.mlp_forward(_view(z, 0)).cpu().numpy()
    rows = np.array(sorted(odd))
    same = np.setdiff1d(np.arange(4000), rows)
    np.testing.assert_array_equal(y[same], clean[same])
    few = sim.mlp_forward(_view(z[rows], 0)).cpu().numpy()
    np.testing.assert_array_equal(np.isfinite(y[rows]), np.isfinite(few))
    ok = np.isfinite(few)
    np.testing.assert_allclose(y[rows][ok], few[ok], rtol=1e-5)
    sim.close()
