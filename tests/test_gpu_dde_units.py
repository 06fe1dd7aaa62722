"""Gridding units of the DDE-aware adjoint, where they can go wrong: a tile with one unit and with
several, items that fill a unit or a group exactly, more items than a wavefront scans at once,
tiles on the wrapping edges, each tile side, and a per-block unit of more visibilities than one
group holds; and tiled grids of more than 1024 cells.  Phi^dagger whole and masked against the
oracle's DDE-aware operator, and the batched dual update against the per-block one.
Tolerance: FP32 sums of the oracle's FP64 terms, relative l2 <= 1e-5 as for every operator."""
import numpy as np
import pytest
import torch

import synth
from helpers import rel_l2, to_plan
from oracle import pd as opd
from oracle.dde import DDEMeasurement
from oracle.measurement import Measurement

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def R():
    import paper_1610_08895_amd as R

    assert torch.cuda.is_available()
    return R


def _clusters(n, counts, seed):
    """counts[i] visibilities in a few cells around the i-th place (corner, edge, inner), shuffled."""
    K = 2 * n
    rng = np.random.default_rng(seed)
    places = np.array([[0, 0], [K - 3, K // 2], [K // 2 + 5, K // 4], [K // 4 + 16, K // 4 + 16]])
    kap = np.concatenate([places[i % 4] + rng.uniform(0.0, 6.0, (c, 2)) for i, c in enumerate(counts)])
    uv = 2 * np.pi * kap / K
    uv = np.where(uv >= np.pi, uv - 2 * np.pi, uv).astype(np.float32)
    return uv[rng.permutation(len(uv))], rng


@pytest.mark.parametrize("n,tile,jd,counts,d", [
    (64, 32, 5, (1, 511, 512, 513), 1), (64, 16, 3, (300, 2600, 64, 63), 3), (128, 64, 7, (1500, 900, 1, 40), 2),
    (32, 16, 1, (700, 700, 700, 700), 70), (64, 64, 5, (900, 1300, 10, 5), 130), (1024, 32, 3, (1200, 600, 7, 1), 2)])
def test_dde_gridding_units(R, n, tile, jd, counts, d):
    uv, rng = _clusters(n, counts, n + jd)
    M = len(uv)
    off = np.linspace(0, M, d + 1).astype(np.int64)
    taps = synth.dde_taps(M, jd, rng, strength=0.3)
    dm = DDEMeasurement(Measurement(uv, off, (n, n)), taps)
    plan = R.Plan(n, uv, off, tile=tile)
    plan.set_dde(taps)
    order = plan.order()
    w = rng.standard_normal(M) + 1j * rng.standard_normal(M)
    wt = torch.tensor(to_plan(w, order), dtype=torch.complex64, device="cuda")
    assert rel_l2(plan.phi_adj(wt).cpu().numpy(), dm.phi_adj_real(w)) < TOL
    mask = (np.arange(d) % 3 != 1).astype(np.uint8)
    xm = plan.phi_adj(wt, mask=torch.tensor(mask, device="cuda")).cpu().numpy()
    assert rel_l2(xm, dm.phi_adj_real(w, blocks=np.flatnonzero(mask))) < TOL
    # a mask without an active block leaves nothing of the last call behind
    none = plan.phi_adj(wt, mask=torch.zeros(d, dtype=torch.uint8, device="cuda"))
    assert not none.any()


@pytest.mark.parametrize("n", [64, 1024])
def test_dde_batched_steps_equal_per_block_steps(R, n):
    """Blocks of 1300 and more visibilities on one tile: a per-block unit of two groups.  Both forms
    sum the same FP32 terms in another order: 12 steps stay within 1e-5."""
    uv, rng = _clusters(n, (2700, 900, 300, 5), n)
    M, d = len(uv), 2
    off = np.array([0, M // 2, M])
    plan = R.Plan(n, uv, off)
    plan.set_dde(synth.dde_taps(M, 3, rng, strength=0.3))
    y = torch.tensor(rng.standard_normal(M) + 1j * rng.standard_normal(M), dtype=torch.complex64, device="cuda")
    prm = opd.default_params(3.0, 1e4)
    sols = [R.PD(plan, R.Sara(n), y, np.full(d, 1.0), prm.tau, prm.sigma, prm.varsigma, prm.kappa, 3.0, 1e4)
            for _ in range(2)]
    for t in range(12):
        mask = np.array([t % 3 != 1, t % 4 != 2], np.uint8)
        sols[0].step(torch.tensor(mask, device="cuda"))
        sols[1].step_plain(mask)
    for which in (0, 3):
        a, b = (s.get(which).cpu().numpy() for s in sols)
        assert np.linalg.norm(b) > 0 and rel_l2(a, b) < TOL
