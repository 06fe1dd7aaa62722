"""Tiled plans (grids of more than 1024 cells per axis) at few visibilities, where the gridding and
the merging of the tiles' reaches can go wrong: visibilities on both sides of every kind of tile
border (edges, corners, the wrapping ones), pairs of one cell, each tile side, dense tiles in one
unit and in slices, more blocks than a wavefront tests at once; Phi, Phi^dagger whole and masked
against the oracle, and the batched dual update's sum against the per-block one.  Tolerance: FP32
sums of the oracle's FP64 terms, relative l2 <= 1e-5 as for every operator."""
import numpy as np
import pytest
import torch

from helpers import problem, rel_l2, to_plan, to_user
from oracle import pd as opd
from oracle.measurement import Measurement

pytestmark = pytest.mark.gpu
TOL = 1e-5
N = 1024


def _borders(tile, rng):
    """Visibilities in every row and column of cells around a tile corner, the grid's corner and an
    edge's middle, some cells twice, and a dense cluster inside one tile."""
    K = 2 * N
    r = np.arange(-8, 8)
    gy, gx = (a.ravel() for a in np.meshgrid(r, r, indexing="ij"))
    local = np.stack([gy, gx], axis=1)
    at = [(5 * tile, 7 * tile), (0, 0), (K // 2, K // 2), (0, 9 * tile), (3 * tile + tile // 2, 0)]
    cells = np.concatenate([local + np.array(c) for c in at] + [np.repeat(local[:40] + 2 * tile + 8, 60, axis=0)])
    kap = np.mod(cells, K) + rng.uniform(0.0, 1.0, cells.shape)
    uv = 2 * np.pi * kap / K
    return np.where(uv >= np.pi, uv - 2 * np.pi, uv).astype(np.float32)[rng.permutation(len(cells))]


@pytest.mark.parametrize("tile,d,slice_vis", [(16, 3, 0), (32, 1, 0), (32, 5, 300), (64, 70, 0), (64, 2, 500)])
def test_tile_borders(tile, d, slice_vis):
    import paper_1610_08895_amd as R

    rng = np.random.default_rng(tile + d)
    uv = _borders(tile, rng)
    M = len(uv)
    off = np.linspace(0, M, d + 1).astype(np.int64)
    plan = R.Plan(N, uv, off, tile=tile, slice_vis=slice_vis)
    meas, order = Measurement(uv, off, (N, N)), plan.order()
    x = rng.uniform(0.0, 1.0, (N, N))
    y = to_user(plan.phi(torch.tensor(x, dtype=torch.float32, device="cuda")).cpu().numpy(), order)
    assert rel_l2(y, meas.phi(x)) < TOL
    w = rng.standard_normal(M) + 1j * rng.standard_normal(M)
    wt = torch.tensor(to_plan(w, order), dtype=torch.complex64, device="cuda")
    assert rel_l2(plan.phi_adj(wt).cpu().numpy(), meas.phi_adj_real(w)) < TOL
    mask = (np.arange(d) % 3 != 1).astype(np.uint8)
    xm = plan.phi_adj(wt, mask=torch.tensor(mask, device="cuda")).cpu().numpy()
    assert rel_l2(xm, meas.phi_adj_real(w, blocks=np.flatnonzero(mask))) < TOL


@pytest.mark.parametrize("slice_vis", [0, 300])
def test_batched_and_per_block_steps_agree(slice_vis):
    """x and v of 8 steps with changing masks, batched, per block, and batched without masks at
    first (the sum rebuilt): the same FP32 terms in another order, within 1e-5."""
    import paper_1610_08895_amd as R

    M, d = 20000, 4
    _, uv, off = problem(N, M, d, "lognormal", 5)
    rng = np.random.default_rng(6)
    plan = R.Plan(N, uv, off, slice_vis=slice_vis)
    y = torch.tensor(rng.standard_normal(M) + 1j * rng.standard_normal(M), dtype=torch.complex64, device="cuda")
    prm = opd.default_params(3.0, 200.0)
    pds = [R.PD(plan, R.Sara(N), y, np.full(d, 20.0), prm.tau, prm.sigma, prm.varsigma, prm.kappa, 3.0, 200.0)
           for _ in range(3)]
    for t in range(8):
        mask = np.ones(d, np.uint8) if t % 3 == 0 else (rng.uniform(size=d) < 0.6).astype(np.uint8)
        mk = torch.tensor(mask, device="cuda")
        pds[0].step(mk)
        pds[1].step_plain(mask)
        pds[2].step(None if mask.all() else mk)
    for which in (0, 3):
        a, b, c = (pd.get(which).cpu().numpy() for pd in pds)
        assert np.linalg.norm(a) > 0 and rel_l2(b, a) < TOL and rel_l2(c, a) < TOL, which
