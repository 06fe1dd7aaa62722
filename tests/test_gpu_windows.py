"""Windowed plans (grids of up to 1024 cells per axis), where the gridding can go wrong: window
counts around a chunk of 32 and around the four wavefronts' share of it, more segments in a
window than a wavefront holds at once, windows on the grid's wrapping edges, each tile side,
and the largest windowed and the smallest tiled grid; Phi^dagger whole and masked, and the dual
update's sum (batched against per-block), against the oracle.  Tolerance: FP32 sums of the
oracle's FP64 terms, relative l2 <= 1e-5 as for every operator."""
import numpy as np
import pytest
import torch

import synth
from helpers import problem, rel_l2, to_plan, to_user
from oracle.measurement import Measurement

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def R():
    import paper_1610_08895_amd as R

    assert torch.cuda.is_available()
    return R


def _check(R, n, uv, off, tile=32, seed=0):
    rng = np.random.default_rng(seed)
    M, d = uv.shape[0], len(off) - 1
    plan = R.Plan(n, uv, off, tile=tile)
    order = plan.order()
    meas = Measurement(uv, off, (n, n))
    x = synth.sky(n, 5, 10, rng)
    y = to_user(plan.phi(torch.tensor(x, dtype=torch.float32, device="cuda")).cpu().numpy(), order)
    assert rel_l2(y, meas.phi(x)) < TOL
    w = rng.standard_normal(M) + 1j * rng.standard_normal(M)
    wt = torch.tensor(to_plan(w, order), dtype=torch.complex64, device="cuda")
    assert rel_l2(plan.phi_adj(wt).cpu().numpy(), meas.phi_adj_real(w)) < TOL
    mask = (np.arange(d) % 3 != 1).astype(np.uint8)
    xm = plan.phi_adj(wt, mask=torch.tensor(mask, device="cuda")).cpu().numpy()
    assert rel_l2(xm, meas.phi_adj_real(w, blocks=np.flatnonzero(mask))) < TOL


@pytest.mark.parametrize("n,tile", [(16, 16), (32, 32), (64, 64), (256, 16)])
@pytest.mark.parametrize("count", [1, 31, 32, 33, 127, 129, 600])
def test_window_counts(R, n, tile, count):
    """`count` visibilities in each of a few windows (corner, wrapping edge, inner), two blocks."""
    K = 2 * n
    rng = np.random.default_rng(1000 * n + count)
    cells = np.array([[0, 0], [K - 8, K - 8], [K // 2, 8], [K // 2 - 8, K // 2]])
    kap = np.repeat(cells, count, axis=0) + rng.uniform(0.0, 8.0, (4 * count, 2))
    uv = 2 * np.pi * kap / K
    uv = np.where(uv >= np.pi, uv - 2 * np.pi, uv).astype(np.float32)
    M = uv.shape[0]
    uv = uv[rng.permutation(M)]
    _check(R, n, uv, np.array([0, max(1, M // 3), M]), tile=tile, seed=count)


@pytest.mark.parametrize("d", [63, 64, 65, 130])
def test_many_segments_per_window(R, d):
    """Every block in the same few windows: a window has d segments of 1 to 5 visibilities."""
    n, K = 32, 64
    rng = np.random.default_rng(d)
    sizes = rng.integers(1, 6, d)
    M = int(sizes.sum())
    kap = rng.integers(0, 2, (M, 2)) * 8 + rng.uniform(0.0, 8.0, (M, 2))
    _check(R, n, (2 * np.pi * kap / K).astype(np.float32), np.concatenate([[0], np.cumsum(sizes)]), seed=d)


@pytest.mark.parametrize("n", [512, 1024])
def test_largest_windowed_and_smallest_tiled_grid(R, n):
    x, uv, off = problem(n, 60000, 5, "lognormal", 3, outliers=0.2)
    _check(R, n, uv, off, seed=n)


def test_running_sum_of_batched_and_plain_steps(R):
    """The same masked steps through the batched and the per-block gridding: x, v equal to 1e-5."""
    n, M, d = 64, 5000, 6
    x, uv, off = problem(n, M, d, "lognormal", 5)
    plan = R.Plan(n, uv, off)
    rng = np.random.default_rng(6)
    y = torch.tensor(rng.standard_normal(M) + 1j * rng.standard_normal(M), dtype=torch.complex64, device="cuda")
    pds = [R.PD(plan, R.Sara(n), y, np.full(d, 5.0), 0.49, 1.0 / 9.0, 1e-6, 1e-3, 3.0, 300.0) for _ in range(2)]
    for t in range(6):
        mask = (rng.uniform(size=d) < 0.6).astype(np.uint8)
        pds[0].step(torch.tensor(mask, device="cuda"))
        pds[1].step_plain(mask)
    for which in (0, 3):
        a, b = (p.get(which).cpu().numpy() for p in pds)
        assert rel_l2(a, b) < TOL
