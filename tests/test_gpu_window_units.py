"""Dense tiles of the windowed gridding, cut into several units: window counts around the share of a unit,
segments cut where a part ends, parts without visibilities, parts of whole blocks and slice_vis down to
one visibility; Phi^dagger whole and masked against the oracle, twice (the parts' regions are rewritten
by every launch), and the running sum of the batched steps against the per-block ones, whose units are
not cut.  Tolerance: FP32 sums of the oracle's FP64 terms, relative l2 <= 1e-5 as for every operator."""
import numpy as np
import pytest
import torch

from helpers import rel_l2, to_plan
from oracle.measurement import Measurement

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _uv(n, counts, rng):
    """counts[i] visibilities in the i-th of a few windows (grid corner, wrapping edges, inner), shuffled."""
    K = 2 * n
    cells = np.array([[0, 0], [K - 8, K - 8], [K // 2, 8], [K // 2, 0]])
    kap = np.concatenate([cells[i % 4] + rng.uniform(0.0, 8.0, (c, 2)) for i, c in enumerate(counts)])
    uv = 2 * np.pi * kap / K
    return np.where(uv >= np.pi, uv - 2 * np.pi, uv).astype(np.float32)[rng.permutation(len(kap))]


def _check(plan, meas, off, rng):
    M, d = int(off[-1]), len(off) - 1
    w = rng.standard_normal(M) + 1j * rng.standard_normal(M)
    wt = torch.tensor(to_plan(w, plan.order()), dtype=torch.complex64, device="cuda")
    mask = (np.arange(d) % 3 != 1).astype(np.uint8)
    for _ in range(2):
        assert rel_l2(plan.phi_adj(wt).cpu().numpy(), meas.phi_adj_real(w)) < TOL
        xm = plan.phi_adj(wt, mask=torch.tensor(mask, device="cuda")).cpu().numpy()
        assert rel_l2(xm, meas.phi_adj_real(w, blocks=np.flatnonzero(mask))) < TOL
    none = plan.phi_adj(wt, mask=torch.zeros(d, dtype=torch.uint8, device="cuda"))
    assert not none.any()


@pytest.mark.parametrize("n,counts,d", [(64, (2047, 2048, 2049, 1), 3), (256, (4097, 6200, 40, 3), 70),
                                        (512, (1024, 1025, 9000, 2), 1), (512, (5000, 700, 1, 2049), 130)])
def test_parts_of_dense_windows(n, counts, d):
    import paper_1610_08895_amd as R

    rng = np.random.default_rng(n + d)
    uv = _uv(n, counts, rng)
    off = np.linspace(0, len(uv), d + 1).astype(np.int64)
    _check(R.Plan(n, uv, off), Measurement(uv, off, (n, n)), off, rng)


@pytest.mark.parametrize("n", [64, 512])
@pytest.mark.parametrize("slice_vis,bin", [(1, 1), (7, 16), (100, 64), (300, 0)])
def test_slices(n, slice_vis, bin):
    import paper_1610_08895_amd as R

    rng = np.random.default_rng(slice_vis)
    uv, d = _uv(n, (900, 1, 333, 64), rng), 5
    off = np.linspace(0, len(uv), d + 1).astype(np.int64)
    _check(R.Plan(n, uv, off, slice_vis=slice_vis, bin=bin), Measurement(uv, off, (n, n)), off, rng)


@pytest.mark.parametrize("n,slice_vis", [(64, 0), (64, 200), (512, 0)])
def test_running_sum_with_parts(n, slice_vis):
    import paper_1610_08895_amd as R

    rng = np.random.default_rng(n)
    uv, d = _uv(n, (5000, 2500, 1100, 30), rng), 6
    M = len(uv)
    plan = R.Plan(n, uv, np.linspace(0, M, d + 1).astype(np.int64), slice_vis=slice_vis)
    y = torch.tensor(rng.standard_normal(M) + 1j * rng.standard_normal(M), dtype=torch.complex64, device="cuda")
    pds = [R.PD(plan, R.Sara(n), y, np.full(d, 5.0), 0.49, 1.0 / 9.0, 1e-6, 1e-3, 3.0, 300.0) for _ in range(3)]
    for t in range(8):
        mask = np.ones(d, np.uint8) if t % 3 == 0 else (rng.uniform(size=d) < 0.6).astype(np.uint8)
        mk = torch.tensor(mask, device="cuda")
        pds[0].step(mk)
        pds[1].step_plain(mask)
        pds[2].step(None if mask.all() else mk)
    for which in (0, 3):
        a, b, c = (pd.get(which).cpu().numpy() for pd in pds)
        assert np.linalg.norm(a) > 0 and rel_l2(b, a) < TOL and rel_l2(c, a) < TOL, which


def test_a_dense_window_is_not_one_wavefronts_work():
    """2^18 visibilities in one window of a 512^2 image: 6.3 ms as one wavefront's work, 0.1 ms cut into
    parts; the bound lies between, three times below the one and twenty above the other."""
    import paper_1610_08895_amd as R

    n, M = 512, 1 << 18
    rng = np.random.default_rng(0)
    uv = _uv(n, (M,), rng)
    plan = R.Plan(n, uv, [0, M])
    y = torch.ones(M, dtype=torch.complex64, device="cuda")
    x = plan.phi_adj(y)
    best = 1e9
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        plan.phi_adj(y, x)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    assert best < 2.0
