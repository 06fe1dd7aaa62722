"""Windows of the windowed gridding (grids of up to 1024 cells per axis) that hold tens of thousands of
visibilities: the error of Phi^dagger must not grow with their number.  Sums of equal and of equally
signed terms, where rounding errors add up instead of cancelling, and of random ones.  Tolerance, by
the worst case of each part relative to a sum of positive terms: a chunk's 32 multiply-adds 16 * 2^-24
= 1.0e-6, the compensated sum of the chunks and the four windows' and four wavefronts' patches 18 * 2^-24
= 1.1e-6, the kernel's fit 0.2e-6, the packed coordinate's phase at the image edge 0.8e-6, the passes of the
inverse transform about 0.5e-6: 4e-6 in all."""
import numpy as np
import pytest
import torch

from helpers import rel_l2, to_plan
from oracle.measurement import Measurement

pytestmark = pytest.mark.gpu
TOL = 4e-6


@pytest.mark.parametrize("n", [64, 256, 512])
@pytest.mark.parametrize("kind", ["equal", "ones", "random"])
def test_error_does_not_grow_with_a_windows_count(n, kind):
    import paper_1610_08895_amd as R

    K, N = 2 * n, 60000
    rng = np.random.default_rng(n)
    kap = 40 + rng.uniform(0.0, 8.0, (N, 2))  # one window of 8 x 8 cells
    if kind == "equal":
        kap[:] = kap[0]
    uv = (2 * np.pi * kap / K)
    uv = np.where(uv >= np.pi, uv - 2 * np.pi, uv).astype(np.float32)
    w = np.ones(N, np.complex64)
    if kind == "random":
        w = (rng.standard_normal(N) + 1j * rng.standard_normal(N)).astype(np.complex64)
    off = np.array([0, 1000, N])
    plan = R.Plan(n, uv, off)
    meas = Measurement(uv, off, (n, n))
    wt = torch.tensor(to_plan(w, plan.order()), device="cuda")
    w = w.astype(np.complex128)
    assert rel_l2(plan.phi_adj(wt).cpu().numpy(), meas.phi_adj_real(w)) < TOL
    mask = torch.tensor([0, 1], dtype=torch.uint8, device="cuda")
    assert rel_l2(plan.phi_adj(wt, mask=mask).cpu().numpy(), meas.phi_adj_real(w, blocks=[1])) < TOL
