"""Error of the DDE-aware Phi^dagger where many blocks' short items share a scale of the fixed-point
sums.  With N contributions' bounds in reach of a cell (a quarter of a group of 512) the rounding is
1.35e-9 N = 1.7e-7 of the result for random values; the kernel's fit (2e-7), the packed coordinates (2e-7),
the FP32 weights and passes of the inverse transform (2e-7 together) come on top: 9e-7 when all add up,
where a scale from the bounds of a whole group leaves 1.3e-6."""
import numpy as np
import pytest
import torch

import synth
from helpers import rel_l2, to_plan
from oracle.dde import DDEMeasurement
from oracle.measurement import Measurement

pytestmark = pytest.mark.gpu
TOL = 9e-7


@pytest.mark.parametrize("d,jd,tile", [(1, 5, 32), (64, 5, 32), (200, 5, 32), (64, 3, 16), (64, 7, 64)])
def test_short_items_keep_their_bits(d, jd, tile):
    import paper_1610_08895_amd as R

    n, M = 128, 60000
    rng = np.random.default_rng(d + jd)
    uv = synth.uv_coverage(M, rng).astype(np.float32)  # every block over the whole plane
    off = np.linspace(0, M, d + 1).astype(np.int64)
    taps = synth.dde_taps(M, jd, rng, strength=0.3).astype(np.complex64)
    plan = R.Plan(n, uv, off, tile=tile)
    plan.set_dde(taps)
    dm = DDEMeasurement(Measurement(uv, off, (n, n)), taps)
    w = (rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(np.complex64)
    wt = torch.tensor(to_plan(w, plan.order()), device="cuda")
    assert rel_l2(plan.phi_adj(wt).cpu().numpy(), dm.phi_adj_real(w.astype(np.complex128))) < TOL
    mask = (np.arange(d) % 3 != 1).astype(np.uint8)
    xm = plan.phi_adj(wt, mask=torch.tensor(mask, device="cuda")).cpu().numpy()
    assert rel_l2(xm, dm.phi_adj_real(w.astype(np.complex128), blocks=np.flatnonzero(mask))) < TOL
