"""Staging of the filter banks' tiles, where it can go wrong: the smallest images and the deepest
levels (every row and column wraps), one filter length at a time and all of them, and buffers that
are aligned to one float only.  Psi^dagger and Psi against the oracle's filter banks: FP32 sums of
at most 256 products a level, relative l2 <= 1e-6 a level."""
import numpy as np
import pytest
import torch

from helpers import rel_l2
from oracle.wavelets import Sara as OSara

pytestmark = pytest.mark.gpu


def _shifted(a):
    """A contiguous copy of a that starts one float after an aligned address."""
    buf = torch.empty(a.numel() + 1, dtype=torch.float32, device="cuda")
    out = buf[1:].view(a.shape)
    out.copy_(a)
    return out


@pytest.mark.parametrize("n,levels,wavelets", [(4, 1, range(1, 9)), (4, 2, (8,)), (16, 4, range(1, 9)), (64, 6, (1, 7)),
                                               (64, 1, (2,)), (128, 4, (3, 5)), (256, 2, (4, 6)), (1024, 3, (1, 2, 8))])
def test_filter_banks(n, levels, wavelets):
    import paper_1610_08895_amd as R

    rng = np.random.default_rng(n + levels)
    osara = OSara(n, levels, wavelets=tuple(wavelets))
    sara = R.Sara(n, levels, bases=1 | sum(1 << w for w in wavelets))
    x = torch.tensor(rng.standard_normal((n, n)), dtype=torch.float32, device="cuda")
    s = sara.psi_adj(x)
    assert rel_l2(s.cpu().numpy(), osara.adj(x.double().cpu().numpy())) < 1e-6 * levels
    c = torch.tensor(rng.standard_normal(s.shape), dtype=torch.float32, device="cuda")
    y = sara.psi(c)
    assert rel_l2(y.cpu().numpy(), osara.fwd(c.double().cpu().numpy())) < 1e-6 * levels
    assert torch.equal(sara.psi_adj(_shifted(x), _shifted(s)), s)
    assert torch.equal(sara.psi(_shifted(c), _shifted(y)), y)
