"""The reverse sweep of one step on small problems, where the wavelets' kernels ride on those of the
measurement operator, against the same sweep with a launch per stage (a plan whose direction-
dependent effects are the identity takes that route): over the sizes and levels around the rule's
edges, fewer bases, weights, inactive blocks and blocks inside their ball.  Both routes sum the same
FP32 terms in another order: relative l2 <= 1e-5, as for the operators they are made of."""
import numpy as np
import pytest
import torch

from helpers import problem

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("n,levels,bases", [(16, 4, 0), (32, 2, 0), (64, 4, 0b100010010), (64, 1, 0), (128, 4, 0),
                                            (128, 2, 0b110), (64, 3, 0b1), (256, 4, 0)])
@pytest.mark.parametrize("weighted", [False, True])
def test_reverse_sweep_routes_agree(n, levels, bases, weighted):
    import paper_1610_08895_amd as R

    M, d = 9000, 4
    x, uv, off = problem(n, M, d, "lognormal", n + levels)
    sara = R.Sara(n, levels, bases)
    g = torch.Generator(device="cuda").manual_seed(n + levels)

    def rand(*shape, dtype=torch.float32):
        return torch.randn(*shape, dtype=dtype, device="cuda", generator=g)

    y, v, r = (rand(M, dtype=torch.complex64) for _ in range(3))
    x_new, s_new = rand(n, n), 3e-3 * rand(sara.b, n, n)
    bars = [rand(n, n), rand(n, n), rand(sara.b, n, n), rand(M, dtype=torch.complex64)]
    w = torch.rand(sara.b, n, n, device="cuda", generator=g) + 0.1
    mask = torch.tensor([1, 0, 1, 1], dtype=torch.uint8, device="cuda")
    stats = torch.tensor([[4.0, 1.0], [9.0, 1.0], [1.0, 1.0], [100.0, 1.0]], dtype=torch.float64, device="cuda")
    out = []
    for dde in (None, np.ones((M, 1, 1), np.complex64)):
        plan = R.Plan(n, uv, off)
        plan.set_dde(dde)
        pd = R.PD(plan, sara, y, np.full(d, 1.5), 0.49, 1.0 / 9.0, 1e-4, 3e-3, 3.0, 60.0)
        if weighted:
            pd.set(6, w)
        b, pgrad = [t.clone() for t in bars], torch.zeros(2, dtype=torch.float64, device="cuda")
        for _ in range(2):
            pd.step_vjp(mask, x_new, s_new, v, r, stats, *b, pgrad)
        out.append([t.cpu().numpy() for t in b] + [pgrad.cpu().numpy()])
    for i, (a, b) in enumerate(zip(*out)):
        assert np.linalg.norm(b) > 0 and np.linalg.norm(a - b) <= TOL * np.linalg.norm(b), i
    assert 0 < np.count_nonzero(out[0][2]) < out[0][2].size  # the gate closes on some, not on all
