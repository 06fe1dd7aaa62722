"""Copies of the solver state and the permutation between user and plan order, bit for bit:
sizes around the permutation's chunks and their split over the XCDs, and destinations that are
not aligned to the copy kernel's 16-byte words."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_1610_08895_amd as R

    assert torch.cuda.is_available()
    return R


@pytest.mark.parametrize("M,d", [(1, 1), (1023, 3), (1025, 2), (8 * 1024, 5), (8 * 1024 + 1, 1), (70001, 9)])
def test_permute_is_the_plan_order_both_ways(R, M, d):
    rng = np.random.default_rng(M)
    uv = rng.uniform(-np.pi, np.pi, (M, 2)).astype(np.float32)
    plan = R.Plan(32, uv, np.linspace(0, M, d + 1).astype(np.int64))
    order = plan.order()
    y = (rng.standard_normal(M) + 1j * rng.standard_normal(M)).astype(np.complex64)
    t = torch.tensor(y, device="cuda")
    p = plan.permute(t)
    assert np.array_equal(p.cpu().numpy(), y[order])
    out = torch.full((M + 1,), 9j, dtype=torch.complex64, device="cuda")[1:]  # 8-byte aligned only
    assert np.array_equal(plan.permute(p, to_plan=False, out=out).cpu().numpy(), y)


@pytest.mark.parametrize("offset", [0, 1, 2, 4])
def test_state_copies_are_exact_at_any_alignment(R, offset):
    n, M = 32, 1001
    rng = np.random.default_rng(offset)
    uv = rng.uniform(-np.pi, np.pi, (M, 2)).astype(np.float32)
    plan = R.Plan(n, uv, [0, 400, M])
    y = torch.zeros(M, dtype=torch.complex64, device="cuda")
    pd = R.PD(plan, R.Sara(n), y, np.ones(2), 0.49, 1.0 / 9.0, 1e-6, 1e-3, 3.0, 100.0)

    def view(shape, dtype):
        words = 2 if dtype == torch.complex64 else 1
        cnt = int(np.prod(shape))
        buf = torch.full((cnt + offset,), 7.0, dtype=dtype, device="cuda")
        return buf, buf[offset:].view(*shape), words

    for which, shape, dtype in ((0, (n, n), torch.float32), (2, (9, n, n), torch.float32), (3, (M,), torch.complex64)):
        val = torch.tensor(rng.standard_normal(int(np.prod(shape))), device="cuda").to(dtype).view(*shape)
        buf, src, _ = view(shape, dtype)
        src.copy_(val)
        pd.set(which, src)
        buf2, dst, _ = view(shape, dtype)
        pd.get(which, dst)
        assert torch.equal(dst, val)
        assert torch.all(buf2[:offset] == 7.0)
