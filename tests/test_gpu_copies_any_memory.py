"""ri_pd_get and ri_pd_set with buffers that a kernel cannot reach or address by floats: host memory the
GPU does not map, pinned host memory, device memory at an odd byte; and under graph capture.  Bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pd():
    import paper_1610_08895_amd as R

    n, M = 32, 1001
    rng = np.random.default_rng(1)
    uv = rng.uniform(-np.pi, np.pi, (M, 2)).astype(np.float32)
    y = torch.tensor(rng.standard_normal(M) + 1j * rng.standard_normal(M), dtype=torch.complex64, device="cuda")
    pd = R.PD(R.Plan(n, uv, [0, 400, M]), R.Sara(n), y, np.ones(2), 0.49, 1.0 / 9.0, 1e-6, 1e-3, 3.0, 100.0)
    pd.step()
    return pd


def _buffer(kind, nbytes):
    """(address, function returning the bytes, function storing bytes, object to keep)."""
    if kind == "pageable":
        b = np.zeros(nbytes, np.uint8)
        return b.ctypes.data, lambda: b.copy(), lambda v: b.__setitem__(slice(None), v), b
    if kind == "pinned":
        t = torch.zeros(nbytes, dtype=torch.uint8, pin_memory=True)
        return t.data_ptr(), lambda: t.numpy().copy(), lambda v: t.copy_(torch.from_numpy(v)), t
    t = torch.zeros(nbytes + 3, dtype=torch.uint8, device="cuda")[3:]
    return t.data_ptr(), lambda: t.cpu().numpy(), lambda v: t.copy_(torch.from_numpy(v)), t


@pytest.mark.parametrize("kind", ["pageable", "pinned", "odd"])
@pytest.mark.parametrize("which", [0, 2, 3])
def test_get_and_set(pd, kind, which):
    from paper_1610_08895_amd import _lib as L

    lib, stream = L.load(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ref = pd.get(which)
    want = torch.view_as_real(ref).cpu().numpy() if ref.is_complex() else ref.cpu().numpy()
    want = np.ascontiguousarray(want).view(np.uint8).ravel()
    addr, read, write, keep = _buffer(kind, want.size)
    L.check(lib.ri_pd_get(pd._h, which, addr, want.size, stream))
    torch.cuda.synchronize()
    assert np.array_equal(read(), want)
    other = np.random.default_rng(which).standard_normal(want.size // 4).astype(np.float32).view(np.uint8)
    write(other)
    L.check(lib.ri_pd_set(pd._h, which, addr, want.size, stream))
    torch.cuda.synchronize()
    back = pd.get(which)
    back = torch.view_as_real(back) if back.is_complex() else back
    assert np.array_equal(back.cpu().numpy().view(np.uint8).ravel(), other)
    pd.set(which, ref)


def test_get_under_capture(pd):
    out = torch.zeros_like(pd.get(0))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        pd.get(0, out)
    torch.cuda.current_stream().wait_stream(s)
    for k in range(3):
        pd.step()
        g.replay()
        assert torch.equal(out, pd.get(0))
        out.zero_()
