"""Slices and same-cell pairs of tiled plans (grids of more than 1024 cells per axis, the ones whose tiles
are sliced and whose visibilities are paired): iterations of Algorithm 1 with sliced tiles, masked and
rebuilt, and Eq. 13 at x against the oracle, slices down to one visibility, and pairs in items of each
kind (both slot pairs, one, none).  Tolerances: the iterates' relative error grows by at most 1e-5 a step
and the operators' is at most 1e-5, as everywhere."""
import numpy as np
import pytest
import torch

import synth
from helpers import rel_l2, to_plan, to_user
from oracle import pd as opd
from oracle.measurement import Measurement
from oracle.wavelets import Sara as OSara

pytestmark = pytest.mark.gpu
N = 1024
TOL = 1e-5


@pytest.fixture(scope="module")
def R():
    import paper_1610_08895_amd as R

    assert torch.cuda.is_available()
    return R


def _dense(R, M, d, seed, **tune):
    """Blocks over a Gaussian of 32 cells: a few tiles of thousands of visibilities each."""
    rng = np.random.default_rng(seed)
    x = synth.sky(N, 5, 10, rng)
    uv = synth.uv_coverage(M, rng, sigma=np.pi / 32)
    uv, off, _ = synth.partition(uv, d, "lognormal", rng)
    meas = Measurement(uv, off, (N, N))
    y = meas.phi(x)
    sig = synth.noise_sigma(y, 20.0)
    y = y + synth.complex_noise(M, sig, rng)
    plan = R.Plan(N, uv, off, **tune)
    phin = 1.1 * plan.norm(torch.tensor(rng.standard_normal((N, N)), dtype=torch.float32, device="cuda"), 30, 0.0)[0]
    return dict(x=x, off=off, meas=meas, y=y, eps=synth.l2_ball_radii(off, sig), plan=plan, phin=phin,
                order=plan.order(), rng=rng, prm=opd.default_params(3.0, phin),
                y_plan=torch.tensor(to_plan(y, plan.order()), dtype=torch.complex64, device="cuda"))


def _pd(R, S):
    p = S["prm"]
    return R.PD(S["plan"], R.Sara(N), S["y_plan"], S["eps"], p.tau, p.sigma, p.varsigma, p.kappa, 3.0, S["phin"])


def test_iterations_with_slices_match_oracle(R):
    d = 4
    S = _dense(R, 20000, d, 3, slice_vis=300, bin=64)
    pds = [_pd(R, S) for _ in range(2)]  # all-ones masks as masks, and as the rebuilt sum
    yb, osara = opd.split_blocks(S["meas"], S["y"]), OSara(N)
    st = opd.init_state(S["meas"], osara)
    for t in range(4):
        mask = np.ones(d, np.uint8) if t % 2 == 0 else np.array([1, 0, 1, 0], np.uint8)
        opd.iteration(S["meas"], osara, yb, S["eps"], S["prm"], st, mask.astype(bool))
        mk = torch.tensor(mask, device="cuda")
        pds[0].step(mk)
        pds[1].step(None if mask.all() else mk)
        vo = np.concatenate(st.v)
        for pd in pds:
            for which, ref in ((0, st.x), (1, st.xt), (2, st.s)):
                assert rel_l2(pd.get(which).cpu().numpy(), ref) < TOL * (1 + t), (t, which)
            assert rel_l2(to_user(pd.get(3).cpu().numpy(), S["order"]), vo) < TOL * (1 + t), t
    assert np.linalg.norm(vo) > 0


def test_residual_at_x_with_slices(R):
    S = _dense(R, 20000, 5, 17, slice_vis=300, bin=64)
    pd = _pd(R, S)
    x = np.abs(S["x"]).astype(np.float32)
    pd.set(0, torch.tensor(x, device="cuda"))
    ref = opd.residual_norms(S["meas"], x.astype(np.float64), opd.split_blocks(S["meas"], S["y"]))
    assert np.allclose(pd.residual().cpu().numpy()[:, 1], ref ** 2, rtol=1e-4)


def _check_adjoint(plan, meas, off, rng, mask):
    w = rng.standard_normal(int(off[-1])) + 1j * rng.standard_normal(int(off[-1]))
    wt = torch.tensor(to_plan(w, plan.order()), dtype=torch.complex64, device="cuda")
    for _ in range(2):  # slice patches are rewritten by every launch
        assert rel_l2(plan.phi_adj(wt).cpu().numpy(), meas.phi_adj_real(w)) < TOL
        xm = plan.phi_adj(wt, mask=torch.tensor(mask, device="cuda")).cpu().numpy()
        assert rel_l2(xm, meas.phi_adj_real(w, blocks=np.flatnonzero(mask))) < TOL


@pytest.mark.parametrize("slice_vis,bin", [(1, 1), (100, 64), (-1, 64)])
def test_slices_down_to_one_visibility(R, slice_vis, bin):
    rng = np.random.default_rng(7)
    uv = synth.uv_coverage(1500, rng, sigma=np.pi / 64)
    uv, off, _ = synth.partition(uv, 4, "annuli")
    mask = np.ones(len(off) - 1, np.uint8)
    mask[1] = 0
    _check_adjoint(R.Plan(N, uv, off, slice_vis=slice_vis, bin=bin), Measurement(uv, off, (N, N)), off, rng, mask)


@pytest.mark.parametrize("bin", [1024, 600, 320, 64])
def test_same_cell_pairs(R, bin):
    """One to sixteen visibilities to a cell, in blocks of whole runs of cells and one of a visibility."""
    rng = np.random.default_rng(77 + bin)
    cells = rng.integers(0, 40, (700, 2))
    counts = rng.integers(1, 17, 700)
    M = int(counts.sum())
    uv = (2 * np.pi * (np.repeat(cells, counts, axis=0) + rng.uniform(0.0, 1.0, (M, 2))) / (2 * N)).astype(np.float32)
    off = np.array([0, 1, 900, 2100, M])
    plan, meas = R.Plan(N, uv, off, bin=bin), Measurement(uv, off, (N, N))
    x = synth.sky(N, 5, 10, rng)
    y = to_user(plan.phi(torch.tensor(x, dtype=torch.float32, device="cuda")).cpu().numpy(), plan.order())
    assert rel_l2(y, meas.phi(x)) < TOL
    _check_adjoint(plan, meas, off, rng, np.array([1, 0, 1, 1], np.uint8))
