"""Self-energies and Newton solves at the edges of the 128-row tiles:
one row, one short of a tile, exactly one, one more, and several trial energies per pass.

Reference: the same blocks (as the kernels read them) contracted in FP64 by plain torch.  FP64
sums of n positive and negative terms agree to about sqrt(n) 2^-53 of the sum of their absolute
values; 1e-12 of that sum covers every order of summation here (n < 2^24).  FP32 and split-bf16
integrals carry an FP32-accumulated product error of at most nvec 2^-24 of sum_K |B||B| each
(split bf16: 3 2^-18 more), and Sigma is quadratic in them: twice that, relative to the same sum
built from absolute values.
"""
import numpy as np
import pytest
import torch

from tests._blocks import as_float64, blocks_from_numpy

pytestmark = pytest.mark.gpu


def _case(nocc, nvirt, nvec, nsel, prec, seed=3):
    g = np.random.default_rng(seed)
    nmo = nocc + nvirt
    sc = 0.3 / np.sqrt(nvec)
    Bs = g.standard_normal((nvec, nsel, nmo)) * sc
    Bv = g.standard_normal((nvec, nvirt, nocc)) * sc
    eps = np.concatenate([np.sort(g.uniform(-1.5, -0.3, nocc)), np.sort(g.uniform(0.1, 3.0, nvirt))])
    sel = np.arange(nsel, dtype=np.int32) % nmo
    return blocks_from_numpy(Bs, Bv, nocc, sel, prec), eps


def _terms(bs, bv, eps, nocc):
    """(u, d): every term's numerator and energy-free denominator of both families of Eq. (SE)."""
    nmo = bs.shape[0]
    G = torch.matmul(bs, bv.reshape(-1, bv.shape[-1]).T).reshape(nmo, nmo - nocc, nocc)
    x, y = G[:nocc].transpose(0, 1), G[nocc:].permute(2, 0, 1)
    eo, ev = eps[:nocc], eps[nocc:]
    return ((2 * x - x.transpose(1, 2)) * x, ev[:, None, None] - eo[None, :, None] - eo[None, None, :],
            (2 * y - y.transpose(1, 2)) * y, eo[:, None, None] - ev[None, :, None] - ev[None, None, :])


SHAPES = [(1, 1, 17, 2, 1), (5, 127, 33, 3, 3), (128, 129, 70, 2, 9), (129, 20, 64, 2, 16), (16, 257, 40, 1, 4)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("nocc,nvirt,nvec,nsel,T", SHAPES)
def test_sigma_tile_edges(prec, nocc, nvirt, nvec, nsel, T):
    import paper_0912_1459_amd.core as C
    B, eps_h = _case(nocc, nvirt, nvec, nsel, prec)
    eps = torch.tensor(eps_h, device="cuda")
    om = np.linspace(-0.25, 0.05, nsel * T).reshape(nsel, T)
    print("sigma edges", prec, nocc, nvirt, nvec, T, flush=True)
    s, ds = C.sigma2(B, eps, om)
    bs, bv = as_float64(B)
    u = {"fp64": 1e-12, "fp32": 2 * nvec * 2.0 ** -24, "bf16x3": 2 * (nvec * 2.0 ** -24 + 3 * 2.0 ** -18)}[prec]
    for k in range(nsel):
        ux, dx, uy, dy = _terms(bs[k], bv, eps, nocc)
        ax, _, ay, _ = _terms(bs[k].abs(), bv.abs(), eps, nocc)
        # |2x - x'||x| <= 2 x^2 + |x'||x| with the absolute sums
        mx, my = 3 * ax.abs() + ax.abs().transpose(1, 2), 3 * ay.abs() + ay.abs().transpose(1, 2)
        for t in range(T):
            w = om[k, t]
            ref = float((ux / (w + dx)).sum() + (uy / (w + dy)).sum())
            dref = -float((ux / (w + dx) ** 2).sum() + (uy / (w + dy) ** 2).sum())
            b = float((mx / (w + dx).abs()).sum() + (my / (w + dy).abs()).sum())
            db = float((mx / (w + dx) ** 2).sum() + (my / (w + dy) ** 2).sum())
            assert abs(s[k, t] - ref) <= u * b and abs(ds[k, t] - dref) <= u * db, (prec, k, t, s[k, t] - ref, u * b)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("nocc,nvirt,nvec,nsel,T", SHAPES)
def test_residue_mode_equals_recompute(prec, nocc, nvirt, nvec, nsel, T):
    # one Newton step from stored residues and from recomputed integrals: the same sums, with the
    # residues rounded once to the blocks' precision (FP32: 2^-24 of sum |R / d| <= 1e-6 of it)
    import paper_0912_1459_amd.core as C
    B, eps_h = _case(nocc, nvirt, nvec, nsel, prec)
    eps = torch.tensor(eps_h, device="cuda")
    om = np.full(nsel, -0.1)
    print("residue edges", prec, nocc, nvirt, nvec, flush=True)
    a = C.qp_solve(B, eps, omega0=om, conv=0.0, max_iter=1, mode="residues")
    b = C.qp_solve(B, eps, omega0=om, conv=0.0, max_iter=1, mode="recompute")
    tol = 1e-12 if prec == "fp64" else 1e-6
    sig, _ = C.sigma2(B, eps, om[:, None])
    assert np.abs(a.omega - b.omega).max() <= tol * max(1.0, np.abs(sig).max())
    assert np.abs(a.pole - b.pole).max() <= tol
    c = C.qp_solve(B, eps, omega0=om, conv=0.0, max_iter=3, mode="residues")
    d = C.qp_solve(B, eps, omega0=om, conv=0.0, max_iter=3, mode="recompute")
    assert np.abs(c.omega - d.omega).max() <= 10 * tol * max(1.0, np.abs(sig).max())
