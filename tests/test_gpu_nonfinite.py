"""Vanishing denominators and NaN blocks: infinities and NaN reach the outputs they belong to and no
others, and the statuses say so.

Every energy below is a multiple of 2^-20, so the denominators w + e_a - e_i - e_j are exact and one
of them is exactly zero at w = e_q.
"""
import numpy as np
import pytest
import torch

from paper_0912_1459_amd import _lib as A
from tests._blocks import blocks_from_numpy

pytestmark = pytest.mark.gpu

NOCC, NVIRT, NVEC = 12, 21, 19
I0, J0, A0 = 3, 8, 5                       # the pole of orbital 0: e_0 + e_a = e_i + e_j


def _energies():
    g = np.random.default_rng(2)
    grid = lambda lo, hi, n: np.sort(np.round(g.uniform(lo, hi, n) * 2 ** 20)) / 2 ** 20
    eo, ev = grid(-2.0, -0.6, NOCC), grid(0.5, 2.8, NVIRT)
    eo[0] = eo[I0] + eo[J0] - ev[A0]       # moves orbital 0 only
    return np.concatenate([eo, ev])


def _case(sel):
    g = np.random.default_rng(5)
    nmo = NOCC + NVIRT
    Bs = g.standard_normal((NVEC, len(sel), nmo)) * 0.02
    Bv = g.standard_normal((NVEC, NVIRT, NOCC)) * 0.02
    return Bs, Bv, _energies()


def _poles(e, w):
    """How many (a; i <= j) and (i; a <= b) denominators vanish at w."""
    eo, ev = e[:NOCC], e[NOCC:]
    dx = w + ev[:, None, None] - eo[None, :, None] - eo[None, None, :]
    dy = w + eo[:, None, None] - ev[None, :, None] - ev[None, None, :]
    return int((np.triu(dx == 0)).sum()), int((np.triu(dy == 0)).sum())


def test_the_pole_is_exact():
    e = _energies()
    assert _poles(e, e[0]) == (1, 0)
    assert all(_poles(e, e[q]) == (0, 0) for q in range(9, 14))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_sigma_and_solve_at_a_pole(prec):
    import paper_0912_1459_amd.core as C
    sel = [0, 11, 12]
    Bs, Bv, e = _case(sel)
    B = blocks_from_numpy(Bs, Bv, NOCC, sel, prec)
    eps = torch.tensor(e, device="cuda")
    print("pole", prec, flush=True)
    s, ds = C.sigma2(B, eps, e[sel][:, None])
    assert np.isinf(s[0]).all() and np.isneginf(ds[0]).all()
    assert np.isfinite(s[1:]).all() and np.isfinite(ds[1:]).all()
    for mode in ("residues", "recompute"):
        r = C.qp_solve(B, eps, mode=mode)
        assert r.status[0] == A.QP_NONFINITE and r.iters[0] == 1
        assert (r.status[1:] == 0).all() and np.isfinite(r.omega[1:]).all()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_adjoint_at_a_pole(prec):
    # dSigma/dw is -inf, so the pole strength is 0: everything is 0 but what meets the vanishing
    # denominator, which is 0 * inf
    import paper_0912_1459_amd.core as C
    Bs, Bv, e = _case([0])
    B = blocks_from_numpy(Bs, Bv, NOCC, [0], prec)
    print("adjoint at a pole", prec, flush=True)
    gs, gv, ge = C.qp_adjoint(B, torch.tensor(e, device="cuda"), e[:1], np.array([0.7]))
    gs = gs.cpu().numpy().reshape(NOCC + NVIRT, B.ldk)[:, :NVEC]
    gv = gv.cpu().numpy().reshape(NVIRT, NOCC, B.ldk)[:, :, :NVEC]
    ge = ge.cpu().numpy()
    ms, mv, me = np.zeros(gs.shape, bool), np.zeros(gv.shape, bool), np.zeros(ge.shape, bool)
    ms[[I0, J0]] = True
    mv[A0, [I0, J0]] = True
    me[[I0, J0, NOCC + A0]] = True
    for x, m in ((gs, ms), (gv, mv), (ge, me)):
        assert np.isnan(x[m]).all() and (x[~m] == 0).all()


def _dyson(Bs, Bv, e, sel, prec="fp64"):
    import paper_0912_1459_amd.core as C
    return C.dyson_solve(blocks_from_numpy(Bs, Bv, NOCC, sel, prec), torch.tensor(e, device="cuda"))


def test_dyson_at_a_pole():
    # every entry of root 0's matrix is infinite: it is not diagonalised and the root keeps its vector
    sel = [0, 11, 12]
    Bs, Bv, e = _case(sel)
    print("dyson pole", flush=True)
    r = _dyson(Bs, Bv, e, sel)
    assert r.status[0] == A.QP_NONFINITE and r.iters[0] == 1 and not np.isfinite(r.omega[0])
    assert (r.vec[0] == [1.0, 0.0, 0.0]).all()
    assert (r.status[1:] == 0).all() and np.isfinite(r.vec[1:]).all()


@pytest.mark.parametrize("what", ["nan block", "zero block at a pole"])
@pytest.mark.parametrize("nsel", [2, 3, 6])
def test_dyson_nan_matrix_gives_nan_vectors(what, nsel):
    # a NaN in the matrix (from the blocks, or 0 * inf: an orbital without integrals, at another's
    # pole) makes the root's energy, pole strength and vector NaN
    sel = [0, 11, 12, 13, 10, 9][:nsel]
    Bs, Bv, e = _case(sel)
    if what == "nan block":
        Bs[2, nsel - 1, :] = np.nan
    else:
        Bs[:, nsel - 1, :] = 0.0
    print("dyson", what, nsel, flush=True)
    r = _dyson(Bs, Bv, e, sel)
    bad = np.arange(nsel) if what == "nan block" else np.array([0])
    assert (r.status[bad] == A.QP_NONFINITE).all() and (r.iters[bad] == 1).all()
    assert np.isnan(r.omega[bad]).all() and np.isnan(r.pole[bad]).all()
    assert np.isnan(r.vec[bad]).all()
    good = np.setdiff1d(np.arange(nsel), bad)
    assert (r.status[good] == 0).all() and np.isfinite(r.vec[good]).all()
