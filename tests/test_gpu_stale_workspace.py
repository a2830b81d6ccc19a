"""A call's results do not depend on what earlier calls of the same context left in its workspaces."""
import numpy as np
import pytest
import torch

from oracle import selfenergy as SE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbf,nmo,nocc,nvec,sel", [
    (2, 2, 1, 1, [0]), (17, 16, 15, 3, [14, 15]), (33, 31, 5, 70, [4, 5, 30]), (130, 129, 33, 50, [32, 33])])
def test_transform_adjoint_after_nan_coefficients(nbf, nmo, nocc, nvec, sel):
    # a transform of 200 orbitals whose coefficients are all NaN fills the coefficient workspace with
    # NaN; the adjoint's padding (rows nbf .. of its coefficient copy) must not read it.  Bound as in
    # the other tests of the adjoint: 1e-12 of the sum of the absolute terms.
    import paper_0912_1459_amd.core as C
    g = np.random.default_rng(nbf)
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x)).to(device="cuda", dtype=torch.float64)
    ctx = C.Context(0)
    print("adjoint after NaN coefficients", nbf, nmo, nocc, nvec, flush=True)
    nan = torch.full((200, 200), float("nan"), dtype=torch.float64, device="cuda")
    C.transform(dev(g.standard_normal((2, 200 * 201 // 2))), 2, nan, 80, np.arange(80, 90), "fp64", ctx=ctx)
    np_ = nbf * (nbf + 1) // 2
    L, Cm = g.standard_normal((np_, nvec)), g.standard_normal((nbf, nmo))
    gs, gv = g.standard_normal((nvec, len(sel), nmo)), g.standard_normal((nvec, nmo - nocc, nocc))
    Ld = torch.zeros((nvec + 1, np_), dtype=torch.float64, device="cuda")     # one row more: the row stride is np_
    Ld[:nvec] = dev(L.T)
    out = C.transform_adjoint(Ld[:nvec], nvec, dev(Cm), nocc, sel, dev(gs.reshape(nvec, -1).T),
                              dev(gv.reshape(nvec, -1).T), nvec, ctx=ctx).cpu().numpy()
    ref = SE.transform_adjoint(L, Cm, nocc, sel, gs, gv)
    mag = SE.transform_adjoint(np.abs(L), np.abs(Cm), nocc, sel, np.abs(gs), np.abs(gv))
    assert (np.abs(out - ref) <= 1e-12 * mag).all()
