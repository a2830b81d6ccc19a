"""Adjoints at odd sizes: one occupied or one virtual orbital, sizes off every multiple of 16, one
vector, several batches of vectors, repeated and mixed targets, FP32 cotangents.

The transform's adjoint is a sum of products in FP64: 1e-12 of the sum of their absolute values
(n, nvec < 2^13).  The solve's adjoint is compared with the oracle's implicit gradient at the same
energies: FP64 as in test_gpu_adjoint (1e-9 of the largest entry), FP32 and split bf16 1e-4 and
1e-3 (norm), the scale of the products' rounding.
"""
import numpy as np
import pytest
import torch

from oracle import selfenergy as SE
from tests._blocks import as_float64, blocks_from_numpy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
@pytest.mark.parametrize("nbf,nmo,nocc,nvec,sel", [
    (2, 2, 1, 1, [0]), (17, 16, 15, 3, [14, 15, 14]), (33, 31, 1, 70, [0, 1, 30]), (130, 130, 37, 9, [36, 37, 5, 129, 37]),
    (65, 64, 20, 8200, [20])])
def test_transform_adjoint_edges(dt, nbf, nmo, nocc, nvec, sel):
    import paper_0912_1459_amd.core as C
    g = np.random.default_rng(nbf)
    np_ = nbf * (nbf + 1) // 2
    L, Cm = g.standard_normal((np_, nvec)), g.standard_normal((nbf, nmo))
    gs, gv = g.standard_normal((nvec, len(sel), nmo)), g.standard_normal((nvec, nmo - nocc, nocc))
    if dt == torch.float32:
        gs, gv = gs.astype(np.float32).astype(np.float64), gv.astype(np.float32).astype(np.float64)
    ldk = nvec + 5
    pad = lambda x, rows: np.pad(x.reshape(nvec, rows).T, ((0, 0), (0, 5)), constant_values=np.nan)
    dev = lambda x, t=torch.float64: torch.as_tensor(np.ascontiguousarray(x)).to(device="cuda", dtype=t)
    print("transform adjoint edges", dt, nbf, nmo, nocc, nvec, flush=True)
    Ld = torch.zeros((nvec + 1, np_), dtype=torch.float64, device="cuda")     # one row more: the row stride is np_
    Ld[:nvec] = dev(L.T)
    out = C.transform_adjoint(Ld[:nvec], nvec, dev(Cm), nocc, sel, dev(pad(gs, len(sel) * nmo), dt),
                              dev(pad(gv, (nmo - nocc) * nocc), dt), ldk).cpu().numpy()
    ref = SE.transform_adjoint(L, Cm, nocc, sel, gs, gv)
    mag = SE.transform_adjoint(np.abs(L), np.abs(Cm), nocc, sel, np.abs(gs), np.abs(gv))
    assert (np.abs(out - ref) <= 1e-12 * mag).all()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("nocc,nvirt,nvec,nsel,chunk", [
    (1, 1, 3, 2, 0), (5, 33, 17, 3, 2), (37, 21, 130, 4, 0), (130, 7, 40, 2, 1), (300, 4, 20, 2, 0), (16, 144, 64, 5, 0)])
def test_qp_adjoint_edges(prec, nocc, nvirt, nvec, nsel, chunk):
    import paper_0912_1459_amd.core as C
    g = np.random.default_rng(nocc + nvirt)
    nmo = nocc + nvirt
    sc = 0.3 / np.sqrt(nvec)
    B = blocks_from_numpy(g.standard_normal((nvec, nsel, nmo)) * sc, g.standard_normal((nvec, nvirt, nocc)) * sc, nocc,
                          np.arange(nsel) % nmo, prec)
    eps = np.concatenate([np.sort(g.uniform(-1.5, -0.3, nocc)), np.sort(g.uniform(0.1, 3.0, nvirt))])
    om, wbar = g.uniform(-0.2, 0.0, nsel), g.uniform(-1.0, 1.0, nsel)
    print("qp adjoint edges", prec, nocc, nvirt, nvec, flush=True)
    ctx = C.Context(0)
    ctx.set_target_chunk(chunk)
    gs, gv, ge = C.qp_adjoint(B, torch.tensor(eps, device="cuda"), om, wbar, ctx=ctx)
    bs, bv = (t.cpu().numpy() for t in as_float64(B))
    rs, rv, re = np.zeros_like(bs), np.zeros_like(bv), np.zeros(nmo)
    for s in range(nsel):
        q = SE.qp_gradient(np.ascontiguousarray(bs[s].T), np.ascontiguousarray(bv.transpose(2, 0, 1)), eps, nocc,
                           int(B.sel[s]), om[s])
        rs[s] = wbar[s] * q.Bsel_q.T
        rv += wbar[s] * q.Bvo.transpose(1, 2, 0)
        re += wbar[s] * q.eps
    gs = gs.double().cpu().numpy().reshape(nsel, nmo, B.ldk)
    gv = gv.double().cpu().numpy().reshape(nvirt, nocc, B.ldk)
    assert (gs[:, :, nvec:] == 0).all() and (gv[:, :, nvec:] == 0).all()
    ge = ge.cpu().numpy()
    if prec == "fp64":
        big = max(np.abs(rs).max(), np.abs(rv).max())
        assert np.abs(gs[:, :, :nvec] - rs).max() <= 1e-9 * big and np.abs(gv[:, :, :nvec] - rv).max() <= 1e-9 * big
        assert np.abs(ge - re).max() <= 1e-9 * max(1.0, np.abs(re).max())
    else:
        tol = 1e-4 if prec == "fp32" else 1e-3
        for x, r in ((gs[:, :, :nvec], rs), (gv[:, :, :nvec], rv), (ge, re)):
            assert np.linalg.norm(x - r) <= tol * np.linalg.norm(r)
