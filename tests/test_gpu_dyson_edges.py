"""Self-energy matrices at the edges of the pair blocks and element chunks: 1 to 31 orbitals, one to
20 energies per call, tiles of 8 occupied orbitals and chunks of 64 elements cut off anywhere.

Reference: the same blocks contracted in FP64 by plain torch.  FP64: 1e-12 of the sum of absolute
terms; FP32 and split bf16: the integrals' product error (nvec 2^-24, split bf16 3 2^-18 more, of
sum_K |B||B| each), the sum being quadratic in them: twice that.
"""
import numpy as np
import pytest
import torch

from tests._blocks import as_float64, blocks_from_numpy

pytestmark = pytest.mark.gpu


def _matrix(bs, bv, eps, nocc, w):
    n, nmo = bs.shape[0], bs.shape[1]
    G = torch.matmul(bs.reshape(n * nmo, -1), bv.reshape(-1, bv.shape[-1]).T).reshape(n, nmo, nmo - nocc, nocc)
    eo, ev = eps[:nocc], eps[nocc:]
    out, mag = [], []
    for p in (1, 2):
        s = m = 0.0
        for z, d in ((G[:, :nocc].transpose(1, 2), ev[:, None, None] - eo[None, :, None] - eo[None, None, :]),
                     (G[:, nocc:].permute(0, 3, 1, 2), eo[:, None, None] - ev[None, :, None] - ev[None, None, :])):
            zw = (z / (w + d) ** p).reshape(n, -1)
            num = (2 * z - z.transpose(2, 3)).reshape(n, -1)
            s = s + (zw @ num.T.contiguous()) * (1 if p == 1 else -1)
            m = m + zw.abs() @ (2 * z.abs() + z.abs().transpose(2, 3)).reshape(n, -1).T.contiguous()
        out.append(s)
        mag.append(m)
    return out, mag


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("nocc,nvirt,nvec,nsel,T", [
    (1, 1, 3, 1, 1), (7, 9, 17, 2, 8), (9, 23, 33, 6, 9), (65, 3, 40, 17, 20), (8, 64, 64, 31, 16), (10, 30, 20, 12, 3)])
def test_sigma_matrix_edges(prec, nocc, nvirt, nvec, nsel, T):
    import paper_0912_1459_amd.core as C
    g = np.random.default_rng(nocc + nvirt)
    nmo = nocc + nvirt
    sc = 0.3 / np.sqrt(nvec)
    B = blocks_from_numpy(g.standard_normal((nvec, nsel, nmo)) * sc, g.standard_normal((nvec, nvirt, nocc)) * sc, nocc,
                          np.arange(nsel) % nmo, prec)
    eps = torch.tensor(np.concatenate([np.sort(g.uniform(-1.5, -0.3, nocc)), np.sort(g.uniform(0.1, 3.0, nvirt))]),
                       device="cuda")
    om = np.linspace(-0.25, 0.05, T)
    print("sigma matrix edges", prec, nocc, nvirt, nsel, T, flush=True)
    s, ds = C.sigma2_matrix(B, eps, om)
    bs, bv = as_float64(B)
    u = {"fp64": 1e-12, "fp32": 2 * nvec * 2.0 ** -24, "bf16x3": 2 * (nvec * 2.0 ** -24 + 3 * 2.0 ** -18)}[prec]
    for t in range(T):
        ref, _ = _matrix(bs, bv, eps, nocc, om[t])
        # magnitudes from absolute integrals (their product error is relative to those)
        _, mag = _matrix(bs.abs(), bv.abs(), eps, nocc, om[t])
        for got, r, m in ((s[t], ref[0], mag[0]), (ds[t], ref[1], mag[1])):
            m = (m + m.T).cpu().numpy()
            assert (np.abs(got - r.cpu().numpy()) <= u * m).all(), (prec, t)
            assert (got == got.T).all()


@pytest.mark.parametrize("nsel", [1, 2, 3, 16, 17, 31])
def test_dyson_step_equals_host_diagonalisation(nsel):
    # one step of every root from e_q with the unit vector: the matrix at e_q diagonalised by LAPACK.
    # Both are backward stable; eigenvectors move by (rounding)/(gap), so the bar is 1e-13 / gap.
    import paper_0912_1459_amd.core as C
    g = np.random.default_rng(nsel)
    nocc, nvirt, nvec = 20, 24, 30
    nmo = nocc + nvirt
    B = blocks_from_numpy(g.standard_normal((nvec, nsel, nmo)) * 0.02, g.standard_normal((nvec, nvirt, nocc)) * 0.02, nocc,
                          np.arange(4, 4 + nsel), "fp64")
    e = np.concatenate([np.sort(g.uniform(-1.5, -0.3, nocc)), np.sort(g.uniform(0.1, 3.0, nvirt))])
    eps = torch.tensor(e, device="cuda")
    print("dyson step", nsel, flush=True)
    r = C.dyson_solve(B, eps, conv=1e-300, max_iter=1)
    sel = np.arange(4, 4 + nsel)
    s, ds = C.sigma2_matrix(B, eps, e[sel])
    for k in range(nsel):
        lam, V = np.linalg.eigh(np.diag(e[sel]) + s[k])
        j = int(np.argmax(np.abs(V[k])))
        u = V[:, j] * np.sign(V[k, j])
        gap = np.abs(np.delete(lam, j) - lam[j]).min() if nsel > 1 else 1.0
        tol = 1e-13 / gap
        assert np.abs(r.vec[k] - u).max() <= tol
        P = 1.0 / (1.0 - u @ ds[k] @ u)
        assert abs(r.pole[k] - P) <= 10 * tol * max(1.0, np.abs(ds[k]).max())
        assert abs(r.omega[k] - (e[sel[k]] + (lam[j] - e[sel[k]]) * P)) <= 10 * tol * max(1.0, np.abs(ds[k]).max())
    assert (r.iters == 1).all()
