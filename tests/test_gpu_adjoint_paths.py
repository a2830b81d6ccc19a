"""The transform's adjoint on both sides of its choice between the full symmetric cotangent (up to 128
functions, or little work) and the rows of occupied orbitals and targets only.

Reference: C_bar = sum_K L^K C (Bbar^K + Bbar^K^T) by plain torch in FP64; bound as in the other
tests of the adjoint, 1e-12 of the sum of the absolute terms.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _reference(L, Cm, nocc, sel, gs, gv):
    n, nmo = Cm.shape
    nu, mu = np.tril_indices(n)
    out = torch.zeros_like(Cm)
    for k0 in range(0, L.shape[0], 200):
        f = torch.zeros((min(200, L.shape[0] - k0), n, n), dtype=torch.float64, device="cuda")
        f[:, nu, mu] = L[k0:k0 + 200]
        f[:, mu, nu] = L[k0:k0 + 200]
        b = torch.zeros((f.shape[0], nmo, nmo), dtype=torch.float64, device="cuda")
        b[:, nocc:, :nocc] = gv[:, k0:k0 + 200].T.reshape(-1, nmo - nocc, nocc)
        for s, q in enumerate(sel):
            b[:, q, :] += gs[s * nmo:(s + 1) * nmo, k0:k0 + 200].T
        b = b + b.transpose(1, 2)
        out += torch.matmul(f, torch.matmul(Cm, b)).sum(0)
    return out


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
@pytest.mark.parametrize("nbf,nmo,nocc,nvec,sel", [
    (128, 128, 64, 40, [63, 64, 63]), (128, 112, 1, 2100, [0, 111]), (129, 129, 1, 70, [0, 1, 128]),
    (129, 127, 126, 3, [126]), (144, 144, 100, 33, [99, 100]), (130, 128, 30, 600, [29, 30, 127]), (144, 144, 36, 700, [35]),
    (131, 48, 47, 8200, [46, 47]), (260, 257, 33, 90, list(range(20, 45)))])
def test_transform_adjoint_paths(dt, nbf, nmo, nocc, nvec, sel):
    import paper_0912_1459_amd.core as C
    g = torch.Generator(device="cuda").manual_seed(nbf)
    r = lambda *s: torch.randn(s, generator=g, dtype=torch.float64, device="cuda")
    L, Cm = r(nvec, nbf * (nbf + 1) // 2), r(nbf, nmo)
    gs, gv = r(len(sel) * nmo, nvec).to(dt), r((nmo - nocc) * nocc, nvec).to(dt)
    print("transform adjoint paths", dt, nbf, nmo, nocc, nvec, flush=True)
    out = C.transform_adjoint(L, nvec, Cm, nocc, sel, gs, gv, nvec)
    ref = _reference(L, Cm, nocc, sel, gs.double(), gv.double())
    mag = _reference(L.abs(), Cm.abs(), nocc, sel, gs.double().abs(), gv.double().abs())
    assert bool(((out - ref).abs() <= 1e-12 * mag).all())
    torch.cuda.empty_cache()
