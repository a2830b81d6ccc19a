"""The transform's products at the edges of their tiles: block counts that deal to the waves in
2 x 4 parts, in row strips and in column strips, K padding, batches, and blocks stored by the
products themselves (several batches of vectors, scattered and repeated targets).

Reference: C^T L^K C in FP64 by plain torch.  Bound per element, relative to (|C|^T |L^K| |C|): two
products of at most n terms, each with a rounding of 2^-53 (FP64), 2^-24 (FP32), or 2^-24 and
3 2^-18 for the split operands (split bf16), doubled for the two stages; the split output adds
2^-16 of the value.
"""
import numpy as np
import pytest
import torch

from tests._blocks import as_float64

pytestmark = pytest.mark.gpu

U = {"fp64": lambda n: 2 * n * 2.0 ** -53, "fp32": lambda n: 2 * n * 2.0 ** -24 + 2.0 ** -23,
     "bf16x3": lambda n: 2 * (n * 2.0 ** -24 + 3 * 2.0 ** -18) + 2.0 ** -16}


def _square(L, n):
    nu, mu = np.tril_indices(n)
    f = torch.zeros((L.shape[0], n, n), dtype=torch.float64, device=L.device)
    f[:, nu, mu] = L
    f[:, mu, nu] = L
    return f


# (nbf, nmo, nocc, nvec, sel): n of one block, 15 and 17 rows, 130-row T (one block past a tile),
# tiles of 5 and 7 blocks, more vectors than a batch of the smallest shapes holds
CASES = [(2, 2, 1, 3, [0, 1]), (17, 16, 5, 70, [4, 15, 4]), (33, 33, 16, 9, [20, 3]),
         (131, 130, 120, 5, [125, 0, 129, 126, 127, 121, 122, 123, 124, 128]), (208, 200, 79, 4, [80, 81, 79, 7]),
         (70, 64, 3, 5000, [2, 3, 4])]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("nbf,nmo,nocc,nvec,sel", CASES)
def test_transform_edges(prec, nbf, nmo, nocc, nvec, sel):
    import paper_0912_1459_amd.core as C
    g = torch.Generator(device="cuda").manual_seed(nbf)
    np_ = nbf * (nbf + 1) // 2
    L = torch.randn((nvec, np_), generator=g, dtype=torch.float64, device="cuda")
    Cm = torch.randn((nbf, nmo), generator=g, dtype=torch.float64, device="cuda")
    print("transform edges", prec, nbf, nmo, nocc, nvec, flush=True)
    B = C.transform(L, nvec, Cm, nocc, sel, prec)
    bs, bv = as_float64(B)
    worst = 0.0
    for k0 in range(0, nvec, 500):
        full, mag = _square(L[k0:k0 + 500], nbf), _square(L[k0:k0 + 500].abs(), nbf)
        ref = torch.matmul(torch.matmul(Cm.T.contiguous(), full), Cm)
        bnd = U[prec](nbf) * torch.matmul(torch.matmul(Cm.abs().T.contiguous(), mag), Cm.abs())
        for s, q in enumerate(sel):
            d = (bs[s, :, k0:k0 + 500].T - ref[:, q, :]).abs()
            assert bool((d <= bnd[:, q, :]).all()), (prec, "sel", s)
        d = (bv[:, :, k0:k0 + 500].permute(2, 0, 1) - ref[:, nocc:, :nocc]).abs()
        assert bool((d <= bnd[:, nocc:, :nocc]).all()), (prec, "vo")
        worst = max(worst, float((d / bnd[:, nocc:, :nocc]).max()))
    assert bool((B.Bvo.reshape(-1, B.ldk)[:, nvec:] == 0).all())


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("nocc,nvirt,nvec", [(1, 1, 5), (3, 50, 70), (16, 9, 64), (37, 70, 33), (130, 9, 40)])
def test_mp2_edges(prec, nocc, nvirt, nvec):
    # tiles below the block diagonal are left out, whatever the size of a block against a tile.
    # E is quadratic in integrals whose relative error is that of the products (as in the
    # self-energy): 2 u sum of the absolute terms; 1e-12 of it in FP64
    import paper_0912_1459_amd.core as C
    from tests._blocks import blocks_from_numpy
    g = np.random.default_rng(nocc)
    Bv = g.standard_normal((nvec, nvirt, nocc)) * 0.3 / np.sqrt(nvec)
    Bs = g.standard_normal((nvec, 1, nocc + nvirt))
    eps = np.concatenate([np.sort(g.uniform(-1.5, -0.3, nocc)), np.sort(g.uniform(0.1, 3.0, nvirt))])
    B = blocks_from_numpy(Bs, Bv, nocc, [0], prec)
    print("mp2 edges", prec, nocc, nvirt, flush=True)
    e = C.mp2_energy(B, torch.tensor(eps, device="cuda"))
    bv = as_float64(B)[1].reshape(nvirt * nocc, nvec).cpu()
    u = {"fp64": 1e-12, "fp32": 2 * nvec * 2.0 ** -24, "bf16x3": 2 * (nvec * 2.0 ** -24 + 3 * 2.0 ** -18)}[prec]

    def energy(b):
        x = (b @ b.T).reshape(nvirt, nocc, nvirt, nocc)
        eo, ev = torch.tensor(eps[:nocc]), torch.tensor(eps[nocc:])
        d = eo[None, :, None, None] + eo[None, None, None, :] - ev[:, None, None, None] - ev[None, None, :, None]
        return float(((2 * x - x.permute(0, 3, 2, 1)) * x / d).sum()), float((3 * x * x / d).sum())

    ref, bound = energy(bv)[0], abs(energy(bv.abs())[1])
    assert abs(e - ref) <= u * bound
