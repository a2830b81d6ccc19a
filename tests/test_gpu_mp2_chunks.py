"""MP2 energies whose integrals take several chunks of virtuals (4 GiB each at most), the last one short.

37 occupied, 901 virtuals: 33,337 rows, 8.9 GB of integrals in FP64 (chunks of 226, 226, 226 and 223
virtuals), 4.4 GB in FP32 and split bf16 (451 and 450).  Reference: the same blocks contracted in
FP64 by plain torch.  Bounds as for one chunk: E is quadratic in integrals whose relative error is
that of the products, 2 u of the sum of the absolute terms; 1e-12 of it in FP64.
"""
import numpy as np
import pytest
import torch

from tests._blocks import as_float64, blocks_from_numpy

pytestmark = pytest.mark.gpu


def _energy(b, eps, nocc, nvirt):
    eo, ev = eps[:nocc], eps[nocc:]
    e = m = 0.0
    for a0 in range(0, nvirt, 32):
        n = min(32, nvirt - a0)
        x = (b[a0 * nocc:(a0 + n) * nocc] @ b.T).reshape(n, nocc, nvirt, nocc)      # (ai|bj)
        d = eo[None, :, None, None] + eo[None, None, None, :] - ev[a0:a0 + n, None, None, None] - ev[None, None, :, None]
        y = x.permute(0, 3, 2, 1)                                                   # (aj|bi)
        e += float(((2 * x - y) * x / d).sum())
        m += float(((2 * x.abs() + y.abs()) * x.abs() / d.abs()).sum())
    return e, m


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_mp2_in_chunks(prec):
    import paper_0912_1459_amd.core as C
    nocc, nvirt, nvec = 37, 901, 20
    g = np.random.default_rng(9)
    Bv = g.standard_normal((nvec, nvirt, nocc)) * 0.05
    e = np.concatenate([np.sort(g.uniform(-1.5, -0.3, nocc)), np.sort(g.uniform(0.1, 3.0, nvirt))])
    B = blocks_from_numpy(g.standard_normal((nvec, 1, nocc + nvirt)), Bv, nocc, [0], prec)
    eps = torch.tensor(e, device="cuda")
    print("mp2 in chunks", prec, flush=True)
    with C.Context(0) as ctx:
        got = C.mp2_energy(B, eps, ctx=ctx)
    b = as_float64(B)[1].reshape(nvirt * nocc, nvec).contiguous()
    u = {"fp64": 1e-12, "fp32": 2 * nvec * 2.0 ** -24, "bf16x3": 2 * (nvec * 2.0 ** -24 + 3 * 2.0 ** -18)}[prec]
    ref, _ = _energy(b, eps, nocc, nvirt)
    _, mag = _energy(b.abs(), eps, nocc, nvirt)
    assert abs(got - ref) <= u * mag
