"""Calls whose work items pass the 2^32 threads of one launch dimension, or come near it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_sigma_of_more_tasks_than_one_launch_holds():
    # 128 occupied, 1024 virtuals, 1300 targets: 4,659,200 off-diagonal tile pairs of 1024 threads
    # each (2^32 threads are 4,194,304 of them); in chunks of 100 targets every launch is far below
    # the limit and each target's sums are the same
    import paper_0912_1459_amd.core as C
    from paper_0912_1459_amd import _lib as A
    nocc, nvirt, nsel, nvec = 128, 1024, 1300, 8
    nmo = nocc + nvirt
    g = torch.Generator(device="cuda").manual_seed(1)
    r = lambda n: torch.randn((n, nvec), generator=g, dtype=torch.float64, device="cuda") * 0.02
    B = C.BBlocks(A.PREC_FP64, r(nsel * nmo), r(nvirt * nocc), nvec, nvec, nmo, nocc,
                  (np.arange(nsel) % nmo).astype(np.int32))
    eps = torch.cat([torch.linspace(-1.5, -0.3, nocc, dtype=torch.float64), torch.linspace(0.1, 3.0, nvirt, dtype=torch.float64)])
    eps = eps.cuda()
    om = np.linspace(-0.2, 0.05, nsel)[:, None]
    print("sigma, 1300 targets in one call", flush=True)
    a = C.sigma2(B, eps, om, ctx=C.Context(0))
    ctx = C.Context(0)
    ctx.set_target_chunk(100)
    b = C.sigma2(B, eps, om, ctx=ctx)
    assert np.isfinite(a[0]).all()
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
