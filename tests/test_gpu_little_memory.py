"""Calls on a device that is nearly full take smaller pieces instead of failing.

Most of the device's memory is taken by one allocation; what is left holds the call in pieces but not
at its usual size.  The results are those of a call with room: the pieces change no MP2 pair sum, and
regroup the adjoint's sum over the vectors (1e-12 of the sum of absolute terms).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


class _Full:
    """All but `left` bytes of the free device memory, taken for a while."""

    def __init__(self, left):
        self.left = left

    def __enter__(self):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        self.t = torch.empty(torch.cuda.mem_get_info()[0] - self.left, dtype=torch.uint8, device="cuda")

    def __exit__(self, *exc):
        del self.t
        torch.cuda.empty_cache()


def _blocks(nocc, nvirt, nvec):
    import paper_0912_1459_amd.core as C
    from paper_0912_1459_amd import _lib as A
    g = torch.Generator(device="cuda").manual_seed(nocc)
    r = lambda rows: torch.randn((rows, 64), generator=g, dtype=torch.float64, device="cuda") * 0.02
    V, S = r(nvirt * nocc), r(nocc + nvirt)
    V[:, nvec:] = 0
    S[:, nvec:] = 0
    eps = torch.cat([torch.linspace(-1.5, -0.3, nocc, dtype=torch.float64), torch.linspace(0.1, 3.0, nvirt, dtype=torch.float64)])
    return C.BBlocks(A.PREC_FP64, S, V, nvec, 64, nocc + nvirt, nocc, np.zeros(1, np.int32)), eps.cuda()


def test_mp2_in_smaller_chunks():
    # 23,000 rows: 4.2 GB of integrals (4.8 with the workspace's headroom) in one chunk, 2.4 in two
    import paper_0912_1459_amd.core as C
    B, eps = _blocks(50, 460, 40)
    ref = C.mp2_energy(B, eps, ctx=C.Context(0))
    print("mp2, 3.5 GiB left", flush=True)
    with C.Context(0) as ctx, _Full(7 << 29):
        e = C.mp2_energy(B, eps, ctx=ctx)
        assert ctx.workspace_bytes() < 7 << 29
        assert C.mp2_energy(B, eps, ctx=ctx) == e
    assert e == ref


def test_transform_adjoint_in_smaller_batches():
    # 300 functions, 60 occupied, 2000 vectors: 2.4 GB for a batch of 1398 vectors, 1.2 for 699
    import paper_0912_1459_amd.core as C
    n, nocc, nvec, sel = 300, 60, 2000, [58, 59, 60]
    g = torch.Generator(device="cuda").manual_seed(4)
    r = lambda *s: torch.randn(s, generator=g, dtype=torch.float64, device="cuda")
    L, Cm, gs, gv = r(nvec, n * (n + 1) // 2), r(n, n), r(len(sel) * n, nvec), r((n - nocc) * nocc, nvec)
    with C.Context(0) as ctx:
        ref = C.transform_adjoint(L, nvec, Cm, nocc, sel, gs, gv, nvec, ctx=ctx)
        mag = C.transform_adjoint(L.abs(), nvec, Cm.abs(), nocc, sel, gs.abs(), gv.abs(), nvec, ctx=ctx)
    print("transform adjoint, 1.5 GiB left", flush=True)
    with C.Context(0) as ctx, _Full(3 << 29):
        out = C.transform_adjoint(L, nvec, Cm, nocc, sel, gs, gv, nvec, ctx=ctx)
        assert ctx.workspace_bytes() < 3 << 29
        assert torch.equal(C.transform_adjoint(L, nvec, Cm, nocc, sel, gs, gv, nvec, ctx=ctx), out)
    assert bool(((out - ref).abs() <= 1e-12 * mag).all())
