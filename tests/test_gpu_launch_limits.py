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


def _nan(*shape):
    """Memory of this size that holds NaN goes back to the allocator."""
    torch.cuda.empty_cache()
    torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")


def test_transform_padding_of_more_than_2_32_entries():
    # 529 + 1564 rows of 2^21 - 3 padding entries each (17.6 GB in FP32), in one launch of both blocks
    import paper_0912_1459_amd.core as C
    n, nocc, nsel, nvec, ldk = 46, 23, 34, 3, 2 ** 21
    g = torch.Generator(device="cuda").manual_seed(2)
    L = torch.randn((nvec, n * (n + 1) // 2), generator=g, dtype=torch.float64, device="cuda")
    Cm = torch.randn((n, n), generator=g, dtype=torch.float64, device="cuda")
    ref = C.transform(L, nvec, Cm, nocc, np.arange(nsel), "fp32")
    _nan(nsel * n, ldk)
    print("transform, rows of 2^21", flush=True)
    B = C.transform(L, nvec, Cm, nocc, np.arange(nsel), "fp32", ldk=ldk)
    for x, r in ((B.Bsel, ref.Bsel), (B.Bvo, ref.Bvo)):
        assert torch.equal(x[:, :nvec], r[:, :nvec])
        assert not bool(x[:, nvec:].any())
    del B, x
    torch.cuda.empty_cache()


def test_adjoint_of_more_than_2_32_entries():
    # Bsel_bar of 2116 rows of 2^21 (17.7 GB in FP32)
    import paper_0912_1459_amd.core as C
    from paper_0912_1459_amd import _lib as A
    n, nocc, nsel, nvec, ldk = 46, 23, 46, 5, 2 ** 21
    g = torch.Generator(device="cuda").manual_seed(3)
    r = lambda rows: torch.randn((rows, 64), generator=g, dtype=torch.float32, device="cuda") * 0.02
    S, V = r(nsel * n), r((n - nocc) * nocc)
    S[:, nvec:] = 0
    V[:, nvec:] = 0
    eps = torch.cat([torch.linspace(-1.5, -0.3, nocc, dtype=torch.float64), torch.linspace(0.1, 3.0, n - nocc, dtype=torch.float64)])
    eps, om, wb, sel = eps.cuda(), np.linspace(-0.2, 0.05, nsel), np.linspace(-1.0, 1.0, nsel), np.arange(nsel, dtype=np.int32)
    ref = C.qp_adjoint(C.BBlocks(A.PREC_FP32, S, V, nvec, 64, n, nocc, sel), eps, om, wb)
    SL, VL = (torch.zeros((x.shape[0], ldk), dtype=torch.float32, device="cuda") for x in (S, V))
    SL[:, :64] = S
    VL[:, :64] = V
    x = torch.full((nsel * n, ldk), float("nan"), dtype=torch.float32, device="cuda")
    del x
    print("adjoint, rows of 2^21", flush=True)
    got = C.qp_adjoint(C.BBlocks(A.PREC_FP32, SL, VL, nvec, ldk, n, nocc, sel), eps, om, wb)
    for x, r in zip(got[:2], ref[:2]):
        assert torch.equal(x[:, :nvec], r[:, :nvec])
        assert not bool(x[:, nvec:].any())
    assert torch.equal(got[2], ref[2])
    del got, x, SL, VL
    torch.cuda.empty_cache()


def test_adjoint_of_the_most_pairs():
    # 1020 occupied, 2056 virtuals: 2,097,120 = 65535 * 32 rows of Bvo, the most that a transpose takes;
    # the parts of the sum over them must not be padded past that.  Checked by what holds exactly:
    # a common shift of the energies (sum of eps_bar = omega_bar), and Sigma's degree two in either
    # block (sum of Bsel_bar Bsel = sum of Bvo_bar Bvo = 2 omega_bar P Sigma).  The sums have 4e9
    # positive and negative terms: 1e-9 of the largest is far above their rounding
    import paper_0912_1459_amd.core as C
    from paper_0912_1459_amd import _lib as A
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 130 << 30:
        pytest.skip("needs 130 GiB of device memory")
    nocc, nvirt, nvec, ldk = 1020, 2056, 2, 64
    g = torch.Generator(device="cuda").manual_seed(6)

    def block(rows):
        x = torch.zeros((rows, ldk), dtype=torch.float64, device="cuda")
        x[:, :nvec] = torch.rand((rows, nvec), generator=g, dtype=torch.float64, device="cuda") * 1e-2
        return x
    S, V = block(nocc + nvirt), block(nvirt * nocc)
    eps = torch.cat([torch.linspace(-1.5, -0.3, nocc, dtype=torch.float64), torch.linspace(0.1, 3.0, nvirt, dtype=torch.float64)]).cuda()
    B = C.BBlocks(A.PREC_FP64, S, V, nvec, ldk, nocc + nvirt, nocc, np.array([nocc - 1], np.int32))
    om, wb = np.array([-0.2]), np.array([0.75])
    print("adjoint of 2,097,120 pairs", flush=True)
    with C.Context(0) as ctx:
        gs, gv, ge = C.qp_adjoint(B, eps, om, wb, ctx=ctx)
        s, ds = C.sigma2(B, eps, om[:, None], ctx=ctx)
    want = 2.0 * wb[0] / (1.0 - ds[0, 0]) * s[0, 0]
    for x, y in ((gs, S), (gv, V)):
        assert abs(float((x * y).sum()) - want) <= 1e-9 * float((x * y).abs().sum())
    assert abs(float(ge.sum()) - wb[0]) <= 1e-9 * float(ge.abs().sum())
    del gs, gv, S, V, B
    torch.cuda.empty_cache()
