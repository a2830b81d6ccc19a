// Adjoints of the quasi-particle solve and of the AO->MO transform.
//
// The converged energy w* solves F(w, theta) = e_q + Sigma_qq(w; theta) - w = 0
// (Eq. (qpapp) of the paper); implicit differentiation gives
//   dw*/dtheta = P dF/dtheta,   P = 1 / (1 - Sigma'(w*))   (pole strength, Eq. (ps)).
// With g = (q r|a j) = G[s][r][a*nocc+j] (Eq. (aomo)) the self-energy Eq. (SE)
// depends on each integral through its own term and its exchange partner:
//   dSigma/dx_{a;ij} = (4 x_{a;ij} - 2 x_{a;ji}) / d_{a;ij},  same for y.
// Since G = Bsel Bvo^T:
//   Bsel_bar[s] = W[s] Bvo            (W = omega_bar P dSigma/dG)
//   Bvo_bar     = sum_s W[s]^T Bsel[s]
// and the energies enter through the denominators and e_q itself.
// Transform adjoint: B^K = C^T L^K C gives C_bar = sum_K L^K C (Bbar^K + Bbar^K^T).  Bbar has only the
// rows of the targets and the virtual-occupied block, so with the rows x = occupied orbitals and
// targets, Z^K[x][r] their cotangents (occupied i: Bvo_bar[a][i] at r = a; target s: Bsel_bar[s][r]),
// T^K_x = L^K C_x and Y^K_x = sum_r C_r Z^K[x][r]:
//   C_bar_r += sum_K sum_x T^K_x Z^K[x][r]   and   C_bar_x += sum_K L^K Y^K_x,
// 4 n nx (n + nvirt) operations per vector against 4 n^3 for the full symmetric Bbar (n = 480, 120
// occupied: 0.45 of it; 960: 0.26), every product K-contiguous.  Both sums run over the vectors
// inside the products, a run of vectors per workgroup, and the runs are added in order.
#include "cds_internal.h"

#include <cmath>
#include <vector>

int cds_gemm_ex(cds_ctx *ctx, int prec, const GemmDesc &d, const void *Alo, const void *Blo);
int cds_sigma_eval_internal(cds_ctx *ctx, int prec, int64_t nvec, int64_t ldk, int nmo, int nocc,
                            int nsel, const void *Bsel, const void *Bvo, const double *eps,
                            const double *h_omega, int T, double *h_out);
int cds_contract_internal(cds_ctx *ctx, int prec, int64_t nvec, int64_t ldk, int nmo, int nocc,
                          int nsel, const void *Bsel, const void *Bvo, int s0, int nsc, void *G);
int cds_grad_epilogue_internal(cds_ctx *ctx, int prec, int nmo, int nocc, int nsc, const void *G,
                               const double *eps, const double *d_omega, const double *d_gscale,
                               void *W, double *epsA, double *epsB);
int cds_sigma_from_g_internal(cds_ctx *ctx, int prec, int nmo, int nocc, int nsc, const void *G,
                              const double *eps, const double *d_omega, double *d_out);

namespace {

// bf16 hi/lo planes -> float
__global__ void planes_to_float_kernel(const __bf16 *__restrict__ b, int64_t n, float *__restrict__ out)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) out[t] = (float)b[t] + (float)b[n + t];
}

template <typename T>
__global__ void zero_cols_kernel(T *__restrict__ B, int64_t nrows, int64_t ldk, int64_t c0)
{
    int64_t npad = ldk - c0;
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nrows * npad) return;
    int64_t r = t / npad;
    B[r * ldk + c0 + (t - r * npad)] = (T)0;
}

// eps_bar[r] = sum over targets and blocks of the energy partials, + P*omega_bar on e_q
// eps_bar[r]: one workgroup per orbital r; the threads take the (target, virtual) partials in a
// fixed stride, four loads in flight at a time, and the workgroup sums them in a fixed order
__global__ __launch_bounds__(256) void eps_bar_kernel(const double *__restrict__ epsA, const double *__restrict__ epsB,
                                                      int nsel, int nocc, int nvirt, const int32_t *__restrict__ sel,
                                                      const double *__restrict__ gscale, double *__restrict__ out)
{
    __shared__ double sh[4];
    const int r = blockIdx.x;
    const int64_t per = (int64_t)nvirt * (nocc + 1);
    double acc = 0.0;
    if (r < nocc) {
        const int64_t n = (int64_t)nsel * nvirt;                 // (target, virtual) pairs
        constexpr int U = 4;
        for (int64_t q0 = threadIdx.x; q0 < n; q0 += (int64_t)U * 256) {
            double va[U], vb[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = q0 + (int64_t)u * 256 < n ? q0 + (int64_t)u * 256 : n - 1;
                const int64_t s = q / nvirt, a = q - s * nvirt;
                const int64_t off = s * per + a * (nocc + 1) + r;
                va[u] = epsA[off];
                vb[u] = epsB[off];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (q0 + (int64_t)u * 256 < n) acc += va[u] + vb[u];
        }
    } else {
        for (int s = threadIdx.x; s < nsel; s += 256) {
            const int64_t off = (int64_t)s * per + (int64_t)(r - nocc) * (nocc + 1) + nocc;
            acc += epsA[off] + epsB[off];
        }
    }
    for (int s = threadIdx.x; s < nsel; s += 256)
        if (sel[s] == r) acc += gscale[s];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[r] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// CX[x][nu] = C[nu][sel or occupied orbital of row x] (x < nocc: occupied x; xo <= x < xo + nsel:
// target x - xo; other rows and nu >= nbf: 0), and Ccat[nu][c] = C[nu][nocc + c] for c < nvirt,
// C[nu][c - ap] for ap <= c < ap + nocc, else 0
__global__ void coef_adj_kernel(const double *__restrict__ C, int nbf, int nmo, int nocc, int nsel,
                                const int32_t *__restrict__ sel, int np_, int xo, int xp, int ap, int cp,
                                double *__restrict__ CX, double *__restrict__ Ccat)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, n1 = (int64_t)xp * np_;
    if (t < n1) {
        const int x = (int)(t / np_), nu = (int)(t - (int64_t)x * np_);
        const int q = x < nocc ? x : (x >= xo && x < xo + nsel ? sel[x - xo] : -1);
        CX[t] = q >= 0 && nu < nbf ? C[(int64_t)nu * nmo + q] : 0.0;
    } else if (t - n1 < (int64_t)nbf * cp) {
        const int64_t u = t - n1;
        const int nu = (int)(u / cp), c = (int)(u - (int64_t)nu * cp);
        const int q = c < nmo - nocc ? nocc + c : (c >= ap && c < ap + nocc ? c - ap : -1);
        Ccat[u] = q >= 0 ? C[(int64_t)nu * nmo + q] : 0.0;
    }
}

// out[z oz + kb ok + x] = in[z iz + x ix + kb] (FP64) for kb < nkb, x < nx, and 0 for nx <= x < nxp:
// 32 x 32 tiles through LDS, every load of a thread in flight before its stores
template <typename BT>
__global__ __launch_bounds__(256) void bar_transpose_kernel(const BT *__restrict__ in, int64_t iz, int64_t ix, int nkb,
                                                            int nx, int nxp, int64_t oz, int64_t ok,
                                                            double *__restrict__ out)
{
    __shared__ double t[32][33];
    const int x0 = blockIdx.y * 32, k0 = blockIdx.x * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const BT *src = in + blockIdx.z * iz;
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int x = x0 + ty + 8 * u, k = k0 + tx;
        v[u] = x < nx && k < nkb ? (double)src[x * ix + k] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) t[ty + 8 * u][tx] = v[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = k0 + ty + 8 * u, x = x0 + tx;
        if (k < nkb && x < nxp) out[blockIdx.z * oz + k * ok + x] = t[tx][ty + 8 * u];
    }
}

// C_bar[mu][r] from the summed products: virtual columns Pv, occupied columns Po, and the columns
// of P2 (occupied x at x, target s at xo + s)
__global__ void cbar_kernel(const double *__restrict__ Pv, const double *__restrict__ Po, const double *__restrict__ P2,
                            int nbf, int nmo, int nocc, int nsel, const int32_t *__restrict__ sel, int xo, int xp,
                            double *__restrict__ out)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nbf * nmo) return;
    const int64_t mu = t / nmo;
    const int r = (int)(t - mu * nmo);
    double v = r < nocc ? Po[mu * nocc + r] + P2[mu * xp + r] : Pv[mu * (nmo - nocc) + r - nocc];
    for (int s = 0; s < nsel; ++s)
        if (sel[s] == r) v += P2[mu * xp + xo + s];
    out[t] = v;
}

// out[e] (+)= sum_{b < nb} part[b][e], b in increasing order
__global__ void sum_parts_kernel(const double *__restrict__ part, int nb, int64_t ne, int accumulate,
                                 double *__restrict__ out)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= ne) return;
    // in order, eight loads in flight at a time
    constexpr int U = 8;
    double acc = accumulate ? out[e] : 0.0;
    for (int b0 = 0; b0 < nb; b0 += U) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = b0 + u < nb ? part[(int64_t)(b0 + u) * ne + e] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (b0 + u < nb) acc += v[u];
    }
    out[e] = acc;
}

// Lu[kb][mu][nu] (nu padded to np_) in FP64
__global__ void unpack64_kernel(const double *__restrict__ L, int64_t ldl, int64_t k0, int nkb, int nbf,
                                int np_, double *__restrict__ out)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t per = (int64_t)nbf * np_;
    if (t >= per * nkb) return;
    int kb = (int)(t / per);
    int64_t rem = t - (int64_t)kb * per;
    int mu = (int)(rem / np_), nu = (int)(rem - (int64_t)mu * np_);
    double v = 0.0;
    if (nu < nbf) {
        int a = mu < nu ? mu : nu, b = mu < nu ? nu : mu;
        v = L[(k0 + kb) * ldl + (int64_t)b * (b + 1) / 2 + a];
    }
    out[t] = v;
}

}  // namespace

extern "C" int cds_qp_adjoint(cds_ctx *ctx, int32_t prec, int64_t nvec, int64_t ldk, int32_t nmo,
                              int32_t nocc, int32_t nsel, const int32_t *h_sel, const void *Bsel,
                              const void *Bvo, const double *eps, const double *h_omega,
                              const double *h_omega_bar, void *Bsel_bar, void *Bvo_bar, double *eps_bar)
{
    CDS_CALL(cds_enter(ctx));
    CDS_REQUIRE(ctx, prec == CDS_PREC_FP64 || prec == CDS_PREC_FP32 || prec == CDS_PREC_BF16X3,
                "unknown precision %d", prec);
    CDS_REQUIRE(ctx, nmo >= 2 && nocc >= 1 && nocc < nmo && nocc <= 1024, "bad nocc/nmo");
    CDS_REQUIRE(ctx, nsel >= 1 && h_sel && h_omega && h_omega_bar, "bad targets");
    CDS_REQUIRE(ctx, nvec >= 1 && ldk >= nvec, "need nvec >= 1, ldk >= nvec");
    CDS_REQUIRE(ctx, prec != CDS_PREC_BF16X3 || ldk % 64 == 0, "BF16X3 needs ldk % 64 == 0");
    CDS_REQUIRE(ctx, Bsel && Bvo && eps && Bsel_bar && Bvo_bar && eps_bar, "NULL pointer");
    for (int s = 0; s < nsel; ++s)
        CDS_REQUIRE(ctx, h_sel[s] >= 0 && h_sel[s] < nmo, "h_sel[%d] out of range", s);
    CdsTimer tall;
    CDS_CALL(cds_timer_start(ctx, &tall));
    const int nvirt = nmo - nocc;
    const int64_t nvo = (int64_t)nvirt * nocc, nselr = (int64_t)nsel * nmo;

    // the pole strengths at the converged energies come from each chunk's integrals (below)
    std::vector<double> out((size_t)nsel * 2), hscale(nsel);

    // working copies: float operands for BF16X3 (planes -> float)
    const int gprec = prec == CDS_PREC_FP64 ? CDS_PREC_FP64 : CDS_PREC_FP32;
    const size_t es = prec == CDS_PREC_FP64 ? 8 : 4;
    const void *Bs = Bsel, *Bv = Bvo;
    void *tmp;
    size_t nB = (size_t)(nselr + nvo) * ldk;
    size_t small = (size_t)nsel * 8 * 5 + (size_t)nsel * 4 + 256;
    size_t epsbytes = (size_t)2 * nsel * nvirt * (nocc + 1) * 8;
    CDS_CALL(cds_ws(ctx, WS_AD_TMP, (prec == CDS_PREC_BF16X3 ? nB * 4 : 0) + small + epsbytes, &tmp));
    unsigned char *tp = (unsigned char *)tmp;
    if (prec == CDS_PREC_BF16X3) {
        float *fs = (float *)tp, *fv = fs + nselr * ldk;
        hipLaunchKernelGGL(planes_to_float_kernel, dim3((unsigned)cds_ceil_div(nselr * ldk, 256)), dim3(256),
                           0, ctx->stream, (const __bf16 *)Bsel, nselr * ldk, fs);
        hipLaunchKernelGGL(planes_to_float_kernel, dim3((unsigned)cds_ceil_div(nvo * ldk, 256)), dim3(256), 0,
                           ctx->stream, (const __bf16 *)Bvo, nvo * ldk, fv);
        CDS_LAUNCHED(ctx);
        Bs = fs;
        Bv = fv;
        tp += nB * 4;
    }
    double *d_omega = (double *)tp;
    double *d_scale = d_omega + nsel;
    double *d_sig = d_scale + nsel;                    // [nsel][2]: Sigma, Sigma'
    int32_t *d_sel = (int32_t *)(d_sig + 2 * nsel);
    double *epsA = (double *)(tp + small);
    double *epsB = epsA + (size_t)nsel * nvirt * (nocc + 1);
    CDS_HIP(ctx, hipMemcpyAsync(d_omega, h_omega, (size_t)nsel * 8, hipMemcpyHostToDevice, ctx->stream));
    CDS_HIP(ctx, hipMemcpyAsync(d_sel, h_sel, (size_t)nsel * 4, hipMemcpyHostToDevice, ctx->stream));

    // chunks of targets: G, W and W^T each nsc * nmo * nvo, at most 12 GiB each (few, large
    // chunks: the product over nvo below has only nsc * nmo / 128 tile rows)
    size_t per = (size_t)nmo * nvo * es;
    int csz = (int)std::max<size_t>(1, ((size_t)12 << 30) / std::max<size_t>(per, 1));
    if (ctx->target_chunk > 0) csz = std::min(csz, ctx->target_chunk);
    csz = std::min(csz, (int)nsel);
    void *G, *W;
    CDS_CALL(cds_ws(ctx, WS_SG_G, (size_t)csz * per, &G));
    CDS_CALL(cds_ws(ctx, WS_AD_G, (size_t)csz * per, &W));
    // K-contiguous copies of the operands the two products read across K (the GEMM's fast path
    // loads rows along K): Bvo^T [nvec][nvo], then per chunk W^T [nvo][nsc*nmo] and the chunk's
    // Bsel^T [nvec][nsc*nmo]
    void *BvT, *WT, *BsT;
    CDS_CALL(cds_ws(ctx, WS_AD_T1, (size_t)nvec * nvo * es, &BvT));
    CDS_CALL(cds_ws(ctx, WS_AD_T2, (size_t)csz * per, &WT));
    CDS_CALL(cds_ws(ctx, WS_AD_T3, (size_t)nvec * csz * nmo * es, &BsT));
    CDS_CALL(cds_transpose(ctx, (int)es, nvo, nvec, Bv, ldk, BvT, nvo));
    for (int s0 = 0; s0 < nsel; s0 += csz) {
        const int nsc = std::min(csz, nsel - s0);
        CDS_CALL(cds_contract_internal(ctx, prec, nvec, ldk, nmo, nocc, nsel, Bsel, Bvo, s0, nsc, G));
        // P_s = 1 / (1 - Sigma'(w*_s)) from the same integrals, then the weights' scale
        CDS_CALL(cds_sigma_from_g_internal(ctx, prec, nmo, nocc, nsc, G, eps, d_omega + s0, d_sig + 2 * s0));
        CDS_HIP(ctx, hipMemcpyAsync(out.data() + 2 * s0, d_sig + 2 * s0, (size_t)nsc * 2 * 8, hipMemcpyDeviceToHost,
                                    ctx->stream));
        CDS_HIP(ctx, hipStreamSynchronize(ctx->stream));
        for (int s = s0; s < s0 + nsc; ++s) hscale[s] = h_omega_bar[s] / (1.0 - out[2 * s + 1]);
        CDS_HIP(ctx, hipMemcpyAsync(d_scale + s0, hscale.data() + s0, (size_t)nsc * 8, hipMemcpyHostToDevice,
                                    ctx->stream));
        CDS_CALL(cds_grad_epilogue_internal(ctx, prec, nmo, nocc, nsc, G, eps, d_omega + s0, d_scale + s0, W,
                                            epsA + (size_t)s0 * nvirt * (nocc + 1),
                                            epsB + (size_t)s0 * nvirt * (nocc + 1)));
        // Bsel_bar[s0..] = W Bvo :  (nsc*nmo) x nvec, reduction over nvo
        GemmDesc d1 = {};
        d1.M = (int64_t)nsc * nmo; d1.N = nvec; d1.K = nvo; d1.batch = 1;
        d1.A = W; d1.sAm = nvo; d1.sAk = 1;
        d1.B = BvT; d1.sBk = 1; d1.sBn = nvo;
        d1.C = (unsigned char *)Bsel_bar + (size_t)s0 * nmo * ldk * es; d1.sCm = ldk; d1.sCn = 1;
        d1.alpha = 1.0; d1.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, gprec, d1, nullptr, nullptr));
        // Bvo_bar += W^T Bsel[s0..] : nvo x nvec, reduction over nsc*nmo
        const int64_t kc = (int64_t)nsc * nmo;
        CDS_CALL(cds_transpose(ctx, (int)es, kc, nvo, W, nvo, WT, kc));
        CDS_CALL(cds_transpose(ctx, (int)es, kc, nvec, (const unsigned char *)Bs + (size_t)s0 * nmo * ldk * es, ldk,
                               BsT, kc));
        GemmDesc d2 = {};
        d2.M = nvo; d2.N = nvec; d2.K = kc; d2.batch = 1;
        d2.A = WT; d2.sAm = kc; d2.sAk = 1;
        d2.B = BsT; d2.sBk = 1; d2.sBn = kc;
        d2.C = Bvo_bar; d2.sCm = ldk; d2.sCn = 1;
        d2.alpha = 1.0; d2.beta = s0 == 0 ? 0.0 : 1.0;
        CDS_CALL(cds_gemm_ex(ctx, gprec, d2, nullptr, nullptr));
    }
    if (ldk > nvec) {
        if (gprec == CDS_PREC_FP64) {
            hipLaunchKernelGGL(zero_cols_kernel<double>, dim3((unsigned)cds_ceil_div(nselr * (ldk - nvec), 256)),
                               dim3(256), 0, ctx->stream, (double *)Bsel_bar, nselr, ldk, nvec);
            hipLaunchKernelGGL(zero_cols_kernel<double>, dim3((unsigned)cds_ceil_div(nvo * (ldk - nvec), 256)),
                               dim3(256), 0, ctx->stream, (double *)Bvo_bar, nvo, ldk, nvec);
        } else {
            hipLaunchKernelGGL(zero_cols_kernel<float>, dim3((unsigned)cds_ceil_div(nselr * (ldk - nvec), 256)),
                               dim3(256), 0, ctx->stream, (float *)Bsel_bar, nselr, ldk, nvec);
            hipLaunchKernelGGL(zero_cols_kernel<float>, dim3((unsigned)cds_ceil_div(nvo * (ldk - nvec), 256)),
                               dim3(256), 0, ctx->stream, (float *)Bvo_bar, nvo, ldk, nvec);
        }
        CDS_LAUNCHED(ctx);
    }
    hipLaunchKernelGGL(eps_bar_kernel, dim3((unsigned)nmo), dim3(256), 0, ctx->stream,
                       (const double *)epsA, (const double *)epsB, nsel, nocc, nvirt, (const int32_t *)d_sel,
                       (const double *)d_scale, eps_bar);
    CDS_LAUNCHED(ctx);
    CDS_CALL(cds_timer_stop(ctx, &tall, &ctx->stats.t_adjoint_ms));
    CDS_CALL(cds_timers_flush(ctx));
    return CDS_OK;
}

extern "C" int cds_transform_adjoint(cds_ctx *ctx, int32_t prec, int32_t nbf, int64_t nvec,
                                     const double *L, int64_t ldl, const double *C, int32_t nmo,
                                     int32_t nocc, int32_t nsel, const int32_t *h_sel, int64_t ldk,
                                     const void *Bsel_bar, const void *Bvo_bar, double *C_bar)
{
    CDS_CALL(cds_enter(ctx));
    CDS_REQUIRE(ctx, prec == CDS_PREC_FP64 || prec == CDS_PREC_FP32 || prec == CDS_PREC_BF16X3,
                "unknown precision %d", prec);
    CDS_REQUIRE(ctx, nbf >= 1 && nmo >= 2 && nmo <= nbf && nocc >= 1 && nocc < nmo, "bad sizes");
    CDS_REQUIRE(ctx, nsel >= 1 && h_sel, "bad targets");
    CDS_REQUIRE(ctx, nvec >= 1 && ldk >= nvec && ldl >= cds_npairs(nbf), "bad nvec/ldk/ldl");
    CDS_REQUIRE(ctx, L && C && Bsel_bar && Bvo_bar && C_bar, "NULL pointer");
    for (int s = 0; s < nsel; ++s)
        CDS_REQUIRE(ctx, h_sel[s] >= 0 && h_sel[s] < nmo, "h_sel[%d] out of range", s);
    CdsTimer tall;
    CDS_CALL(cds_timer_start(ctx, &tall));
    const int nvirt = nmo - nocc;
    auto up16 = [](int64_t n) { return (int)(cds_ceil_div(n, 16) * 16); };
    const int np_ = up16(nbf);
    const int xo = up16(nocc), selp = up16(nsel), xp = xo + selp;    // rows x: occupied, then targets
    const int ap = up16(nvirt), cp = ap + up16(nocc);                // columns: virtual, then occupied
    // vectors per batch: the largest of the batch's arrays stays below 1 GiB
    const int64_t per = 8 * std::max<int64_t>((int64_t)nbf * np_, std::max<int64_t>((int64_t)xp * np_, (int64_t)nmo * xp));
    const int kb = (int)std::min<int64_t>(std::min<int64_t>(nvec, 8192), std::max<int64_t>(1, (int64_t)(1ull << 30) / per));
    // runs of vectors per product, so that each product launches about 1024 tiles
    auto run_of = [&](int64_t n) {
        const int64_t tiles = cds_ceil_div(nbf, 128) * cds_ceil_div(n, 128);
        return std::max<int64_t>(1, kb * tiles / 1024);
    };
    const int64_t rv = run_of(nvirt), ro = run_of(nocc), r2 = run_of(xp);
    auto runs = [](int64_t nkb, int64_t run) { return cds_ceil_div(nkb, run); };
    const int64_t npart = std::max({runs(kb, rv) * nbf * nvirt, runs(kb, ro) * nbf * nocc, runs(kb, r2) * nbf * xp});
    void *wl, *wt, *wz, *wy, *wc, *wp;
    CDS_CALL(cds_ws(ctx, WS_TR_UNPACK, (size_t)kb * nbf * np_ * 8, &wl));
    CDS_CALL(cds_ws(ctx, WS_TR_T, (size_t)kb * nbf * xp * 8, &wt));                       // T[mu][kb][x]
    const size_t nzv = (size_t)nvirt * kb * xp, nzo = (size_t)nocc * kb * selp;           // Zv[a][kb][x], Zo[r][kb][s]
    const size_t nzr = (size_t)nocc * kb * ap, nzs = (size_t)nsel * kb * cp;              // Zr[i][kb][a], Zs[s][kb][c]
    CDS_CALL(cds_ws(ctx, WS_AD_TMP2, (nzv + nzo + nzr + nzs) * 8, &wz));
    CDS_CALL(cds_ws(ctx, WS_AD_T1, (size_t)xp * kb * np_ * 8, &wy));                      // Y[x][kb][nu]
    const size_t ncx = (size_t)xp * np_, nccat = (size_t)nbf * cp, nsum = (size_t)nbf * (nmo + xp);
    CDS_CALL(cds_ws(ctx, WS_TR_CX, (ncx + nccat + nsum) * 8 + (size_t)nsel * 4 + 64, &wc));
    CDS_CALL(cds_ws(ctx, WS_AD_TMP, (size_t)npart * 8, &wp));
    double *Lu = (double *)wl, *T = (double *)wt, *Y = (double *)wy, *part = (double *)wp;
    double *Zv = (double *)wz, *Zo = Zv + nzv, *Zr = Zo + nzo, *Zs = Zr + nzr;
    double *CX = (double *)wc, *Ccat = CX + ncx, *Pv = Ccat + nccat, *Po = Pv + (size_t)nbf * nvirt, *P2 = Po + (size_t)nbf * nocc;
    int32_t *dsel = (int32_t *)(P2 + (size_t)nbf * xp);
    CDS_HIP(ctx, hipMemcpyAsync(dsel, h_sel, (size_t)nsel * 4, hipMemcpyHostToDevice, ctx->stream));
    const int64_t ncoef = (int64_t)(ncx + nccat);
    hipLaunchKernelGGL(coef_adj_kernel, dim3((unsigned)cds_ceil_div(ncoef, 256)), dim3(256), 0, ctx->stream, C, nbf, nmo,
                       nocc, nsel, (const int32_t *)dsel, np_, xo, xp, ap, cp, CX, Ccat);
    CDS_LAUNCHED(ctx);
    const size_t bes = prec == CDS_PREC_FP64 ? 8 : 4;
    // out[z][kb][x] from the rows z * iz + x * ix of a cotangent block, columns k0 ..
    auto bars = [&](const void *blk, int64_t row0, int64_t iz, int64_t ix, int nz, int nx, int nxp, double *out, int64_t oz,
                    int64_t ok, int64_t k0, int nkb) -> int {
        const dim3 g((unsigned)cds_ceil_div(nkb, 32), (unsigned)cds_ceil_div(nxp, 32), (unsigned)nz);
        const void *src = (const unsigned char *)blk + (size_t)(row0 * ldk + k0) * bes;
        if (prec == CDS_PREC_FP64)
            hipLaunchKernelGGL(bar_transpose_kernel<double>, g, dim3(256), 0, ctx->stream, (const double *)src, iz * ldk,
                               ix * ldk, nkb, nx, nxp, oz, ok, out);
        else
            hipLaunchKernelGGL(bar_transpose_kernel<float>, g, dim3(256), 0, ctx->stream, (const float *)src, iz * ldk,
                               ix * ldk, nkb, nx, nxp, oz, ok, out);
        CDS_LAUNCHED(ctx);
        return CDS_OK;
    };
    // sum over the vectors of a batch: out[m][n] (+)= sum_kb sum_k A[m][kb][k] B[n][kb][k]
    auto summed = [&](int64_t N, int64_t K, int nkb, int64_t run, const double *A, int64_t sAm, int64_t sAb,
                      const double *B, int64_t sBn, int64_t sBb, bool more, double *out) -> int {
        GemmDesc g = {};
        g.M = nbf; g.N = N; g.K = K; g.batch = nkb; g.bacc = run;
        g.A = A; g.sAm = sAm; g.sAk = 1; g.sAb = sAb;
        g.B = B; g.sBn = sBn; g.sBk = 1; g.sBb = sBb;
        g.C = part; g.sCm = N; g.sCn = 1; g.sCb = nbf * N;
        g.alpha = 1.0; g.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, CDS_PREC_FP64, g, nullptr, nullptr));
        const int64_t ne = nbf * N;
        hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)cds_ceil_div(ne, 256)), dim3(256), 0, ctx->stream,
                           (const double *)part, (int)runs(nkb, run), ne, more ? 1 : 0, out);
        CDS_LAUNCHED(ctx);
        return CDS_OK;
    };
    for (int64_t k0 = 0; k0 < nvec; k0 += kb) {
        const int nkb = (int)std::min<int64_t>(kb, nvec - k0);
        const int64_t n1 = (int64_t)nkb * nbf * np_;
        hipLaunchKernelGGL(unpack64_kernel, dim3((unsigned)cds_ceil_div(n1, 256)), dim3(256), 0, ctx->stream, L,
                           ldl, k0, nkb, nbf, np_, Lu);
        CDS_LAUNCHED(ctx);
        // T[mu][kb][x] = sum_nu L^K[mu][nu] CX[x][nu]
        GemmDesc gt = {};
        gt.M = nbf; gt.N = xp; gt.K = np_; gt.batch = nkb;
        gt.A = Lu; gt.sAm = np_; gt.sAk = 1; gt.sAb = (int64_t)nbf * np_;
        gt.B = CX; gt.sBn = np_; gt.sBk = 1; gt.sBb = 0;
        gt.C = T; gt.sCm = (int64_t)nkb * xp; gt.sCn = 1; gt.sCb = xp;
        gt.alpha = 1.0; gt.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, CDS_PREC_FP64, gt, nullptr, nullptr));
        // the cotangents with x along the rows (Zv: virtual columns a, occupied rows then targets; Zo:
        // the targets' occupied columns), then C_bar_r += sum T Z
        const int64_t zs = (int64_t)nkb * xp;
        CDS_CALL(bars(Bvo_bar, 0, nocc, 1, nvirt, nocc, xo, Zv, zs, xp, k0, nkb));
        CDS_CALL(bars(Bsel_bar, nocc, 1, nmo, nvirt, nsel, selp, Zv + xo, zs, xp, k0, nkb));
        CDS_CALL(bars(Bsel_bar, 0, 1, nmo, nocc, nsel, selp, Zo, (int64_t)nkb * selp, selp, k0, nkb));
        CDS_CALL(summed(nvirt, xp, nkb, rv, T, zs, xp, Zv, zs, xp, k0 > 0, Pv));
        CDS_CALL(summed(nocc, selp, nkb, ro, T + xo, zs, xp, Zo, (int64_t)nkb * selp, selp, k0 > 0, Po));
        // the cotangents with r along the rows, Y[x][kb][nu] = sum_r Z[x][kb][r] C[nu][r], then
        // C_bar_x += sum L Y
        CDS_CALL(bars(Bvo_bar, 0, 1, nocc, nocc, nvirt, ap, Zr, (int64_t)nkb * ap, ap, k0, nkb));
        CDS_CALL(bars(Bsel_bar, nocc, nmo, 1, nsel, nvirt, ap, Zs, (int64_t)nkb * cp, cp, k0, nkb));
        CDS_CALL(bars(Bsel_bar, 0, nmo, 1, nsel, nocc, cp - ap, Zs + ap, (int64_t)nkb * cp, cp, k0, nkb));
        GemmDesc gy = {};
        gy.M = (int64_t)nocc * nkb; gy.N = np_; gy.K = ap; gy.batch = 1;
        gy.A = Zr; gy.sAm = ap; gy.sAk = 1;
        gy.B = Ccat; gy.sBn = cp; gy.sBk = 1;
        gy.C = Y; gy.sCm = np_; gy.sCn = 1;
        gy.alpha = 1.0; gy.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, CDS_PREC_FP64, gy, nullptr, nullptr));
        gy.M = (int64_t)nsel * nkb; gy.K = cp;
        gy.A = Zs; gy.sAm = cp;
        gy.C = Y + (int64_t)xo * nkb * np_;
        CDS_CALL(cds_gemm_ex(ctx, CDS_PREC_FP64, gy, nullptr, nullptr));
        CDS_CALL(summed(xp, np_, nkb, r2, Lu, np_, (int64_t)nbf * np_, Y, (int64_t)nkb * np_, np_, k0 > 0, P2));
    }
    const int64_t ne = (int64_t)nbf * nmo;
    hipLaunchKernelGGL(cbar_kernel, dim3((unsigned)cds_ceil_div(ne, 256)), dim3(256), 0, ctx->stream, (const double *)Pv,
                       (const double *)Po, (const double *)P2, nbf, nmo, nocc, nsel, (const int32_t *)dsel, xo, xp, C_bar);
    CDS_LAUNCHED(ctx);
    CDS_CALL(cds_timer_stop(ctx, &tall, &ctx->stats.t_adjoint_ms));
    return CDS_OK;
}
