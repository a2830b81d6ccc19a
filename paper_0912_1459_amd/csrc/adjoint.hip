// Adjoints of the quasi-particle solve and of the AO->MO transform.
//
// The converged energy w* solves F(w, theta) = e_q + Sigma_qq(w; theta) - w = 0
// (Eq. (qpapp) of the paper); implicit differentiation gives
//   dw*/dtheta = P dF/dtheta,   P = 1 / (1 - Sigma'(w*))   (pole strength, Eq. (ps)).
// With g = (q r|a j) = G[s][r][a*nocc+j] (Eq. (aomo)) the self-energy Eq. (SE)
// depends on each integral through its own term and its exchange partner:
//   dSigma/dx_{a;ij} = (4 x_{a;ij} - 2 x_{a;ji}) / d_{a;ij},  same for y.
// Since G = Bsel Bvo^T, with W = dSigma/dG and the scale omega_bar_s P_s of each target:
//   Bsel_bar[s] = scale_s W[s] Bvo
//   Bvo_bar     = sum_s W[s]^T (scale_s Bsel[s])
// and the energies enter through the denominators and e_q itself (FP32: the scale is in the stored
// weights).  Only W^T is written, [v][(s, r)]:
// the first product reads it m-contiguous, the second K-contiguous.
// Transform adjoint: B^K = C^T L^K C gives C_bar = sum_K L^K C (Bbar^K + Bbar^K^T).  Bbar has only the
// rows of the targets and the virtual-occupied block, so with the rows x = occupied orbitals and
// targets, Z^K[x][r] their cotangents (occupied i: Bvo_bar[a][i] at r = a; target s: Bsel_bar[s][r]),
// T^K_x = L^K C_x and Y^K_x = sum_r C_r Z^K[x][r]:
//   C_bar_r += sum_K sum_x T^K_x Z^K[x][r]   and   C_bar_x += sum_K L^K Y^K_x,
// 4 n nx (n + nvirt) operations per vector against 4 n^3 for the full symmetric Bbar (n = 480, 120
// occupied: 0.45 of it; 960: 0.26), every product K-contiguous.  Both sums run over the vectors
// inside the products, a run of vectors per workgroup, and the runs are added in order.  Small
// systems form the full symmetric Bbar instead (transform_adjoint_full).
#include "cds_internal.h"

#include <cmath>
#include <cstring>
#include <vector>

int cds_gemm_ex(cds_ctx *ctx, int prec, const GemmDesc &d, const void *Alo, const void *Blo);
int cds_contract_internal(cds_ctx *ctx, int prec, int64_t nvec, int64_t ldk, int nmo, int nocc,
                          int nsel, const void *Bsel, const void *Bvo, int s0, int nsc, void *G);

namespace {

// bf16 hi/lo planes -> float
__global__ void planes_to_float_kernel(const __bf16 *__restrict__ b, int64_t n, float *__restrict__ out)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) out[t] = (float)b[t] + (float)b[n + t];
}

// B[r][c] = 0 for r < nrows, c0 <= c < ld
template <typename T>
__global__ void zero_cols_kernel(T *__restrict__ B, int64_t nrows, int64_t ld, int64_t c0)
{
    int64_t npad = ld - c0;
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nrows * npad) return;
    int64_t r = t / npad;
    B[r * ld + c0 + (t - r * npad)] = (T)0;
}

template <typename T>
int zero_cols(cds_ctx *ctx, T *B, int64_t nrows, int64_t ld, int64_t c0)
{
    if (nrows <= 0 || ld <= c0) return CDS_OK;
    hipLaunchKernelGGL(zero_cols_kernel<T>, dim3((unsigned)cds_ceil_div(nrows * (ld - c0), 256)), dim3(256), 0, ctx->stream,
                       B, nrows, ld, c0);
    CDS_LAUNCHED(ctx);
    return CDS_OK;
}

template <int NTH>
__device__ __forceinline__ double block_sum(double v, double *sh)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < NTH / 64; ++k) s += sh[k];   // fixed order
    return s;
}

// Weights and energy partials of a chunk of targets.  Both kernels read every integral once, both
// exchange partners together, and write W^T in runs of consecutive r: HBM traffic is one read of G
// and one write of W^T.  (Separate kernels for Sigma', W with a thread per row, and a transposed
// copy of W took 3.2 ms for 480 orbitals, 12 targets FP64; these take 1.1 ms.)  FP32 weights are
// rounded with their scale, which needs the partials of the whole target first: two passes there,
// the first without the weights, the second without the partials.
enum : int { W_WEIGHTS = 1, W_PARTIALS = 2 };
struct WArgs {
    const void *G;          // integrals of the chunk [sc][nmo][nvo]
    void *WT;               // weights [nvo][kc_pad], column s * nmo + r
    int nmo, nocc, nvirt;
    int64_t nvo, ldw;
    const double *eps, *omega;      // omega: [sc]
    const double *scale;            // [sc], or null: the weights' factor
    double *epsA;           // [sc][nvirt][nocc + 1]: part A by virtual a: each e_i, then e_a
    double *epsBi;          // [sc][pairs of virtual tiles][nocc]: part B, each e_i
    double *epsBv;          // [sc][pairs][2 * WB]: part B, e_a of the pair's two tiles
    int npairs, p0;         // pairs of virtual tiles, first pair of this launch
};

// part A (fixed virtual a = blockIdx.x, target blockIdx.y), X[i][j] = (qi|aj), d = w + e_a - e_i - e_j:
// 32 x 32 tile pairs (IB <= JB) of X and its transpose through LDS.  W_ij = (4 x - 2 x') / d; with
// u = (2 x - x') x and t_ij = (u_ij + u_ji) / d^2 (symmetric), e_i gets sum_j t_ij and e_a
// -sum_ij u_ij / d^2.
template <typename GT, int WHAT>
__global__ __launch_bounds__(256) void weights_a_kernel(WArgs e)
{
    __shared__ double sh[4];
    __shared__ double eo[1024], ei[1024];
    __shared__ double t1[32][33], t2[32][33];
    const int a = blockIdx.x, s = blockIdx.y, nocc = e.nocc;
    for (int i = threadIdx.x; i < nocc; i += 256) {
        eo[i] = e.eps[i];
        ei[i] = 0.0;
    }
    const double d0 = e.omega[s] + e.eps[nocc + a], gs = e.scale ? e.scale[s] : 1.0;
    const GT *G = (const GT *)e.G + (int64_t)s * e.nmo * e.nvo + (int64_t)a * nocc;     // + i*nvo + j
    GT *WT = (GT *)e.WT + (int64_t)a * nocc * e.ldw + (int64_t)s * e.nmo;               // + j*ldw + i
    double ea = 0.0;
    const int nb = (nocc + 31) / 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int IB = 0; IB < nb; ++IB)
        for (int JB = IB; JB < nb; ++JB) {
            // all loads out before the first is waited for: no branch around them (see part B)
            GT v1[4], v2[4];
            bool in1[4], in2[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = ty + 8 * u;
                const int i1 = IB * 32 + r, j1 = JB * 32 + tx, i2 = JB * 32 + r, j2 = IB * 32 + tx;
                in1[u] = i1 < nocc && j1 < nocc;
                in2[u] = i2 < nocc && j2 < nocc;
                v1[u] = G[in1[u] ? (int64_t)i1 * e.nvo + j1 : 0];                             // X[i1][j1]
                v2[u] = G[in2[u] ? (int64_t)i2 * e.nvo + j2 : 0];                             // X[i2][j2]
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                t1[ty + 8 * u][tx] = in1[u] ? (double)v1[u] : 0.0;
                t2[ty + 8 * u][tx] = in2[u] ? (double)v2[u] : 0.0;
            }
            __syncthreads();
            // element (i, j) = (IB*32 + tx, JB*32 + cj): the weights of both partners, W_ij along i
            // straight out, W_ji (along j) and t_ij back into the tiles
            double tv[4], wv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int cj = ty + 8 * u, i = IB * 32 + tx, j = JB * 32 + cj;
                const bool in = i < nocc && j < nocc;
                const double x = t1[tx][cj], xt = t2[cj][tx];
                const double id = in ? 1.0 / (d0 - eo[i] - eo[j]) : 0.0;
                const double uu = (2.0 * x - xt) * x, ut = (2.0 * xt - x) * xt;
                tv[u] = in ? (uu + ut) * id * id : 0.0;
                wv[u] = gs * (4.0 * xt - 2.0 * x) * id;
                // off the diagonal tile both partners are counted here
                ea -= in ? (IB == JB ? uu : uu + ut) * id * id : 0.0;
                if (WHAT & W_WEIGHTS && in) WT[(int64_t)j * e.ldw + i] = (GT)(gs * (4.0 * x - 2.0 * xt) * id);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (WHAT & W_PARTIALS) t1[tx][ty + 8 * u] = tv[u];
                if (WHAT & W_WEIGHTS) t2[tx][ty + 8 * u] = wv[u];        // W_ji at [i][j]
            }
            __syncthreads();
            if (WHAT & W_WEIGHTS && IB != JB)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = IB * 32 + ty + 8 * u, j = JB * 32 + tx;
                    if (i < nocc && j < nocc) WT[(int64_t)i * e.ldw + j] = (GT)t2[ty + 8 * u][tx];
                }
            if (!(WHAT & W_PARTIALS)) continue;
            // row sums of t to e_i, and off the diagonal tile its column sums to e_j
            if (threadIdx.x < 32) {
                double v = 0.0;
                for (int c = 0; c < 32; ++c) v += t1[threadIdx.x][c];
                if (IB * 32 + (int)threadIdx.x < nocc) ei[IB * 32 + threadIdx.x] += v;
            } else if (threadIdx.x >= 64 && threadIdx.x < 96 && IB != JB) {
                double v = 0.0;
                for (int r = 0; r < 32; ++r) v += t1[r][threadIdx.x - 64];
                if (JB * 32 + (int)threadIdx.x - 64 < nocc) ei[JB * 32 + threadIdx.x - 64] += v;
            }
        }
    if (!(WHAT & W_PARTIALS)) return;
    __syncthreads();
    double *dst = e.epsA + ((int64_t)s * e.nvirt + a) * (nocc + 1);
    for (int i = threadIdx.x; i < nocc; i += 256) dst[i] = ei[i];
    ea = block_sum<256>(ea, sh);
    if (threadIdx.x == 0) dst[nocc] = ea;
}

// part B, Y_i[a][b] = (qa|ib) = G[nocc + a][b nocc + i], d = w + e_i - e_a - e_b: a pair of tiles of WB
// virtuals (TA <= TB) and all i, WB at a time.  e_i gets -sum_ab u_ab / d^2 and e_a sum_b (u_ab +
// u_ba) / d^2.
constexpr int WB = 16, WB_A = WB * WB + 1;      // LDS: [a][b][i], rows of a padded to an odd stride

template <typename GT, int WHAT>
__global__ __launch_bounds__(256) void weights_b_kernel(WArgs e)
{
    __shared__ double y1[WB * WB_A], y2[WB * WB_A];
    __shared__ double sb[WB][WB + 1];
    const int s = blockIdx.y, nocc = e.nocc, nvirt = e.nvirt;
    const int pr = e.p0 + (int)blockIdx.x;                           // the pair
    int TA = 0, p = pr;
    const int nt = (nvirt + WB - 1) / WB;
    while (p >= nt - TA) p -= nt - TA++;
    const int TB = TA + p;
    const bool diag = TA == TB;
    const int a0 = TA * WB, b0 = TB * WB;
    const int lo = threadIdx.x & 15, hi = threadIdx.x >> 4;
    const GT *G = (const GT *)e.G + (int64_t)s * e.nmo * e.nvo;
    GT *WT = (GT *)e.WT + (int64_t)s * e.nmo + nocc;                 // + (b nocc + i) ldw + a
    const double *ev = e.eps + nocc;
    double ea[WB];                                                   // e_a of the pair's first tile
    for (int a = 0; a < WB; ++a) ea[a] = 0.0;
    double eb = 0.0;                                                 // e_b, b = b0 + hi
    const double w0 = e.omega[s], vb = ev[min(b0 + hi, nvirt - 1)], gs = e.scale ? e.scale[s] : 1.0;
    for (int i0 = 0; i0 < nocc; i0 += WB) {
        // thread (b, i) = (hi, lo): every a of the first tile and both partners
        const int i = i0 + lo, b = b0 + hi;
        const bool inb = i < nocc && b < nvirt;
        const double wi = w0 + e.eps[min(i, nocc - 1)] - vb;
        // all loads out before the first is waited for: no branch around them (a branch holds the
        // conversion of a masked FP32 load too, so that each waited for its own: both passes 16.1 ms
        // for 960 orbitals, 16 targets, where the one FP64 pass took 6.2)
        GT yv[WB], yw[WB];
#pragma unroll
        for (int a = 0; a < WB; ++a) {
            const bool in = inb && a0 + a < nvirt;
            yv[a] = G[in ? (int64_t)(nocc + a0 + a) * e.nvo + (int64_t)b * nocc + i : 0];
            yw[a] = G[in ? (int64_t)(nocc + b) * e.nvo + (int64_t)(a0 + a) * nocc + i : 0];
        }
        double si = 0.0;
        __syncthreads();                                             // the tiles of the last round are written out
#pragma unroll
        for (int a = 0; a < WB; ++a) {
            const bool in = inb && a0 + a < nvirt;
            const double id = in ? 1.0 / (wi - ev[min(a0 + a, nvirt - 1)]) : 0.0;
            const double y = in ? (double)yv[a] : 0.0, yt = in ? (double)yw[a] : 0.0;
            const double u = (2.0 * y - yt) * y * id * id, ut = (2.0 * yt - y) * yt * id * id;
            si -= diag ? u : u + ut;
            ea[a] += u + ut;
            eb += u + ut;
            if (WHAT & W_WEIGHTS) {
                y1[a * WB_A + hi * WB + lo] = gs * (4.0 * y - 2.0 * yt) * id;
                y2[a * WB_A + hi * WB + lo] = gs * (4.0 * yt - 2.0 * y) * id;
            }
        }
        if (WHAT & W_PARTIALS) sb[lo][hi] = si;
        __syncthreads();
        // W^T rows (b, i), 16 consecutive a; rows (a, i), 16 consecutive b (thread (i, r) = (hi, lo))
        const int io = i0 + hi;
        if (WHAT & W_WEIGHTS && io < nocc) {
#pragma unroll 4
            for (int c = 0; c < WB; ++c)
                if (a0 + lo < nvirt && b0 + c < nvirt)
                    WT[((int64_t)(b0 + c) * nocc + io) * e.ldw + a0 + lo] = (GT)y1[lo * WB_A + c * WB + hi];
            if (!diag)
#pragma unroll 4
                for (int c = 0; c < WB; ++c)
                    if (b0 + lo < nvirt && a0 + c < nvirt)
                        WT[((int64_t)(a0 + c) * nocc + io) * e.ldw + b0 + lo] = (GT)y2[c * WB_A + lo * WB + hi];
        }
        if (WHAT & W_PARTIALS && threadIdx.x < WB && i0 + (int)threadIdx.x < nocc) {
            double v = 0.0;
            for (int c = 0; c < WB; ++c) v += sb[threadIdx.x][c];
            e.epsBi[((int64_t)s * e.npairs + pr) * nocc + i0 + threadIdx.x] = v;
        }
    }
    if (!(WHAT & W_PARTIALS)) return;
    // e_a: over the 256 threads; e_b: over the 16 threads of b (off the diagonal: the second tile)
    __syncthreads();
#pragma unroll
    for (int a = 0; a < WB; ++a) y1[a * WB_A + threadIdx.x] = ea[a];
    y2[threadIdx.x] = eb;
    __syncthreads();
    if (threadIdx.x < WB) {
        double v = 0.0, x = 0.0;
        for (int c = 0; c < 256; ++c) v += y1[threadIdx.x * WB_A + c];
        for (int c = 0; c < WB; ++c) x += y2[threadIdx.x * WB + c];
        double *dst = e.epsBv + ((int64_t)s * e.npairs + pr) * 2 * WB;
        dst[threadIdx.x] = v;
        dst[WB + threadIdx.x] = diag ? 0.0 : x;
    }
}

// both parts for nsc targets; part B's pairs in launches of at most 2^31 threads (92,673 virtuals
// have 2^24 pairs)
template <typename GT, int WHAT>
int weights(cds_ctx *ctx, WArgs w, int nsc)
{
    hipLaunchKernelGGL((weights_a_kernel<GT, WHAT>), dim3((unsigned)w.nvirt, (unsigned)nsc), dim3(256), 0, ctx->stream, w);
    constexpr int most = 1 << 23;
    for (w.p0 = 0; w.p0 < w.npairs; w.p0 += most)
        hipLaunchKernelGGL((weights_b_kernel<GT, WHAT>), dim3((unsigned)std::min(most, w.npairs - w.p0), (unsigned)nsc), dim3(256), 0,
                           ctx->stream, w);
    CDS_LAUNCHED(ctx);
    return CDS_OK;
}

// scale[s] = omega_bar_s / (1 - Sigma'_s): Sigma' is the sum of part A's e_a and part B's e_i partials
// (each is -sum u / d^2)
__global__ __launch_bounds__(256) void scale_kernel(const double *__restrict__ epsA, const double *__restrict__ epsBi,
                                                    int nocc, int nvirt, int npairs, const double *__restrict__ omega_bar,
                                                    double *__restrict__ scale)
{
    __shared__ double sh[4];
    const int s = blockIdx.x;
    double v = 0.0;
    for (int a = threadIdx.x; a < nvirt; a += 256) v += epsA[((int64_t)s * nvirt + a) * (nocc + 1) + nocc];
    const int64_t n = (int64_t)npairs * nocc;
    constexpr int U = 4;
    for (int64_t q0 = threadIdx.x; q0 < n; q0 += U * 256) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = q0 + u * 256 < n ? epsBi[s * n + q0 + u * 256] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) v += x[u];
    }
    v = block_sum<256>(v, sh);
    if (threadIdx.x == 0) scale[s] = omega_bar[s] / (1.0 - v);
}

// eps_bar[r] = sum_s scale_s (the energy partials of r) + scale_s on e_q: one workgroup per orbital,
// partials in a fixed stride, four loads in flight at a time, summed in a fixed order
__global__ __launch_bounds__(256) void eps_bar_kernel(const double *__restrict__ epsA, const double *__restrict__ epsBi,
                                                      const double *__restrict__ epsBv, int nsel, int nocc, int nvirt,
                                                      int npairs, const int32_t *__restrict__ sel,
                                                      const double *__restrict__ scale, double *__restrict__ out)
{
    __shared__ double sh[4];
    const int r = blockIdx.x, nt = (nvirt + WB - 1) / WB;
    const int ta = (r - nocc) / WB, la = (r - nocc) % WB;            // r >= nocc: its tile and place
    const int per = r < nocc ? nvirt + npairs : nt + 1;              // partials of r per target
    const int64_t n = (int64_t)nsel * per;
    constexpr int U = 4;
    double acc = 0.0;
    for (int64_t q0 = threadIdx.x; q0 < n; q0 += (int64_t)U * 256) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = q0 + (int64_t)u * 256 < n ? q0 + (int64_t)u * 256 : n - 1;
            const int64_t s = q / per;
            const int k = (int)(q - s * per);
            if (r < nocc) {
                v[u] = k < nvirt ? epsA[(s * nvirt + k) * (nocc + 1) + r] : epsBi[(s * npairs + k - nvirt) * nocc + r];
            } else if (k == nt) {
                v[u] = epsA[(s * nvirt + r - nocc) * (nocc + 1) + nocc];
            } else {
                // tile pair (min(ta, k), max(ta, k)): first place where ta is the smaller
                const int lo = ta < k ? ta : k, hi = ta < k ? k : ta;
                const int64_t pr = (int64_t)lo * nt - (int64_t)lo * (lo - 1) / 2 + (hi - lo);
                v[u] = epsBv[(s * npairs + pr) * 2 * WB + (ta <= k ? 0 : WB) + la];
            }
            v[u] *= scale[s];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (q0 + (int64_t)u * 256 < n) acc += v[u];
    }
    for (int s = threadIdx.x; s < nsel; s += 256)
        if (sel[s] == r) acc += scale[s];
    acc = block_sum<256>(acc, sh);
    if (threadIdx.x == 0) out[r] = acc;
}

// B[row][n] = scale[row / per] (1 without scale) sum_b part[b][row][n] in order, n < nvec; 0 for nvec <= n < ldk
template <typename T>
__global__ __launch_bounds__(256) void sum_scaled_kernel(const T *__restrict__ part, int nb, int64_t rows, int64_t nvec,
                                                         int64_t per, const double *__restrict__ scale,
                                                         T *__restrict__ B, int64_t ldk)
{
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < rows * ldk; t += (int64_t)gridDim.x * 256) {
        const int64_t row = t / ldk, n = t - row * ldk;
        double v = 0.0;
        if (n < nvec) {
            for (int b = 0; b < nb; ++b) v += (double)part[(int64_t)b * rows * nvec + row * nvec + n];
            if (scale) v *= scale[row / per];
        }
        B[t] = (T)v;
    }
}

// CX[x][nu] = C[nu][sel or occupied orbital of row x] (x < nocc: occupied x; xo <= x < xo + nsel:
// target x - xo; other rows and nu >= nbf: 0), and Ccat[nu][c] = C[nu][nocc + c] for c < nvirt,
// C[nu][c - ap] for ap <= c < ap + nocc, else 0 (and 0 for nbf <= nu < np_: the product with it
// reads np_ rows, and columns of Y that are not 0 there would meet the zeros of L as NaN)
__global__ void coef_adj_kernel(const double *__restrict__ C, int nbf, int nmo, int nocc, int nsel,
                                const int32_t *__restrict__ sel, int np_, int xo, int xp, int ap, int cp,
                                double *__restrict__ CX, double *__restrict__ Ccat)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, n1 = (int64_t)xp * np_;
    if (t < n1) {
        const int x = (int)(t / np_), nu = (int)(t - (int64_t)x * np_);
        const int q = x < nocc ? x : (x >= xo && x < xo + nsel ? sel[x - xo] : -1);
        CX[t] = q >= 0 && nu < nbf ? C[(int64_t)nu * nmo + q] : 0.0;
    } else if (t - n1 < (int64_t)np_ * cp) {
        const int64_t u = t - n1;
        const int nu = (int)(u / cp), c = (int)(u - (int64_t)nu * cp);
        const int q = c < nmo - nocc ? nocc + c : (c >= ap && c < ap + nocc ? c - ap : -1);
        Ccat[u] = q >= 0 && nu < nbf ? C[(int64_t)nu * nmo + q] : 0.0;
    }
}

// out[z oz + kb ok + x] = in[z iz + x ix + kb] (FP64) for kb < nkb, x < nx, and 0 for nx <= x < nxp, for
// the six pieces of a batch's cotangents in one launch, z running through them (gradients of 47
// orbitals, FP32, against the full symmetric cotangent: 610 / 537 us with six launches, with one
// launch and one copy of the solve's inputs 630 / 678 us on a slower box): 32 x 32 tiles through LDS,
// every load of a thread in flight before its stores
struct BarPiece {
    const void *in;
    int64_t iz, ix, oz, ok;
    int nz, nx, nxp;
    double *out;
};
constexpr int BAR_PIECES = 6;
struct BarArgs {
    BarPiece p[BAR_PIECES];
};

template <typename BT>
__global__ __launch_bounds__(256) void bar_transpose_kernel(BarArgs a, int nkb, int nz)
{
    __shared__ double t[32][33];
    const int x0 = blockIdx.y * 32, k0 = blockIdx.x * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int zz = blockIdx.z; zz < nz; zz += gridDim.z) {
        int z = zz, q = 0;
        while (z >= a.p[q].nz) z -= a.p[q++].nz;
        const BarPiece &e = a.p[q];
        if (x0 >= e.nxp) continue;                                   // (the same for the whole workgroup)
        const BT *src = (const BT *)e.in + z * e.iz;
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int x = x0 + ty + 8 * u, k = k0 + tx;
            v[u] = x < e.nx && k < nkb ? (double)src[x * e.ix + k] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) t[ty + 8 * u][tx] = v[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + ty + 8 * u, x = x0 + tx;
            if (k < nkb && x < e.nxp) e.out[z * e.oz + k * e.ok + x] = t[tx][ty + 8 * u];
        }
    }
}

// The full symmetric cotangent of small systems: S[kb][p][q] = Bbar^K[p][q] + Bbar^K[q][p] (FP64),
// Bbar scattered from the sel and vo blocks, and 0 for the columns nbf <= nu < np_ of Wt[kb][p][nu],
// which the product that forms Wt does not write
template <typename BT>
__global__ __launch_bounds__(256) void sym_bar_kernel(const BT *__restrict__ bsel, const BT *__restrict__ bvo, int64_t ldk,
                                                      int64_t k0, int nkb, int nbf, int np_, int nmo, int nocc, int nsel,
                                                      const int32_t *__restrict__ sel, double *__restrict__ S,
                                                      double *__restrict__ Wt)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int per = nmo * (nmo + np_ - nbf);
    if (t >= (int64_t)per * nkb) return;
    const int kb = (int)(t / per), e = (int)(t - (int64_t)kb * per);
    const int p = e / (nmo + np_ - nbf), q = e - p * (nmo + np_ - nbf);
    if (q >= nmo) {
        Wt[((int64_t)kb * nmo + p) * np_ + nbf + q - nmo] = 0.0;
        return;
    }
    const int64_t K = k0 + kb;
    double v = 0.0;
    for (int s = 0; s < nsel; ++s) {
        if (sel[s] == p) v += (double)bsel[((int64_t)s * nmo + q) * ldk + K];
        if (sel[s] == q) v += (double)bsel[((int64_t)s * nmo + p) * ldk + K];
    }
    if (p >= nocc && q < nocc) v += (double)bvo[((int64_t)(p - nocc) * nocc + q) * ldk + K];
    if (q >= nocc && p < nocc) v += (double)bvo[((int64_t)(q - nocc) * nocc + p) * ldk + K];
    S[((int64_t)kb * nmo + p) * nmo + q] = v;
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

    // working copies: float operands for BF16X3 (planes -> float)
    const int gprec = prec == CDS_PREC_FP64 ? CDS_PREC_FP64 : CDS_PREC_FP32;
    const size_t es = prec == CDS_PREC_FP64 ? 8 : 4;
    const void *Bs = Bsel, *Bv = Bvo;
    void *tmp;
    size_t nB = (size_t)(nselr + nvo) * ldk;
    const int nt = (nvirt + WB - 1) / WB, npairs = nt * (nt + 1) / 2;
    size_t small = (size_t)nsel * 8 * 3 + (size_t)nsel * 4 + 256;
    size_t epsbytes = (size_t)nsel * 8 * ((size_t)nvirt * (nocc + 1) + (size_t)npairs * (nocc + 2 * WB));
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
    double *d_obar = d_omega + nsel;
    int32_t *d_sel = (int32_t *)(d_obar + nsel);       // (to here: one copy from the host)
    double *d_scale = (double *)(d_sel + nsel + nsel % 2);
    double *epsA = (double *)(tp + (small + 7) / 8 * 8);
    double *epsBi = epsA + (size_t)nsel * nvirt * (nocc + 1);
    double *epsBv = epsBi + (size_t)nsel * npairs * nocc;
    std::vector<unsigned char> hin((size_t)nsel * 20);
    std::memcpy(hin.data(), h_omega, (size_t)nsel * 8);
    std::memcpy(hin.data() + (size_t)nsel * 8, h_omega_bar, (size_t)nsel * 8);
    std::memcpy(hin.data() + (size_t)nsel * 16, h_sel, (size_t)nsel * 4);
    CDS_HIP(ctx, hipMemcpyAsync(d_omega, hin.data(), hin.size(), hipMemcpyHostToDevice, ctx->stream));

    // chunks of targets: G and W^T each nsc * nmo * nvo, at most 12 GiB each (few, large chunks: the
    // product over nvo below has only nsc * nmo / 128 tile rows)
    const size_t per = (size_t)nmo * nvo * es;
    int csz = (int)std::max<size_t>(1, ((size_t)12 << 30) / std::max<size_t>(per, 1));
    if (ctx->target_chunk > 0) csz = std::min(csz, ctx->target_chunk);
    csz = std::min(csz, (int)nsel);
    // K padding of the products (their stage holds 16 FP64 or 32 FP32 k): the sum over v in S parts of
    // vp (the tiles of Bsel_bar alone do not fill the chip: 360 of 512 workgroups for 480 orbitals,
    // 12 targets, 930 vectors), the sum over (s, r) to kcp.  S: the fewest rounds of 512 workgroups
    // per part, each part adding a pass over its result.  FP32 sums in one part: its rounding is that
    // of one sum over v of weights rounded with their scale, so the weights pass runs a second time
    // there, once the pole strengths are known
    const int64_t ks = es == 8 ? 16 : 32;
    auto up = [&](int64_t n) { return cds_ceil_div(n, ks) * ks; };
    int S = 1;
    if (es == 8) {
        const int64_t tiles = cds_ceil_div((int64_t)csz * nmo, 128) * cds_ceil_div(nvec, 128);
        double best = 0.0;
        for (int c = 1; c <= 16 && (c == 1 || nvo / c >= 512); ++c) {
            if (c > 1 && c * up(cds_ceil_div(nvo, c)) > (int64_t)65535 * 32) continue;   // (cds_transpose's rows)
            const double cost = (double)cds_ceil_div(tiles * c, 512) / c * (1.0 + 0.01 * c);
            if (c == 1 || cost < best) {
                best = cost;
                S = c;
            }
        }
    }
    const int64_t vp = up(cds_ceil_div(nvo, S)), nvp = S * vp;
    const int64_t kcp = up((int64_t)csz * nmo);
    void *G, *WT, *BvT, *BsT, *part;
    CDS_CALL(cds_ws(ctx, WS_SG_G, (size_t)csz * per, &G));
    CDS_CALL(cds_ws(ctx, WS_AD_G, (size_t)nvp * kcp * es, &WT));
    CDS_CALL(cds_ws(ctx, WS_AD_T1, (size_t)nvec * nvp * es, &BvT));                 // Bvo^T
    CDS_CALL(cds_ws(ctx, WS_AD_T2, (size_t)S * csz * nmo * nvec * es, &part));      // Bsel_bar's parts
    CDS_CALL(cds_ws(ctx, WS_AD_T3, (size_t)nvec * kcp * es, &BsT));                 // the chunk's scaled Bsel^T
    CDS_CALL(cds_transpose(ctx, (int)es, nvo, nvec, Bv, ldk, BvT, nvp));
    for (int s0 = 0; s0 < nsel; s0 += csz) {
        const int nsc = std::min(csz, nsel - s0);
        const int64_t kc = (int64_t)nsc * nmo, kp = up(kc);
        CDS_CALL(cds_contract_internal(ctx, prec, nvec, ldk, nmo, nocc, nsel, Bsel, Bvo, s0, nsc, G));
        WArgs w = {};
        w.G = G;
        w.WT = WT;
        w.nmo = nmo;
        w.nocc = nocc;
        w.nvirt = nvirt;
        w.nvo = nvo;
        w.ldw = kp;
        w.eps = eps;
        w.omega = d_omega + s0;
        w.epsA = epsA + (size_t)s0 * nvirt * (nocc + 1);
        w.epsBi = epsBi + (size_t)s0 * npairs * nocc;
        w.epsBv = epsBv + (size_t)s0 * npairs * 2 * WB;
        w.npairs = npairs;
        if (es == 8) {
            CDS_CALL((weights<double, W_WEIGHTS | W_PARTIALS>(ctx, w, nsc)));
            CDS_CALL(zero_cols(ctx, (double *)WT, nvo, kp, kc));
            CDS_CALL(zero_cols(ctx, (double *)WT + nvo * kp, nvp - nvo, kp, (int64_t)0));
        } else {
            CDS_CALL((weights<float, W_PARTIALS>(ctx, w, nsc)));
        }
        hipLaunchKernelGGL(scale_kernel, dim3((unsigned)nsc), dim3(256), 0, ctx->stream, (const double *)w.epsA,
                           (const double *)w.epsBi, nocc, nvirt, npairs, (const double *)d_obar + s0, d_scale + s0);
        if (es == 4) {
            w.scale = d_scale + s0;
            CDS_CALL((weights<float, W_WEIGHTS>(ctx, w, nsc)));
            CDS_CALL(zero_cols(ctx, (float *)WT, nvo, kp, kc));
            CDS_CALL(zero_cols(ctx, (float *)WT + nvo * kp, nvp - nvo, kp, (int64_t)0));
        }
        CDS_LAUNCHED(ctx);
        // Bsel_bar[s0..] = scale W Bvo :  (nsc*nmo) x nvec, reduction over nvo in S parts
        GemmDesc d1 = {};
        d1.M = kc; d1.N = nvec; d1.K = vp; d1.batch = S; d1.ka = 1;
        d1.A = WT; d1.sAm = 1; d1.sAk = kp; d1.sAb = vp * kp;
        d1.B = BvT; d1.sBk = 1; d1.sBn = nvp; d1.sBb = vp;
        d1.C = part; d1.sCm = nvec; d1.sCn = 1; d1.sCb = kc * nvec;
        d1.alpha = 1.0; d1.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, gprec, d1, nullptr, nullptr));
        const dim3 gs(cds_stride_grid(kc * ldk));
        void *out = (unsigned char *)Bsel_bar + (size_t)s0 * nmo * ldk * es;
        if (es == 8)
            hipLaunchKernelGGL(sum_scaled_kernel<double>, gs, dim3(256), 0, ctx->stream, (const double *)part, S, kc, nvec,
                               (int64_t)nmo, (const double *)d_scale + s0, (double *)out, ldk);
        else
            hipLaunchKernelGGL(sum_scaled_kernel<float>, gs, dim3(256), 0, ctx->stream, (const float *)part, S, kc, nvec,
                               (int64_t)nmo, (const double *)nullptr, (float *)out, ldk);
        CDS_LAUNCHED(ctx);
        // Bvo_bar += W^T (scale Bsel[s0..]) : nvo x nvec, reduction over nsc*nmo
        CDS_CALL(cds_transpose(ctx, (int)es, kc, nvec, (const unsigned char *)Bs + (size_t)s0 * nmo * ldk * es, ldk,
                               BsT, kp, es == 8 ? d_scale + s0 : nullptr, nmo));
        GemmDesc d2 = {};
        d2.M = nvo; d2.N = nvec; d2.K = kp; d2.batch = 1;
        d2.A = WT; d2.sAm = kp; d2.sAk = 1;
        d2.B = BsT; d2.sBk = 1; d2.sBn = kp;
        d2.C = Bvo_bar; d2.sCm = ldk; d2.sCn = 1;
        d2.alpha = 1.0; d2.beta = s0 == 0 ? 0.0 : 1.0;
        CDS_CALL(cds_gemm_ex(ctx, gprec, d2, nullptr, nullptr));
    }
    if (es == 8) CDS_CALL(zero_cols(ctx, (double *)Bvo_bar, nvo, ldk, nvec));
    else CDS_CALL(zero_cols(ctx, (float *)Bvo_bar, nvo, ldk, nvec));
    hipLaunchKernelGGL(eps_bar_kernel, dim3((unsigned)nmo), dim3(256), 0, ctx->stream, (const double *)epsA,
                       (const double *)epsBi, (const double *)epsBv, nsel, nocc, nvirt, npairs, (const int32_t *)d_sel,
                       (const double *)d_scale, eps_bar);
    CDS_LAUNCHED(ctx);
    CDS_CALL(cds_timer_stop(ctx, &tall, &ctx->stats.t_adjoint_ms));
    CDS_CALL(cds_timers_flush(ctx));
    return CDS_OK;
}

namespace {

// C_bar = sum_K L^K (C S^K), S^K = Bbar^K + Bbar^K^T in full: two products and three small kernels
int transform_adjoint_full(cds_ctx *ctx, int prec, int nbf, int64_t nvec, const double *L, int64_t ldl, const double *C, int nmo,
                           int nocc, int nsel, const int32_t *h_sel, int64_t ldk, const void *Bsel_bar, const void *Bvo_bar,
                           double *C_bar)
{
    const int np_ = (int)(cds_ceil_div(nbf, 32) * 32);
    // vectors per batch: enough that the first product launches about 2048 tiles, the unpacked batch
    // below 1 GiB (C_bar sums the vectors in order whatever the batch)
    const int64_t tiles = cds_ceil_div(nmo, 128) * cds_ceil_div(nbf, 128);
    int64_t kbw = std::max<int64_t>(64, cds_ceil_div(2048, tiles));
    kbw = std::min<int64_t>(kbw, std::max<int64_t>(1, (int64_t)((1ull << 30) / ((size_t)nbf * np_ * 8))));
    const int kb = (int)std::min<int64_t>(kbw, nvec);
    void *wl, *ws, *wk, *wsel, *wp;
    CDS_CALL(cds_ws(ctx, WS_TR_UNPACK, (size_t)kb * nbf * np_ * 8, &wl));
    CDS_CALL(cds_ws(ctx, WS_AD_TMP2, (size_t)kb * nmo * nmo * 8, &ws));
    CDS_CALL(cds_ws(ctx, WS_TR_T, (size_t)kb * nmo * np_ * 8, &wk));
    CDS_CALL(cds_ws(ctx, WS_TR_CX, (size_t)nsel * 4 + 64, &wsel));
    CDS_CALL(cds_ws(ctx, WS_AD_TMP, (size_t)kb * nbf * nmo * 8, &wp));
    CDS_HIP(ctx, hipMemcpyAsync(wsel, h_sel, (size_t)nsel * 4, hipMemcpyHostToDevice, ctx->stream));
    for (int64_t k0 = 0; k0 < nvec; k0 += kb) {
        const int nkb = (int)std::min<int64_t>(kb, nvec - k0);
        CDS_CALL(cds_unpack64(ctx, L, ldl, k0, nkb, nbf, np_, (double *)wl));
        const dim3 g((unsigned)cds_ceil_div((int64_t)nkb * nmo * (nmo + np_ - nbf), 256));
        if (prec == CDS_PREC_FP64)
            hipLaunchKernelGGL(sym_bar_kernel<double>, g, dim3(256), 0, ctx->stream, (const double *)Bsel_bar,
                               (const double *)Bvo_bar, ldk, k0, nkb, nbf, np_, nmo, nocc, nsel, (const int32_t *)wsel,
                               (double *)ws, (double *)wk);
        else
            hipLaunchKernelGGL(sym_bar_kernel<float>, g, dim3(256), 0, ctx->stream, (const float *)Bsel_bar,
                               (const float *)Bvo_bar, ldk, k0, nkb, nbf, np_, nmo, nocc, nsel, (const int32_t *)wsel,
                               (double *)ws, (double *)wk);
        CDS_LAUNCHED(ctx);
        // Wt[kb][p][nu] = sum_r S[kb][p][r] C[nu][r]   (S symmetric; both operands K-contiguous)
        GemmDesc g1 = {};
        g1.M = nmo; g1.N = nbf; g1.K = nmo; g1.batch = nkb;
        g1.A = ws; g1.sAm = nmo; g1.sAk = 1; g1.sAb = (int64_t)nmo * nmo;
        g1.B = C; g1.sBn = nmo; g1.sBk = 1; g1.sBb = 0;
        g1.C = wk; g1.sCm = np_; g1.sCn = 1; g1.sCb = (int64_t)nmo * np_;
        g1.alpha = 1.0; g1.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, CDS_PREC_FP64, g1, nullptr, nullptr));
        // part[kb][mu][p] = sum_nu Lu[kb][mu][nu] Wt[kb][p][nu], then C_bar (+)= sum_kb part[kb]
        GemmDesc g2 = {};
        g2.M = nbf; g2.N = nmo; g2.K = np_; g2.batch = nkb;
        g2.A = wl; g2.sAm = np_; g2.sAk = 1; g2.sAb = (int64_t)nbf * np_;
        g2.B = wk; g2.sBn = np_; g2.sBk = 1; g2.sBb = (int64_t)nmo * np_;
        g2.C = wp; g2.sCm = nmo; g2.sCn = 1; g2.sCb = (int64_t)nbf * nmo;
        g2.alpha = 1.0; g2.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, CDS_PREC_FP64, g2, nullptr, nullptr));
        const int64_t ne = (int64_t)nbf * nmo;
        hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)cds_ceil_div(ne, 256)), dim3(256), 0, ctx->stream,
                           (const double *)wp, nkb, ne, k0 > 0 ? 1 : 0, C_bar);
        CDS_LAUNCHED(ctx);
    }
    return CDS_OK;
}

}  // namespace

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
    // Small systems take the full symmetric cotangent: five launches against twelve, and products that
    // one tile per vector holds save nothing by leaving rows out.  Per call, full / rows only, nocc =
    // n / 4, 2 targets: 8 functions, 24 vectors 32 / 58 us; 45, 135: 55 / 102; 96, 288: 113 / 196; 128,
    // 896: 370 / 447; 130, 130: 210 / 171 (nmo off the multiples of 16 takes the general product);
    // 144, 432 (5.2e9 operations): 317 / 330; 160, 480 (7.9e9): 370 / 373; 192, 576 (16e9): 703 / 536
    if (nbf <= 128 || (nmo % 16 == 0 && 4.0 * nmo * nbf * (double)nbf * (double)nvec < 5.5e9)) {
        CDS_CALL(transform_adjoint_full(ctx, prec, nbf, nvec, L, ldl, C, nmo, nocc, nsel, h_sel, ldk, Bsel_bar, Bvo_bar, C_bar));
        CDS_CALL(cds_timer_stop(ctx, &tall, &ctx->stats.t_adjoint_ms));
        return CDS_OK;
    }
    auto up16 = [](int64_t n) { return (int)(cds_ceil_div(n, 16) * 16); };
    const int np_ = (int)(cds_ceil_div(nbf, 32) * 32);
    const int xo = up16(nocc), selp = up16(nsel), xp = xo + selp;    // rows x: occupied, then targets
    const int ap = up16(nvirt), cp = ap + up16(nocc);                // columns: virtual, then occupied
    // vectors per batch: the largest of the batch's arrays stays below 1 GiB
    const int64_t per = 8 * std::max<int64_t>((int64_t)nbf * np_, std::max<int64_t>((int64_t)xp * np_, (int64_t)nmo * xp));
    int kb = (int)std::min<int64_t>(std::min<int64_t>(nvec, 8192), std::max<int64_t>(1, (int64_t)(1ull << 30) / per));
    // runs of vectors per product, so that each product launches about 1024 tiles
    auto run_of = [&](int64_t n) {
        const int64_t tiles = cds_ceil_div(nbf, 128) * cds_ceil_div(n, 128);
        return std::max<int64_t>(1, kb * tiles / 1024);
    };
    auto runs = [](int64_t nkb, int64_t run) { return cds_ceil_div(nkb, run); };
    int64_t rv, ro, r2;
    size_t nzv, nzo, nzr, nzs;                                                          // see below
    void *wl, *wt, *wz, *wy, *wc, *wp;
    auto alloc = [&]() -> int {
        rv = run_of(nvirt), ro = run_of(nocc), r2 = run_of(xp);
        nzv = (size_t)nvirt * kb * xp, nzo = (size_t)nocc * kb * selp;                  // Zv[a][kb][x], Zo[r][kb][s]
        nzr = (size_t)nocc * kb * ap, nzs = (size_t)nsel * kb * cp;                     // Zr[i][kb][a], Zs[s][kb][c]
        const int64_t npart = std::max({runs(kb, rv) * nbf * nvirt, runs(kb, ro) * nbf * nocc, runs(kb, r2) * nbf * xp});
        CDS_CALL(cds_ws(ctx, WS_TR_UNPACK, (size_t)kb * nbf * np_ * 8, &wl));
        CDS_CALL(cds_ws(ctx, WS_TR_T, (size_t)kb * nbf * xp * 8, &wt));                 // T[mu][kb][x]
        CDS_CALL(cds_ws(ctx, WS_AD_TMP2, (nzv + nzo + nzr + nzs) * 8, &wz));
        CDS_CALL(cds_ws(ctx, WS_AD_T1, (size_t)xp * kb * np_ * 8, &wy));                // Y[x][kb][nu]
        return cds_ws(ctx, WS_AD_TMP, (size_t)npart * 8, &wp);
    };
    // smaller batches where the device has no room for these
    int rc = alloc();
    while (rc == CDS_ENOMEM && kb > 1) {
        for (const int slot : {WS_TR_UNPACK, WS_TR_T, WS_AD_TMP2, WS_AD_T1, WS_AD_TMP}) CDS_CALL(cds_ws_release(ctx, slot));
        kb = (kb + 1) / 2;
        rc = alloc();
    }
    CDS_CALL(rc);
    ctx->err.clear();
    const size_t ncx = (size_t)xp * np_, nccat = (size_t)np_ * cp, nsum = (size_t)nbf * (nmo + xp);
    CDS_CALL(cds_ws(ctx, WS_TR_CX, (ncx + nccat + nsum) * 8 + (size_t)nsel * 4 + 64, &wc));
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
    auto bar = [&](const void *blk, int64_t row0, int64_t iz, int64_t ix, int nz, int nx, int nxp, double *out, int64_t oz,
                   int64_t ok, int64_t k0) {
        return BarPiece{(const unsigned char *)blk + (size_t)(row0 * ldk + k0) * bes, iz * ldk, ix * ldk, oz, ok, nz, nx, nxp,
                        out};
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
        CDS_CALL(cds_unpack64(ctx, L, ldl, k0, nkb, nbf, np_, Lu));
        // T[mu][kb][x] = sum_nu L^K[mu][nu] CX[x][nu]
        GemmDesc gt = {};
        gt.M = nbf; gt.N = xp; gt.K = np_; gt.batch = nkb;
        gt.A = Lu; gt.sAm = np_; gt.sAk = 1; gt.sAb = (int64_t)nbf * np_;
        gt.B = CX; gt.sBn = np_; gt.sBk = 1; gt.sBb = 0;
        gt.C = T; gt.sCm = (int64_t)nkb * xp; gt.sCn = 1; gt.sCb = xp;
        gt.alpha = 1.0; gt.beta = 0.0;
        CDS_CALL(cds_gemm_ex(ctx, CDS_PREC_FP64, gt, nullptr, nullptr));
        // the cotangents with x along the rows (Zv: virtual columns a, occupied rows then targets; Zo:
        // the targets' occupied columns) and with r along the rows (Zr, Zs)
        const int64_t zs = (int64_t)nkb * xp;
        const BarArgs ba = {{bar(Bvo_bar, 0, nocc, 1, nvirt, nocc, xo, Zv, zs, xp, k0),
                             bar(Bsel_bar, nocc, 1, nmo, nvirt, nsel, selp, Zv + xo, zs, xp, k0),
                             bar(Bsel_bar, 0, 1, nmo, nocc, nsel, selp, Zo, (int64_t)nkb * selp, selp, k0),
                             bar(Bvo_bar, 0, 1, nocc, nocc, nvirt, ap, Zr, (int64_t)nkb * ap, ap, k0),
                             bar(Bsel_bar, nocc, nmo, 1, nsel, nvirt, ap, Zs, (int64_t)nkb * cp, cp, k0),
                             bar(Bsel_bar, 0, nmo, 1, nsel, nocc, cp - ap, Zs + ap, (int64_t)nkb * cp, cp, k0)}};
        int nz = 0, nxm = 0;
        for (const BarPiece &e : ba.p) {
            nz += e.nz;
            nxm = std::max(nxm, e.nxp);
        }
        const dim3 gb((unsigned)cds_ceil_div(nkb, 32), (unsigned)cds_ceil_div(nxm, 32), (unsigned)std::min(nz, 65535));
        if (prec == CDS_PREC_FP64)
            hipLaunchKernelGGL(bar_transpose_kernel<double>, gb, dim3(256), 0, ctx->stream, ba, nkb, nz);
        else
            hipLaunchKernelGGL(bar_transpose_kernel<float>, gb, dim3(256), 0, ctx->stream, ba, nkb, nz);
        CDS_LAUNCHED(ctx);
        // C_bar_r += sum T Z
        CDS_CALL(summed(nvirt, xp, nkb, rv, T, zs, xp, Zv, zs, xp, k0 > 0, Pv));
        CDS_CALL(summed(nocc, selp, nkb, ro, T + xo, zs, xp, Zo, (int64_t)nkb * selp, selp, k0 > 0, Po));
        // Y[x][kb][nu] = sum_r Z[x][kb][r] C[nu][r], then C_bar_x += sum L Y
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
