// Non-diagonal second-order self-energy over selected orbitals and the Dyson pole
// search (Sec. II.B of the paper: Eqs. (Dyson), (DysonSol), (DysonSol2); Eq. (SE) is the
// diagonal of this matrix):
//   Sigma_st(w) = sum_{a,i,j} (si|aj) (2(ti|aj) - (tj|ai)) / (w + e_a - e_i - e_j)
//               + sum_{i,a,b} (sa|ib) (2(ta|ib) - (tb|ia)) / (w + e_i - e_a - e_b).
// The integrals of all selected orbitals come from one MFMA contraction
// G[s][r][a*nocc+j] = (s r|a j).  Both families are summed over unordered index pairs
// (d is symmetric in i, j and in a, b): element e = (a; i <= j) or (i; a <= b) carries
//   u_s = (si|aj), v_s = (sj|ai)   resp.   u_s = (sa|ib), v_s = (sb|ia),
// and contributes c_e (2 u_s u_t + 2 v_s v_t - u_s v_t - v_s u_t) / (w + d_e) to Sigma_st,
// with c_e = 1/2 on the diagonal (i = j, a = b) and 1 otherwise: over the pairs (s <= t) and the trial
// energies that is a product num[pair][e] weight[e][energy] summed over the elements, which
// sigma_pairs_kernel gives to FP64 MFMA; per-block partial sums are reduced in a fixed order.
//
// The Dyson search (steps on the device, dyson_step_kernel; the host follows the statuses): one
// root per selected orbital, started at e_q with u = unit vector q; at each step the
// symmetric matrix diag(e_S) + Sigma_SS(w) is diagonalised (Jacobi), the
// eigenvector of largest overlap with the previous one is followed, and
//   w <- w + (lambda - w) P,   P = 1 / (1 - u^T Sigma'(w) u)
// until |dw| <= conv (Eq. (NR)); P is the pole strength.  With one orbital this is Eq. (iter).
#include "cds_internal.h"

#include <cmath>
#include <vector>

int cds_contract_internal(cds_ctx *ctx, int prec, int64_t nvec, int64_t ldk, int nmo, int nocc,
                          int nsel, const void *Bsel, const void *Bvo, int s0, int nsc, void *G);

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int DY_NT = 256;
constexpr int DY_CH = 64;            // elements per chunk
constexpr int DY_P = DY_CH + 2;      // LDS row pitch: 16-byte reads of 8 rows fall into distinct banks
constexpr int DY_MAXSEL = 31;        // selected orbitals
constexpr int DY_TT = 16;            // trial energies per launch
constexpr int DY_BLOCKS = 512;       // workgroups (two per CU)
constexpr size_t DY_G_MAX = (size_t)16 << 30;

__device__ __forceinline__ int64_t tri_hi(int64_t x)
{
    // largest b with b(b+1)/2 <= x
    int64_t b = (int64_t)((sqrt(8.0 * (double)x + 1.0) - 1.0) * 0.5);
    if (b * (b + 1) / 2 > x) --b;
    if ((b + 1) * (b + 2) / 2 <= x) ++b;
    return b;
}

// Chunks of 64 elements, taken in turn by the workgroups: part A, virtual a, an 8 x 8 tile of (i, j)
// (IB <= JB); then part B, virtual a, 64 consecutive (b, i) of row a (chunks wholly below b = a are
// passed over).  Both families' integrals are read in runs: u of part B 512 bytes, of part A 64
// bytes, v at least 64 bytes (elements in the order (i <= j; a), (a <= b; i) read 8 bytes per line:
// 894 us per launch for 16 of 240 orbitals, 120 occupied; this order and the MFMA form 490 us for twice the energies).
// A chunk's u and v of every orbital and its weights are staged in LDS; a wave owns blocks of 16
// pairs: lane (r, g) forms num of pair r for elements 8h + 2g and 8h + 2g + 1 (MFMA operand A) and
// reads the same elements' weights of energy column r (operand B).  Columns: 2t Sigma, 2t + 1 Sigma'.
// NB: pair blocks per wave (4 waves); NC: column blocks of 8 energies.
template <typename GT, int NB, int NC>
__global__ __launch_bounds__(DY_NT, 2) void sigma_pairs_kernel(const GT *__restrict__ G, int nsel, int nmo, int nocc,
                                                              int nvirt, int64_t nvo, const double *__restrict__ eps,
                                                              const double *__restrict__ omega,
                                                              const int *__restrict__ list, int T, int64_t nchA,
                                                              int64_t nch, int nchB, double *__restrict__ part)
{
    extern __shared__ __align__(16) double lds[];
    double *su = lds, *sv = su + nsel * DY_P, *sw = sv + nsel * DY_P;      // [nsel][DY_P] x 2, [16 NC][DY_P]
    int64_t *ou = (int64_t *)(sw + 16 * NC * DY_P), *ov = ou + DY_CH;
    double *sd = (double *)(ov + DY_CH), *sc = sd + DY_CH;
    const int npair = nsel * (nsel + 1) / 2;
    const int64_t gstride = (int64_t)nmo * nvo;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane >> 4, r16 = lane & 15;
    // pair of this lane in each block of its wave (blocks wave, wave + 4, ...): LDS rows of s and t
    int as[NB], at[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int P = min((wave + 4 * b) * 16 + r16, npair - 1);
        const int t = (int)tri_hi(P);
        as[b] = (P - t * (t + 1) / 2) * DY_P + 2 * g;
        at[b] = t * DY_P + 2 * g;
    }
    doublex4 acc[NB][NC];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[b][c] = doublex4{0.0, 0.0, 0.0, 0.0};
    const int nt8 = (nocc + 7) / 8, ntri = nt8 * (nt8 + 1) / 2;
    for (int64_t c = blockIdx.x; c < nch; c += gridDim.x) {
        const bool partA = c < nchA;
        int a, JB = 0, IB = 0;
        int64_t q0 = 0;
        if (partA) {
            a = (int)(c / ntri);
            const int p = (int)(c - (int64_t)a * ntri);
            JB = (int)tri_hi(p);
            IB = p - JB * (JB + 1) / 2;
        } else {
            const int64_t f = c - nchA;
            a = (int)(f / nchB);
            q0 = (f - (int64_t)a * nchB) * DY_CH;
            if (q0 + DY_CH <= (int64_t)a * nocc) continue;         // wholly below b = a
        }
        __syncthreads();                                           // the last chunk is read
        if (threadIdx.x < DY_CH) {
            const int l = threadIdx.x;
            int64_t offu = 0, offv = 0;
            double d = 0.0, ce = 0.0;
            if (partA) {
                const int i = IB * 8 + (l >> 3), j = JB * 8 + (l & 7);
                if (j < nocc && i <= j) {
                    offu = i * nvo + (int64_t)a * nocc + j;
                    offv = j * nvo + (int64_t)a * nocc + i;
                    d = eps[nocc + a] - eps[i] - eps[j];
                    ce = i == j ? 0.5 : 1.0;
                }
            } else {
                const int64_t q = q0 + l;
                const int b = (int)(q / nocc), i = (int)(q - (int64_t)b * nocc);
                if (b < nvirt && b >= a) {
                    offu = (nocc + a) * nvo + q;
                    offv = (int64_t)(nocc + b) * nvo + (int64_t)a * nocc + i;
                    d = eps[i] - eps[nocc + a] - eps[nocc + b];
                    ce = a == b ? 0.5 : 1.0;
                }
            }
            ou[l] = offu;
            ov[l] = offv;
            sd[l] = d;
            sc[l] = ce;
        }
        __syncthreads();
        {
            // every gathered load of a thread in flight before its LDS stores; elements that do not
            // count (weight 0) read as 0
            constexpr int QN = (DY_MAXSEL * DY_CH + DY_NT - 1) / DY_NT;
            const int l = threadIdx.x & (DY_CH - 1), s0 = threadIdx.x / DY_CH;
            const bool on = sc[l] != 0.0;
            const GT *pu = G + ou[l], *pv = G + ov[l];
            double gu[QN], gv[QN];
#pragma unroll
            for (int u = 0; u < QN; ++u) {
                const int s = s0 + 4 * u;
                const bool ok = on && s < nsel;
                gu[u] = ok ? (double)pu[s * gstride] : 0.0;
                gv[u] = ok ? (double)pv[s * gstride] : 0.0;
            }
            // weights: thread (l, t) of energies t = s0, s0 + 4, ...
#pragma unroll
            for (int t = s0; t < 8 * NC; t += 4) {
                const double inv = on && t < T ? 1.0 / (omega[list ? list[t] : t] + sd[l]) : 0.0;
                const double w = sc[l] * inv;
                sw[2 * t * DY_P + l] = w;
                sw[(2 * t + 1) * DY_P + l] = -w * inv;
            }
#pragma unroll
            for (int u = 0; u < QN; ++u) {
                const int s = s0 + 4 * u;
                if (s < nsel) {
                    su[s * DY_P + l] = gu[u];
                    sv[s * DY_P + l] = gv[u];
                }
            }
        }
        __syncthreads();
        for (int h = 0; h < DY_CH / 8; ++h) {
            double2 w[NC];
#pragma unroll
            for (int cb = 0; cb < NC; ++cb)
                w[cb] = *reinterpret_cast<const double2 *>(sw + (16 * cb + r16) * DY_P + 2 * g + 8 * h);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (NB > 1 && (wave + 4 * b) * 16 >= npair) continue;
                const double2 us = *reinterpret_cast<const double2 *>(su + as[b] + 8 * h);
                const double2 vs = *reinterpret_cast<const double2 *>(sv + as[b] + 8 * h);
                const double2 ut = *reinterpret_cast<const double2 *>(su + at[b] + 8 * h);
                const double2 vt = *reinterpret_cast<const double2 *>(sv + at[b] + 8 * h);
                const double nx = 2.0 * (us.x * ut.x + vs.x * vt.x) - us.x * vt.x - vs.x * ut.x;
                const double ny = 2.0 * (us.y * ut.y + vs.y * vt.y) - us.y * vt.y - vs.y * ut.y;
#pragma unroll
                for (int cb = 0; cb < NC; ++cb) {
                    acc[b][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(nx, w[cb].x, acc[b][cb], 0, 0, 0);
                    acc[b][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ny, w[cb].y, acc[b][cb], 0, 0, 0);
                }
            }
        }
    }
    // lane (r16, g): column r16 of pairs 16 block + g + 4e
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int cb = 0; cb < NC; ++cb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int P = (wave + 4 * b) * 16 + g + 4 * e;
                if (P < npair) part[((int64_t)blockIdx.x * npair + P) * (16 * NC) + 16 * cb + r16] = acc[b][cb][e];
            }
}

// out[q] = sum_b part[b][q], q over pairs x columns: one wave per output, lane l sums
// blocks l, l+64, ... in order, then a fixed shuffle tree (deterministic)
__global__ void pairs_reduce_kernel(const double *__restrict__ part, int nblk, int64_t nq, double *__restrict__ out)
{
    const int64_t q = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (q >= nq) return;                                   // whole waves leave together
    double a = 0.0;
    for (int b = l; b < nblk; b += 64) a += part[(int64_t)b * nq + q];
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if (l == 0) out[q] = a;
}

// One Newton step of the Dyson search for the roots act[blockIdx.x]: the matrix diag(e_S) + Sigma_SS(w)
// of the root's energy (columns 2t, 2t + 1 of the reduced sums) is diagonalised by parallel-ordered
// Jacobi sweeps in LDS (round-robin rounds of disjoint rotations), the eigenvector of largest
// overlap with the previous one is followed, and w <- w + (lambda - w) P.  A workgroup per root:
// the host did them one after the other (16 roots of 16 orbitals: about 450 us per solve).
struct DyRoots {
    double *w, *pole, *U;        // [n], [n], [n][n]: row k = tracked vector of root k
    int *status, *iters;         // [n]
    const double *eS;            // [n]
};

__global__ __launch_bounds__(256) void dyson_step_kernel(int n, const double *__restrict__ sums, int ncol,
                                                         const int *__restrict__ act, double conv, int it, DyRoots d)
{
    __shared__ double A[DY_MAXSEL + 1][DY_MAXSEL + 2], V[DY_MAXSEL + 1][DY_MAXSEL + 2];
    __shared__ double rc[(DY_MAXSEL + 1) / 2], rs[(DY_MAXSEL + 1) / 2], red[2][DY_MAXSEL + 1], ov[DY_MAXSEL + 1], un[DY_MAXSEL + 1];
    __shared__ uchar2 pq[DY_MAXSEL][(DY_MAXSEL + 1) / 2];      // round r's i-th pair
    __shared__ int jbest;
    const int t = blockIdx.x, k = act[t], tid = threadIdx.x;
    for (int e = tid; e < n * n; e += 256) {
        const int i = e / n, j = e - i * n, hi = max(i, j), lo = min(i, j);
        A[i][j] = sums[(int64_t)(hi * (hi + 1) / 2 + lo) * ncol + 2 * t] + (i == j ? d.eS[i] : 0.0);
        V[i][j] = i == j ? 1.0 : 0.0;
    }
    const int m = n + (n & 1), half = m / 2;      // players of the round robin (an odd n sits one out)
    // round r: (m-1, r) and ((r + i) mod (m-1), (r - i) mod (m-1)), i = 1 .. half - 1
    for (int e = tid; e < (m - 1) * half; e += 256) {
        const int r = e / half, i = e - r * half;
        const int x = i == 0 ? m - 1 : (r + i) % (m - 1), y = i == 0 ? r : (r + m - 1 - i) % (m - 1);
        pq[r][i] = make_uchar2((unsigned char)min(x, y), (unsigned char)max(x, y));
    }
    for (int sweep = 0; sweep < 100; ++sweep) {
        __syncthreads();
        double off = 0.0, tot = 0.0;
        for (int e = tid; e < n * n; e += 256) {
            const int i = e / n, j = e - i * n;
            const double x = A[i][j] * A[i][j];
            tot += x;
            if (i != j) off += x;
        }
        // fixed order: lanes by butterfly, then the four waves
        for (int o = 32; o > 0; o >>= 1) {
            off += __shfl_xor(off, o, 64);
            tot += __shfl_xor(tot, o, 64);
        }
        if ((tid & 63) == 0) {
            red[0][tid >> 6] = off;
            red[1][tid >> 6] = tot;
        }
        __syncthreads();
        off = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
        tot = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
        // a matrix of infinities leaves here, undiagonalised (inf <= inf); one with a NaN does not: its
        // rotations make the energy and the vector NaN, all of it within two sweeps (the first makes
        // two whole rows and columns NaN, the second every pair they are in)
        if (off <= 1e-30 * tot || off == 0.0) break;
        if (sweep == 2 && tot != tot) break;
        for (int r = 0; r < m - 1; ++r) {
            if (tid < half) {
                const int p = pq[r][tid].x, q = pq[r][tid].y;
                double c = 1.0, s = 0.0;
                if (q < n && A[p][q] != 0.0) {
                    const double theta = (A[q][q] - A[p][p]) / (2.0 * A[p][q]);
                    const double tn = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                    c = 1.0 / sqrt(tn * tn + 1.0);
                    s = tn * c;
                }
                rc[tid] = c;
                rs[tid] = s;
            }
            __syncthreads();
            for (int e = tid; e < half * n * 2; e += 256) {      // columns p, q of A and V
                const int i = e / (2 * n), rem = e - i * 2 * n, x = rem >> 1;
                const int p = pq[r][i].x, q = pq[r][i].y;
                if (q >= n || rs[i] == 0.0) continue;
                double(*M)[DY_MAXSEL + 2] = rem & 1 ? V : A;
                const double a = M[x][p], b = M[x][q];
                M[x][p] = rc[i] * a - rs[i] * b;
                M[x][q] = rs[i] * a + rc[i] * b;
            }
            __syncthreads();
            for (int e = tid; e < half * n; e += 256) {          // rows p, q of A
                const int i = e / n, x = e - i * n;
                const int p = pq[r][i].x, q = pq[r][i].y;
                if (q >= n || rs[i] == 0.0) continue;
                const double a = A[p][x], b = A[q][x];
                A[p][x] = rc[i] * a - rs[i] * b;
                A[q][x] = rs[i] * a + rc[i] * b;
            }
            __syncthreads();
        }
    }
    if (tid < n) {
        double v = 0.0;
        for (int i = 0; i < n; ++i) v += V[i][tid] * d.U[(int64_t)k * n + i];
        ov[tid] = v;
    }
    __syncthreads();
    if (tid == 0) {
        int jb = 0;
        double best = -1.0;
        for (int j = 0; j < n; ++j)
            if (fabs(ov[j]) > best) {
                best = fabs(ov[j]);
                jb = j;
            }
        jbest = jb;
    }
    __syncthreads();
    const int jb = jbest;
    if (tid < n) un[tid] = (ov[jb] >= 0.0 ? 1.0 : -1.0) * V[tid][jb];
    __syncthreads();
    if (tid < n) {
        d.U[(int64_t)k * n + tid] = un[tid];
        double v = 0.0;
        for (int j = 0; j < n; ++j) {
            const int hi = max(tid, j), lo = min(tid, j);
            v += sums[(int64_t)(hi * (hi + 1) / 2 + lo) * ncol + 2 * t + 1] * un[j];
        }
        red[0][tid] = un[tid] * v;
    }
    __syncthreads();
    if (tid == 0) {
        double sp = 0.0;
        for (int i = 0; i < n; ++i) sp += red[0][i];
        const double P = 1.0 / (1.0 - sp), w = d.w[k], wn = w + (A[jb][jb] - w) * P;
        d.pole[k] = P;
        d.iters[k] = it;
        d.w[k] = wn;
        if (!isfinite(wn) || !isfinite(P)) d.status[k] = CDS_QP_NONFINITE;
        else if (fabs(wn - w) <= conv) d.status[k] = CDS_QP_CONVERGED;
    }
}

// the roots still iterating, in order; first: the state is set up (w = e_q, unit vectors)
__global__ __launch_bounds__(64) void dyson_list_kernel(int n, int first, const double *__restrict__ eps,
                                                        const int *__restrict__ sel, double *__restrict__ eS, DyRoots d,
                                                        int *__restrict__ act)
{
    const int k = threadIdx.x;                    // n <= DY_MAXSEL
    if (first && k < n) {
        d.w[k] = eS[k] = eps[sel[k]];
        d.pole[k] = __builtin_nan("");
        d.status[k] = -1;
        d.iters[k] = 0;
        for (int i = 0; i < n; ++i) d.U[k * n + i] = i == k ? 1.0 : 0.0;
    }
    const bool on = k < n && (first || d.status[k] < 0);
    const unsigned long long m = __ballot(on);
    if (on) act[__popcll(m & ((1ull << k) - 1))] = k;
}

struct DyState {
    int prec, nmo, nocc, nvirt, nsel;
    int64_t nvo;
    void *G;
    const double *eps;
    double *d_omega, *part, *out;
    int nblk, nchB;
    int64_t nchA, nch;
};

int dy_setup(cds_ctx *ctx, int32_t prec, int64_t nvec, int64_t ldk, int32_t nmo, int32_t nocc, int32_t nsel,
             const int32_t *h_sel, const void *Bsel, const void *Bvo, const double *eps, DyState &S)
{
    CDS_REQUIRE(ctx, prec == CDS_PREC_FP64 || prec == CDS_PREC_FP32 || prec == CDS_PREC_BF16X3,
                "unknown precision %d", prec);
    CDS_REQUIRE(ctx, nmo >= 2 && nocc >= 1 && nocc < nmo, "need 1 <= nocc < nmo");
    CDS_REQUIRE(ctx, nsel >= 1 && nsel <= DY_MAXSEL && h_sel, "need 1 <= nsel <= %d and h_sel", DY_MAXSEL);
    CDS_REQUIRE(ctx, nvec >= 1 && ldk >= nvec && ldk % 64 == 0, "need 1 <= nvec <= ldk, ldk a multiple of 64");
    CDS_REQUIRE(ctx, Bsel && Bvo && eps, "NULL pointer");
    for (int s = 0; s < nsel; ++s)
        CDS_REQUIRE(ctx, h_sel[s] >= 0 && h_sel[s] < nmo, "h_sel[%d] out of range", s);
    S.prec = prec;
    S.nmo = nmo;
    S.nocc = nocc;
    S.nvirt = nmo - nocc;
    S.nsel = nsel;
    S.nvo = (int64_t)S.nvirt * nocc;
    S.eps = eps;
    const size_t gs = prec == CDS_PREC_FP64 ? 8 : 4;
    const size_t gbytes = (size_t)nsel * nmo * S.nvo * gs;
    CDS_REQUIRE(ctx, gbytes <= DY_G_MAX, "integrals of the selected orbitals exceed %zu bytes", DY_G_MAX);
    CDS_CALL(cds_ws(ctx, WS_DY_G, gbytes, &S.G));
    const int64_t nt8 = cds_ceil_div(nocc, 8);
    S.nchA = S.nvirt * (nt8 * (nt8 + 1) / 2);
    S.nchB = (int)cds_ceil_div(S.nvo, DY_CH);
    S.nch = S.nchA + (int64_t)S.nvirt * S.nchB;
    S.nblk = (int)std::min<int64_t>(DY_BLOCKS, S.nch);
    const int npair = nsel * (nsel + 1) / 2;
    void *w;
    const size_t nq = (size_t)npair * DY_TT * 2;
    CDS_CALL(cds_ws(ctx, WS_DY_PART, ((size_t)S.nblk * nq + nq + DY_TT) * 8, &w));
    S.part = (double *)w;
    S.out = S.part + (size_t)S.nblk * nq;
    S.d_omega = S.out + nq;
    // all selected orbitals' integrals in one contraction
    CDS_CALL(cds_contract_internal(ctx, prec, nvec, ldk, nmo, nocc, nsel, Bsel, Bvo, 0, nsel, S.G));
    return CDS_OK;
}

template <typename GT, int NC>
void dy_launch(cds_ctx *ctx, const DyState &S, int T, const double *omega, const int *list)
{
    const size_t lds = ((size_t)(2 * S.nsel + 16 * NC) * DY_P + 4 * DY_CH) * 8;
    const int nb = (int)cds_ceil_div(cds_ceil_div(S.nsel * (S.nsel + 1) / 2, 16), 4);   // pair blocks per wave
    const auto k = nb <= 1 ? sigma_pairs_kernel<GT, 1, NC> : nb <= 2 ? sigma_pairs_kernel<GT, 2, NC>
                 : nb <= 3 ? sigma_pairs_kernel<GT, 3, NC> : nb <= 5 ? sigma_pairs_kernel<GT, 5, NC>
                           : sigma_pairs_kernel<GT, 8, NC>;
    hipLaunchKernelGGL(k, dim3((unsigned)S.nblk), dim3(DY_NT), lds, ctx->stream, (const GT *)S.G, S.nsel, S.nmo, S.nocc,
                       S.nvirt, S.nvo, S.eps, omega, list, T, S.nchA, S.nch, S.nchB, S.part);
}

int dy_cols(int T) { return T <= 8 ? 16 : 32; }

// the pairs' sums S.out [pair][dy_cols(T)] at T <= DY_TT device energies: omega[t], or omega[list[t]]
int dy_sums(cds_ctx *ctx, const DyState &S, int T, const double *omega, const int *list)
{
    const int64_t nq = (int64_t)(S.nsel * (S.nsel + 1) / 2) * dy_cols(T);
    if (S.prec == CDS_PREC_FP64) {
        if (T <= 8) dy_launch<double, 1>(ctx, S, T, omega, list);
        else dy_launch<double, 2>(ctx, S, T, omega, list);
    } else {
        if (T <= 8) dy_launch<float, 1>(ctx, S, T, omega, list);
        else dy_launch<float, 2>(ctx, S, T, omega, list);
    }
    CDS_LAUNCHED(ctx);
    hipLaunchKernelGGL(pairs_reduce_kernel, dim3((unsigned)cds_ceil_div(nq, 4)), dim3(256), 0, ctx->stream,
                       (const double *)S.part, S.nblk, nq, S.out);
    CDS_LAUNCHED(ctx);
    return CDS_OK;
}

// Sigma_SS and Sigma'_SS at up to DY_TT trial energies -> host (T x nsel x nsel each)
int dy_eval(cds_ctx *ctx, const DyState &S, int T, const double *h_w, double *h_sig, double *h_dsig)
{
    const int npair = S.nsel * (S.nsel + 1) / 2, ncol = dy_cols(T);
    const int64_t nq = (int64_t)npair * ncol;
    void *hp;
    CDS_CALL(cds_pinned(ctx, (size_t)npair * 2 * DY_TT * 8 + 256, &hp));
    double *hb = (double *)hp;
    for (int t = 0; t < DY_TT; ++t) hb[t] = h_w[t < T ? t : T - 1];
    CDS_HIP(ctx, hipMemcpyAsync(S.d_omega, hb, DY_TT * 8, hipMemcpyHostToDevice, ctx->stream));
    CDS_CALL(dy_sums(ctx, S, T, S.d_omega, nullptr));
    CDS_HIP(ctx, hipMemcpyAsync(hb, S.out, (size_t)nq * 8, hipMemcpyDeviceToHost, ctx->stream));
    CDS_HIP(ctx, hipStreamSynchronize(ctx->stream));
    const int n = S.nsel;
    for (int P = 0; P < npair; ++P) {
        int t2 = 0;
        while ((t2 + 1) * (t2 + 2) / 2 <= P) ++t2;
        const int s = P - t2 * (t2 + 1) / 2;
        for (int t = 0; t < T; ++t) {
            const double v = hb[(size_t)P * ncol + 2 * t], dv = hb[(size_t)P * ncol + 2 * t + 1];
            h_sig[(size_t)t * n * n + (size_t)s * n + t2] = h_sig[(size_t)t * n * n + (size_t)t2 * n + s] = v;
            h_dsig[(size_t)t * n * n + (size_t)s * n + t2] = h_dsig[(size_t)t * n * n + (size_t)t2 * n + s] = dv;
        }
    }
    return CDS_OK;
}

}  // namespace

extern "C" int cds_sigma2_matrix(cds_ctx *ctx, int32_t prec, int64_t nvec, int64_t ldk, int32_t nmo,
                                 int32_t nocc, int32_t nsel, const int32_t *h_sel, const void *Bsel,
                                 const void *Bvo, const double *eps, int32_t T, const double *h_omega,
                                 double *h_sigma, double *h_dsigma)
{
    CDS_CALL(cds_enter(ctx));
    CDS_REQUIRE(ctx, T >= 1 && T <= 1024 && h_omega && h_sigma && h_dsigma, "need 1 <= T <= 1024 and host arrays");
    DyState S;
    CdsTimer tm;
    CDS_CALL(cds_timer_start(ctx, &tm));
    CDS_CALL(dy_setup(ctx, prec, nvec, ldk, nmo, nocc, nsel, h_sel, Bsel, Bvo, eps, S));
    const size_t nn = (size_t)nsel * nsel;
    for (int t0 = 0; t0 < T; t0 += DY_TT) {
        const int nt = std::min(DY_TT, T - t0);
        CDS_CALL(dy_eval(ctx, S, nt, h_omega + t0, h_sigma + t0 * nn, h_dsigma + t0 * nn));
    }
    CDS_CALL(cds_timer_stop(ctx, &tm, &ctx->stats.t_dyson_ms));
    CDS_CALL(cds_timers_flush(ctx));
    return CDS_OK;
}

extern "C" int cds_dyson_solve(cds_ctx *ctx, int32_t prec, int64_t nvec, int64_t ldk, int32_t nmo, int32_t nocc,
                               int32_t nsel, const int32_t *h_sel, const void *Bsel, const void *Bvo,
                               const double *eps, double conv, int32_t max_iter, double *h_omega, double *h_pole,
                               double *h_vec, int32_t *h_iters, int32_t *h_status)
{
    CDS_CALL(cds_enter(ctx));
    CDS_REQUIRE(ctx, conv > 0.0 && max_iter >= 1, "need conv > 0 and max_iter >= 1");
    CDS_REQUIRE(ctx, h_omega && h_pole && h_vec && h_iters && h_status, "NULL host pointer");
    DyState S;
    CdsTimer tm;
    CDS_CALL(cds_timer_start(ctx, &tm));
    CDS_CALL(dy_setup(ctx, prec, nvec, ldk, nmo, nocc, nsel, h_sel, Bsel, Bvo, eps, S));
    const int n = nsel;
    // the roots' state, read back whole after every step: w, P, the vectors, status, steps; then the
    // orbitals' own energies, their numbers and the list of roots still iterating
    const size_t state = (size_t)n * (2 + n) * 8 + (size_t)2 * n * 4;
    void *wr, *hp;
    CDS_CALL(cds_ws(ctx, WS_AD_TMP2, state + (size_t)n * 16 + 64, &wr));
    CDS_CALL(cds_pinned(ctx, state + (size_t)n * 4, &hp));
    DyRoots R;
    R.w = (double *)wr;
    R.pole = R.w + n;
    R.U = R.pole + n;
    R.status = (int *)(R.U + (size_t)n * n);
    R.iters = R.status + n;
    double *d_eS = (double *)(R.iters + n);
    R.eS = d_eS;
    int *d_sel = (int *)(d_eS + n), *d_act = d_sel + n;
    std::copy(h_sel, h_sel + n, (int32_t *)hp);
    CDS_HIP(ctx, hipMemcpyAsync(d_sel, hp, (size_t)n * 4, hipMemcpyHostToDevice, ctx->stream));
    const double *hw = (const double *)hp, *hP = hw + n, *hU = hP + n;
    const int *hs = (const int *)(hU + (size_t)n * n), *hi = hs + n;
    int nact = n, nlist = -1;                     // roots still iterating, and in the device's list
    for (int it = 1; it <= max_iter && nact > 0; ++it) {
        if (nlist != nact) {                      // (a root that ended never comes back)
            hipLaunchKernelGGL(dyson_list_kernel, dim3(1), dim3(64), 0, ctx->stream, n, it == 1 ? 1 : 0, eps,
                               (const int *)d_sel, d_eS, R, d_act);
            CDS_LAUNCHED(ctx);
            nlist = nact;
        }
        for (int b0 = 0; b0 < nact; b0 += DY_TT) {
            const int nt = std::min(DY_TT, nact - b0);
            CDS_CALL(dy_sums(ctx, S, nt, R.w, d_act + b0));
            hipLaunchKernelGGL(dyson_step_kernel, dim3((unsigned)nt), dim3(256), 0, ctx->stream, n, (const double *)S.out,
                               dy_cols(nt), (const int *)d_act + b0, conv, it, R);
            CDS_LAUNCHED(ctx);
        }
        CDS_HIP(ctx, hipMemcpyAsync(hp, wr, state, hipMemcpyDeviceToHost, ctx->stream));
        CDS_HIP(ctx, hipStreamSynchronize(ctx->stream));
        nact = 0;
        for (int k = 0; k < n; ++k) nact += hs[k] < 0;
    }
    for (int k = 0; k < n; ++k) {
        h_omega[k] = hw[k];
        h_pole[k] = hP[k];
        h_iters[k] = hi[k];
        h_status[k] = hs[k] < 0 ? CDS_QP_MAX_ITER : hs[k];
        for (int i = 0; i < n; ++i) h_vec[(size_t)k * n + i] = hU[(size_t)k * n + i];
    }
    CDS_CALL(cds_timer_stop(ctx, &tm, &ctx->stats.t_dyson_ms));
    CDS_CALL(cds_timers_flush(ctx));
    return CDS_OK;
}
