// GP hyperparameter marginalisation on gfx950 (Sec. 5 "Gaussian process" experiments; App.
// "Gaussian Process Hyperparameter Marginalization"): the likelihood of a candidate
// u = log theta, theta = (sigma_f, l_1, l_2, l_p, P, sigma_n), is the log marginal likelihood
//   log N(y; 0, K + sigma_n^2 I),  K_ab = sigma_f^2 exp(-1/2 sum_j (a_j-b_j)^2 / l_j^2
//                                               - 2 sum_j sin^2(pi (a_j-b_j)/P) / l_p^2)
// over n <= 256 observations with 2-D inputs (a squared-exponential times a periodic kernel,
// each a product over the input dimensions).
//
// One workgroup of 8 waves evaluates one candidate at a time.  The kernel matrix is built as
// 16x16 tiles of the lower triangle, transposed, in the accumulator layout of the 16x16x4 MFMA
// (tile t is held by wave t mod 8 in registers) and factorised by a right-looking blocked
// Cholesky.  For each block column J the wave that holds the diagonal tile brings it up to date
// and eliminates it with one row per lane: 16 lanes its rows, 16 more the rows of the identity,
// which come out as the columns of the inverse factor.  Every tile below is then multiplied by
// that inverse on MFMA.  A transposed accumulator is laid out as an operand of the next product
// (lane l, register r: row l & 15, k-step r), so the panel goes from the registers to LDS and
// back as whole 16- and 32-byte pieces.  While one wave eliminates, the others bring the later
// columns' tiles up to date, and one of them takes the forward solve a block column behind:
// z_J = L_JJ^{-1} y_J, y_I -= L_IJ z_J, one row per lane.
//   log L = -|z|^2 / 2 - sum_i log L_ii - n/2 log(2 pi).
// A pivot that is not positive makes the factorisation fail (FP64: log L = -inf).
//
// The order of every FP64 sum is fixed, by explicit fused operations where the compiler could
// choose: the prior reaches sigma_f^2 / sigma_n^2 = 1e8, where another rounding of an entry, a
// root or a product moves log L by 1e-9 of itself, and results are to stay what they are.
//
// What bounds it at n = 256 (about 250,000 cycles an evaluation): the chain of 16 block columns,
// each about 3,000 cycles to bring the diagonal tile up to date and into rows, 4,000 for its 16
// dependent pivots and 1,800 for the panel, then the entries' exponentials (50,000) and what the
// updates leave uncovered.  500 chains of 30 steps: 25.9 ms a pass with one wave factoring, then
// inverting, each diagonal tile and the tiles in a layout that had to be turned for every product,
// 16.4 here; at n = 100 in the FP32 mode 5.3 and 3.7 ms.  (n, the tile indices and the LDS address
// have to be wave-uniform values to the compiler: as vector values the indices came back from
// scratch memory for every tile, 25.3 ms.)
//
//  k_hrss_gp   one HRSS chain per workgroup (App. A.6), candidates evaluated one at a time
//  k_eval_gp   one point per workgroup (initial live set, tests)
#include "nss_chol.hpp"
#include "nss_internal.hpp"
#include "nss_rng.hpp"
#include "nss_wave.hpp"

#include <math.h>

namespace nss {

namespace {

constexpr int kGpWaves = 8;                                           // per workgroup
constexpr int kGpThreads = 64 * kGpWaves;
constexpr int kGpMaxTiles = 136;                                      // 16 * 17 / 2
constexpr int kGpSlots = kGpMaxTiles / kGpWaves;                      // tiles per wave
constexpr int kFrag = 256;             // a tile in LDS as an operand: lane l's four values at 4 l
constexpr int kGpD = 6;                                               // hyperparameters

// LDS: inputs and targets (FP64), reduction slots, then the factorisation's tiles in T
constexpr int kOffXs = 0;                                             // double [256][2]
constexpr int kOffYs = kOffXs + 2 * kGpMaxObs * 8;                    // double [256]
constexpr int kOffMisc = kOffYs + kGpMaxObs * 8;                      // double [16], int flag
constexpr int kOffChain = kOffMisc + 256;                             // chain point, direction
constexpr int kOffSc = kOffChain + 128;                               // double [256][4]
constexpr int kOffT = kOffSc + 4 * kGpMaxObs * 8;
template <typename T>
constexpr int kGpInv = sizeof(T) == 4 ? 16 : 2;   // inverse factors kept (the FP32 solve reads all)
template <typename T>
constexpr int gp_lds_bytes()
{
    // two columns of tiles (the one being written and the one being read), the diagonal tile, the
    // inverse factors, the right-hand side and z; the FP32 refinement adds alpha and the partial
    // products of a block step
    return kOffT + (int)sizeof(T) * (2 * 16 * kFrag + (1 + kGpInv<T>) * kTile + 2 * kGpMaxObs) +
           (sizeof(T) == 4 ? 4 * (kGpMaxObs + 16 * 16) : 0);
}

struct GpTheta {
    double sf2, il1, il2, ilp2, iper, sn2;
};

__device__ __forceinline__ GpTheta gp_theta(const double *u)
{
    GpTheta h;
    h.sf2 = exp(2.0 * u[0]);
    h.il1 = exp(-u[1]);
    h.il2 = exp(-u[2]);
    h.ilp2 = exp(-2.0 * u[3]);
    h.iper = exp(-u[4]);
    h.sn2 = exp(2.0 * u[5]);
    return h;
}

// sin(u - v) from p = (sin, cos) u, q = (sin, cos) v
__device__ __forceinline__ double sin_diff(double2 p, double2 q)
{
    return fma(p.x, q.y, -(p.y * q.x));
}

// The kernel at input differences d1, d2, with s1, s2 the sines of pi d / P.
template <typename T>
__device__ __forceinline__ T gp_cov(double d1, double d2, double s1, double s2, const GpTheta &h)
{
    if constexpr (sizeof(T) == 8) {
        const double a1 = d1 * h.il1, a2 = d2 * h.il2;
        const double a = fma(a1, a1, a2 * a2), s = fma(s1, s1, s2 * s2);
        return h.sf2 * exp(fma(a, -0.5, -(h.ilp2 * (s + s))));
    } else {
        const float a1 = (float)(d1 * h.il1), a2 = (float)(d2 * h.il2);
        const float f1 = (float)s1, f2 = (float)s2;
        return (float)h.sf2 *
               expf(-0.5f * (a1 * a1 + a2 * a2) - 2.0f * (f1 * f1 + f2 * f2) * (float)h.ilp2);
    }
}

// Entry (row, col) of the padded covariance: identity outside the n observations, zero above
// the diagonal (never read as data).  sin(pi (a - b) / P) = s_a c_b - c_a s_b from the per-point
// sc[i] = (sin, cos)(pi x_i1 / P), (sin, cos)(pi x_i2 / P), so an entry costs one exponential.
template <typename T>
__device__ __forceinline__ T gp_entry(const double *xs, const double *sc, int n, int row, int col,
                                      const GpTheta &h)
{
    if (row >= n || col >= n) return (row == col) ? T(1) : T(0);
    if (col > row) return T(0);
    // (the combined sine of a point and itself is a rounding error, not 0: below l_p = 1e-15 its
    // square counts)
    if (row == col) return (T)h.sf2 + (T)h.sn2;
    const double2 *pa = (const double2 *)(sc + 4 * row), *pb = (const double2 *)(sc + 4 * col);
    return gp_cov<T>(xs[2 * row] - xs[2 * col], xs[2 * row + 1] - xs[2 * col + 1],
                     sin_diff(pa[0], pb[0]), sin_diff(pa[1], pb[1]), h);
}

// sum_c a_c b_c as a row of sixteen lanes' pairwise exchanges give it to its first lane, the first
// exchange's sum fused with the lane's own product
template <typename T>
__device__ __forceinline__ T dot16(const T (&a)[16], const T (&b)[16])
{
    auto f = [&](int i, int j) { return fma(a[i], b[i], a[j] * b[j]); };
    return ((f(0, 1) + f(2, 3)) + (f(7, 6) + f(5, 4))) +
           ((f(15, 14) + f(13, 12)) + (f(8, 9) + f(10, 11)));
}

// -|z|^2 / 2 - sum_i log L_ii of N(y; 0, K_theta + sigma_n^2 I) at u = log theta with the
// factorisation in T.  Called by every thread of the workgroup with the same u (the result is
// uniform); the inputs and targets must be staged at kOffXs / kOffYs.  failed = a pivot was not
// positive.
//
// A function of its own rather than inlined in the chain's loop: there, the loop's state and what
// the compiler hoists out of it (addresses, the math functions' constants) took registers that
// the tiles need, and came back from scratch memory inside the entries' loop.
typedef __attribute__((address_space(3))) unsigned char *lds_ptr;
struct GpPoint {
    double u[kGpD];
};
struct GpResult {
    double L;
    int failed;
};
template <typename T>
__device__ __attribute__((noinline)) GpResult gp_eval_at(GpPoint pt, int n, lds_ptr lds)
{
    // (arguments arrive in vector registers)
    lds = (lds_ptr)(uintptr_t)(unsigned)uniform_i((int)(unsigned)(uintptr_t)lds);
    n = uniform_i(n);
    unsigned char *smem = (unsigned char *)lds;
    const double *u = pt.u;
    typedef Mf<T> M;
    typedef typename M::v4 v4;
    const double *xs = (const double *)(smem + kOffXs);
    const double *ys = (const double *)(smem + kOffYs);
    double *red = (double *)(smem + kOffMisc);   // log det / 2, |z|^2, partial sums, pivots' products
    int *flag = (int *)(red + 16);
    double *sc = (double *)(smem + kOffSc);
    T *pan = (T *)(smem + kOffT);    // [2][16] panel tiles
    T *dg = pan + 2 * 16 * kFrag;    // the diagonal tile, in rows
    T *li = dg + kTile;              // [kGpInv] inverse factors, in rows
    T *yb = li + kGpInv<T> * kTile;
    T *zb = yb + kGpMaxObs;
    constexpr bool refine = sizeof(T) == 4;
    // FP32 refinement: alpha = L^{-T} z, the partial products of one block step
    float *alpha = (float *)(zb + kGpMaxObs);
    float *part = alpha + kGpMaxObs;
    // the thread index, opaque to the compiler in each evaluation and each block column: keeps
    // the many lane-derived masks and LDS addresses of the unrolled code below from being hoisted
    // out of the loops around it, where they would hold registers across all of it
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane0 = tid & 63, w = uniform_i(tid >> 6);
    const int NT = (n + 15) >> 4, NTT = NT * (NT + 1) / 2;
    const GpTheta h = gp_theta(u);

    for (int i = tid; i < 16 * NT; i += kGpThreads) yb[i] = (i < n) ? (T)ys[i] : T(0);
    for (int i = tid; i < n; i += kGpThreads) {
        double s0, c0, s1, c1;
        sincospi(xs[2 * i] * h.iper, &s0, &c0);
        sincospi(xs[2 * i + 1] * h.iper, &s1, &c1);
        sc[4 * i] = s0; sc[4 * i + 1] = c0; sc[4 * i + 2] = s1; sc[4 * i + 3] = c1;
    }
    if (tid == 0) { *flag = 0; red[0] = red[1] = 0.0; }
    __syncthreads();

    // The wave's tiles, four at a time through its share of the panel buffers: the entries' code
    // then stands in a loop over tiles, with a lane's four entries side by side, instead of once
    // per register slot.  Lane l, register r of tile (I, K): row 16 I + (l & 15), column
    // 16 K + M::row(l, r).
    int tI[kGpSlots], tK[kGpSlots];
    v4 acc[kGpSlots];
#pragma unroll
    for (int s0 = 0; s0 < kGpSlots; s0 += 4) {
        T *stage = pan + 4 * w * kFrag + 4 * lane0;
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {
            const int t = w + kGpWaves * (s0 + q);
            if (s0 + q >= kGpSlots || t >= NTT) break;
            const int l = lane0;
            int I, K;
            tile_ik(t, I, K);
            const int row = 16 * I + (l & 15);
            v4 e;
            if (I > K && 16 * I + 16 <= n) {   // all observations, all below the diagonal
                const double2 xr = *(const double2 *)(xs + 2 * row);
                const double2 r1 = *(const double2 *)(sc + 4 * row);
                const double2 r2 = *(const double2 *)(sc + 4 * row + 2);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int col = 16 * K + M::row(l, r);
                    const double2 xc = *(const double2 *)(xs + 2 * col);
                    const double2 c1 = *(const double2 *)(sc + 4 * col);
                    const double2 c2 = *(const double2 *)(sc + 4 * col + 2);
                    e[r] = gp_cov<T>(xr.x - xc.x, xr.y - xc.y, sin_diff(r1, c1), sin_diff(r2, c2), h);
                }
            } else {
#pragma unroll 1
                for (int r = 0; r < 4; ++r) {
                    const T v = gp_entry<T>(xs, sc, n, row, 16 * K + M::row(l, r), h);
                    e[0] = r == 0 ? v : e[0];
                    e[1] = r == 1 ? v : e[1];
                    e[2] = r == 2 ? v : e[2];
                    e[3] = r == 3 ? v : e[3];
                }
            }
            *(v4 *)(stage + q * kFrag) = e;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int s = s0 + q;
            if (s < kGpSlots) {
                const int t = w + kGpWaves * s;
                int I = -1, K = -1;
                if (t < NTT) {
                    tile_ik(t, I, K);
                    acc[s] = *(const v4 *)(stage + q * kFrag);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[s][r] = T(0);
                }
                tI[s] = uniform_i(I);
                tK[s] = uniform_i(K);
            }
        }
    }
    // Block column J = 0..NT: the elimination of column J, the update of the later tiles by column
    // J - 1 and the forward solve of block J - 1 side by side, then the panel of column J.
    for (int J = 0;; ++J) {
        int l = lane0;
        asm volatile("" : "+v"(l));
        T *cur = pan + (J & 1) * 16 * kFrag;
        const T *prv = pan + ((J & 1) ^ 1) * 16 * kFrag;   // column J - 1 of the factor
        // A_IK^T -= L_K,J-1 L_I,J-1^T
        auto multiply = [&](v4 &a, const v4 &oK, const v4 &oI) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a = M::mma(oK[ks], -oI[ks], a);
        };
        auto operand = [&](int I) { return *(const v4 *)(prv + I * kFrag + 4 * l); };
        const int tJ = J * (J + 3) / 2;                    // the diagonal tile
        const int pw = tJ & (kGpWaves - 1);
        if (J < NT && w == pw) {
#pragma unroll
            for (int s = 0; s < kGpSlots; ++s) {
                if (w + kGpWaves * s == tJ) {
                    if (J > 0) {
                        const v4 o = operand(J);
                        multiply(acc[s], o, o);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) dg[(l & 15) * kTileLd + M::row(l, r)] = acc[s][r];
                }
            }
            wave_sync();
            T a[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const T v = dg[(l & 15) * kTileLd + c];
                a[c] = !(l & 16) ? v : (l & 15) == c ? T(1) : T(0);
            }
            double p0, p1;
            int bad;
            eliminate<T>(a, p0, p1, bad);
            if ((l >> 4) == 1) {   // lane 16 + c: column c of the inverse
                T *lj = li + (J & (kGpInv<T> - 1)) * kTile + (l & 15);
#pragma unroll
                for (int r = 0; r < 16; ++r) lj[r * kTileLd] = a[r];
            }
            if (l == 0) {
                red[10 + (J & 1)] = p0;
                red[12 + (J & 1)] = p1;
                if (bad) *flag = 1;
            }
        }
        if (J > 0) {
            if (w == ((pw + 2) & (kGpWaves - 1))) {
                // the forward solve of block J - 1, one row per lane
                const int j0 = 16 * (J - 1);
                T a[16], b[16];
                if (l < 16) {
                    const T *lj = li + ((J - 1) & (kGpInv<T> - 1)) * kTile + l * kTileLd;
#pragma unroll
                    for (int c = 0; c < 16; ++c) { a[c] = lj[c]; b[c] = yb[j0 + c]; }
                    zb[j0 + l] = dot16<T>(a, b);
                }
                wave_sync();
#pragma unroll
                for (int c = 0; c < 16; ++c) b[c] = zb[j0 + c];
                double q2 = fma((double)b[0], (double)b[0], (double)b[1] * (double)b[1]);
#pragma unroll
                for (int c = 2; c < 16; ++c) q2 = fma((double)b[c], (double)b[c], q2);
                double ld = log(red[10 + ((J - 1) & 1)]);
                if (refine) ld = 0.5 * (ld + log(red[12 + ((J - 1) & 1)]));
                if (l == 0) {
                    red[0] += ld;
                    red[1] += q2;
                }
                for (int i = l; i < 16 * (NT - J); i += 64) {
                    const T *fr = prv + (J + (i >> 4)) * kFrag + 4 * (i & 15);
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const v4 o = *(const v4 *)(fr + 64 * g);
#pragma unroll
                        for (int r = 0; r < 4; ++r) a[M::row(16 * g, r)] = o[r];
                    }
                    yb[16 * J + i] -= dot16<T>(a, b);
                }
            }
            // the tiles of this and the later columns take column J - 1, two at a time
#pragma unroll
            for (int s = 0; s < kGpSlots; s += 2) {
                const int s1 = s + 1 < kGpSlots ? s + 1 : s;
                const bool b0 = tK[s] >= J && w + kGpWaves * s != tJ;
                const bool b1 = s1 > s && tK[s1] >= J && w + kGpWaves * s1 != tJ;
                if (b0 || b1) {   // (a tile that is not due reads its own operands, unused)
                    const v4 i0 = operand(max(tI[s], 0)), k0 = operand(max(tK[s], 0));
                    const v4 i1 = operand(max(tI[s1], 0)), k1 = operand(max(tK[s1], 0));
                    if (b0) multiply(acc[s], k0, i0);
                    if (b1) multiply(acc[s1], k1, i1);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        if (J == NT) break;
        // the panel: L_IJ^T = L_JJ^{-1} A_IJ^T
        T lf[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            lf[ks] = li[(J & (kGpInv<T> - 1)) * kTile + (l & 15) * kTileLd + M::row(l, ks)];
#pragma unroll
        for (int s = 0; s < kGpSlots; ++s) {
            if (tK[s] == J && tI[s] > J) {
                v4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = T(0);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) o = M::mma(lf[ks], acc[s][ks], o);
                *(v4 *)(cur + tI[s] * kFrag + 4 * l) = o;
                if constexpr (refine) acc[s] = o;   // kept for the solve
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    }
    if constexpr (refine) {
        // alpha = L^{-T} z, block rows from the last: alpha_J = L_JJ^{-T} (z_J - sum_{I > J}
        // L_IJ^T alpha_I), the products L_IJ^T alpha_I from the tiles' owners
        for (int J = NT - 1; J >= 0; --J) {
            int l = lane0;
            asm volatile("" : "+v"(l));
#pragma unroll
            for (int s = 0; s < kGpSlots; ++s) {
                if (tK[s] == J && tI[s] > J) {
                    const float al = alpha[16 * tI[s] + (l & 15)];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = row_sum16((float)acc[s][r] * al);
                        if ((l & 15) == 0) part[16 * tI[s] + M::row(l, r)] = v;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
            if (w == 0) {   // lane i: component i
                const int i = l & 15;
                float wv = zb[16 * J + i], a0 = 0.f, a1 = 0.f;
                for (int I = J + 1; I < NT; ++I) wv -= part[16 * I + i];
#pragma unroll
                for (int c = 0; c < 16; c += 2) {
                    a0 += (float)li[J * kTile + c * kTileLd + i] * readlane_t(wv, c);
                    a1 += (float)li[J * kTile + (c + 1) * kTileLd + i] * readlane_t(wv, c + 1);
                }
                if (l < 16) alpha[16 * J + l] = a0 + a1;
            }
            __syncthreads();
        }
    }
    const double ld = red[0];
    double q = red[1];
    const int failed = *flag;
    if constexpr (refine) {
        // y^T K^{-1} y from the FP32 solve alpha, with the entries in FP64:
        // 2 y^T alpha - alpha^T K alpha = y^T K^{-1} y - |alpha - K^{-1} y|_K^2, exact up to a
        // term of second order in the solve's error
        double s2 = 0.0;
        const int ne = n * (n + 1) / 2;
        for (int e = tid; e < ne; e += kGpThreads) {
            int i = (int)((sqrt(8.0 * (double)e + 1.0) - 1.0) * 0.5);
            while (i * (i + 1) / 2 > e) --i;
            while ((i + 1) * (i + 2) / 2 <= e) ++i;
            const int jj = e - i * (i + 1) / 2;
            const double kij = gp_entry<double>(xs, sc, n, i, jj, h);
            const double t = (double)alpha[i] * (double)alpha[jj] * kij;
            s2 += (i == jj) ? t : 2.0 * t;
        }
        for (int i = tid; i < n; i += kGpThreads) s2 -= 2.0 * ys[i] * (double)alpha[i];
        s2 = wave_sum(s2);
        __syncthreads();
        if ((tid & 63) == 0) red[2 + w] = s2;
        __syncthreads();
        double qv = 0.0;
#pragma unroll
        for (int v = 0; v < kGpWaves; ++v) qv -= red[2 + v];
        q = qv;
    }
    __syncthreads();   // the LDS slots are reused by the next evaluation
    return GpResult{fma(q, -0.5, -ld), failed};
}

// n/2 log(2 pi), rounded: log L of a chain's point is the evaluator's value less this
__device__ __forceinline__ double gp_norm(int n)
{
    double c = 0.5 * (double)n * LOG_2PI;
    asm volatile("" : "+v"(c));   // (not fused with the subtraction)
    return c;
}

template <typename T>
__device__ __forceinline__ double gp_eval(const double *u, int n, unsigned char *smem, bool &failed)
{
    GpPoint pt;
#pragma unroll
    for (int a = 0; a < kGpD; ++a) pt.u[a] = u[a];
    // (opaque: known to be the kernel's dynamic LDS in every call, its address would be looked up in
    // a table in memory wherever the evaluator uses it)
    lds_ptr lds = (lds_ptr)smem;
    asm volatile("" : "+v"(lds));
    const GpResult r = gp_eval_at<T>(pt, n, lds);
    failed = uniform_i(r.failed) != 0;
    return r.L;
}

__device__ __forceinline__ void gp_stage(const DevProblem &P, unsigned char *smem)
{
    double *xs = (double *)(smem + kOffXs);
    double *ys = (double *)(smem + kOffYs);
    for (int i = threadIdx.x; i < 2 * P.gp_n; i += blockDim.x) xs[i] = P.gp_x[i];
    for (int i = threadIdx.x; i < P.gp_n; i += blockDim.x) ys[i] = P.gp_y[i];
}

// Mixed precision: the FP32 estimate decides unless it lies within this band of L*; then (and
// when the FP32 factorisation breaks down) the FP64 value decides.  After the refinement the
// error is that of the FP32 log-determinant, which grows with the condition number, bounded
// by n s with s = (sigma_f^2 + sigma_n^2) / sigma_n^2 (the noise floor bounds the smallest
// eigenvalue of the covariance, its trace the largest).  Beyond n s = kGpMaxCond the FP32
// factor is not trusted and the FP64 value decides.
constexpr double kGpMaxCond = 1e5;
__device__ __forceinline__ double gp_cond(const DevProblem &P, const double *u)
{
    const double sf2 = exp(2.0 * u[0]), sn2 = exp(2.0 * u[5]);
    return (sf2 + sn2) / sn2 * (double)P.gp_n;
}
// beyond the bound the candidate is evaluated in FP64 only (no FP32 attempt)
__device__ __forceinline__ bool gp_illcond(const DevProblem &P, const double *u)
{
    return !(gp_cond(P, u) <= kGpMaxCond);
}
__device__ __forceinline__ bool gp_near(double L32, double Lstar, const DevProblem &P,
                                        const double *u)
{
    const double cond = gp_cond(P, u);
    if (!(cond <= kGpMaxCond)) return true;
    const double band = (double)P.guard_rel * fabs(L32) + (double)P.guard_abs +
                        (double)P.guard_kappa * cond;
    return !(fabs(L32 - Lstar) > band);
}

}  // namespace

template <int MODE>
__global__ __launch_bounds__(kGpThreads) void k_eval_gp(Launch Lc, const double *X, int ld, int n,
                                                        double *out, int from_run)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    unsigned long long *nonfinite = nullptr;
    if (from_run) { X = R.X; ld = R.m_pad; n = R.m; out = R.logL; nonfinite = R.ctr + 5; }
    const int i = bm.y;
    if (i >= n) return;
    gp_stage(P, smem);
    double u[kGpD];
#pragma unroll
    for (int a = 0; a < kGpD; ++a) u[a] = X[(size_t)a * ld + i];
    __syncthreads();
    bool failed = false;
    double L;
    if constexpr (MODE == MODE_FP64) L = gp_eval<double>(u, P.gp_n, smem, failed);
    else L = gp_eval<float>(u, P.gp_n, smem, failed);
    L = fma(-0.5 * (double)P.gp_n, LOG_2PI, L);
    if (threadIdx.x == 0) {
        unsigned long long nf = 0;
        out[i] = failed ? -INFINITY : sanitize(L, nf);
        if (nf && nonfinite) atomicAdd(nonfinite, nf);
    }
}

template <int MODE>
__global__ __launch_bounds__(kGpThreads) void k_hrss_gp(Launch Lc)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    if (R.iscal[0] || R.iscal[2] <= 0) return;
    const int j = bm.y;
    if (j >= R.k) return;
    const int tid = threadIdx.x, n = P.gp_n;
    double *sx0 = (double *)(smem + kOffChain);   // current point of the chain
    double *sv = sx0 + 8;                         // direction of the current step
    gp_stage(P, smem);
    const double Lstar = R.scal[0];
    const int t0 = R.iscal[1], nsurv = R.iscal[2];
    const uint32_t it = (uint32_t)R.iscal[3] + 1u;
    const double width = R.width;
    const int p = R.p, cap_out = R.stepout_cap, cap_sh = R.shrink_cap;
    const bool box = (P.prior_kind == PRIOR_BOX);

    double ur, unused;
    draw2(R.key0, R.key1, PUR_RESAMPLE, (uint32_t)j, it, 0u, 0u, ur, unused);
    int qi = (int)floor(ur * (double)nsurv);
    if (qi > nsurv - 1) qi = nsurv - 1;
    const int parent = R.perm[t0 + qi];
    if (tid == 0) R.parents[j] = parent;
    if (tid < kGpD) sx0[tid] = R.X[(size_t)tid * R.m_pad + parent];
    double logL0 = R.logL[parent];
    int exact0 = 1;
    // The walk's state is the same in every thread; outcomes are made uniform where they are
    // taken, so that it sits in scalar registers across the evaluation, whose tiles need the
    // vector ones.  Thread 0 publishes the counters.
    unsigned long long c_evals = 0, c_tests = 0, c_prej = 0, c_outcap = 0, c_shcap = 0,
                       c_nonfin = 0, c_rc = 0, c_viol = 0, c_wait = 0;
    const double norm = gp_norm(n);
    __syncthreads();

    // log prior density (Gaussian prior; the box prior is uniform on its support)
    auto logprior = [&](const double *x) -> double {
        double lp = 0.0;
#pragma unroll
        for (int a = 0; a < kGpD; ++a) {
            const double zt = (x[a] - P.pa[a]) / P.pb[a];
            lp += -0.5 * zt * zt;
        }
        return lp + P.logprior_norm;
    };

    // The chain as one loop with a single evaluation site: each pass picks the next test of the
    // current phase, evaluates it and advances.
    enum { PH_NEW = 0, PH_LEFT = 1, PH_RIGHT = 2, PH_SHRINK = 3, PH_FINAL = 4 };
    int phase = PH_NEW, st = 0, nl = 0, nr = 0, ns = 0;
    double tL = 0.0, tR = 0.0, logy = -INFINITY;
    for (;;) {
        if (phase == PH_NEW) {
            if (st == p) {
                if (MODE == MODE_FP64 || exact0) break;
                phase = PH_FINAL;   // stored log-likelihoods are FP64
                __syncthreads();    // the last accepted point is in sx0 for every wave
            } else {
                __syncthreads();   // every thread is done with the previous direction
                if (tid == 0) {
                    // direction z ~ N(0, I), v = Lsig z / |z|
                    double z[kGpD];
#pragma unroll
                    for (int q = 0; q < kGpD / 2; ++q) {
                        double ua, ub;
                        draw2(R.key0, R.key1, PUR_DIR, (uint32_t)j, it, (uint32_t)st,
                              (uint32_t)q, ua, ub);
                        box_muller(ua, ub, z[2 * q], z[2 * q + 1]);
                    }
                    double nz = 0.0;
#pragma unroll
                    for (int a = 0; a < kGpD; ++a) nz += z[a] * z[a];
                    nz = sqrt(nz);
                    for (int a = 0; a < kGpD; ++a) {
                        double s2 = 0.0;
                        for (int b = 0; b <= a; ++b) s2 += R.Lsig[a * P.D + b] * z[b];
                        sv[a] = s2 / nz;
                    }
                }
                __syncthreads();
                double U, uh;
                draw2(R.key0, R.key1, PUR_STEP, (uint32_t)j, it, (uint32_t)st, 0u, U, uh);
                logy = box ? -INFINITY : logprior(sx0) + log(uh);
                tL = -width * U;
                tR = tL + width;
                nl = nr = ns = 0;
                phase = PH_LEFT;
                continue;
            }
        }
        double t = 0.0;
        if (phase == PH_LEFT) {
            if (nl >= cap_out) { ++c_outcap; phase = PH_RIGHT; continue; }
            t = tL;
        } else if (phase == PH_RIGHT) {
            if (nr >= cap_out) { ++c_outcap; phase = PH_SHRINK; continue; }
            t = tR;
        } else if (phase == PH_SHRINK) {
            if (ns >= cap_sh) {
                // null move
                ++c_shcap;
                if (R.trace && tid == 0) {
                    int *tr = R.trace + ((size_t)j * p + st) * 4;
                    tr[0] = nl; tr[1] = nr; tr[2] = ns; tr[3] = 0;
                }
                ++st;
                phase = PH_NEW;
                continue;
            }
            double us, un2;
            draw2(R.key0, R.key1, PUR_SHRINK, (uint32_t)j, it, (uint32_t)st, (uint32_t)ns, us, un2);
            t = tL + us * (tR - tL);
        }
        double y[kGpD];
#pragma unroll
        for (int a = 0; a < kGpD; ++a) y[a] = (phase == PH_FINAL) ? sx0[a] : fma(t, sv[a], sx0[a]);
        int in = 1;
        if (phase != PH_FINAL) {
            ++c_tests;
            if (box) {
#pragma unroll
                for (int a = 0; a < kGpD; ++a) in &= (y[a] >= P.pa[a] && y[a] <= P.pb[a]) ? 1 : 0;
            } else {
                in = logprior(y) > logy ? 1 : 0;
            }
        }
        in = uniform_i(in);
        int r = 0, exact = 1;
        double L = -INFINITY;
        if (!in) {
            ++c_prej;
        } else {
            // the single evaluation site
            bool failed = false;
            if (P.gp_give_up) {
                failed = true;
                ++c_wait;
            } else if constexpr (MODE == MODE_FP64) {
                L = gp_eval<double>(y, n, smem, failed) - norm;
            } else {
                int need64 = (phase == PH_FINAL);
                if (!need64 && uniform_i(gp_illcond(P, y))) {   // FP64 only, no FP32 attempt
                    need64 = 1;
                    ++c_rc;
                } else if (!need64) {
                    L = gp_eval<float>(y, n, smem, failed) - norm;
                    need64 = uniform_i(failed || !(L == L) || gp_near(L, Lstar, P, y));
                    if (need64) ++c_rc; else exact = 0;
                }
                if (need64) L = gp_eval<double>(y, n, smem, failed) - norm;
            }
            if (failed) L = -INFINITY;
            if (phase == PH_FINAL) {
                logL0 = L;
                if (!(logL0 > Lstar)) ++c_viol;
                break;
            }
            ++c_evals;
            const int nf = uniform_i((L != L || L == INFINITY) ? 1 : 0);
            if (nf) L = -INFINITY;
            c_nonfin += nf;
            r = uniform_i(L > Lstar ? 1 : 0);
        }
        if (phase == PH_LEFT) {
            if (r) { tL -= width; ++nl; } else phase = PH_RIGHT;
        } else if (phase == PH_RIGHT) {
            if (r) { tR += width; ++nr; } else phase = PH_SHRINK;
        } else {
            ++ns;
            if (r) {
                // every thread has passed the evaluation's barriers: sx0 is free to update
                if (tid < kGpD) sx0[tid] = fma(t, sv[tid], sx0[tid]);
                logL0 = L;
                exact0 = exact;
                if (R.trace && tid == 0) {
                    int *tr = R.trace + ((size_t)j * p + st) * 4;
                    tr[0] = nl; tr[1] = nr; tr[2] = ns; tr[3] = 1;
                }
                ++st;
                phase = PH_NEW;
            } else {
                tL = t < 0.0 ? t : tL;
                tR = t < 0.0 ? tR : t;
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        const int slot = R.perm[j];
#pragma unroll
        for (int a = 0; a < kGpD; ++a) R.X[(size_t)a * R.m_pad + slot] = sx0[a];
        R.logL[slot] = logL0;
        atomicAdd(&R.ctr[0], c_evals);
        atomicAdd(&R.ctr[1], c_tests);
        atomicAdd(&R.ctr[2], c_prej);
        atomicAdd(&R.ctr[3], c_outcap);
        atomicAdd(&R.ctr[4], c_shcap);
        atomicAdd(&R.ctr[5], c_nonfin);
        atomicAdd(&R.ctr[6], c_rc);
        atomicAdd(&R.ctr[7], c_viol);
        if (c_wait) atomicAdd(&R.ctr[10], c_wait);
    }
}

template <typename F>
static hipError_t gp_lds(F *f, size_t bytes)
{
    return hipFuncSetAttribute((const void *)f, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

hipError_t launch_hrss_gp(const Launch &L, int mode, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    const size_t lds = (size_t)(gp_lds_bytes<double>() > gp_lds_bytes<float>() ? gp_lds_bytes<double>()
                                                                               : gp_lds_bytes<float>());
    if (mode == MODE_FP64) {
        hipError_t e = gp_lds(k_hrss_gp<MODE_FP64>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_hrss_gp<MODE_FP64>, dim3(L.nblocks), dim3(kGpThreads), lds, s, L);
    } else if (mode == MODE_FP32) {
        hipError_t e = gp_lds(k_hrss_gp<MODE_FP32>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_hrss_gp<MODE_FP32>, dim3(L.nblocks), dim3(kGpThreads), lds, s, L);
    } else {
        return hipErrorNotSupported;
    }
    return hipGetLastError();
}

hipError_t launch_eval_gp(const Launch &L, int mode, const double *X, int ld, int n, double *out,
                          int from_run, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    const size_t lds = (size_t)(gp_lds_bytes<double>() > gp_lds_bytes<float>() ? gp_lds_bytes<double>()
                                                                               : gp_lds_bytes<float>());
    if (mode == MODE_FP64) {
        hipError_t e = gp_lds(k_eval_gp<MODE_FP64>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_eval_gp<MODE_FP64>, dim3(L.nblocks), dim3(kGpThreads), lds, s, L, X,
                           ld, n, out, from_run);
    } else if (mode == MODE_FP32) {
        hipError_t e = gp_lds(k_eval_gp<MODE_FP32>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_eval_gp<MODE_FP32>, dim3(L.nblocks), dim3(kGpThreads), lds, s, L, X,
                           ld, n, out, from_run);
    } else {
        return hipErrorNotSupported;
    }
    return hipGetLastError();
}

}  // namespace nss
