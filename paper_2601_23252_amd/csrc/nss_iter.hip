// gfx950 kernels of an outer iteration beside the chains:
//
//  k_select      delete-k: sort (logL, index), threshold L*, unrolled evidence update of the
//                k deaths, dead record, termination flag (Sec. 2.1; App. D.2.1)
//  k_cov/k_chol  whitening: survivors' covariance + jitter, lower Cholesky factor (Sec. 3.2)
//  k_dirs        every chain's directions and step uniforms of the iteration
//  k_smc         adaptive tempered SMC: next temperature, resampling
//  k_logz        final live-set contribution to the evidence (Sec. 2.1)
#include "nss_chol.hpp"
#include "nss_internal.hpp"
#include "nss_rng.hpp"
#include "nss_tiles.hpp"
#include "nss_wave.hpp"

#include <math.h>
#include <type_traits>

namespace nss {

// ------------------------------------------------------------------------------------------
// delete-k, threshold, unrolled evidence, termination (one workgroup of 1024 threads)
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long key_of(double x)
{
    if (x == 0.0) x = 0.0;  // -0 -> +0
    const unsigned long long b = __double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double val_of(unsigned long long k)
{
    const unsigned long long b = (k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k;
    return __longlong_as_double(b);
}

// Block reductions over up to 16 waves; red has >= 32 doubles.  Each wave's value goes to LDS and
// every row of 16 lanes reduces them again.
__device__ __forceinline__ double wave_value(const double *red, int below, double none)
{
    const int i = threadIdx.x & 15;
    return i < below ? red[i] : none;
}
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum_fast(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return row_sum16(wave_value(red, (int)(blockDim.x >> 6), 0.0));
}
__device__ __forceinline__ void block_sum2(double &a, double &b, double *red)
{
    a = wave_sum_fast(a);
    b = wave_sum_fast(b);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = a;
        red[16 + (threadIdx.x >> 6)] = b;
    }
    __syncthreads();
    a = row_sum16(wave_value(red, (int)(blockDim.x >> 6), 0.0));
    b = row_sum16(wave_value(red + 16, (int)(blockDim.x >> 6), 0.0));
}
__device__ __forceinline__ double block_max(double v, double *red)
{
    v = row_max16(v);
    v = fmax(v, __shfl_xor(v, 16, 64));
    v = fmax(v, __shfl_xor(v, 32, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return row_max16(wave_value(red, (int)(blockDim.x >> 6), -INFINITY));
}
// Exclusive prefix sum over the block; all: the block's sum.
__device__ __forceinline__ double block_exscan(double v, double *red, double &all)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    double inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double t = __shfl_up(inc, o, 64);
        if (l >= o) inc += t;
    }
    __syncthreads();
    if (l == 63) red[w] = inc;
    __syncthreads();
    all = row_sum16(wave_value(red, (int)(blockDim.x >> 6), 0.0));
    return row_sum16(wave_value(red, w, 0.0)) + inc - v;
}

// packed lower-triangular index e = a(a+1)/2 + b  ->  (a, b)
__device__ __forceinline__ void unpack_tri(int e, int &a, int &b)
{
    a = (int)((sqrt(8.0 * e + 1.0) - 1.0) * 0.5);
    while (a * (a + 1) / 2 > e) --a;
    while ((a + 1) * (a + 2) / 2 <= e) ++a;
    b = e - a * (a + 1) / 2;
}

__device__ __forceinline__ double lse2(double a, double b)
{
    if (a == -INFINITY) return b;
    if (b == -INFINITY) return a;
    const double mx = fmax(a, b);
    return mx + log(exp(a - mx) + exp(b - mx));
}

// A lane's value at lane ^ S: moves within a row of 16 lanes where they exist (xor 4 = a mirror
// of eight, then of four), else through LDS.
template <int S>
__device__ __forceinline__ unsigned xor_lane(unsigned v)
{
    auto dpp = [](unsigned x, auto c) {
        return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, decltype(c)::value, 0xF, 0xF, false);
    };
    if constexpr (S == 1) return dpp(v, std::integral_constant<int, DPP_XOR1>{});
    else if constexpr (S == 2) return dpp(v, std::integral_constant<int, DPP_XOR2>{});
    else if constexpr (S == 4)
        return dpp(dpp(v, std::integral_constant<int, DPP_HMIR>{}), std::integral_constant<int, 0x1B>{});
    else if constexpr (S == 8) return dpp(v, std::integral_constant<int, 0x128>{});   // row_ror:8
    else return __shfl_xor(v, S, 64);
}
// Compare-exchange of a bitonic stage with the element S lanes away (element i0 + 64 e in
// register e of the lane).
template <int S, int E>
__device__ __forceinline__ void exchange_lanes(unsigned long long (&key)[E], int (&idx)[E], int i0,
                                               int size)
{
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned long long ko = (unsigned long long)xor_lane<S>((unsigned)(key[e] >> 32)) << 32 |
                                      xor_lane<S>((unsigned)key[e]);
        const int io = (int)xor_lane<S>((unsigned)idx[e]);
        const int i = i0 + 64 * e;
        const bool keep_min = ((i & S) == 0) == ((i & size) == 0);
        const bool less = ko < key[e] || (ko == key[e] && io < idx[e]);
        if (less == keep_min) { key[e] = ko; idx[e] = io; }
    }
}

// Sorts (logL, index) of a run by a bitonic network on registers: wave w holds elements
// 64 E w .. 64 E (w + 1) - 1, lane l of it 64 e + l in register e.  Exchanges at a distance below
// 64 are lane moves, up to 64 E register swaps, and only the longer ones (ten of the 66 stages at
// 2048 points) go through LDS and its barriers.  The sorted keys and indices are left in LDS.
template <int E>
__device__ __forceinline__ void sort_live(const DevRun &R, int m, unsigned long long *skey,
                                          int *sidx)
{
    const int tid = threadIdx.x, i0 = (tid >> 6) * 64 * E + (tid & 63);
    const auto logL = as_global((const double *)R.logL);
    int NP = 64;
    while (NP < m) NP <<= 1;
    unsigned long long key[E];
    int idx[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + 64 * e;
        key[e] = i < m ? key_of(logL[i]) : ~0ull;
        idx[e] = i < m ? i : 0x7FFFFFFF - kSelectThreads * E + i;   // (padding, in order)
    }
    for (int size = 2; size <= NP; size <<= 1) {
        for (int stride = size >> 1; stride >= 64 * E; stride >>= 1) {
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) { skey[i0 + 64 * e] = key[e]; sidx[i0 + 64 * e] = idx[e]; }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int i = i0 + 64 * e;
                const unsigned long long ko = skey[i ^ stride];
                const int io = sidx[i ^ stride];
                const bool keep_min = ((i & stride) == 0) == ((i & size) == 0);
                const bool less = ko < key[e] || (ko == key[e] && io < idx[e]);
                if (less == keep_min) { key[e] = ko; idx[e] = io; }
            }
        }
#pragma unroll
        for (int q = E / 2; q >= 1; q >>= 1) {
            if (size < 128 * q) continue;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (e & q) continue;
                const bool asc = ((i0 + 64 * e) & size) == 0;
                const bool gt = key[e] > key[e ^ q] || (key[e] == key[e ^ q] && idx[e] > idx[e ^ q]);
                if (gt == asc) {
                    const unsigned long long k = key[e];
                    const int i = idx[e];
                    key[e] = key[e ^ q]; idx[e] = idx[e ^ q];
                    key[e ^ q] = k; idx[e ^ q] = i;
                }
            }
        }
        if (size >= 64) exchange_lanes<32, E>(key, idx, i0, size);
        if (size >= 32) exchange_lanes<16, E>(key, idx, i0, size);
        if (size >= 16) exchange_lanes<8, E>(key, idx, i0, size);
        if (size >= 8) exchange_lanes<4, E>(key, idx, i0, size);
        if (size >= 4) exchange_lanes<2, E>(key, idx, i0, size);
        exchange_lanes<1, E>(key, idx, i0, size);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) { skey[i0 + 64 * e] = key[e]; sidx[i0 + 64 * e] = idx[e]; }
}

// E: elements per thread (1024 E >= m).
template <int E>
__global__ __launch_bounds__(kSelectThreads) void k_select(Launch Lc, int op)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const DevRun R = Lc.R[Lc.map[blockIdx.x].x];
    if (R.iscal[0]) return;
    const int m = R.m, k = R.k, tid = threadIdx.x;
    constexpr int NK = kSelectThreads * E;
    unsigned long long *key = (unsigned long long *)smem;
    int *idx = (int *)(key + NK);
    double *red = (double *)(idx + NK);
    int *st0 = (int *)(red + 32);
    const auto scal = as_global(R.scal);
    const auto ctr = as_global(R.ctr);
    const double logZ0 = scal[1], logX0 = scal[2], M0 = scal[3];   // (on their way early)
    const long long nd0 = (long long)ctr[9];
    if (tid == 0) *st0 = m;
    sort_live<E>(R, m, key, idx);
    __syncthreads();
    const auto perm = as_global(R.perm);
    for (int t = tid; t < m; t += kSelectThreads) perm[t] = idx[t];
    const double Lstar = val_of(key[k - 1]);
    for (int t = k + tid; t < m; t += kSelectThreads)   // the first point above L*
        if (val_of(key[t]) > Lstar && !(val_of(key[t - 1]) > Lstar)) *st0 = t;
    if (op == 2) {
        __syncthreads();
        if (tid == 0) {
            R.scal[0] = Lstar;
            R.iscal[1] = *st0;
            R.iscal[2] = m - *st0;
        }
        return;
    }
    // unrolled deaths j = 1..k at live counts n_j = m - j + 1
    const int per = (k + kSelectThreads - 1) / kSelectThreads;   // deaths per thread, at most E
    const int j0 = tid * per;
    double inv[E], lw[E], Lv[E], ssum = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int jj = j0 + e + 1;
        inv[e] = (e < per && jj <= k) ? 1.0 / (double)(m - jj + 1) : 0.0;
        ssum += inv[e];
    }
    double S_k;
    double lmax = -INFINITY, run = block_exscan(ssum, red, S_k);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        lw[e] = -INFINITY; Lv[e] = 0.0;
        if (inv[e] > 0.0) {
            Lv[e] = val_of(key[j0 + e]);
            lw[e] = Lv[e] + (logX0 - run) + log(-expm1(-inv[e]));
            run += inv[e];
            lmax = fmax(lmax, lw[e]);
        }
    }
    const double mx = block_max(lmax, red);
    double esum = 0.0, lsum = 0.0;   // sums of exp(lw - mx) and of it times logL
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (lw[e] != -INFINITY) {
            const double x = exp(lw[e] - mx);
            esum += x;
            lsum += x * Lv[e];
        }
    block_sum2(esum, lsum, red);
    const double lse_new = (mx == -INFINITY) ? -INFINITY : mx + log(esum);
    const double logZ1 = lse2(logZ0, lse_new);
    const double msum = (mx == -INFINITY) ? 0.0 : exp(mx - logZ1) * lsum;
    const double M1 = (logZ0 == -INFINITY ? 0.0 : exp(logZ0 - logZ1) * M0) + msum;
    const double logX1 = logX0 - S_k;
    // dead record
    const auto dead = as_global(R.dead);
    for (int t = tid; t < k; t += kSelectThreads)
        if (nd0 + t < R.dead_cap) dead[nd0 + t] = val_of(key[t]);
    if (R.deadx) {   // NS_FLAG_RECORD_POINTS: the dead points' coordinates, point-major [n][d]
        const int d = Lc.P[Lc.map[blockIdx.x].x].d;
        for (long long e = tid; e < (long long)k * d; e += blockDim.x) {
            const int t = (int)(e / d), a = (int)(e - (long long)t * d);
            if (nd0 + t < R.dead_cap)
                R.deadx[(nd0 + t) * d + a] = R.X[(size_t)a * R.m_pad + idx[t]];
        }
    }
    __syncthreads();
    if (tid == 0) {
        const int t0 = *st0;
        const double maxL = val_of(key[m - 1]);
        int done = (R.term_on && (logX1 + maxL - logZ1 < R.log_term)) ? 1 : 0;
        R.scal[0] = Lstar; R.scal[1] = logZ1; R.scal[2] = logX1; R.scal[3] = M1;
        R.iscal[1] = t0;
        R.iscal[2] = m - t0;
        if (!done && m - t0 <= 0) { R.iscal[4] = 1; done = 1; }
        R.iscal[0] = done;
        if (op == 1) R.iscal[3] += 1;
        R.ctr[9] = (unsigned long long)(nd0 + k);
    }
}

// ------------------------------------------------------------------------------------------
// whitening: survivors' covariance (one-pass about a fixed shift c = the best live point),
// partial sums over groups of survivors, then a single-workgroup reduction + Cholesky
// ------------------------------------------------------------------------------------------
// grid (tile, group); tile = lower 16x16 block (ta >= tb).  part2[g][tile][256], part1[g][D]
__global__ __launch_bounds__(256) void k_cov(Launch Lc)
{
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    if (R.iscal[0]) return;
    // frozen whitening: the first iteration's factor, or one the caller supplied, is kept
    if (R.freeze && (R.iscal[3] > 0 || R.iscal[6])) return;
    const int d = P.d;
    const int nt = P.D / 16, ntile = nt * (nt + 1) / 2;
    const int G = R.covG;
    double *part1 = R.part1, *part2 = R.part2;
    const int tile = bm.y % ntile, g = bm.y / ntile, tid = threadIdx.x;
    int ta, tb;
    unpack_tri(tile, ta, tb);
    const auto X = as_global((const double *)R.X);
    const auto perm = as_global((const int *)R.perm);
    const int off = R.smc ? 0 : R.k;   // SMC: every particle
    const int n = R.m - off;
    const int s0 = (int)((long long)n * g / G), s1 = (int)((long long)n * (g + 1) / G);
    const int cidx = perm[R.m - 1];
    // up to 64 survivors at a time, 16 coordinates of tile a and 16 of tile b each: a thread's
    // eight elements, their indices and shifts are requested together
    __shared__ double ca[64][17], cb[64][17];
    const int c = tid & 31;
    const int coord = (c < 16) ? ta * 16 + c : tb * 16 + (c - 16);
    const auto col = X + (size_t)(coord < d ? coord : 0) * R.m_pad;
    const double shift = col[cidx];
    double acc = 0.0, acc1 = 0.0;
    for (int sb = s0; sb < s1; sb += 64) {
        const int ns = (s1 - sb < 64) ? s1 - sb : 64;
        int pi[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int s = (tid >> 5) + 8 * q;
            pi[q] = perm[off + sb + (s < ns ? s : 0)];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int s = (tid >> 5) + 8 * q;
            const double v = (s < ns && coord < d) ? col[pi[q]] - shift : 0.0;
            if (c < 16) ca[s][c] = v; else cb[s][c - 16] = v;
        }
        __syncthreads();
        for (int s = 0; s < ns; ++s) acc += ca[s][tid & 15] * cb[s][tid >> 4];
        if (ta == tb && tid < 16)
            for (int s = 0; s < ns; ++s) acc1 += ca[s][tid];
        __syncthreads();
    }
    part2[((size_t)g * ntile + tile) * 256 + tid] = acc;
    if (ta == tb && tid < 16) part1[(size_t)g * P.D + ta * 16 + tid] = acc1;
}

// The factor of runs up to D = 128, one workgroup of eight waves per run: tile t of the lower
// triangle in wave t mod 8's registers; for each block column its tiles, up to date, go to LDS
// and are eliminated with one row per lane (the diagonal tile's rows in a wave's first lanes, 48
// rows below it in the others), while the other waves' tiles take the previous column on MFMA.
// Bound by the pivots' dependent chain, about 4,000 cycles per 16 columns, and two barriers a
// block column.  d = 5, 32, 50, 64: 8.1, 15.7, 25 and 39 us; a column at a time with three barriers
// each took 10.8, 32.6, 62 and 101.  The sums, products, roots and quotients are those of that
// column-by-column factor in its order, bit for bit: with fewer survivors than dimensions the
// covariance is singular but for the jitter and its last columns are rounding errors, which the
// chains' steps follow (a factor of other roundings moved such runs' points by 1e-7).
constexpr int kCholThreads = 512, kCholWaves = 8;
constexpr int kCholSlots = 5;            // 36 tiles at D = 128
constexpr size_t kCholLds = (2 * 8 * kTile + 128 + 32) * 8 + 16;
__global__ __launch_bounds__(kCholThreads) void k_chol(Launch Lc)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem &P = Lc.P[bm.x];
    const DevRun &R = Lc.R[bm.x];
    if (P.D > 128 || R.iscal[0]) return;
    if (R.freeze && (R.iscal[3] > 0 || R.iscal[6])) return;
    typedef Mf<double>::v4 v4;
    double *pan = (double *)smem;            // [2][8] tiles
    double *mc = pan + 2 * 8 * kTile;        // mean - shift, [128]
    double *red = mc + 128;                  // [32]
    int *fail = (int *)(red + 32);
    const int G = R.covG, D = P.D, d = P.d;
    const int ntile = (D / 16) * (D / 16 + 1) / 2;
    const auto part1 = as_global((const double *)R.part1), part2 = as_global((const double *)R.part2);
    const auto Lsig = as_global(R.Lsig), Lpk = as_global(R.Lpk);
    const int n = R.smc ? R.m : R.m - R.k;
    const int tid = threadIdx.x, l = tid & 63, w = uniform_i(tid >> 6);
    const int NT = (d + 15) >> 4, NTT = NT * (NT + 1) / 2;
    if (tid < 16 * NT) {
        double s = 0.0;
        if (tid < d) for (int g = 0; g < G; ++g) s += part1[(size_t)g * D + tid];
        mc[tid] = s / n;
    }
    if (tid == 0) *fail = 0;
    // sum of a tile's products over the groups: element (row, col) of tile t
    auto summed = [&](int t, int row, int col) -> double {
        const auto src = part2 + (size_t)t * 256 + col * 16 + row;
        double s = 0.0;
#pragma unroll 4
        for (int g = 0; g < G; ++g) s += src[(size_t)g * ntile * 256];
        return s;
    };
    // the jitter, 1e-12 * tr / d: the trace as a sum over lanes a = 0..127 and their two waves
    auto jitter = [&](double v) -> double {
        v = wave_sum(v);
        __syncthreads();
        if (l == 0) red[w] = v;
        __syncthreads();
        return 1e-12 * (red[0] + red[1]) / d;
    };
    auto variance = [&](int a) -> double {   // without the jitter
        const int I = a >> 4;
        return summed(I * (I + 1) / 2 + I, a & 15, a & 15) / n - mc[a] * mc[a];
    };
    if (R.diag) {   // the diagonal metric: square roots of the (jittered) variances
        __syncthreads();
        const double v = tid < d ? variance(tid) : 0.0;
        const double vj = v + jitter(v);
        if (tid < d && !(vj > 0.0)) *fail = 1;
        __syncthreads();
        if (tid < d) {
            const double x = *fail ? (v > 0.0 ? sqrt(v) : 1.0) : sqrt(vj);
            Lsig[tid * D + tid] = x;
            Lpk[tid * (tid + 1) / 2 + tid] = x;
        }
        if (tid == 0 && *fail) atomicAdd(&R.ctr[8], 1ull);
        return;
    }
    int tI[kCholSlots], tK[kCholSlots];
    v4 acc[kCholSlots];
#pragma unroll
    for (int s = 0; s < kCholSlots; ++s) {
        const int t = w + kCholWaves * s;
        int I = -1, K = -1;
        if (t < NTT) tile_ik(t, I, K);
        tI[s] = I;
        tK[s] = K;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = Mf<double>::row(l, r), col = l & 15;
            acc[s][r] = (I >= 0 && 16 * I + row < d && 16 * K + col < d) ? summed(t, row, col) : 0.0;
        }
    }
    __syncthreads();   // mc
    double *diag = pan;
#pragma unroll
    for (int s = 0; s < kCholSlots; ++s) {
        if (tI[s] < 0) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = 16 * tI[s] + Mf<double>::row(l, r), b = 16 * tK[s] + (l & 15);
            if (a < d && b < d) {
                acc[s][r] = acc[s][r] / n - mc[a] * mc[b];
                if (a == b) diag[a] = acc[s][r];
            } else if (a == b) {
                acc[s][r] = 1.0;   // padded coordinates: identity (never stored)
            }
        }
    }
    __syncthreads();
    const double jit = jitter(tid < d ? diag[tid] : 0.0);
#pragma unroll
    for (int s = 0; s < kCholSlots; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = Mf<double>::row(l, r);
            if (tI[s] >= 0 && tI[s] == tK[s] && row == (l & 15) && 16 * tI[s] + row < d)
                acc[s][r] += jit;
        }
    for (int J = 0; J < NT; ++J) {
        double *cur = pan + (J & 1) * 8 * kTile;
        const double *prv = pan + ((J & 1) ^ 1) * 8 * kTile;   // column J - 1 of the factor
        auto update = [&](v4 &a, int I, int K) {
            const double *pI = prv + I * kTile + (l & 15) * kTileLd + (l >> 4);
            const double *pK = prv + K * kTile + (l & 15) * kTileLd + (l >> 4);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a = Mf<double>::mma(-pI[4 * ks], pK[4 * ks], a);
        };
#pragma unroll
        for (int s = 0; s < kCholSlots; ++s)
            if (tK[s] == J) {
                if (J > 0) update(acc[s], tI[s], J);
                store_tile<double>(acc[s], cur + tI[s] * kTile, l);
            }
        __syncthreads();
        const int rows = 16 * (NT - 1 - J);
        if (w == 0 || 48 * w < rows) {
            const int below = 48 * w + (l - 16);
            const bool prow = l >= 16 && below < rows;
            const int a0 = 16 * J + (l < 16 ? l : (prow ? 16 + below : 0));
            double *rp = cur + (a0 >> 4) * kTile + (a0 & 15) * kTileLd;
            double a[16], p0, p1;
            int bad;
#pragma unroll
            for (int c = 0; c < 16; ++c) a[c] = rp[c];
            eliminate<double, true>(a, p0, p1, bad);
            if (w == 0 && l == 0 && bad) *fail = 1;
            if (prow || (w == 0 && l < 16)) {
                const int ro = a0 * (a0 + 1) / 2;
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    const int b = 16 * J + c;
                    if (prow) rp[c] = a[c];
                    if (a0 < d && b <= a0) {
                        Lsig[a0 * D + b] = a[c];
                        Lpk[ro + b] = a[c];
                    }
                }
            }
        }
        if (J > 0) {
#pragma unroll
            for (int s = 0; s < kCholSlots; ++s)
                if (tK[s] > J) update(acc[s], tI[s], tK[s]);
        }
        __syncthreads();
    }
    if (*fail) {
        // diagonal fallback: square roots of the variances
        for (int e = tid; e < d * d; e += kCholThreads) {
            const int a = e / d, b = e - a * d;
            if (b < a) { Lsig[a * D + b] = 0.0; Lpk[a * (a + 1) / 2 + b] = 0.0; }
        }
        if (tid < d) {
            const double v = variance(tid), x = v > 0.0 ? sqrt(v) : 1.0;
            Lsig[tid * D + tid] = x;
            Lpk[tid * (tid + 1) / 2 + tid] = x;
        }
        if (tid == 0) atomicAdd(&R.ctr[8], 1ull);
    }
}

// The factor of runs above D = 128, worked in place in the run's packed factor (global memory,
// coherent within the workgroup across its barriers).
__global__ __launch_bounds__(1024) void k_chol_wide(Launch Lc)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    if (P.D <= 128 || R.iscal[0]) return;
    if (R.freeze && (R.iscal[3] > 0 || R.iscal[6])) return;
    const int G = R.covG, ntile = (P.D / 16) * (P.D / 16 + 1) / 2;
    const double *part1 = R.part1, *part2 = R.part2;
    const int D = P.D, d = P.d, tid = threadIdx.x;
    double *A = R.Lpk;                       // packed lower triangle, D(D+1)/2
    double *mc = (double *)smem;             // mean - shift, [D]
    double *red = mc + D;                    // [32]
    int *fail = (int *)(red + 32);
    const int n = R.smc ? R.m : R.m - R.k;
    for (int a = tid; a < D; a += blockDim.x) {
        double s = 0.0;
        if (a < d) for (int g = 0; g < G; ++g) s += part1[(size_t)g * D + a];
        mc[a] = s / n;
    }
    if (tid == 0) *fail = 0;
    __syncthreads();
    const int np = D * (D + 1) / 2;
    for (int e = tid; e < np; e += blockDim.x) {
        int a, b;  // a >= b
        unpack_tri(e, a, b);
        double v = 0.0;
        if (a < d && b < d && (a == b || !R.diag)) {   // the diagonal metric needs variances only
            const int ta = a >> 4, tb = b >> 4;
            const int tile = ta * (ta + 1) / 2 + tb;
            const int off = (b & 15) * 16 + (a & 15);
            double s = 0.0;
            for (int g = 0; g < G; ++g) s += part2[((size_t)g * ntile + tile) * 256 + off];
            v = s / n - mc[a] * mc[b];
        } else if (a == b) {
            v = 1.0;  // padded coordinates: identity (never used, keeps the factor regular)
        }
        A[e] = v;
    }
    __syncthreads();
    // jitter: 1e-12 * tr / d on the diagonal
    double tr = 0.0;
    for (int a = tid; a < d; a += blockDim.x) tr += A[a * (a + 1) / 2 + a];
    tr = block_sum(tr, red);
    for (int a = tid; a < d; a += blockDim.x) A[a * (a + 1) / 2 + a] += 1e-12 * tr / d;
    __syncthreads();
    // right-looking Cholesky on the packed lower triangle; for the diagonal metric it reduces
    // to the square roots of the (jittered) variances, taken directly
    if (R.diag) {
        for (int a = tid; a < d; a += blockDim.x) {
            const double v = A[a * (a + 1) / 2 + a];
            if (!(v > 0.0)) *fail = 1;
            else A[a * (a + 1) / 2 + a] = sqrt(v);
        }
        __syncthreads();
    } else
    for (int j = 0; j < d; ++j) {
        const double ajj = A[j * (j + 1) / 2 + j];
        if (!(ajj > 0.0)) { if (tid == 0) *fail = 1; break; }
        const double ljj = sqrt(ajj);
        __syncthreads();
        for (int i = j + 1 + tid; i < d; i += blockDim.x) A[i * (i + 1) / 2 + j] /= ljj;
        __syncthreads();
        if (tid == 0) A[j * (j + 1) / 2 + j] = ljj;
        const int rem = d - j - 1;
        for (int e = tid; e < rem * rem; e += blockDim.x) {
            const int ii = e / rem, r2 = e - ii * rem;
            if (r2 > ii) continue;
            const int i = j + 1 + ii, l2 = j + 1 + r2;
            A[i * (i + 1) / 2 + l2] -= A[i * (i + 1) / 2 + j] * A[l2 * (l2 + 1) / 2 + j];
        }
        __syncthreads();
    }
    __syncthreads();
    const int failed = *fail;
    if (failed) {
        // diagonal fallback: sqrt of the (jittered) variances, recomputed from the partials
        for (int e = tid; e < np; e += blockDim.x) A[e] = 0.0;
        __syncthreads();
        for (int a = tid; a < d; a += blockDim.x) {
            const int ta = a >> 4;
            const int tile = ta * (ta + 1) / 2 + ta;
            const int off = (a & 15) * 16 + (a & 15);
            double s = 0.0;
            for (int g = 0; g < G; ++g) s += part2[((size_t)g * ntile + tile) * 256 + off];
            const double v = s / n - mc[a] * mc[a];
            A[a * (a + 1) / 2 + a] = (v > 0.0) ? sqrt(v) : 1.0;
        }
        if (tid == 0) atomicAdd(&R.ctr[8], 1ull);
    }
    __syncthreads();
    for (int a = d; a < D; ++a)
        if (tid == 0) A[a * (a + 1) / 2 + a] = 0.0;  // padded coordinates never move
    for (int e = tid; e < np; e += blockDim.x) {
        int a, b;
        unpack_tri(e, a, b);
        R.Lpk[e] = (a < d && b < d) ? A[e] : 0.0;
    }
    for (int e = tid; e < D * D; e += blockDim.x) {
        const int a = e / D, b = e - a * D;
        R.Lsig[e] = (b <= a && a < d) ? A[a * (a + 1) / 2 + b] : 0.0;
    }
}

// ------------------------------------------------------------------------------------------
// directions of every chain and step of the iteration (they do not depend on the chains'
// outcomes): z ~ N(0, I_d) from Philox purpose DIR, v = L z / |z| (unit Mahalanobis length;
// random-walk runs: the proposal step v = s L z), dirbuf[(j p + s) D + a], zero for a >= d.
// 64 directions per workgroup (32 from D = 128).
// ------------------------------------------------------------------------------------------
// directions per k_dirs workgroup: 64, or 32 from D = 128 (at 320 their normals fill the LDS)
__host__ __device__ constexpr int dir_rows(int D) { return D > 64 ? 32 : 64; }
__host__ __device__ inline int dirs_lds_bytes(int D)
{
    const int rows = dir_rows(D);
    return al16(rows * (D + 1) * 8) + rows * 8 + rows * kStepU * 8 + 2 * rows * 4;
}

// The normals and uniforms are drawn by all threads; V = L Z is one small FP64 MFMA product per
// workgroup.  The row tiles of L go to the waves in pairs (t, NT - 1 - t) of equal triangular work,
// each with all the workgroup's directions or its share of them, so that L is read once per
// workgroup (as the A operand, from the run's row-major factor; the normals in LDS are the B
// operand, lane l: direction 16 g + (l & 15), coordinate 4 ks + (l >> 4)).  Register i of a tile's
// result is V[16 t + (l >> 4) + 4 i][16 g + (l & 15)]; the results go back through the normals'
// rows so that the stores to the direction buffer are whole rows.  What bounds it is the vector
// arithmetic of the generator, log, sine and cosine, then the product and the stores, one after the
// other in a workgroup: 32 directions a workgroup at D >= 128 keep four workgroups on a compute
// unit at different ones (64: 3.75 ms against 3.56 for 64 runs of d <= 128 and 250 chains; with L
// read by every wave for 16 directions, as before, 5.59 ms; 1.25e6 directions of d = 100: 1.88 ms
// then, 1.10 now).
template <int D>
__global__ __launch_bounds__(256) void k_dirs(Launch Lc)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    if (R.iscal[0] || R.iscal[2] <= 0) return;
    constexpr int LDZ = D + 1, ROWS = dir_rows(D);
    double *zs = (double *)smem;
    double *nz = zs + ROWS * LDZ;
    double *udraw = nz + ROWS;              // [ROWS][kStepU] raw uniforms
    int *rj = (int *)(udraw + ROWS * kStepU);   // chain of each row (-1 past the end)
    int *rs = rj + ROWS;                    // step of each row
    const int tid = threadIdx.x, d = P.d, p = R.p;
    const long long total = (long long)R.k * p;
    const long long base = (long long)bm.y * ROWS;
    const uint32_t it = (uint32_t)R.iscal[3] + 1u;
    if (tid < ROWS) {
        const long long idx = base + tid;
        int j = -1, st = 0;
        if (idx < total) { j = (int)(idx / p); st = (int)(idx - (long long)j * p); }
        rj[tid] = j;
        rs[tid] = st;
    }
    __syncthreads();
    const int nq = (d + 1) >> 1;
    for (int i = tid; i < ROWS * nq; i += 256) {
        const int r = i / nq, q = i - r * nq;
        const int j = rj[r];
        if (j < 0) continue;
        double ua, ub, z0, z1;
        draw2(R.key0, R.key1, PUR_DIR, (uint32_t)j, it, (uint32_t)rs[r], (uint32_t)q, ua, ub);
        box_muller(ua, ub, z0, z1);
        zs[r * LDZ + 2 * q] = z0;
        if (2 * q + 1 < d) zs[r * LDZ + 2 * q + 1] = z1;
    }
    // The step's uniforms: ubuf[0] = tL0 = -w U, ubuf[1] = the height uniform uh (purpose
    // STEP), ubuf[2 + i] = the uniform of the i-th shrink proposal (purpose SHRINK, draw i).
    for (int i = tid; i < ROWS * kStepU; i += 256) {
        const int r = i / kStepU, q = i - r * kStepU;
        const int j = rj[r], st = rs[r];
        if (j < 0) continue;
        double ua, ub;
        if (q < 2) {
            draw2(R.key0, R.key1, PUR_STEP, (uint32_t)j, it, (uint32_t)st, 0u, ua, ub);
            udraw[r * kStepU + q] = (q == 0) ? ua : ub;
        } else {
            draw2(R.key0, R.key1, PUR_SHRINK, (uint32_t)j, it, (uint32_t)st, (uint32_t)(q - 2), ua, ub);
            udraw[r * kStepU + q] = ua;
        }
    }
    __syncthreads();
    if (tid < ROWS && rj[tid] >= 0) {
        const double *u = udraw + tid * kStepU;
        const auto o = as_global(R.ubuf) + (base + tid) * kStepU;
        o[0] = -R.width * u[0];
        for (int q = 1; q < kStepU; ++q) o[q] = u[q];
    }
    const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
    // |z| of 16 directions a wave: four partial sums per direction, then lane exchanges; HRSS
    // scales to unit Mahalanobis length, the random walk by the proposal's s
    if (16 * w < ROWS) {
        const int r = 16 * w + li;
        double s2 = 0.0;
        for (int a = lk; a < d; a += 4) {
            const double z = zs[r * LDZ + a];
            s2 += z * z;
        }
        s2 += __shfl_xor(s2, 16, 64);
        s2 += __shfl_xor(s2, 32, 64);
        if (lk == 0) nz[r] = sqrt(s2);
    }
    constexpr int NT = D / 16, NPR = NT / 2, NG = ROWS / 16;   // row tiles, pairs, column groups
    constexpr int WPP = NPR < 4 ? 4 / NPR : 1;                 // waves per pair
    constexpr int GPW = NG / WPP < 1 ? 1 : NG / WPP;           // column groups per wave
    constexpr int PPW = (NPR + 3) / 4;                         // pairs per wave
    const auto L = as_global((const double *)R.Lsig) + li * D + lk;
    d4 acc[PPW][2][GPW];
    const int g0 = (w % WPP) * GPW;
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
        const int pr = w / WPP + 4 * q;
#pragma unroll
        for (int g = 0; g < GPW; ++g) acc[q][0][g] = acc[q][1][g] = (d4){0.0, 0.0, 0.0, 0.0};
        if (pr >= NPR) continue;
        const int ta = pr, tb = NT - 1 - pr;
        const auto La = L + 16 * ta * D, Lb = L + 16 * tb * D;
        const int na = 4 * ta + 4, nb = 4 * tb + 4;            // L is zero above its diagonal
        // four k-steps of both tiles requested at a time
        for (int k0 = 0; k0 < nb; k0 += 4) {
            double a0[4], a1[4], z[GPW][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a1[i] = Lb[4 * (k0 + i)];
                a0[i] = k0 < na ? La[4 * (k0 + i)] : 0.0;
#pragma unroll
                for (int g = 0; g < GPW; ++g) {
                    const int bb = 4 * (k0 + i) + lk;
                    z[g][i] = bb < d ? zs[(16 * (g0 + g) + li) * LDZ + bb] : 0.0;
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int g = 0; g < GPW; ++g) {
                    acc[q][1][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[i], z[g][i], acc[q][1][g], 0, 0, 0);
                    if (k0 < na)
                        acc[q][0][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[i], z[g][i], acc[q][0][g], 0, 0, 0);
                }
        }
    }
    __syncthreads();   // every wave has read the normals
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
        const int pr = w / WPP + 4 * q;
        if (pr >= NPR) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int t = h ? NT - 1 - pr : pr;
#pragma unroll
            for (int g = 0; g < GPW; ++g) {
                const int r = 16 * (g0 + g) + li;
                const double n = nz[r], sc = R.rw ? R.width : 1.0 / n;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int a = 16 * t + lk + 4 * i;
                    const double y = acc[q][h][g][i];
                    double v = y * sc;
                    if (!R.rw) v = fma(fma(-v, n, y), sc, v);   // the quotient y / n
                    zs[r * LDZ + a] = a < d ? v : 0.0;
                }
            }
        }
    }
    __syncthreads();
    const auto out = as_global(R.dirbuf) + base * D;
    const long long left = total - base;
    const int nrow = left < ROWS ? (int)left : ROWS;
    for (int e = tid; e < nrow * D; e += 256) {
        const int rr = e / D, a = e - rr * D;
        out[e] = zs[rr * LDZ + a];
    }
}

// ------------------------------------------------------------------------------------------
// adaptive tempered SMC (the slice-sampling mutation runs in k_hrss with R.smc set)
// ------------------------------------------------------------------------------------------
// One workgroup per run.  op 0: start at beta = 0 (identity order, log Z = 0).  op 1 (the
// start of a step): the next inverse temperature by 50 bisection steps on the ESS of the
// incremental weights exp((b - beta) (logL - max logL)) (target rho m, or beta = 1), the log
// mean incremental weight added to log Z, systematic resampling with one uniform (purpose
// RESAMPLE, counter (0, step)) against the cumulative normalised weights, and the gather of
// the resampled particles into slots 0..m-1.  op 2 (the end of a step): the step count, and
// done once beta = 1.  scal[0] = beta, scal[1] = log Z; iscal[5] = this step reached beta = 1.
// The step's draws (resampling, directions, chains) use iteration number iscal[3] + 1.
constexpr int kSmcPer = kMaxLive / kSelectThreads;   // particles per thread, contiguous

__global__ __launch_bounds__(kSelectThreads) void k_smc(Launch Lc, int op)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[32];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    const int m = R.m, tid = threadIdx.x;
    if (op == 0) {
        for (int i = tid; i < m; i += blockDim.x) R.perm[i] = i;
        if (tid == 0) {
            R.scal[0] = 0.0; R.scal[1] = 0.0; R.scal[2] = 0.0; R.scal[3] = 0.0;
            R.iscal[1] = 0; R.iscal[2] = m; R.iscal[5] = 0;
        }
        return;
    }
    if (op == 2) {   // the step's draws used iteration number iscal[3] + 1
        if (tid == 0 && !R.iscal[0]) {
            R.iscal[3] += 1;
            if (R.iscal[5]) R.iscal[0] = 1;
        }
        return;
    }
    if (R.iscal[0]) return;
    double *cum = (double *)smem;                         // [m]
    int *par = (int *)(smem + (size_t)kMaxLive * 8);      // [m]
    const double beta = R.scal[0];
    // particle tid + 1024 q in register q: every thread has its share at any m
    double Lr[kSmcPer];
    double lmax = -INFINITY;
    const int nq = (m + kSelectThreads - 1) / kSelectThreads;
#pragma unroll
    for (int q = 0; q < kSmcPer; ++q) {
        const int i = tid + q * kSelectThreads;
        Lr[q] = (i < m) ? R.logL[i] : -INFINITY;
        lmax = fmax(lmax, Lr[q]);
    }
    lmax = block_max(lmax, red);
    if (!(lmax > -INFINITY)) {   // every particle has log L = -inf: nothing to weigh
        if (tid == 0) { R.iscal[4] = 1; R.iscal[0] = 1; }
        return;
    }
    auto ess = [&](double b) -> double {
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int q = 0; q < kSmcPer; ++q) {
            if (q < nq && Lr[q] > -INFINITY) {
                const double e = exp((b - beta) * (Lr[q] - lmax));
                s1 += e;
                s2 += e * e;
            }
        }
        block_sum2(s1, s2, red);
        return s1 * s1 / s2;
    };
    const double target = R.ess_frac * m;
    double nb = 1.0;
    if (ess(1.0) < target) {
        double lo = beta, hi = 1.0;
        for (int t = 0; t < 50; ++t) {
            const double mid = 0.5 * (lo + hi);
            if (ess(mid) >= target) lo = mid; else hi = mid;
        }
        nb = lo > beta ? lo : hi;
    }
    const double db = nb - beta;
    // cumulative weights in particle order: slices of 1024, each scanned from the last one's end
    double sw = 0.0;
#pragma unroll
    for (int q = 0; q < kSmcPer; ++q) {
        if (q >= nq) break;
        const int i = tid + q * kSelectThreads;
        const double wt = (Lr[q] > -INFINITY) ? exp(db * (Lr[q] - lmax)) : 0.0;
        double all;
        const double pre = block_exscan(wt, red, all);
        if (i < m) cum[i] = sw + (pre + wt);
        sw += all;
    }
    __syncthreads();
    for (int i = tid; i < m; i += blockDim.x) cum[i] /= sw;
    const uint32_t it = (uint32_t)R.iscal[3] + 1u;
    double u, unused;
    draw2(R.key0, R.key1, PUR_RESAMPLE, 0u, it, 0u, 0u, u, unused);
    __syncthreads();
    // parent of slot j: the first particle whose cumulative weight reaches (u + j) / m
    for (int j = tid; j < m; j += blockDim.x) {
        const double pos = (u + j) / m;
        int lo = 0, hi = m - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cum[mid] >= pos) hi = mid; else lo = mid + 1;
        }
        par[j] = lo;
        R.parents[j] = lo;
    }
    __syncthreads();
    // gather through the scratch copy, then back into the live arrays
    const int d = P.d;
    const auto X = as_global(R.X), Xt = as_global(R.Xtmp), lg = as_global(R.logL), lt = as_global(R.Ltmp);
    const size_t ld = R.m_pad;
    for (int j = tid; j < m; j += blockDim.x) {
        const int pj = par[j];
        lt[j] = lg[pj];
#pragma unroll 8
        for (int a = 0; a < d; ++a) Xt[a * ld + j] = X[a * ld + pj];
    }
    __syncthreads();
    for (int j = tid; j < m; j += blockDim.x) {   // (each thread reads back what it wrote)
        lg[j] = lt[j];
#pragma unroll 8
        for (int a = 0; a < d; ++a) X[a * ld + j] = Xt[a * ld + j];
    }
    if (tid == 0) {
        R.scal[0] = nb;
        R.scal[1] += db * lmax + log(sw) - log((double)m);
        R.iscal[1] = 0;
        R.iscal[2] = m;
        R.iscal[5] = (nb == 1.0) ? 1 : 0;
    }
}

// ------------------------------------------------------------------------------------------
// final live-set contribution (non-destructive): scal[4..6] = ln Z, sqrt(H/m), H
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_logz(Launch Lc)
{
    const DevRun R = Lc.R[Lc.map[blockIdx.x].x];
    __shared__ double red[32];
    const int m = R.m, k = R.k, n = m - k, tid = threadIdx.x;
    double mx = -INFINITY;
    for (int t = k + tid; t < m; t += blockDim.x) mx = fmax(mx, R.logL[R.perm[t]]);
    mx = block_max(mx, red);
    double s = 0.0;
    for (int t = k + tid; t < m; t += blockDim.x) s += exp(R.logL[R.perm[t]] - mx);
    s = block_sum(s, red);
    const double logZ = R.scal[1], logX = R.scal[2], M = R.scal[3];
    const double lme = mx + log(s) - log((double)n);
    const double zf = lse2(logZ, logX + lme);
    double mt = 0.0;
    for (int t = k + tid; t < m; t += blockDim.x) {
        const double L = R.logL[R.perm[t]];
        const double lw = logX - log((double)n) + L;
        if (lw != -INFINITY) mt += exp(lw - zf) * L;
    }
    mt = block_sum(mt, red);
    if (tid == 0) {
        const double Mf = (logZ == -INFINITY ? 0.0 : exp(logZ - zf) * M) + mt;
        const double H = Mf - zf;
        R.scal[4] = zf;
        R.scal[5] = sqrt(H > 0.0 ? H / m : 0.0);
        R.scal[6] = H;
    }
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
int dirs_rows(int D) { return dir_rows(D); }

template <typename F>
static hipError_t set_lds(F *f, size_t bytes)
{
    return hipFuncSetAttribute((const void *)f, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

hipError_t launch_smc(const Launch &L, int op, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    const size_t lds = (size_t)kMaxLive * 12;
    hipError_t e = set_lds(k_smc, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_smc, dim3(L.nblocks), dim3(kSelectThreads), lds, s, L, op);
    return hipGetLastError();
}

template <int E>
static hipError_t select_t(const Launch &L, int op, hipStream_t s)
{
    const size_t lds = (size_t)kSelectThreads * E * 12 + 32 * 8 + 16;
    hipError_t e = set_lds(k_select<E>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_select<E>, dim3(L.nblocks), dim3(kSelectThreads), lds, s, L, op);
    return hipGetLastError();
}

hipError_t launch_select(const Launch &L, int op, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    if (L.max_m <= kSelectThreads) return select_t<1>(L, op, s);
    if (L.max_m <= 2 * kSelectThreads) return select_t<2>(L, op, s);
    if (L.max_m <= 4 * kSelectThreads) return select_t<4>(L, op, s);
    return select_t<8>(L, op, s);
}

hipError_t launch_cov(const Launch &cov, const Launch &one, int D, hipStream_t s)
{
    if (one.nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cov, dim3(cov.nblocks), dim3(256), 0, s, cov);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = set_lds(k_chol, kCholLds)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_chol, dim3(one.nblocks), dim3(kCholThreads), kCholLds, s, one);
    if ((e = hipGetLastError()) != hipSuccess || D <= 128) return e;
    const size_t lds = (size_t)(D + 32) * 8 + 16;
    if ((e = set_lds(k_chol_wide, lds)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_chol_wide, dim3(one.nblocks), dim3(1024), lds, s, one);
    return hipGetLastError();
}

template <int D>
static hipError_t dirs_t(const Launch &L, hipStream_t s)
{
    const size_t lds = (size_t)dirs_lds_bytes(D);
    hipError_t e = set_lds(k_dirs<D>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dirs<D>, dim3(L.nblocks), dim3(256), lds, s, L);
    return hipGetLastError();
}

hipError_t launch_dirs(const Launch &L, int D, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    if (D == 32) return dirs_t<32>(L, s);
    if (D == 64) return dirs_t<64>(L, s);
    if (D == 128) return dirs_t<128>(L, s);
    if (D == 320) return dirs_t<320>(L, s);
    return hipErrorInvalidValue;
}

hipError_t launch_logz(const Launch &L, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_logz, dim3(L.nblocks), dim3(1024), 0, s, L);
    return hipGetLastError();
}
}  // namespace nss
