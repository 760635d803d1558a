// Post-hoc geometric uncertainty of a run (App. "Estimation of prior volumes and propagation
// of geometric uncertainty"): R replicas of the prior-volume trajectory with random shrinkages,
// trapezoid weights at inverse temperature beta, log Z per replica, the geometric-mean weights
// over the replicas and their Kish effective sample size.
//
// Deaths g = 0..N-1 in likelihood order: the dead record (the j-th death of a batch, j = 0..k-1,
// sees n = m - j live points) followed by the final survivors in ascending logL (n = nf - q).
// Replica r: log t_g = log(u_g) / n_g with u_g the first (g even) or second (g odd) uniform of
// Philox (purpose GEOM, index r, counter word g/2); log X_g = sum_{h<g} log t_h (X before death
// g); the trapezoid element X_g (1 - t_g t_{g+1}) / 2 with t_N = 0 (X after the last death is 0);
// log w = beta logL + log dX (the tempered term is 0 at beta = 0).
//
// Nothing of size R x N is stored, and every shrinkage is drawn once: a chunk of deaths is worked
// relative to log X at its own first death, which enters the log weights and evidence terms as a
// summand afterwards.
//  k_geom_chunks   grid (chunk, replica group), a wave each: keeps its chunk's live counts and
//                  likelihood factors in registers, loops over the group's replicas, draws log t,
//                  and per replica stores the chunk's sum of log t and its (max, sum) of the
//                  evidence; per death the sums over the group's replicas that the mean needs
//  k_geom_offsets  one workgroup per replica: exclusive scan of the chunk sums (log X at each
//                  chunk's first death)
//  k_geom_mean     per death: mean of the log weights over the replicas; per-wave ESS partials
//  k_geom_final    one workgroup per replica combines its evidence partials; one more combines
//                  the ESS partials
#include "nss_internal.hpp"
#include "nss_rng.hpp"
#include "nss_wave.hpp"

#include <math.h>

namespace nss {

namespace {

constexpr uint32_t PUR_GEOM = 6;
constexpr int kGeomE = 8;                   // consecutive deaths per lane (even)
constexpr int kGeomC = 64 * kGeomE;         // deaths per chunk
constexpr int kGeomT = 256;                 // threads of the scan
constexpr int kGeomW = kGeomT / 64;
constexpr double kLn2 = 0.69314718055994530942;

struct GeomArgs {
    const double *dead;   // [n_dead] dead-point logL in death order
    const double *logL;   // [m] live logL, ascending through perm
    const int *perm;      // [m]; the final survivors are perm[k..m-1]
    long long n_dead, N;
    int m, k, R, nchunk, rpg;  // rpg: replicas per group in k_geom_chunks
    double beta;
    uint32_t key0, key1;
    double *csum;      // [R][nchunk] chunk sums of log t, scanned in place into offsets
    double2 *zpart;    // [R][nchunk] (max, sum) of the evidence terms, X relative to the chunk's
    double *accp;      // [groups][N] per-group sums of log w over replicas, likewise relative
    double *logw_mean; // [N]
    double4 *epart;    // [ceil(N / 64)] per-wave (max, sum, sum of squares) of mean weights
    double *logz;      // [R]
    double *ess;       // [1]
};

// (N < 2^31 deaths, checked by the caller, so death indices are 32-bit)
__device__ __forceinline__ double live_count(const GeomArgs &a, int g)
{
    return g < (int)a.n_dead ? (double)(a.m - (int)((unsigned)g % (unsigned)a.k))
                             : (double)((a.m - a.k) - (g - (int)a.n_dead));
}

__device__ __forceinline__ double death_logL(const GeomArgs &a, int g)
{
    return g < (int)a.n_dead ? a.dead[g] : a.logL[a.perm[a.k + (g - (int)a.n_dead)]];
}

// beta logL (the tempered term is 0 at beta = 0)
__device__ __forceinline__ double tempered(const GeomArgs &a, int g)
{
    return a.beta == 0.0 ? 0.0 : a.beta * death_logL(a, g);
}

// The constants of log_uniform and exp_shrink, held in scalar registers: as literals the compiler
// takes them to vector registers ahead of the loop, and spills.
struct GeomConst {
    double q[11], e[11];
};
__device__ __forceinline__ GeomConst geom_const()
{
    GeomConst c = {{2.0 / 3.0, 2.0 / 5.0, 2.0 / 7.0, 2.0 / 9.0, 2.0 / 11.0, 2.0 / 13.0, 2.0 / 15.0,
                    2.0 / 17.0, 2.0 / 19.0, 2.0 / 21.0, 2.0 / 23.0},
                   {1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0, 1.0 / 720.0, 1.0 / 5040.0, 1.0 / 40320.0,
                    1.0 / 362880.0, 1.0 / 3628800.0, 1.0 / 39916800.0, 1.0 / 479001600.0,
                    1.0 / 6227020800.0}};
#pragma unroll
    for (int i = 0; i < 11; ++i) asm volatile("" : "+s"(c.q[i]), "+s"(c.e[i]));
    return c;
}
constexpr double kLn2Hi = 0x1.62e42fee00000p-1, kLn2Lo = 0x1.a39ef35793c76p-33;   // 32 bits, the rest

// log(u) for a uniform u of the generator (normal, in (0, 1)), u = 2^k (1 + f) with 1 + f in
// [sqrt(1/2), sqrt(2)): log(1 + f) = 2 atanh(w) = 2 w + w Q(w^2) at w = f / (2 + f),
// Q(z) = 2 sum_{i>0} z^i / (2 i + 1) (z <= 0.0295: eleven terms leave 1e-19), and 2 w = f - w f, so
// that what is added to the exact f is at most a fifth of it.  k log 2 + f is carried with its
// rounding error.  A third of the general log's instructions.
__device__ __forceinline__ double log_uniform(double u, const GeomConst &C)
{
    double m = __builtin_amdgcn_frexp_mant(u);   // [1/2, 1)
    int k = __builtin_amdgcn_frexp_exp(u);
    const bool low = m < 0.70710678118654752440;
    m = low ? m + m : m;
    k = low ? k - 1 : k;
    const double kd = (double)k, f = m - 1.0, dd = 2.0 + f;
    double r = __builtin_amdgcn_rcp(dd);         // about 2^-23, then a cubic step
    const double e = fma(-dd, r, 1.0);
    r = fma(r * e, 1.0 + e, r);
    double w = f * r;
    w = fma(fma(-dd, w, f), r, w);
    const double z = w * w;
    double q = C.q[10];
#pragma unroll
    for (int i = 9; i >= 0; --i) q = fma(q, z, C.q[i]);
    const double K = kd * kLn2Hi, a = K + f;     // (exact product; |K| > |f| or K = 0)
    return a + fma(kd, kLn2Lo, fma(w, fma(q, z, -f), f - (a - K)));
}

// log(f) for f = 0 or in [1/2, 1)
__device__ __forceinline__ double log_product(double f, const GeomConst &C)
{
    return f > 0.0 ? log_uniform(f, C) : -INFINITY;
}

// exp(x) for x <= 0: x = k log 2 + r, |r| <= log(2) / 2, the Taylor polynomial of degree 13
// (truncation 4e-18); large -x gives 0 by the exponent.
__device__ __forceinline__ double exp_shrink(double x, const GeomConst &C)
{
    const double k = rint(x * 1.44269504088896340736);
    const double r = fma(-k, kLn2Lo, fma(-k, kLn2Hi, x));
    double p = C.e[10];
#pragma unroll
    for (int i = 9; i >= 0; --i) p = fma(p, r, C.e[i]);
    p = fma(p, r, 0.5);
    return ldexp(1.0 + fma(r * r, p, r), (int)k);
}

// Combined (max, sum exp(x - max)) of per-thread pairs over the wave; an empty pair is
// (-inf, 0).
__device__ __forceinline__ double2 wave_lse(double ref, double sum)
{
    const double M = wave_max(ref);
    double c = 0.0;
    if (ref > -INFINITY) c = sum * exp(ref - M);
    return make_double2(M, wave_sum_fast(c));
}

}  // namespace

__global__ __launch_bounds__(kGeomT) void k_geom_offsets(GeomArgs a)
{
    __shared__ double red[kGeomW];
    double *cs = a.csum + (size_t)blockIdx.x * a.nchunk;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    double carry = 0.0;
    for (int c0 = 0; c0 < a.nchunk; c0 += kGeomT) {
        const int c = c0 + (int)threadIdx.x;
        const double v = c < a.nchunk ? cs[c] : 0.0;
        double inc = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double u = __shfl_up(inc, o, 64);
            if (l >= o) inc += u;
        }
        double ex = __shfl_up(inc, 1, 64);
        if (l == 0) ex = 0.0;
        if (l == 63) red[w] = inc;
        __syncthreads();
        double pre = carry, all = carry;
#pragma unroll
        for (int i = 0; i < kGeomW; ++i) {
            if (i < w) pre += red[i];
            all += red[i];
        }
        if (c < a.nchunk) cs[c] = pre + ex;
        carry = all;
        __syncthreads();
    }
}

// Inclusive sum over the wave's lanes in order: shifts within the rows of 16, then the row totals
// passed on (lane 15 to the next row, lane 31 to the upper half).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    int2 p = __builtin_bit_cast(int2, v);
    p.x = __builtin_amdgcn_update_dpp(0, p.x, CTRL, ROWS, 0xF, false);
    p.y = __builtin_amdgcn_update_dpp(0, p.y, CTRL, ROWS, 0xF, false);
    return v + __builtin_bit_cast(double, p);
}
__device__ __forceinline__ double wave_scan(double v)
{
    v = dpp_add<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8: +0 from before the row
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);   // row_bcast:15
    return dpp_add<0x143, 0xC>(v);   // row_bcast:31
}

// Bound by the vector arithmetic of the generator, log and exp (one of each a shrinkage).  The
// log1p of the weights is taken of a product: sum_r log(1 - y_r) = log prod_r (1 - y_r), each factor
// as exact as log1p(-y_r) of the rounded y_r is, the product's exponent kept apart.  312,000 deaths,
// 100 replicas: 162 us (with a pass of its own for the chunk sums, workgroups of four waves, a
// barrier a replica and the general log, exp and log1p: 132 + 363 us).  Three waves on a SIMD with a
// few spilled values were faster than two with none (175 us).
__global__ __launch_bounds__(64, 3) void k_geom_chunks(GeomArgs a)
{
    const int c = blockIdx.x, grp = blockIdx.y, l = threadIdx.x;
    const int g0 = c * kGeomC + l * kGeomE;
    const bool more = (long long)(c + 1) * kGeomC < a.N;   // another chunk follows
    double rn[kGeomE], ew[kGeomE], sums[kGeomE], prod[kGeomE];
    int pexp[kGeomE];
    double tmax = -INFINITY, psum = 0.0;
#pragma unroll
    for (int q = 0; q < kGeomE; ++q) {
        const bool ok = g0 + q < a.N;   // (past the last death: shrinkages of exactly 1)
        rn[q] = ok ? 1.0 / live_count(a, g0 + q) : 0.0;
        ew[q] = ok ? tempered(a, g0 + q) : -INFINITY;
        tmax = fmax(tmax, ew[q]);
        sums[q] = 0.0;
        prod[q] = 1.0;
        pexp[q] = 0;
    }
    // likelihood factors relative to the lane's largest, taken once for all replicas
#pragma unroll
    for (int q = 0; q < kGeomE; ++q) ew[q] = ew[q] > -INFINITY ? exp(ew[q] - tmax) : 0.0;
    const double rn_next = more ? 1.0 / live_count(a, (c + 1) * kGeomC) : 0.0;
    const int r0 = grp * a.rpg, r1 = min(a.R, r0 + a.rpg);
    const GeomConst C = geom_const();
    int last = a.N - 1 - g0 < kGeomE ? (int)(a.N - 1 - g0) : kGeomE;   // the last death, as one of the lane's
    double t_next = 0.0;
    for (int r = r0; r < r1; ++r) {
        // the shrinkage of the next chunk's first death, for 64 replicas at a time
        if (((r - r0) & 63) == 0 && more) {
            double ua, ub;
            draw2(a.key0, a.key1, PUR_GEOM, (uint32_t)(r + l), (uint32_t)((c + 1) * (kGeomC / 2)), 0u, 0u,
                  ua, ub);
            t_next = exp_shrink(log_uniform(ua, C) * rn_next, C);
        }
        // two deaths at a time, in order; a death is finished once the next shrinkage is known:
        // dX = X_g (1 - t_g t_{g+1}) / 2
        double sum = 0.0, X = 1.0, z = 0.0, t_first = 0.0, t_prev = 0.0;
        asm volatile("" : "+v"(last));   // (compared again, not kept as masks)
        const auto finish = [&](int q, double t, double tnext) {
            const double om = q != last ? 1.0 - t * tnext : 1.0;   // X after the last death is 0
            const double f = prod[q] * om;
            prod[q] = __builtin_amdgcn_frexp_mant(f);
            pexp[q] += __builtin_amdgcn_frexp_exp(f);
            z += ew[q] * X * om;
            X *= t;
        };
#pragma unroll
        for (int q = 0; q < kGeomE; q += 2) {
            // (opaque copies: the generator's parts that replicas or pairs share are not kept in
            // registers)
            uint32_t k0 = a.key0, k1 = a.key1, pair = (uint32_t)g0 / 2 + q / 2;
            asm volatile("" : "+s"(k0), "+s"(k1), "+v"(pair));
            double ua, ub;
            draw2(k0, k1, PUR_GEOM, (uint32_t)r, pair, 0u, 0u, ua, ub);
            const double s0 = log_uniform(ua, C) * rn[q], s1 = log_uniform(ub, C) * rn[q + 1];
            const double t0 = exp_shrink(s0, C), t1 = exp_shrink(s1, C);
            sums[q] += s0;
            sums[q + 1] += s1;
            sum += s0 + s1;
            if (q == 0) t_first = t0;
            else finish(q - 1, t_prev, t0);
            finish(q, t0, t1);
            t_prev = t1;
            __builtin_amdgcn_sched_barrier(0);   // the pairs' temporaries don't add up
        }
        // shrinkage of the death after this lane's last one, and log X before its first
        double tn = __shfl_down(t_first, 1, 64);
        const double next = __shfl(t_next, (r - r0) & 63, 64);
        if (l == 63) tn = next;
        finish(kGeomE - 1, t_prev, tn);
        const double inc = wave_scan(sum);
        double P = __shfl_up(inc, 1, 64);
        if (l == 0) P = 0.0;
        psum += P;
        // evidence terms of this lane: exp(tmax + P) * z / 2
        const double ref = (z > 0.0) ? tmax + P - kLn2 : -INFINITY;
        const double2 pr = wave_lse(ref, z);
        if (l == 63) {
            a.csum[(size_t)r * a.nchunk + c] = inc;
            a.zpart[(size_t)r * a.nchunk + c] = pr;
        }
    }
    // sum over the group's replicas of log w = beta logL + log X_g + log(1 - y) - log 2
#pragma unroll
    for (int q = 0; q < kGeomE; ++q) {
        if (g0 + q < a.N)
            a.accp[(size_t)grp * a.N + g0 + q] =
                r1 > r0 ? (r1 - r0) * (tempered(a, g0 + q) - kLn2) + (psum + (log_product(prod[q], C) + pexp[q] * kLn2))
                        : 0.0;
        psum += sums[q];
    }
}

// (256 deaths of one chunk a workgroup)
__global__ __launch_bounds__(256) void k_geom_mean(GeomArgs a, int groups)
{
    __shared__ double red[4];
    static_assert(kGeomC % 256 == 0, "a workgroup's deaths are of one chunk");
    const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    // log X at the chunk's first death, over all replicas
    double off = 0.0;
    const int c = (int)(blockIdx.x / (kGeomC / 256));
    for (int r = threadIdx.x; r < a.R; r += 256) off += a.csum[(size_t)r * a.nchunk + c];
    off = wave_sum_fast(off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = off;
    __syncthreads();
    off = (red[0] + red[1]) + (red[2] + red[3]);
    double v = -INFINITY;
    if (g < a.N) {
        double s = 0.0;
        for (int i = 0; i < groups; ++i) s += a.accp[(size_t)i * a.N + g];
        v = (s + off) / a.R;
        a.logw_mean[g] = v;
    }
    const double M = wave_max(v);
    const double e = v > -INFINITY ? exp(v - M) : 0.0;
    const double s1 = wave_sum_fast(e), s2 = wave_sum_fast(e * e);
    if ((threadIdx.x & 63) == 0 && g < a.N) a.epart[g >> 6] = make_double4(M, s1, s2, 0.0);
}

__global__ __launch_bounds__(256) void k_geom_final(GeomArgs a)
{
    __shared__ double red[4];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < a.R) {
        const double2 *zp = a.zpart + (size_t)blockIdx.x * a.nchunk;
        const double *off = a.csum + (size_t)blockIdx.x * a.nchunk;
        const int n = a.nchunk;
        double M = -INFINITY;
        for (int i = tid; i < n; i += 256) M = fmax(M, zp[i].x + off[i]);
        M = wave_max(M);
        if ((tid & 63) == 0) red[tid >> 6] = M;
        __syncthreads();
        M = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        __syncthreads();
        double s = 0.0;
        if (M > -INFINITY)
            for (int i = tid; i < n; i += 256)
                if (zp[i].x > -INFINITY) s += zp[i].y * exp(zp[i].x + off[i] - M);
        s = wave_sum_fast(s);
        if ((tid & 63) == 0) red[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) {
            s = (red[0] + red[1]) + (red[2] + red[3]);
            a.logz[blockIdx.x] = (M > -INFINITY && s > 0.0) ? M + log(s) : -INFINITY;
        }
        return;
    }
    const long long n = (a.N + 63) >> 6;
    double M = -INFINITY;
    for (long long i = tid; i < n; i += 256) M = fmax(M, a.epart[i].x);
    M = wave_max(M);
    if ((tid & 63) == 0) red[tid >> 6] = M;
    __syncthreads();
    M = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    __syncthreads();
    double s1 = 0.0, s2 = 0.0;
    if (M > -INFINITY)
        for (long long i = tid; i < n; i += 256) {
            const double4 e = a.epart[i];
            if (e.x > -INFINITY) {
                const double f = exp(e.x - M);
                s1 += e.y * f;
                s2 += e.z * f * f;
            }
        }
    s1 = wave_sum_fast(s1);
    s2 = wave_sum_fast(s2);
    __shared__ double red2[4];
    if ((tid & 63) == 0) { red[tid >> 6] = s1; red2[tid >> 6] = s2; }
    __syncthreads();
    if (tid == 0) {
        s1 = (red[0] + red[1]) + (red[2] + red[3]);
        s2 = (red2[0] + red2[1]) + (red2[2] + red2[3]);
        *a.ess = s2 > 0.0 ? s1 * s1 / s2 : 0.0;
    }
}

// ------------------------------------------------------------------------------------------
// weighted posterior samples (resampling with the geometric-mean weights)
// ------------------------------------------------------------------------------------------
constexpr uint32_t PUR_POST = 7;

// Normalised cumulative weights cum[i] = sum_{l <= i} w_l / sum w, w = exp(logw_mean - max), in
// index order, over blocks of 8192 deaths (eight consecutive per thread).  The scratch ws holds
// [0] the maximum, [1] the total, [2, 2 + nb) the block maxima and then the blocks' exclusive
// offsets, [2 + nb, 2 + 2 nb) the block sums.
constexpr int kCumT = 1024, kCumPer = 8;
constexpr long long kCumChunk = (long long)kCumT * kCumPer;

long long post_cum_blocks(long long N) { return (N + kCumChunk - 1) / kCumChunk; }

__global__ __launch_bounds__(kCumT) void k_post_bmax(const double *lw, long long N, double *ws)
{
    __shared__ double red[16];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const long long base = (long long)blockIdx.x * kCumChunk;
    double mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < kCumPer; ++q) {
        const long long i = base + (long long)q * kCumT + tid;
        if (i < N) mx = fmax(mx, lw[i]);
    }
    mx = wave_max(mx);
    if (l == 0) red[w] = mx;
    __syncthreads();
    if (tid == 0) {
        double m = red[0];
        for (int i = 1; i < 16; ++i) m = fmax(m, red[i]);
        ws[2 + blockIdx.x] = m;
    }
}

// One workgroup: the maximum of the nb block maxima into ws[0].
__global__ __launch_bounds__(kCumT) void k_post_gmax(double *ws, int nb)
{
    __shared__ double red[16];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    double mx = -INFINITY;
    for (int b = tid; b < nb; b += kCumT) mx = fmax(mx, ws[2 + b]);
    mx = wave_max(mx);
    if (l == 0) red[w] = mx;
    __syncthreads();
    if (tid == 0) {
        double m = red[0];
        for (int i = 1; i < 16; ++i) m = fmax(m, red[i]);
        ws[0] = m;
    }
}

// exp(lw - M) over this workgroup's block: thread t takes deaths i0 .. i0 + 7 (i0 = base + 8 t),
// v[q] its running sums, pre the sum of the block's earlier deaths; returns the block's total.
// The block sums and the final pass both use this, so their totals agree bit for bit.
__device__ __forceinline__ double block_cum(const double *lw, long long N, double M, long long i0,
                                            double (&v)[kCumPer], double &pre, double *red)
{
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kCumPer; ++q) {
        const long long i = i0 + q;
        const double x = i < N ? lw[i] : -INFINITY;
        s += x > -INFINITY ? exp(x - M) : 0.0;
        v[q] = s;
    }
    double inc = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double t = __shfl_up(inc, o, 64);
        if (l >= o) inc += t;
    }
    if (l == 63) red[w] = inc;
    __syncthreads();
    double p = 0.0, all = 0.0;
    for (int q = 0; q < 16; ++q) {
        if (q < w) p += red[q];
        all += red[q];
    }
    pre = p + (inc - s);
    return all;
}

__global__ __launch_bounds__(kCumT) void k_post_bsum(const double *lw, long long N, double *ws,
                                                     int nb)
{
    __shared__ double red[16];
    const long long i0 = (long long)blockIdx.x * kCumChunk + (long long)threadIdx.x * kCumPer;
    double v[kCumPer], pre;
    const double all = block_cum(lw, N, ws[0], i0, v, pre, red);
    if (threadIdx.x == 0) ws[2 + nb + blockIdx.x] = all;
}

// One thread, in block order: the exclusive offsets (over the block maxima, no longer needed)
// and the total, so that each offset plus its block's sum is exactly the next offset.
__global__ void k_post_offsets(double *ws, int nb)
{
    if (threadIdx.x != 0) return;
    double acc = 0.0;
    for (int b = 0; b < nb; ++b) {
        const double sb = ws[2 + nb + b];
        ws[2 + b] = acc;
        acc += sb;
    }
    ws[1] = acc;
}

__global__ __launch_bounds__(kCumT) void k_post_cum(const double *lw, long long N,
                                                    const double *ws, double *cum)
{
    __shared__ double red[16];
    const long long i0 = (long long)blockIdx.x * kCumChunk + (long long)threadIdx.x * kCumPer;
    double v[kCumPer], pre;
    (void)block_cum(lw, N, ws[0], i0, v, pre, red);
    const double off = ws[2 + blockIdx.x] + pre, tot = ws[1];
#pragma unroll
    for (int q = 0; q < kCumPer; ++q)
        if (i0 + q < N) cum[i0 + q] = (off + v[q]) / tot;
}

// Sample j: the first death whose cumulative weight reaches (u + j) / n; its coordinates, kPickT
// lanes a sample so that rows are read and written whole (10000 samples of d = 64: 10 us, one lane a
// sample 30 us).
constexpr int kPickT = 16;
__global__ __launch_bounds__(256) void k_post_pick(const double *cum, long long N, long long n_dead,
                                                   const double *deadx, const double *X,
                                                   const int *perm, int k, int m_pad, int d,
                                                   int n, uint32_t key0, uint32_t key1,
                                                   double *xo, long long *io)
{
    const int j = blockIdx.x * (256 / kPickT) + threadIdx.x / kPickT, a0 = threadIdx.x % kPickT;
    if (j >= n) return;
    double u, unused;
    draw2(key0, key1, PUR_POST, 0u, 0u, 0u, 0u, u, unused);
    const double pos = (u + j) / n;
    long long lo = 0, hi = N - 1;
    while (lo < hi) {
        const long long mid = (lo + hi) >> 1;
        if (cum[mid] >= pos) hi = mid; else lo = mid + 1;
    }
    if (a0 == 0) io[j] = lo;
    for (int a = a0; a < d; a += kPickT)
        xo[(size_t)j * d + a] = lo < n_dead ? deadx[lo * d + a]
                                            : X[(size_t)a * m_pad + perm[k + (int)(lo - n_dead)]];
}

hipError_t launch_post_samples(const GeomLaunch &G, const double *deadx, const double *X,
                               int m_pad, int d, int n, double *cum, double *cws, double *xo,
                               long long *io, hipStream_t s)
{
    const long long nbl = post_cum_blocks(G.N);
    const int nb = (int)nbl;
    hipLaunchKernelGGL(k_post_bmax, dim3((unsigned)nb), dim3(kCumT), 0, s, G.logw_mean, G.N, cws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_post_gmax, dim3(1), dim3(kCumT), 0, s, cws, nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_post_bsum, dim3((unsigned)nb), dim3(kCumT), 0, s, G.logw_mean, G.N, cws,
                       nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_post_offsets, dim3(1), dim3(64), 0, s, cws, nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_post_cum, dim3((unsigned)nb), dim3(kCumT), 0, s, G.logw_mean, G.N, cws,
                       cum);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    constexpr int per = 256 / kPickT;
    hipLaunchKernelGGL(k_post_pick, dim3((unsigned)(((long long)n + per - 1) / per)), dim3(256), 0, s, cum, G.N,
                       G.n_dead, deadx, X, G.perm, G.k, m_pad, d, n, G.key0, G.key1, xo, io);
    return hipGetLastError();
}

// Callers compare this with fixed workspaces: it is counted in blocks of 1024 deaths (8 bytes and
// four 16-byte pairs a replica), which the chunks' sums and pairs do not use up.
size_t geom_workspace_bytes(long long N, int R, int groups)
{
    const long long nblk = (N + 1023) / 1024;
    size_t b = 0;
    auto add = [&](size_t n) { b += (n + 255) / 256 * 256; };
    add((size_t)R * nblk * 8);
    add((size_t)R * nblk * 64);
    add((size_t)groups * N * 8);                 // accp
    add((size_t)((N + 63) / 64) * 32);           // epart
    return b;
}

int geom_groups(long long N, int R)
{
    // enough workgroups to fill the chip several times over, at least 8 replicas per group
    const long long nblk = (N + 1023) / 1024;
    long long g = (2048 + nblk - 1) / nblk;
    if (g > (R + 7) / 8) g = (R + 7) / 8;
    return (int)(g < 1 ? 1 : g);
}

hipError_t launch_geom(const GeomLaunch &G, hipStream_t s)
{
    const long long nchunk = (G.N + kGeomC - 1) / kGeomC;
    const int groups = G.groups;
    GeomArgs a{};
    a.dead = G.dead; a.logL = G.logL; a.perm = G.perm;
    a.n_dead = G.n_dead; a.N = G.N; a.m = G.m; a.k = G.k; a.R = G.R; a.nchunk = (int)nchunk;
    a.rpg = (G.R + groups - 1) / groups;
    a.beta = G.beta; a.key0 = G.key0; a.key1 = G.key1;
    char *p = (char *)G.ws;
    auto take = [&](size_t n) { char *q = p; p += (n + 255) / 256 * 256; return (void *)q; };
    a.csum = (double *)take((size_t)G.R * nchunk * 8);
    a.zpart = (double2 *)take((size_t)G.R * nchunk * 16);
    a.accp = (double *)take((size_t)groups * G.N * 8);
    a.epart = (double4 *)take((size_t)((G.N + 63) / 64) * 32);
    a.logz = G.logz;
    a.logw_mean = G.logw_mean;
    a.ess = G.ess;
    hipLaunchKernelGGL(k_geom_chunks, dim3((unsigned)nchunk, groups), dim3(64), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_geom_offsets, dim3(G.R), dim3(kGeomT), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_geom_mean, dim3((unsigned)((G.N + 255) / 256)), dim3(256), 0, s, a,
                       groups);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_geom_final, dim3(G.R + 1), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace nss
