// gfx950 HRSS chains evaluated along each step's line: likelihoods of quadratic forms (Gaussian
// mixtures), and those summed over a candidate's coordinates (Neal's funnel, Gaussian-Rastrigin).
//
// A step's candidates all lie on x + t v, and a form |W (x + t v - mu)|^2 is on that line the
// parabola a + 2 b t + g t^2 with a = |W (x - mu)|^2, b = W (x - mu) . W v, g = |W v|^2.  The
// directions of an iteration do not depend on the chains' outcomes, so a chain takes fifteen
// steps at a time: with u_n = W v_n for the block's directions and u_15 = W (x - mu) at the
// block's start, the Gram matrix G = u^T u holds every scalar the fifteen steps need.  After a
// move by t along v_s the row of u_15 becomes G[15][n] + t G[s][n]; no vector is touched.  All
// arithmetic is FP64, so the kernel serves every precision of the interface: its decisions are
// the FP64 ones.  Each block starts from its own point, so rounding does not build up over a
// chain, and the chain's final point is evaluated by the batched FP64 tile for the stored logL.
//
// One wave runs one chain (up to four per workgroup) with no barrier until the end.  A block's
// products run on v_mfma_f64_16x16x4: W as the A operand, the sixteen columns as B; the result
// of that product is already laid out as both operands of G = u^T u (lane l, register i of
// column block jb holds element [16 jb + 4 i + (l >> 4)][l & 15], which is k-step 4 jb + i of
// an A or a B operand), so no data moves between the two products.
//
// While walking, lane l stands for column l & 15 and forms (l >> 4) + 4 q: sixteen candidates
// are tested at a time, each form of a candidate in its own lane, and the lanes' votes are
// folded to a bit per candidate.  A mixture is above L* when any component alone is, and is not
// when every one is below L* - log K; only between the two is the sum of exponentials taken.
//
// The walk is a chain of dependent scalar-sized operations, so its length is what a step costs.
// The first pass of a step tests both ends twice and four shrink proposals of each of the three
// likeliest outcomes (neither end, or one of them once, expands); their t do not depend on the
// point, so a block's are laid out at its start, and nine steps of ten end with that pass.  The
// row of u_15 is kept shifted so that the current step's column is column 0 (row shifts and row
// broadcasts instead of trips through LDS), and whole-wave values move by lane reads.
//
// The Gaussian-Rastrigin likelihood has no parabola: a candidate's four lanes sum |y|^2 and
// cos(2 pi y) over a quarter of the coordinates each, y = x + t v from LDS, with no barrier and no
// reduction over the wave.  cos(2 pi y) is sin(2 pi s), s = 1/4 - |y - rint(y)|, by its Taylor
// polynomial of degree 21 (truncation 1.3e-18 on |s| <= 1/4).  At d = 100, 500 chains of 2500
// steps: 25.4 ms a launch with points and 7.4 here; a pass takes 3,000 cycles of FP64 arithmetic,
// eight polynomials side by side for their latency (two: 8.6 ms).
//
// The funnel's radius is a parabola too, but exp(-v) weighs it by up to e^20 in the neck, where it
// is far smaller than at a point in the mouth, and a parabola's rounding is relative to the larger
// one (1e-6 of log L at v = -18).  A candidate whose log L lies within 1e-13 of the terms so weighed
// (their rounding over a block is below 1e-14) of L* has its radius summed from its coordinates, in
// the way of the Rastrigin sums; the tempered slices, which go on from the value itself, and the
// random walk, whose products such sums cost no more than, always.
//
// The random walk's proposals x + u_n are the same products at t = 1: a block's fifteen are tested
// at once from the current point, and again after each acceptance, their moves in registers for
// the box (d = 50, 500 chains of 250 steps: 364 us a launch with points, 122 here; 175 with the
// block's proposals copied and tested against the box one by one).
//
// What it replaces evaluated every candidate as a point, in a tile shared by a workgroup's
// chains, at two barriers and two to three tiles a step.  One launch with points and here:
// d = 5, 50 chains of 25 steps 241 and 33 us; d = 32, 500 chains of 160 steps (BF16x3 points)
// 1561 and 178 us; 8 components at d = 64, 1000 chains of 320 steps in FP64 7800 and 855 us.
// (Without the planned first pass, the shifted row and the fragments requested ahead: 56, 301
// and 1900 us.)  One wave per SIMD runs at those sizes, so the bound is the walk's length, about
// 2,500 cycles a step; at 8 components the products take as long again, twice what the FP64
// matrix rate allows (W's fragments come from L2 for every wave; more sums side by side on the
// matrix unit changed nothing).
#include "nss_internal.hpp"
#include "nss_rng.hpp"
#include "nss_tiles.hpp"
#include "nss_wave.hpp"

#include <math.h>
#include <type_traits>

namespace nss {

constexpr int kLineB = 15;              // steps per block (the sixteenth column is the point)
constexpr int kLineLd = 17;             // row stride of a Gram matrix in LDS
constexpr int kLineSide = 8;            // stepping-out tests per end and pass
constexpr int kLineForms = 16;          // most components

// LDS of one workgroup (byte offsets; identical on host): per chain the forms' Gram matrices
// (the last one the Gaussian prior's), the point, the block's step uniforms, its first passes'
// t, and the shrink uniforms of a later pass; the final points' FP64 tile overlays the Gram
// matrices.
struct LineLayout {
    int gram, x, v, us, tt, su, chain;  // per-chain offsets and stride (v: the direction where
                                        // candidates are points, the walk's block of proposals)
    int mu, pa, ipb;                    // the workgroup's means and Gaussian prior (1 / std)
    int cand, q, L, mask, total;
};
__host__ __device__ inline LineLayout line_layout(int D, int K, int lik, bool box, bool rw)
{
    const int forms = (lik == LIK_MIXTURE ? K : lik == LIK_FUNNEL && !rw ? 1 : 0) + (box ? 0 : 1);
    LineLayout o;
    int off = 0;
    o.gram = off; off += al16(forms * 16 * kLineLd * 8);
    o.x = off; off += al16(D * 8);
    o.v = off; off += rw ? al16(kLineB * (D + 1) * 8) : lik != LIK_MIXTURE ? al16(D * 8) : 0;
    o.us = off; off += 16 * kStepU * 8;
    o.tt = off; off += 16 * 16 * 8;
    o.su = off; off += 16 * 8;
    o.chain = al16(off);
    int t = 0;
    o.cand = t; t += al16(kRows * (D + 1) * 8);
    o.q = t; t += al16(kRows * q_stride(D, K) * 8);
    o.L = t; t += al16(kRows * 8);
    o.mask = t; t += al16(kRows * 4);
    off = kMaxChainsPerWG * o.chain;
    o.mu = off; off += lik == LIK_MIXTURE ? K * D * 8 : 0;
    o.pa = off; off += D * 8;
    o.ipb = off; off += D * 8;
    o.total = off > t ? off : t;
    return o;
}
size_t line_lds_bytes(int D, int K, int lik, int box, int rw)
{
    return (size_t)line_layout(D, K, lik, box != 0, rw != 0).total;
}

// Bits of a ballot folded over the four rows: bit c = some lane of column c voted.
__device__ __forceinline__ unsigned fold_rows(unsigned long long b)
{
    const unsigned h = (unsigned)b | (unsigned)(b >> 32);
    return (h | (h >> 16)) & 0xFFFFu;
}
// Minimum over the wave of floats that are not negative (ordered as their bits are; a negative
// one counts as large): DPP within a row, then the last lanes of rows 0 and 2 into the rows after
// them and lane 31 into the upper half; lane 63 has the result.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_min(unsigned v)
{
    return min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float wave_min_pos(float x)
{
    unsigned v = __builtin_bit_cast(unsigned, x);
    v = dpp_min<DPP_XOR1, 0xF>(v);
    v = dpp_min<DPP_XOR2, 0xF>(v);
    v = dpp_min<DPP_HMIR, 0xF>(v);
    v = dpp_min<DPP_RMIR, 0xF>(v);
    v = dpp_min<0x142, 0xA>(v);   // row_bcast:15
    v = dpp_min<0x143, 0xC>(v);   // row_bcast:31
    float m = __builtin_bit_cast(float, __builtin_amdgcn_readlane((int)v, 63));
    asm volatile("" : "+v"(m));
    return m;
}
#define DPP_BCAST0 0x150   /* row_newbcast:0, the row's first lane to all of it */
#define DPP_ROL1 0x12F     /* row_ror:15, lane i takes lane i + 1 of its row */
// The value of one lane (the same index in every lane), in vector registers: a compare of a
// value known to be uniform has been compiled into a scalar select on a stale condition code,
// so the value is made opaque.
__device__ __forceinline__ double lane_value(double v, int lane)
{
    double r = readlane_d(v, uniform_i(lane));
    asm volatile("" : "+v"(r));
    return r;
}

// sum of cos(2 pi y[i]) (see above; y - rint(y) and, from 1/8 up, 1/4 minus it are exact): the
// polynomials of U values side by side, for the length of their chains
template <int U>
__device__ __forceinline__ double cos_2pi(const double (&y)[U])
{
    constexpr double kC[11] = {0.0011309237482517963, -0.012031585942120627, 0.10422916220813984,
                                -0.7181223017785006, 3.819952584848282, -15.09464257682299,
                                42.058693944897655, -76.70585975306139, 81.60524927607506,
                                -41.34170224039976, 6.283185307179586};
    double s[U], z[U], p[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        s[i] = 0.25 - fabs(y[i] - rint(y[i]));
        z[i] = s[i] * s[i];
        p[i] = kC[0];
    }
#pragma unroll
    for (int k = 1; k < 11; ++k)
#pragma unroll
        for (int i = 0; i < U; ++i) p[i] = fma(p[i], z[i], kC[k]);
    double c = 0.0;
#pragma unroll
    for (int i = 0; i < U; ++i) c = fma(p[i], s[i], c);
    return c;
}

// The chains' kernels: slices under L > L*, tempered slices (no constraint), the random walk.
enum { LINE_SLICE = 0, LINE_TEMPERED = 1, LINE_WALK = 2 };

// NR: forms per lane (components 4 q + row, q < NR); KIND: as above;
// BOX: the prior is a box.
template <int D, int LIK, int NR, int KIND, bool BOX, int OCC>
__global__ __launch_bounds__(256, OCC) void k_hrss_line(Launch Lc, int fp64)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    if (R.iscal[0] || R.iscal[2] <= 0) return;
    constexpr int NA = (D + 63) / 64;
    constexpr int NJB = D / 16, NKS = D / 4, LDV = D + 1;   // LDV: row stride of the walk's proposals
    constexpr bool MIX = LIK == LIK_MIXTURE, RG = LIK == LIK_RG;
    constexpr bool TEMP = KIND == LINE_TEMPERED, RW = KIND == LINE_WALK;
    constexpr bool FORM = MIX || (LIK == LIK_FUNNEL && KIND == LINE_SLICE);   // parabolas
    const LineLayout lay = line_layout(D, P.K, LIK, BOX, RW);
    const int tid = threadIdx.x, w = uniform_i(tid >> 6), l = tid & 63;
    const int col = l & 15, row = l >> 4;
    const int d = P.d, K = MIX ? P.K : FORM ? 1 : 0, C = R.C, p = R.p;
    const double Lstar = R.scal[0], beta = Lstar;   // tempered: the inverse temperature
    const int t0 = R.iscal[1], nsurv = R.iscal[2];
    const uint32_t it = (uint32_t)R.iscal[3] + 1u;
    const double width = R.width;
    const int cap_out = R.stepout_cap, cap_sh = R.shrink_cap;

    unsigned char *mine = smem + w * lay.chain;
    double *gram = (double *)(mine + lay.gram);
    double *xs = (double *)(mine + lay.x);
    double *vs = (double *)(mine + lay.v);
    double *us = (double *)(mine + lay.us);
    double *tt = (double *)(mine + lay.tt);
    double *su = (double *)(mine + lay.su);
    double *gpri = gram + K * 16 * kLineLd;   // the Gaussian prior's form

    double *smu = (double *)(smem + lay.mu), *spa = (double *)(smem + lay.pa),
           *sipb = (double *)(smem + lay.ipb);
    if constexpr (MIX)
        for (int i = tid; i < K * D; i += 256) smu[i] = as_global(P.mu)[i];
    if constexpr (!BOX)
        for (int i = tid; i < D; i += 256) {
            spa[i] = as_global(P.pa)[i];
            sipb[i] = 1.0 / as_global(P.pb)[i];
        }

    const int j = bm.y * C + w;
    const bool has_chain = w < C && j < R.k;
    double x0r[NA], vr[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) { x0r[i] = 0.0; vr[i] = 0.0; }
    double logL0 = -INFINITY;
    bool moved = false;
    int parent = j;   // tempered SMC: the resampled particle j, gathered into slot j
    unsigned long long c_evals = 0, c_tests = 0, c_outcap = 0, c_shcap = 0, c_viol = 0;

    __syncthreads();
    if (has_chain) {
        if constexpr (!TEMP) {
            double u, unused;
            draw2(R.key0, R.key1, PUR_RESAMPLE, (uint32_t)j, it, 0u, 0u, u, unused);
            int qi = (int)floor(u * (double)nsurv);
            if (qi > nsurv - 1) qi = nsurv - 1;
            parent = R.perm[t0 + qi];
            if (l == 0) R.parents[j] = parent;
        }
        // the prior's box of the lane's coordinates, and a distance to its faces that rounding
        // of y = x + t v is small against
        double par[NA], pbr[NA], near_[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int a = l + 64 * i;
            par[i] = -INFINITY; pbr[i] = INFINITY; near_[i] = -1.0;
            if (a < d) {
                x0r[i] = R.X[(size_t)a * R.m_pad + parent];
                if (BOX) {
                    par[i] = P.pa[a];
                    pbr[i] = P.pb[a];
                    near_[i] = 1e-9 * fmax(fabs(par[i]), fabs(pbr[i]));
                }
            }
        }
        logL0 = R.logL[parent];
        double cst[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int c = 4 * q + row;
            cst[q] = MIX ? (c < K ? P.cst[c] : -INFINITY) : 0.0;
        }
        // below this a component cannot make the mixture exceed L* together with the others
        const double Lamb = MIX && K > 1 ? Lstar - log((double)K) - 1e-6
                            : RG         ? Lstar - log(2.0) - 1e-6
                                         : INFINITY;
        const auto dirs = as_global((const double *)R.dirbuf) + (size_t)j * p * D;
        const auto ub = as_global((const double *)R.ubuf) + (size_t)j * p * kStepU;
        const bool xcol = col == 15;
        // the first pass needs room for two expansions of an end and four proposals
        const bool fast = cap_out >= 2 && cap_sh >= 4;

        // the step's direction (lane l: coordinates l, l + 64, ...), one step ahead, and the next
        // block's columns (lane: column col, coordinates 4 ks + row) and uniforms, loaded while
        // the current block is walked
        double pv[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) pv[i] = (l + 64 * i < D) ? dirs[l + 64 * i] : 0.0;
        double b[MIX ? NKS : 1], pus[2];
        auto fetch_block = [&](int s0) {
            const int nb = min(kLineB, p - s0);
            const bool dcol = col < nb;
            const auto vrow = dirs + (size_t)(s0 + (dcol ? col : 0)) * D + row;
            if constexpr (MIX) {
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) b[ks] = dcol ? vrow[4 * ks] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
                pus[i] = l + 64 * i < nb * kStepU ? ub[(size_t)s0 * kStepU + l + 64 * i] : 0.5;
        };
        fetch_block(0);
        // W column blocks in pairs (pr, NJB - 1 - pr) of equal triangular work, taken in
        // chunks of at most 20 fragments, the next chunk's requested before this one's
        // products (a trip to L2 costs about what the products of a chunk take), and the next
        // block's first before the walk
        constexpr int NPR = NJB / 2, NF = 4 * (NJB + 1), NCH = NF > 20 ? 2 : 1;
        constexpr int CH = NF / NCH, NSEQ = NPR * NCH;   // chunks per component
        double wa[CH], wb[CH];
        // fragment f of pair pr: column block j0 or j1 in turn while both have k-steps
        auto frag = [](int pr, int f, int &jb, int &ks, bool &lo) {
            const int n0 = 4 * (pr + 1);
            lo = f < 2 * n0 && !(f & 1);
            jb = lo ? pr : NJB - 1 - pr;
            ks = f < 2 * n0 ? f >> 1 : f - n0;
        };
        auto load = [&](double *wf, int c, int sq) {
            const auto src = as_global(P.wf64) +
                             (size_t)(c < K ? c : K - 1) * NJB * NKS * 64 + l;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                int jb, ks;
                bool lo;
                frag(sq / NCH, (sq % NCH) * CH + i, jb, ks, lo);
                wf[i] = src[(jb * NKS + ks) * 64];
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        // (not where the walk's own values leave no registers for it)
        constexpr bool AHEAD = MIX && (RW ? D < 128 : NR == 1 || (NR == 2 && !TEMP));
        if constexpr (AHEAD) load(wa, 0, 0);

        for (int s0 = 0; s0 < p; s0 += kLineB) {
            const int nb = min(kLineB, p - s0);
            // ---- the block's products ----
#pragma unroll
            for (int i = 0; i < NA; ++i) if (l + 64 * i < D) xs[l + 64 * i] = x0r[i];
            us[l] = pus[0];
            us[l + 64] = pus[1];
            if constexpr (RW && MIX) {
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
                    if (col < kLineB) vs[col * LDV + 4 * ks + row] = b[ks];
            } else if constexpr (RW) {
#pragma unroll
                for (int c = 0; c < kLineB; ++c)
#pragma unroll
                    for (int i = 0; i < NA; ++i)
                        if (l + 64 * i < D)
                            vs[c * LDV + l + 64 * i] = dirs[(size_t)(s0 + min(c, nb - 1)) * D + l + 64 * i];
            }
            wave_sync();
            if constexpr (MIX && !AHEAD) load(wa, 0, 0);
            if constexpr (!RW) {
                // t of the first passes: columns 0, 1 the left end's next tests, 2, 3 the right
                // end's, then four proposals after no expansion, one left, one right (four steps at
                // a time, one per row)
                for (int s4 = 0; s4 < nb; s4 += 4) {
                    const double *uq = us + (s4 + row) * kStepU;
                    const double tl = uq[0], tr = tl + width;
                    const int hyp = (col >> 2) - 1;
                    double sL = hyp == 1 ? tl - width : tl, sR = hyp == 2 ? tr + width : tr;
                    double t = col == 0 ? tl : (col == 1 ? tl - width : (col == 2 ? tr : tr + width));
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const double tq = fma(uq[2 + q], sR - sL, sL);
                        if (col >= 4 && (col & 3) == q) t = tq;
                        if (tq < 0.0) sL = tq; else sR = tq;
                    }
                    tt[(s4 + row) * 16 + col] = t;
                }
            }
            double luh = 0.0;
            if (TEMP || !BOX) luh = log(us[col * kStepU + 1]);
            typedef double d4v __attribute__((ext_vector_type(4)));
            auto put = [&](double *g, const d4v &G) {
#pragma unroll
                for (int i = 0; i < 4; ++i) g[(row + 4 * i) * kLineLd + col] = G[i];
            };
            if constexpr (MIX) {
                d4v G, a0, a1;
                auto mul = [&](const double *wf, int sq) {
                    if (sq % NCH == 0) a0 = a1 = (d4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int i = 0; i < CH; ++i) {
                        int jb, ks;
                        bool lo;
                        frag(sq / NCH, (sq % NCH) * CH + i, jb, ks, lo);
                        if (lo) a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(wf[i], b[ks], a0, 0, 0, 0);
                        else a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(wf[i], b[ks], a1, 0, 0, 0);
                    }
                    if (sq % NCH == NCH - 1) {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            G = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[i], a0[i], G, 0, 0, 0);
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            G = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[i], a1[i], G, 0, 0, 0);
                    }
                };
                auto begin = [&](int c) {   // the point's column, less the component's mean
                    G = (d4v){0.0, 0.0, 0.0, 0.0};
                    const double *mu = smu + c * D + row;
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks)
                        if (xcol) b[ks] = xs[4 * ks + row] - mu[4 * ks];
                };
                if constexpr (NSEQ == 1) {
                    for (int c = 0; c < K; c += 2) {
                        load(wb, c + 1, 0);
                        begin(c);
                        mul(wa, 0);
                        put(gram + c * 16 * kLineLd, G);
                        if (c + 1 < K) {
                            load(wa, c + 2 < K ? c + 2 : 0, 0);
                            begin(c + 1);
                            mul(wb, 0);
                            put(gram + (c + 1) * 16 * kLineLd, G);
                        } else if (AHEAD && c > 0) {
                            load(wa, 0, 0);
                        }
                    }
                } else {
                    for (int c = 0; c < K; ++c) {
                        begin(c);
#pragma unroll
                        for (int sq = 0; sq < NSEQ; sq += 2) {
                            load(wb, c, sq + 1);
                            mul(wa, sq);
                            load(wa, sq + 2 < NSEQ ? c : (c + 1 < K ? c + 1 : 0), sq + 2 < NSEQ ? sq + 2 : 0);
                            mul(wb, sq + 1);
                        }
                        put(gram + c * 16 * kLineLd, G);
                    }
                }
                if (!BOX) {
                    d4v Gp = (d4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) {
                        const int kk = 4 * ks + row;
                        const double bb = kk < d ? (xcol ? xs[kk] - spa[kk] : b[ks]) * sipb[kk] : 0.0;
                        Gp = __builtin_amdgcn_mfma_f64_16x16x4f64(bb, bb, Gp, 0, 0, 0);
                    }
                    put(gpri, Gp);
                }
            } else if (FORM || !BOX) {
                // the funnel's form: the coordinates after the first (and the Gaussian prior's)
                const bool dcol = col < nb;
                const auto vrow = dirs + (size_t)(s0 + (dcol ? col : 0)) * D;
                d4v G = (d4v){0.0, 0.0, 0.0, 0.0}, Gp = (d4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll 16
                for (int ks = 0; ks < NKS; ++ks) {
                    const int kk = 4 * ks + row;
                    const double bv = dcol ? vrow[kk] : (xcol ? xs[kk] : 0.0);
                    const double bb = kk > 0 ? bv : 0.0;
                    if (FORM) G = __builtin_amdgcn_mfma_f64_16x16x4f64(bb, bb, G, 0, 0, 0);
                    if (!BOX) {
                        const double bp = kk < d ? (xcol ? bv - spa[kk] : bv) * sipb[kk] : 0.0;
                        Gp = __builtin_amdgcn_mfma_f64_16x16x4f64(bp, bp, Gp, 0, 0, 0);
                    }
                }
                if (FORM) put(gram, G);
                if (!BOX) put(gpri, Gp);
            }
            wave_sync();
            // the point's products with the directions (row 15; column 0 is the current step's),
            // and its own square
            double h[NR], aa[NR], hp = 0.0;
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                const int c = 4 * q + row;
                const double *g15 = gram + ((c < K ? c : 0) * 16 + 15) * kLineLd;
                h[q] = FORM ? g15[col] : 0.0;
                aa[q] = FORM ? g15[15] : 0.0;
            }
            if (!BOX) hp = gpri[15 * kLineLd + col];
            if (s0 + kLineB < p) fetch_block(s0 + kLineB);
            unsigned n_tests = 0, n_evals = 0;

            if constexpr (RW) {
                // ---- the block's proposals ----
                // x + v_c for every proposal c at once (t = 1), from the current point: up to the
                // first acceptance they are the tests the walk makes; then the point's products
                // move by that proposal's row and the later proposals are tested again
                double dg[NR], dgp = 0.0, v0c = 0.0;
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    const int c = 4 * q + row < K ? 4 * q + row : 0;
                    dg[q] = MIX ? gram[(c * 16 + col) * kLineLd + col] : 0.0;
                }
                if (!BOX) dgp = gpri[col * kLineLd + col];
                if constexpr (!MIX) v0c = vs[min(col, kLineB - 1) * LDV];
                // the proposals' moves of the lane's coordinates (a padded coordinate's is 0 and
                // its box open) and the longest
                double vb[BOX ? kLineB : 1][NA], big[NA];
                if constexpr (BOX) {
#pragma unroll
                    for (int i = 0; i < NA; ++i) {
                        big[i] = 0.0;
#pragma unroll
                        for (int c = 0; c < kLineB; ++c) {
                            vb[c][i] = l + 64 * i < D && c < nb ? vs[c * LDV + l + 64 * i] : 0.0;
                            big[i] = fmax(big[i], fabs(vb[c][i]));
                        }
                    }
                }
                for (int at = 0; at < nb;) {
                    const unsigned todo = ((1u << nb) - 1u) & ~((1u << at) - 1u);
                    unsigned okm = todo, in;
                    if constexpr (BOX) {
                        // (rounding is monotone: where the longest move stays inside, all do)
                        bool all = true;
#pragma unroll
                        for (int i = 0; i < NA; ++i)
                            all = all && x0r[i] + big[i] <= pbr[i] && x0r[i] - big[i] >= par[i];
                        if (!__all(all)) {
                            unsigned ok = 0;
#pragma unroll
                            for (int c = 0; c < kLineB; ++c) {
                                bool ib = true;
#pragma unroll
                                for (int i = 0; i < NA; ++i) {
                                    const double y = x0r[i] + vb[c][i];
                                    ib = ib && y >= par[i] && y <= pbr[i];
                                }
                                ok |= (__all(ib) ? 1u : 0u) << c;
                            }
                            okm = todo & ok;
                        }
                    } else {
                        okm &= (unsigned)__ballot(-0.5 * fma(2.0, hp, dgp) > luh);
                    }
                    if constexpr (MIX) {
                        double lc[NR];
                        bool hit = false, amb = false;
#pragma unroll
                        for (int q = 0; q < NR; ++q) {
                            lc[q] = cst[q] - 0.5 * (aa[q] + fma(2.0, h[q], dg[q]));
                            hit = hit || lc[q] > Lstar;
                            amb = amb || lc[q] > Lamb;
                        }
                        in = fold_rows(__ballot(hit));
                        const unsigned doubt = fold_rows(__ballot(amb)) & ~in & okm;
                        if (doubt) {
                            double se = 0.0;
#pragma unroll
                            for (int q = 0; q < NR; ++q) se += exp(lc[q] - Lstar);
                            se += __shfl_xor(se, 16, 64);
                            se += __shfl_xor(se, 32, 64);
                            in |= (unsigned)__ballot(se > 1.0) & doubt;
                        }
                    } else {
                        double s2 = 0.0;
                        const double *vc = vs + min(col, kLineB - 1) * LDV;
                        for (int a = row ? row : 4; a < d; a += 4) {
                            const double y = xs[a] + vc[a];
                            s2 = fma(y, y, s2);
                        }
                        s2 += __shfl_xor(s2, 16, 64);
                        s2 += __shfl_xor(s2, 32, 64);
                        const double vv = lane_value(x0r[0], 0) + v0c;
                        const double Lc = -vv * vv / 18.0 - 0.5 * (LOG_2PI + log(9.0)) -
                                          0.5 * exp(-vv) * s2 -
                                          (double)(d - 1) * 0.5 * (vv + LOG_2PI);
                        in = (unsigned)__ballot(Lc > Lstar);
                    }
                    const unsigned ac = in & okm;
                    const int s = ac ? __builtin_ctz(ac) : nb - 1;
                    const unsigned cons = todo & ((2u << s) - 1u);
                    n_tests += __builtin_popcount(cons);
                    n_evals += __builtin_popcount(cons & okm);
                    if (R.trace && l < 16 && ((cons >> l) & 1u)) {
                        int *tr = R.trace + ((size_t)j * p + s0 + l) * 4;
                        tr[0] = 0; tr[1] = 0; tr[2] = (okm >> l) & 1u; tr[3] = ac && l == s;
                    }
                    if (ac) {
                        moved = true;
#pragma unroll
                        for (int i = 0; i < NA; ++i)
                            if (l + 64 * i < D) x0r[i] += vs[s * LDV + l + 64 * i];
                        if constexpr (MIX) {
#pragma unroll
                            for (int q = 0; q < NR; ++q) {
                                const int c = 4 * q + row < K ? 4 * q + row : 0;
                                const double hs = __shfl(h[q], (l & 48) | s, 64);
                                aa[q] += fma(2.0, hs, __shfl(dg[q], (l & 48) | s, 64));
                                h[q] += gram[(c * 16 + s) * kLineLd + col];
                            }
                        } else {
                            wave_sync();
#pragma unroll
                            for (int i = 0; i < NA; ++i) if (l + 64 * i < D) xs[l + 64 * i] = x0r[i];
                            wave_sync();
                        }
                        if (!BOX) hp += gpri[s * kLineLd + col];
                    }
                    at = s + 1;
                }
                c_tests += n_tests;
                c_evals += n_evals;
                wave_sync();   // the block's LDS is rewritten
                continue;
            }

            // ---- the block's steps ----
            float size = (float)aa[0];   // what the form's rounding is relative to (funnel)
            double tn = tt[col], grn[NR], gpn = 0.0;   // the next step's, read ahead
#pragma unroll
            for (int q = 0; q < NR; ++q)
                grn[q] = FORM ? gram[((4 * q + row < K ? 4 * q + row : 0) * 16) * kLineLd + col] : 0.0;
            if (!BOX) gpn = gpri[col];
            for (int sb = 0; sb < nb; ++sb) {
                const int st = s0 + sb;
#pragma unroll
                for (int i = 0; i < NA; ++i) vr[i] = pv[i];
                if (st + 1 < p) {
                    const auto nx = dirs + (size_t)(st + 1) * D;
#pragma unroll
                    for (int i = 0; i < NA; ++i) if (l + 64 * i < D) pv[i] = nx[l + 64 * i];
                }
                // the step's parabolas a + b2 t + g t^2 and the row of the update
                double b2[NR], g[NR], gr[NR];
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    gr[q] = grn[q];
                    g[q] = dppd<DPP_BCAST0>(gr[q]);
                    b2[q] = 2.0 * dppd<DPP_BCAST0>(h[q]);
                }
                double bp2 = 0.0, gp = 0.0, grp = 0.0, lu = 0.0;
                if (!BOX) {
                    grp = gpn;
                    gp = dppd<DPP_BCAST0>(grp);
                    bp2 = 2.0 * dppd<DPP_BCAST0>(hp);
                }
                if (TEMP || !BOX) lu = lane_value(luh, sb);
                const double tf = tn;
                {
                    // (step 15 of a full block reads row 15, unused)
                    const int sn = sb + 1;
                    tn = tt[sn * 16 + col];
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                        const int c = 4 * q + row < K ? 4 * q + row : 0;
                        if (FORM) grn[q] = gram[(c * 16 + sn) * kLineLd + min(sn + col, 15)];
                    }
                    if (!BOX) gpn = gpri[sn * kLineLd + min(sn + col, 15)];
                }
                double v0 = 0.0, x00 = 0.0;
                if constexpr (LIK == LIK_FUNNEL) {
                    v0 = lane_value(vr[0], 0);
                    x00 = lane_value(x0r[0], 0);
                }
                // the point and the direction, for the coordinate sums
                auto spread = [&]() {
                    const bool sum0 = RG || l > 0;   // (not the funnel's v)
#pragma unroll
                    for (int i = 0; i < NA; ++i)
                        if (l + 64 * i < D) {
                            xs[l + 64 * i] = i > 0 || sum0 ? x0r[i] : 0.0;
                            vs[l + 64 * i] = i > 0 || sum0 ? vr[i] : 0.0;
                        }
                    wave_sync();
                };
                if constexpr (!FORM) spread();
                // box prior: t inside [tin0, tin1] keeps every coordinate in the box whatever
                // the rounding of x + t v, t outside [tou0, tou1] puts one out; the margins
                // cover the FP32 quotients and, away from the faces, the rounding of y.  The
                // quotients are taken where FP32's range holds them (distances below 1e30 by the
                // caller's check of the box, |v| in [1e-30, 1e30), the smallest quotient 1e-30;
                // an infinite one is a coordinate that rests, or lies beyond every t)
                float tin0 = -INFINITY, tin1 = INFINITY, tou0 = -INFINITY, tou1 = INFINITY;
                if (BOX) {
                    float m0 = INFINITY, m1 = INFINITY;
                    bool face = false;
#pragma unroll
                    for (int i = 0; i < NA; ++i) {
                        const bool pos = vr[i] > 0.0;
                        const double hi = pbr[i] - x0r[i], lo = x0r[i] - par[i];
                        const float va = fabsf((float)vr[i]), rv = __builtin_amdgcn_rcpf(va);
                        constexpr unsigned v0 = __builtin_bit_cast(unsigned, 1e-30f),
                                           v1 = __builtin_bit_cast(unsigned, 1e30f);
                        const bool range = __builtin_bit_cast(unsigned, va) - v0 < v1 - v0;
                        face = face || !(hi > near_[i]) || !(lo > near_[i]) ||
                               !(range || vr[i] == 0.0);
                        m1 = fminf(m1, (float)(pos ? hi : lo) * rv);
                        m0 = fminf(m0, (float)(pos ? lo : hi) * rv);
                    }
                    face = face || fminf(m0, m1) < 1e-30f;
                    m1 = wave_min_pos(m1);
                    m0 = wave_min_pos(m0);
                    tin1 = m1 * (1.f - 2e-5f);
                    tin0 = -m0 * (1.f - 2e-5f);
                    tou1 = m1 * (1.f + 2e-5f);
                    tou0 = -m0 * (1.f + 2e-5f);
                    if (__any(face)) {   // decided coordinate by coordinate
                        tin0 = INFINITY; tin1 = -INFINITY;
                        tou0 = -INFINITY; tou1 = INFINITY;
                    }
                }
                // Sixteen candidates, column c at this lane's t: okm the bits that pass the
                // prior, the result those inside the slice; vm = the candidates wanted.
                double Lv = 0.0;   // tempered: log L of the lane's candidate
                auto test = [&](double t, unsigned vm, unsigned &okm) -> unsigned {
                    unsigned in;
                    const double lp = -0.5 * (t * fma(t, gp, bp2));   // log Pi(y) - log Pi(x)
                    if (BOX) {
                        const unsigned inb = (unsigned)__ballot(t >= (double)tin0 && t <= (double)tin1) & vm;
                        okm = inb;
                        if (inb != vm) {
                            const unsigned out = (unsigned)__ballot(t < (double)tou0 || t > (double)tou1);
                            unsigned ask = vm & ~inb & ~out & 0xFFFFu;
                            while (ask) {   // within a margin of the box's faces
                                const int s = __builtin_ctz(ask);
                                ask &= ask - 1u;
                                const double ts = lane_value(t, s);
                                bool ib = true;
#pragma unroll
                                for (int i = 0; i < NA; ++i) {
                                    const double y = fma(ts, vr[i], x0r[i]);
                                    if (l + 64 * i < d) ib = ib && y >= par[i] && y <= pbr[i];
                                }
                                okm |= (__all(ib) ? 1u : 0u) << s;
                            }
                        }
                    } else {
                        okm = TEMP ? vm : ((unsigned)__ballot(lp > lu) & vm);
                    }
                    if constexpr (MIX) {
                        double lc[NR];
                        bool hit = false, amb = false;
#pragma unroll
                        for (int q = 0; q < NR; ++q) {
                            lc[q] = cst[q] - 0.5 * fma(t, fma(t, g[q], b2[q]), aa[q]);
                            hit = hit || lc[q] > Lstar;
                            amb = amb || lc[q] > Lamb;
                        }
                        if constexpr (TEMP) {
                            double mx = lc[0];
#pragma unroll
                            for (int q = 1; q < NR; ++q) mx = fmax(mx, lc[q]);
                            mx = fmax(mx, __shfl_xor(mx, 16, 64));
                            mx = fmax(mx, __shfl_xor(mx, 32, 64));
                            double se = 0.0;
#pragma unroll
                            for (int q = 0; q < NR; ++q) se += lc[q] > -INFINITY ? exp(lc[q] - mx) : 0.0;
                            se += __shfl_xor(se, 16, 64);
                            se += __shfl_xor(se, 32, 64);
                            Lv = mx == -INFINITY ? -INFINITY : mx + log(se);
                        } else {
                            in = fold_rows(__ballot(hit));
                            const unsigned doubt = fold_rows(__ballot(amb)) & ~in & okm;
                            if (doubt) {
                                double se = 0.0;
#pragma unroll
                                for (int q = 0; q < NR; ++q) se += exp(lc[q] - Lstar);
                                se += __shfl_xor(se, 16, 64);
                                se += __shfl_xor(se, 32, 64);
                                in |= (unsigned)__ballot(se > 1.0) & doubt;
                            }
                        }
                    } else if constexpr (RG) {
                        double s2 = 0.0, sc = 0.0;
                        // the lane's coordinates 8 i + 2 row, + 1: four i at a time, then one
                        auto add = [&](int a, auto n) {
                            constexpr int U = 2 * decltype(n)::value;
                            double y[U];
#pragma unroll
                            for (int i = 0; i < U / 2; ++i) {
                                const double2 x2 = *(const double2 *)(xs + a + 8 * i);
                                const double2 v2 = *(const double2 *)(vs + a + 8 * i);
                                y[2 * i] = fma(t, v2.x, x2.x);
                                y[2 * i + 1] = fma(t, v2.y, x2.y);
                            }
                            double q0 = 0.0, q1 = 0.0;
#pragma unroll
                            for (int i = 0; i < U / 2; ++i) {
                                q0 = fma(y[2 * i], y[2 * i], q0);
                                q1 = fma(y[2 * i + 1], y[2 * i + 1], q1);
                            }
                            s2 += q0 + q1;
                            sc += cos_2pi<U>(y);
                        };
                        int a = 2 * row;
                        for (; a + 25 < d; a += 32) add(a, std::integral_constant<int, 4>{});
                        for (; a + 1 < d; a += 8) add(a, std::integral_constant<int, 1>{});
                        if (a < d) {
                            const double y[1] = {fma(t, vs[a], xs[a])};
                            s2 = fma(y[0], y[0], s2);
                            sc += cos_2pi<1>(y);
                        }
                        s2 += __shfl_xor(s2, 16, 64);
                        sc += __shfl_xor(sc, 16, 64);
                        s2 += __shfl_xor(s2, 32, 64);
                        sc += __shfl_xor(sc, 32, 64);
                        const double tf = P.rg_la - 0.5 * s2;
                        const double tg = P.rg_l1a - P.rg_amp * d + P.rg_amp * sc;
                        const double mx = fmax(tf, tg);
                        if constexpr (TEMP) {
                            Lv = mx + log(exp(tf - mx) + exp(tg - mx));
                        } else {
                            in = (unsigned)__ballot(mx > Lstar) & 0xFFFFu;
                            const unsigned doubt = (unsigned)__ballot(mx > Lamb) & ~in & okm;
                            if (doubt)
                                in |= (unsigned)__ballot(exp(tf - Lstar) + exp(tg - Lstar) > 1.0) &
                                      doubt;
                        }
                    } else {
                        const double vv = fma(t, v0, x00), ew = 0.5 * exp(-vv);
                        const double rest = -vv * vv / 18.0 - 0.5 * (LOG_2PI + log(9.0)) -
                                            (double)(d - 1) * 0.5 * (vv + LOG_2PI);
                        auto radius2 = [&]() -> double {   // the lane's coordinates 8 i + 2 row, + 1
                            double q0 = 0.0, q1 = 0.0;
                            // (rarely run beside the parabola: registers before speed)
                            constexpr int kUnroll = FORM ? 1 : 4;
#pragma unroll kUnroll
                            for (int a = 2 * row; a < d; a += 8) {   // (zero from d up)
                                const double2 x2 = *(const double2 *)(xs + a);
                                const double2 v2 = *(const double2 *)(vs + a);
                                const double y0 = fma(t, v2.x, x2.x), y1 = fma(t, v2.y, x2.y);
                                q0 = fma(y0, y0, q0);
                                q1 = fma(y1, y1, q1);
                            }
                            double s2 = q0 + q1;
                            s2 += __shfl_xor(s2, 16, 64);
                            s2 += __shfl_xor(s2, 32, 64);
                            return s2;
                        };
                        if constexpr (FORM) {
                            const double tb = t * b2[0], tg = t * t * g[0];
                            Lv = rest - ew * (aa[0] + tb + tg);
                            in = (unsigned)__ballot(Lv > Lstar);
                            // (in FP32: too large a term makes it infinite, and everything doubtful)
                            const float slack = (float)ew * (size + (float)(fabs(tb) + tg)) * 1e-13f;
                            const unsigned doubt =
                                (unsigned)__ballot(!(fabs(Lv - Lstar) > (double)slack)) & okm;
                            if (doubt) {
                                spread();
                                Lv = rest - ew * radius2();
                                in = (in & ~doubt) | ((unsigned)__ballot(Lv > Lstar) & doubt);
                                wave_sync();
                            }
                        } else {
                            Lv = rest - ew * radius2();
                            in = (unsigned)__ballot(Lv > Lstar);
                        }
                    }
                    if constexpr (TEMP)
                        in = (unsigned)__ballot((BOX ? 0.0 : lp) + beta * (Lv - logL0) > lu);
                    return in & okm;
                };
                auto tally = [&](unsigned cons, unsigned okm) {
                    n_tests += __builtin_popcount(cons);
                    n_evals += __builtin_popcount(cons & okm);
                };

                const double *uq = us + sb * kStepU;
                int nl = 0, nr = 0, ns = 0, acc = 0;
                bool la = cap_out > 0, ra = la, open = true;
                double tL = 0.0, tR = 0.0, ta = 0.0;
                if (fast) {
                    unsigned okm;
                    const unsigned in = test(tf, 0xFFFFu, okm);
                    const unsigned le = in & 3u, re = (in >> 2) & 3u;
                    nl = le == 3u ? 2 : (int)(le & 1u);
                    nr = re == 3u ? 2 : (int)(re & 1u);
                    la = nl == 2;
                    ra = nr == 2;
                    // a second test of an end is made where its first was inside
                    unsigned cons = 5u | ((le & 1u) << 1) | ((re & 1u) << 3);
                    if (nl + nr <= 1) {   // one of the three outcomes that were planned
                        const int s = 4 + 4 * nl + 8 * nr;
                        const unsigned f = (in >> s) & 0xFu;
                        ns = __builtin_ctz(f | 8u) + 1;
                        cons |= ((1u << ns) - 1u) << s;
                        if (f) {
                            acc = 1;
                            ta = lane_value(tf, s + ns - 1);
                            if constexpr (TEMP) logL0 = lane_value(Lv, s + ns - 1);
                            open = false;
                        }
                    }
                    tally(cons, okm);
                } else if (cap_out <= 0) {
                    c_outcap += 2;
                }
                if (open) {
                    tL = uq[0];
                    tR = tL + width;
                    for (int i = 0; i < nl; ++i) tL -= width;
                    for (int i = 0; i < nr; ++i) tR += width;
                    if (la && nl >= cap_out) { la = false; ++c_outcap; }
                    if (ra && nr >= cap_out) { ra = false; ++c_outcap; }
                    // stepping out: the next eight positions of both ends at once
                    while (la || ra) {
                        const int nsl = la ? min(kLineSide, cap_out - nl) : 0;
                        const int nsr = ra ? min(kLineSide, cap_out - nr) : 0;
                        const double step = col < kLineSide ? -width : width;
                        double t = col < kLineSide ? tL : tR;
#pragma unroll
                        for (int i = 1; i < kLineSide; ++i) if ((col & 7) >= i) t += step;
                        const unsigned ml = (1u << nsl) - 1u, mr = (1u << nsr) - 1u;
                        unsigned okm;
                        const unsigned in = test(t, ml | (mr << kLineSide), okm);
                        // leading inside tests of each end
                        const int na = __builtin_ctz(~(in & ml));
                        const int nc = __builtin_ctz(~((in >> kLineSide) & mr));
                        if (la) {
                            tally(((2u << na) - 1u) & ml, okm);
                            if (na > 0) tL = lane_value(t, min(na, 7)) - (na == 8 ? width : 0.0);
                            nl += na;
                            if (na < nsl) la = false;
                            else if (nl >= cap_out) { la = false; ++c_outcap; }
                        }
                        if (ra) {
                            tally(((2u << nc) - 1u) & mr, okm >> kLineSide);
                            if (nc > 0) tR = lane_value(t, 8 + min(nc, 7)) + (nc == 8 ? width : 0.0);
                            nr += nc;
                            if (nc < nsr) ra = false;
                            else if (nr >= cap_out) { ra = false; ++c_outcap; }
                        }
                    }
                    // the proposals that the first pass rejected
                    for (int q = 0; q < ns; ++q) {
                        const double tq = fma(uq[2 + q], tR - tL, tL);
                        if (tq < 0.0) tL = tq; else tR = tq;
                    }
                    // shrinking: the next sixteen proposals, if every earlier one is rejected
                    while (!acc && ns < cap_sh) {
                        const int np = min(16, cap_sh - ns);
                        double u, unused;
                        draw2(R.key0, R.key1, PUR_SHRINK, (uint32_t)j, it, (uint32_t)st,
                              (uint32_t)(ns + col), u, unused);
                        if (l < 16) su[l] = u;
                        wave_sync();
                        double sL = tL, sR = tR, t = 0.0;
                        for (int q = 0; q < 16; ++q) {
                            const double tq = fma(su[q], sR - sL, sL);
                            if (col == q) t = tq;
                            if (tq < 0.0) sL = tq; else sR = tq;
                        }
                        wave_sync();
                        const unsigned pm = (1u << np) - 1u;
                        unsigned okm;
                        const unsigned in = test(t, pm, okm);
                        if (in) {
                            const int q = __builtin_ctz(in);
                            tally((2u << q) - 1u, okm);
                            ta = lane_value(t, q);
                            if constexpr (TEMP) logL0 = lane_value(Lv, q);
                            ns += q + 1;
                            acc = 1;
                        } else {
                            tally(pm, okm);
                            ns += np;
                            tL = sL;
                            tR = sR;
                        }
                    }
                }
                if (acc) {
                    moved = true;
#pragma unroll
                    for (int i = 0; i < NA; ++i) x0r[i] = fma(ta, vr[i], x0r[i]);
                    if (LIK == LIK_FUNNEL) size += (float)(fabs(ta * b2[0]) + ta * ta * g[0]);
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                        aa[q] = fma(ta, fma(ta, g[q], b2[q]), aa[q]);
                        h[q] = fma(ta, gr[q], h[q]);
                    }
                    if (!BOX) hp = fma(ta, grp, hp);
                } else {
                    ++c_shcap;
                }
#pragma unroll
                for (int q = 0; q < NR; ++q) h[q] = dppd<DPP_ROL1>(h[q]);
                if (!BOX) hp = dppd<DPP_ROL1>(hp);
                if (R.trace && l == 0) {
                    int *tr = R.trace + ((size_t)j * p + st) * 4;
                    tr[0] = nl; tr[1] = nr; tr[2] = ns; tr[3] = acc;
                }
            }
            c_tests += n_tests;
            c_evals += n_evals;
            wave_sync();   // the block's LDS is rewritten
        }
    }

    // stored log-likelihoods: each chain's final point through the batched FP64 tile
    __syncthreads();
    Tile T{};
    T.cand = (double *)(smem + lay.cand);
    T.mu64 = (double *)P.mu;
    T.cst = (double *)P.cst;
    T.q = (double *)(smem + lay.q);
    T.L = (double *)(smem + lay.L);
    T.mask = (int *)(smem + lay.mask);
    for (int i = tid; i < kRows * (D + 1); i += 256) T.cand[i] = 0.0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NA; ++i)
        if (l + 64 * i < D) T.cand[w * (D + 1) + l + 64 * i] = has_chain ? x0r[i] : 0.0;
    if (tid < kRows) T.mask[tid] = tid < kMaxChainsPerWG && tid < C && bm.y * C + tid < R.k;
    __syncthreads();
    eval64<D, LIK>(P, T, T.mask, T.L);
    if (has_chain) {
        unsigned long long nonfin = 0;
        // (in FP64 a chain that never moved keeps its parent's value)
        if (moved || !fp64) logL0 = sanitize(T.L[w], nonfin);
        if (!TEMP && moved && !(logL0 > Lstar)) {
            // a form's last bits let in a point on the contour: the chain keeps its parent
            ++c_viol;
            logL0 = R.logL[parent];
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if (l + 64 * i < d) x0r[i] = R.X[(size_t)(l + 64 * i) * R.m_pad + parent];
        }
        const int slot = TEMP ? j : R.perm[j];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int a = l + 64 * i;
            if (a < d) R.X[(size_t)a * R.m_pad + slot] = x0r[i];
        }
        if (l == 0) {
            R.logL[slot] = logL0;
            atomicAdd(&R.ctr[0], c_evals);
            atomicAdd(&R.ctr[1], c_tests);
            atomicAdd(&R.ctr[2], c_tests - c_evals);
            atomicAdd(&R.ctr[3], c_outcap);
            atomicAdd(&R.ctr[4], c_shcap);
            atomicAdd(&R.ctr[7], c_viol);
        }
    }
}

template <int D, int LIK, int NR, int KIND, bool BOX, int OCC>
static hipError_t line_l(const Launch &L, int fp64, hipStream_t s)
{
    const size_t lds = line_lds_bytes(D, L.max_K, LIK, BOX, KIND == LINE_WALK);
    auto f = k_hrss_line<D, LIK, NR, KIND, BOX, OCC>;
    hipError_t e = hipFuncSetAttribute((const void *)f,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(f, dim3(L.nblocks), dim3(256), lds, s, L, fp64);
    return hipGetLastError();
}

// Workgroups per CU of the register allocation: a mixture's W fragments in flight do not fit 256
// registers at D = 64 and 128, and a launch that leaves one workgroup per CU loses nothing by
// taking more.
template <int D, int LIK, int NR, int KIND, bool BOX>
static hipError_t line_b(const Launch &L, int fp64, int occ, hipStream_t s)
{
    if constexpr (LIK == LIK_MIXTURE && D >= 64)
        if (occ == 1) return line_l<D, LIK, NR, KIND, BOX, 1>(L, fp64, s);
    return line_l<D, LIK, NR, KIND, BOX, 2>(L, fp64, s);
}

template <int D, int LIK, int NR>
static hipError_t line_t(const Launch &L, int kind, int box, int fp64, int occ, hipStream_t s)
{
    if constexpr (LIK != LIK_RG)
        if (kind == LINE_WALK)
            return box ? line_b<D, LIK, NR, LINE_WALK, true>(L, fp64, occ, s)
                       : line_b<D, LIK, NR, LINE_WALK, false>(L, fp64, occ, s);
    if (kind == LINE_TEMPERED)
        return box ? line_b<D, LIK, NR, LINE_TEMPERED, true>(L, fp64, occ, s)
                   : line_b<D, LIK, NR, LINE_TEMPERED, false>(L, fp64, occ, s);
    if (kind == LINE_SLICE)
        return box ? line_b<D, LIK, NR, LINE_SLICE, true>(L, fp64, occ, s)
                   : line_b<D, LIK, NR, LINE_SLICE, false>(L, fp64, occ, s);
    return hipErrorInvalidValue;
}

template <int D>
static hipError_t line_d(const Launch &L, int lik, int kind, int box, int fp64, int occ,
                         hipStream_t s)
{
    if (lik == LIK_FUNNEL) return line_t<D, LIK_FUNNEL, 1>(L, kind, box, fp64, occ, s);
    if (lik == LIK_RG) return line_t<D, LIK_RG, 1>(L, kind, box, fp64, occ, s);
    if constexpr (D <= 128) {
        if (L.max_K <= 4) return line_t<D, LIK_MIXTURE, 1>(L, kind, box, fp64, occ, s);
        if (L.max_K <= 8) return line_t<D, LIK_MIXTURE, 2>(L, kind, box, fp64, occ, s);
        if (L.max_K <= kLineForms) return line_t<D, LIK_MIXTURE, 4>(L, kind, box, fp64, occ, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_hrss_line(const Launch &L, int D, int lik, int smc, int rw, int box, int fp64,
                            int occ, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    const int kind = rw ? LINE_WALK : smc ? LINE_TEMPERED : LINE_SLICE;
    if (D == 32) return line_d<32>(L, lik, kind, box, fp64, occ, s);
    if (D == 64) return line_d<64>(L, lik, kind, box, fp64, occ, s);
    if (D == 128) return line_d<128>(L, lik, kind, box, fp64, occ, s);
    if (D == 320) return line_d<320>(L, lik, kind, box, fp64, occ, s);
    return hipErrorInvalidValue;
}

}  // namespace nss
