// gfx950 HRSS chains whose likelihood is a function of quadratic forms (Gaussian mixtures,
// Neal's funnel), evaluated along each step's line.
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
#include "nss_internal.hpp"
#include "nss_rng.hpp"
#include "nss_tiles.hpp"
#include "nss_wave.hpp"

#include <math.h>

namespace nss {

constexpr int kLineB = 15;              // steps per block (the sixteenth column is the point)
constexpr int kLineLd = 17;             // row stride of a Gram matrix in LDS
constexpr int kLineSide = 8;            // stepping-out tests per end and pass
constexpr int kLineForms = 16;          // most components

// LDS of one workgroup (byte offsets; identical on host): per chain the forms' Gram matrices
// (the last one the Gaussian prior's), the point, the block's step uniforms and the shrink
// uniforms of a pass past the buffer; the final points' FP64 tile overlays the Gram matrices.
struct LineLayout {
    int gram, x, us, su, chain;         // per-chain offsets and stride
    int cand, q, L, mask, total;
};
__host__ __device__ inline LineLayout line_layout(int D, int K, int lik)
{
    const int forms = (lik == LIK_MIXTURE ? K : 1) + 1;
    LineLayout o;
    int off = 0;
    o.gram = off; off += al16(forms * 16 * kLineLd * 8);
    o.x = off; off += al16(D * 8);
    o.us = off; off += kLineB * kStepU * 8;
    o.su = off; off += 16 * 8;
    o.chain = al16(off);
    int t = 0;
    o.cand = t; t += al16(kRows * (D + 1) * 8);
    o.q = t; t += al16(kRows * q_stride(D, K) * 8);
    o.L = t; t += al16(kRows * 8);
    o.mask = t; t += al16(kRows * 4);
    o.total = kMaxChainsPerWG * o.chain > t ? kMaxChainsPerWG * o.chain : t;
    return o;
}
size_t line_lds_bytes(int D, int K, int lik) { return (size_t)line_layout(D, K, lik).total; }

// Bits of a ballot folded over the four rows: bit c = some lane of column c voted.
__device__ __forceinline__ unsigned fold_rows(unsigned long long b)
{
    const unsigned h = (unsigned)b | (unsigned)(b >> 32);
    return (h | (h >> 16)) & 0xFFFFu;
}
__device__ __forceinline__ float wave_minf(float v)
{
    v = fminf(v, dppf<DPP_XOR1>(v)); v = fminf(v, dppf<DPP_XOR2>(v));
    v = fminf(v, dppf<DPP_HMIR>(v)); v = fminf(v, dppf<DPP_RMIR>(v));
    v = fminf(v, __shfl_xor(v, 16, 64));
    return fminf(v, __shfl_xor(v, 32, 64));
}

// NR: forms per lane (components 4 q + row, q < NR); TEMP: tempered SMC slices (no constraint).
template <int D, int LIK, int NR, bool TEMP>
__global__ __launch_bounds__(256, 2) void k_hrss_line(Launch Lc, int fp64)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 bm = Lc.map[blockIdx.x];
    const DevProblem P = Lc.P[bm.x];
    const DevRun R = Lc.R[bm.x];
    if (R.iscal[0] || R.iscal[2] <= 0) return;
    constexpr int NA = (D + 63) / 64;
    constexpr int NJB = D / 16, NKS = D / 4;
    constexpr bool MIX = LIK == LIK_MIXTURE;
    const LineLayout lay = line_layout(D, P.K, LIK);
    const int tid = threadIdx.x, w = uniform_i(tid >> 6), l = tid & 63;
    const int col = l & 15, row = l >> 4;
    const int d = P.d, K = MIX ? P.K : 1, C = R.C, p = R.p;
    const double Lstar = R.scal[0], beta = Lstar;   // tempered: the inverse temperature
    const int t0 = R.iscal[1], nsurv = R.iscal[2];
    const uint32_t it = (uint32_t)R.iscal[3] + 1u;
    const double width = R.width;
    const int cap_out = R.stepout_cap, cap_sh = R.shrink_cap;
    const bool box = P.prior_kind == PRIOR_BOX;

    unsigned char *mine = smem + w * lay.chain;
    double *gram = (double *)(mine + lay.gram);
    double *xs = (double *)(mine + lay.x);
    double *us = (double *)(mine + lay.us);
    double *su = (double *)(mine + lay.su);
    double *gpri = gram + K * 16 * kLineLd;   // the Gaussian prior's form

    const int j = bm.y * C + w;
    const bool has_chain = w < C && j < R.k;
    double x0r[NA], vr[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) { x0r[i] = 0.0; vr[i] = 0.0; }
    double logL0 = -INFINITY;
    bool moved = false;
    unsigned long long c_evals = 0, c_tests = 0, c_outcap = 0, c_shcap = 0, c_viol = 0;

    if (has_chain) {
        int parent = j;   // tempered SMC: the resampled particle j, gathered into slot j
        if constexpr (!TEMP) {
            double u, unused;
            draw2(R.key0, R.key1, PUR_RESAMPLE, (uint32_t)j, it, 0u, 0u, u, unused);
            int qi = (int)floor(u * (double)nsurv);
            if (qi > nsurv - 1) qi = nsurv - 1;
            parent = R.perm[t0 + qi];
            if (l == 0) R.parents[j] = parent;
        }
        // the prior's box of the lane's coordinates, and how far rounding can move y = x + t v
        double par[NA], pbr[NA], slop[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int a = l + 64 * i;
            par[i] = -INFINITY; pbr[i] = INFINITY; slop[i] = 0.0;
            if (a < d) {
                x0r[i] = R.X[(size_t)a * R.m_pad + parent];
                if (box) {
                    par[i] = P.pa[a];
                    pbr[i] = P.pb[a];
                    slop[i] = 4e-15 * fmax(fabs(par[i]), fabs(pbr[i]));
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
        const double Lamb = (MIX && K > 1) ? Lstar - log((double)K) - 1e-6 : INFINITY;
        const double *dirs = R.dirbuf + (size_t)j * p * D;
        const double *ub = R.ubuf + (size_t)j * p * kStepU;
        double pv[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) pv[i] = (l + 64 * i < D) ? dirs[l + 64 * i] : 0.0;

        for (int s0 = 0; s0 < p; s0 += kLineB) {
            const int nb = min(kLineB, p - s0);
            // ---- the block's products ----
#pragma unroll
            for (int i = 0; i < NA; ++i) if (l + 64 * i < D) xs[l + 64 * i] = x0r[i];
            for (int e = l; e < nb * kStepU; e += 64) us[e] = ub[(size_t)s0 * kStepU + e];
            wave_sync();
            const bool dcol = col < nb, xcol = col == 15;
            const double *vrow = dirs + (size_t)(s0 + (dcol ? col : 0)) * D;
            typedef double d4v __attribute__((ext_vector_type(4)));
            auto put = [&](double *g, const d4v &G) {
#pragma unroll
                for (int i = 0; i < 4; ++i) g[(row + 4 * i) * kLineLd + col] = G[i];
            };
            if constexpr (MIX) {
                double b[NKS];   // the directions' columns (the point's column differs per form)
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    const int kk = 4 * ks + row;
                    b[ks] = dcol ? vrow[kk] : (xcol ? xs[kk] : 0.0);
                }
                for (int c = 0; c < K; ++c) {
                    const double *wf = P.wf64 + (size_t)c * NJB * NKS * 64 + l;
                    const double *mu = P.mu + c * D;
                    d4v acc[NJB];
#pragma unroll
                    for (int jb = 0; jb < NJB; ++jb) acc[jb] = (d4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) {
                        const double bb = xcol ? b[ks] - mu[4 * ks + row] : b[ks];
#pragma unroll
                        for (int jb = 0; jb < NJB; ++jb)
                            if (ks < 4 * jb + 4)
                                acc[jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                    wf[((size_t)jb * NKS + ks) * 64], bb, acc[jb], 0, 0, 0);
                    }
                    d4v G = (d4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            G = __builtin_amdgcn_mfma_f64_16x16x4f64(acc[jb][i], acc[jb][i], G, 0, 0, 0);
                    put(gram + c * 16 * kLineLd, G);
                }
                if (!box) {
                    d4v G = (d4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) {
                        const int kk = 4 * ks + row;
                        const double bb = kk < d ? (xcol ? b[ks] - P.pa[kk] : b[ks]) / P.pb[kk] : 0.0;
                        G = __builtin_amdgcn_mfma_f64_16x16x4f64(bb, bb, G, 0, 0, 0);
                    }
                    put(gpri, G);
                }
            } else {
                // the funnel's form: the coordinates after the first
                d4v G = (d4v){0.0, 0.0, 0.0, 0.0}, Gp = (d4v){0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
                for (int ks = 0; ks < NKS; ++ks) {
                    const int kk = 4 * ks + row;
                    const double b = dcol ? vrow[kk] : (xcol ? xs[kk] : 0.0);
                    const double bb = kk > 0 ? b : 0.0;
                    G = __builtin_amdgcn_mfma_f64_16x16x4f64(bb, bb, G, 0, 0, 0);
                    if (!box) {
                        const double bp = kk < d ? (xcol ? b - P.pa[kk] : b) / P.pb[kk] : 0.0;
                        Gp = __builtin_amdgcn_mfma_f64_16x16x4f64(bp, bp, Gp, 0, 0, 0);
                    }
                }
                put(gram, G);
                if (!box) put(gpri, Gp);
            }
            wave_sync();
            // row 15: the point's products with every column; column 15 its own square
            double h[NR], hp = 0.0, luh = 0.0;
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                const int c = 4 * q + row;
                h[q] = (c < K) ? gram[(c * 16 + 15) * kLineLd + col] : 0.0;
            }
            if (!box) hp = gpri[15 * kLineLd + col];
            if (TEMP || !box) luh = log(dcol ? us[col * kStepU + 1] : 1.0);

            // ---- the block's steps ----
            for (int sb = 0; sb < nb; ++sb) {
                const int st = s0 + sb;
#pragma unroll
                for (int i = 0; i < NA; ++i) vr[i] = pv[i];
                if (st + 1 < p) {
                    const double *nx = dirs + (size_t)(st + 1) * D;
#pragma unroll
                    for (int i = 0; i < NA; ++i) if (l + 64 * i < D) pv[i] = nx[l + 64 * i];
                }
                double cu[kStepU];
#pragma unroll
                for (int q = 0; q < kStepU; ++q) cu[q] = us[sb * kStepU + q];
                // the step's parabolas: point, slope, curvature, and the row of the update
                double a[NR], b2[NR], g[NR], gr[NR];
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    const int c = 4 * q + row;
                    const double *gc = gram + ((c < K ? c : 0) * 16 + sb) * kLineLd;
                    gr[q] = gc[col];
                    g[q] = gc[sb];
                    a[q] = __shfl(h[q], (l & 48) | 15, 64);
                    b2[q] = 2.0 * __shfl(h[q], (l & 48) | sb, 64);
                }
                double ap = 0.0, bp2 = 0.0, gp = 0.0, grp = 0.0, lu = 0.0;
                if (!box) {
                    grp = gpri[sb * kLineLd + col];
                    gp = gpri[sb * kLineLd + sb];
                    ap = __shfl(hp, 15, 64);
                    bp2 = 2.0 * __shfl(hp, sb, 64);
                }
                if (TEMP || !box) lu = __shfl(luh, sb, 64);
                double v0 = 0.0, x00 = 0.0;
                if constexpr (!MIX) { v0 = __shfl(vr[0], 0, 64); x00 = __shfl(x0r[0], 0, 64); }
                // box prior: t inside [tin0, tin1] keeps every coordinate in the box whatever
                // the rounding of x + t v, t outside [tou0, tou1] puts one out; the margins
                // cover the FP32 quotients and half a unit in the last place of y
                float tin0 = -INFINITY, tin1 = INFINITY, tou0 = -INFINITY, tou1 = INFINITY;
                if (box) {
                    float i0 = INFINITY, i1 = INFINITY, o0 = INFINITY, o1 = INFINITY;
#pragma unroll
                    for (int i = 0; i < NA; ++i) {
                        // distances to the bound that t > 0 and t < 0 approach
                        const bool pos = vr[i] > 0.0;
                        const double up = pos ? pbr[i] - x0r[i] : x0r[i] - par[i];
                        const double dn = pos ? x0r[i] - par[i] : pbr[i] - x0r[i];
                        const float rv = __builtin_amdgcn_rcpf(fabsf((float)vr[i]));
                        if (fabsf((float)vr[i]) > 1e-30f && up >= 0.0 && dn >= 0.0) {
                            i1 = fminf(i1, (float)(up - slop[i]) * rv);
                            i0 = fminf(i0, (float)(dn - slop[i]) * rv);
                            o1 = fminf(o1, (float)(up + slop[i]) * rv);
                            o0 = fminf(o0, (float)(dn + slop[i]) * rv);
                        } else if (vr[i] != 0.0 || up < 0.0 || dn < 0.0) {
                            i0 = i1 = -1.f;   // decided coordinate by coordinate
                        }
                    }
                    tin1 = wave_minf(i1) * (1.f - 1e-5f);
                    tin0 = -wave_minf(i0) * (1.f - 1e-5f);
                    tou1 = wave_minf(o1) * (1.f + 1e-5f) + 1e-30f;
                    tou0 = -wave_minf(o0) * (1.f + 1e-5f) - 1e-30f;
                }
                // Sixteen candidates, column c at this lane's t: okm the bits that pass the
                // prior, the result those inside the slice; vm = the candidates wanted.
                double Lv = 0.0;   // tempered: log L of the lane's candidate
                auto test = [&](double t, unsigned vm, unsigned &okm) -> unsigned {
                    unsigned in;
                    const double lp = -0.5 * (t * fma(t, gp, bp2));   // log Pi(y) - log Pi(x)
                    if (box) {
                        const unsigned inb = (unsigned)__ballot(t >= (double)tin0 && t <= (double)tin1) & vm;
                        const unsigned out = (unsigned)__ballot(t < (double)tou0 || t > (double)tou1);
                        okm = inb;
                        unsigned ask = vm & ~inb & ~out & 0xFFFFu;
                        while (ask) {   // within a margin of the box's faces
                            const int s = __builtin_ctz(ask);
                            ask &= ask - 1u;
                            const double ts = __shfl(t, s, 64);
                            bool ib = true;
#pragma unroll
                            for (int i = 0; i < NA; ++i) {
                                const double y = fma(ts, vr[i], x0r[i]);
                                if (l + 64 * i < d) ib = ib && y >= par[i] && y <= pbr[i];
                            }
                            okm |= (__all(ib) ? 1u : 0u) << s;
                        }
                    } else {
                        okm = TEMP ? vm : ((unsigned)__ballot(lp > lu) & vm);
                    }
                    if constexpr (MIX) {
                        double lc[NR];
                        bool hit = false, amb = false;
#pragma unroll
                        for (int q = 0; q < NR; ++q) {
                            lc[q] = cst[q] - 0.5 * fma(t, fma(t, g[q], b2[q]), a[q]);
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
                    } else {
                        const double s2 = fmax(fma(t, fma(t, g[0], b2[0]), a[0]), 0.0);
                        const double vv = fma(t, v0, x00);
                        Lv = -vv * vv / 18.0 - 0.5 * (LOG_2PI + log(9.0)) - 0.5 * exp(-vv) * s2
                             - (double)(d - 1) * 0.5 * (vv + LOG_2PI);
                        if constexpr (!TEMP) in = (unsigned)__ballot(Lv > Lstar);
                    }
                    if constexpr (TEMP)
                        in = (unsigned)__ballot((box ? 0.0 : lp) + beta * (Lv - logL0) > lu);
                    return in & okm;
                };
                auto tally = [&](unsigned cons, unsigned okm) {
                    c_tests += __builtin_popcount(cons);
                    c_evals += __builtin_popcount(cons & okm);
                };

                // stepping out: the next eight positions of both ends at once
                double tL = cu[0], tR = tL + width;
                int nl = 0, nr = 0;
                bool la = cap_out > 0, ra = la;
                if (cap_out <= 0) c_outcap += 2;
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
                        if (na > 0) tL = __shfl(t, min(na, 7), 64) - (na == 8 ? width : 0.0);
                        nl += na;
                        if (na < nsl) la = false;
                        else if (nl >= cap_out) { la = false; ++c_outcap; }
                    }
                    if (ra) {
                        tally(((2u << nc) - 1u) & mr, okm >> kLineSide);
                        if (nc > 0) tR = __shfl(t, 8 + min(nc, 7), 64) + (nc == 8 ? width : 0.0);
                        nr += nc;
                        if (nc < nsr) ra = false;
                        else if (nr >= cap_out) { ra = false; ++c_outcap; }
                    }
                }
                // shrinking: the proposals that follow if every earlier one is rejected
                int ns = 0, acc = 0;
                double ta = 0.0;
                while (!acc && ns < cap_sh) {
                    const int avail = ns == 0 ? kStepShrinkU : 16;
                    const int np = min(avail, cap_sh - ns);
                    if (ns > 0) {   // past the buffer: one proposal's uniform per lane
                        double u, unused;
                        draw2(R.key0, R.key1, PUR_SHRINK, (uint32_t)j, it, (uint32_t)st,
                              (uint32_t)(ns + col), u, unused);
                        if (l < 16) su[l] = u;
                        wave_sync();
                    }
                    double sL = tL, sR = tR, t = 0.0;
                    if (ns == 0) {
#pragma unroll
                        for (int q = 0; q < kStepShrinkU; ++q) {
                            const double tq = sL + cu[2 + q] * (sR - sL);
                            if (col == q) t = tq;
                            if (tq < 0.0) sL = tq; else sR = tq;
                        }
                    } else {
                        for (int q = 0; q < 16; ++q) {
                            const double tq = sL + su[q] * (sR - sL);
                            if (col == q) t = tq;
                            if (tq < 0.0) sL = tq; else sR = tq;
                        }
                        wave_sync();
                    }
                    const unsigned pm = (1u << np) - 1u;
                    unsigned okm;
                    const unsigned in = test(t, pm, okm);
                    if (in) {
                        const int q = __builtin_ctz(in);
                        tally((2u << q) - 1u, okm);
                        ta = __shfl(t, q, 64);
                        if constexpr (TEMP) logL0 = __shfl(Lv, q, 64);
                        ns += q + 1;
                        acc = 1;
                    } else {
                        tally(pm, okm);
                        ns += np;
                        tL = sL;
                        tR = sR;
                    }
                }
                if (acc) {
                    moved = true;
#pragma unroll
                    for (int i = 0; i < NA; ++i) x0r[i] = fma(ta, vr[i], x0r[i]);
#pragma unroll
                    for (int q = 0; q < NR; ++q)
                        h[q] = fma(ta, xcol ? fma(ta, g[q], b2[q]) : gr[q], h[q]);
                    if (!box) hp = fma(ta, xcol ? fma(ta, gp, bp2) : grp, hp);
                } else {
                    ++c_shcap;
                }
                if (R.trace && l == 0) {
                    int *tr = R.trace + ((size_t)j * p + st) * 4;
                    tr[0] = nl; tr[1] = nr; tr[2] = ns; tr[3] = acc;
                }
                (void)ap;
            }
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
        if (!TEMP && moved && !(logL0 > Lstar)) ++c_viol;
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

template <int D, int LIK, int NR>
static hipError_t line_t(const Launch &L, int smc, int fp64, hipStream_t s)
{
    const size_t lds = line_lds_bytes(D, L.max_K, LIK);
    auto f = smc ? k_hrss_line<D, LIK, NR, true> : k_hrss_line<D, LIK, NR, false>;
    hipError_t e = hipFuncSetAttribute((const void *)f,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(f, dim3(L.nblocks), dim3(256), lds, s, L, fp64);
    return hipGetLastError();
}

template <int D>
static hipError_t line_d(const Launch &L, int lik, int smc, int fp64, hipStream_t s)
{
    if (lik == LIK_FUNNEL) return line_t<D, LIK_FUNNEL, 1>(L, smc, fp64, s);
    if constexpr (D <= 128) {
        if (L.max_K <= 4) return line_t<D, LIK_MIXTURE, 1>(L, smc, fp64, s);
        if (L.max_K <= 8) return line_t<D, LIK_MIXTURE, 2>(L, smc, fp64, s);
        if (L.max_K <= kLineForms) return line_t<D, LIK_MIXTURE, 4>(L, smc, fp64, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_hrss_line(const Launch &L, int D, int lik, int smc, int fp64, hipStream_t s)
{
    if (L.nblocks <= 0) return hipSuccess;
    if (D == 32) return line_d<32>(L, lik, smc, fp64, s);
    if (D == 64) return line_d<64>(L, lik, smc, fp64, s);
    if (D == 128) return line_d<128>(L, lik, smc, fp64, s);
    if (D == 320) return line_d<320>(L, lik, smc, fp64, s);
    return hipErrorInvalidValue;
}

}  // namespace nss
