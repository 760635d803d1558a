// Blocked Cholesky factorisation shared by the GP likelihood and the whitening: 16x16 tiles of the
// lower triangle in the accumulator layout of the 16x16x4 MFMA, columns of tiles in LDS, and the
// elimination of a block column with one row per lane.
#pragma once
#include "nss_wave.hpp"

namespace nss {

constexpr int kTileLd = 17;              // LDS tile row stride
constexpr int kTile = 16 * kTileLd;

template <typename T> struct Mf;
template <> struct Mf<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(double a, double b, v4 c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // accumulator row of register r in lane l (column l & 15)
    __device__ static int row(int l, int r) { return (l >> 4) + 4 * r; }
};
template <> struct Mf<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(float a, float b, v4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static int row(int l, int r) { return 4 * (l >> 4) + r; }
};

__device__ __forceinline__ double readlane_t(double v, int lane) { return readlane_d(v, lane); }
__device__ __forceinline__ float readlane_t(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// lower tile index t = I (I + 1) / 2 + K  ->  (I, K), K <= I
__device__ __forceinline__ void tile_ik(int t, int &I, int &K)
{
    int i = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while (i * (i + 1) / 2 > t) --i;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    I = i;
    K = t - i * (i + 1) / 2;
}

template <typename T, typename V>
__device__ __forceinline__ void store_tile(const V &acc, T *p, int l)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) p[Mf<T>::row(l, r) * kTileLd + (l & 15)] = acc[r];
}

// 1/sqrt(x) from the hardware estimate r, for a short dependent chain per pivot: with
// e = 1 - x r^2, r (1 + e/2 + 3 e^2/8) has the relative error 5 e^3 / 16 (e is about 2^-23 in FP64;
// FP32 takes Newton's r (1 + e/2)).
__device__ __forceinline__ double rsq_refined(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * r), r, 1.0);
    return fma(r * e, fma(e, 0.375, 0.5), r);
}
__device__ __forceinline__ float rsq_refined(float x)
{
    float r = __builtin_amdgcn_rsqf(x);
    return r * (1.5f - 0.5f * x * r * r);
}
// By two Newton steps r (3/2 - x r^2 / 2) instead (FP32: one): the GP's roots, whose roundings its
// ill-conditioned factors follow.
__device__ __forceinline__ double rsq_newton(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    r *= fma(-r, h * r, 1.5);
    r *= fma(-r, h * r, 1.5);
    return r;
}
__device__ __forceinline__ float rsq_newton(float x) { return rsq_refined(x); }

// Eliminates a block column with one row per lane: a[c] is the lane's row, lane i < 16
// row i of the diagonal tile.  On return lane i < 16 holds row i of the factor (its entries above
// the diagonal are not meaningful), the other lanes their row times the transposed inverse
// factor (of a row of the identity: a column of the inverse).  p0: the product of the pivots'
// roots; in FP32, whose roots are rounded, p0 and p1: of the first and the last eight pivots
// themselves.  bad: a pivot was not positive (the results are then not meaningful).  ROUNDED: the
// roots and quotients are rounded to nearest, as sqrt and / are (about 60 cycles more on a pivot's
// chain), for a matrix whose last pivots are its rounding error: there another rounding is another
// factor.
template <typename T, bool ROUNDED = false>
__device__ __forceinline__ void eliminate(T (&a)[16], double &p0, double &p1, int &bad)
{
    p0 = p1 = 1.0;
    bad = 0;
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
        T piv = readlane_t(a[jj], jj);
        asm volatile("" : "+v"(piv));
        bad |= piv > T(0) ? 0 : 1;
        if constexpr (ROUNDED) {
            const T r = rsq_refined(piv);
            T root = piv * r;
            root = fma(fma(-root, root, piv), T(0.5) * r, root);
            const T inv = fma(fma(-root, r, T(1)), r, r);
            const T q = a[jj] * inv;
            a[jj] = (threadIdx.x & 63) == jj ? root : fma(fma(-q, root, a[jj]), inv, q);
        } else {
            const T r = rsq_newton(piv);
            if (sizeof(T) == 8) p0 *= (double)(piv * r);
            else if (jj < 8) p0 *= (double)piv;
            else p1 *= (double)piv;
            a[jj] *= r;
        }
#pragma unroll
        for (int c = jj + 1; c < 16; ++c) a[c] = fma(-a[jj], readlane_t(a[jj], c), a[c]);
        // every row takes this column now: left to itself the compiler sinks the updates to
        // their columns' turns and keeps all the lane reads until then
#pragma unroll
        for (int c = jj + 1; c < 16; ++c) asm volatile("" : "+v"(a[c]));
    }
}

}  // namespace nss
