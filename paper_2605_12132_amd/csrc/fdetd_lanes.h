// Lane-level building blocks shared by the row-marching kernels: the share of a complex value a lane holds,
// the Horner coefficients, storage layouts and global-memory access.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "fdetd_internal.h"

namespace fdetd {
namespace {

constexpr int WAVE = 64;
constexpr int NXCD = 8;

// The share of one complex value a lane holds: one part (K = 1, FP64 lane pairs) or both (K = 2).
template <typename AR, int K>
struct lv {
    AR p[K];
};
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> operator+(lv<AR, K> a, lv<AR, K> b)
{
#pragma unroll
    for (int c = 0; c < K; ++c) a.p[c] += b.p[c];
    return a;
}
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> operator-(lv<AR, K> a, lv<AR, K> b)
{
#pragma unroll
    for (int c = 0; c < K; ++c) a.p[c] -= b.p[c];
    return a;
}
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> operator*(AR s, lv<AR, K> a)
{
#pragma unroll
    for (int c = 0; c < K; ++c) a.p[c] *= s;
    return a;
}
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> fmav(AR s, lv<AR, K> a, lv<AR, K> acc)
{
#pragma unroll
    for (int c = 0; c < K; ++c) acc.p[c] = fma(s, a.p[c], acc.p[c]);
    return acc;
}
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> zero_lv()
{
    lv<AR, K> z;
#pragma unroll
    for (int c = 0; c < K; ++c) z.p[c] = (AR)0;
    return z;
}
// i * s * x: (re, im) -> (-s im, s re); with lane pairs the partner lane holds the other part
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> times_i(AR s, lv<AR, K> x)
{
    lv<AR, K> r;
    if constexpr (K == 2) {
        r.p[0] = -s * x.p[1];
        r.p[1] = s * x.p[0];
    } else {
        const AR other = __shfl_xor(x.p[0], 1, WAVE);
        r.p[0] = (threadIdx.x & 1) ? s * other : -s * other;
    }
    return r;
}

// A coefficient of the Horner recurrence (dt/(n+1), the source weight -dt 2^-n) given in FP64 and applied
// to values in the arithmetic type AR.  Float arithmetic splits it, c = hi + lo with hi = float(c) and
// lo = float(c - hi), and forms c x as hi x + lo x: the product then carries c to about 2^-48 instead of
// rounding it to 2^-24, which would otherwise shift the effective time step the same way every stage.
template <typename AR>
struct Coef {
    AR hi, lo;
};
template <typename AR>
__device__ __forceinline__ Coef<AR> split_coef(double c)
{
    if constexpr (sizeof(AR) == 8) {
        return Coef<AR>{c, 0.0};
    } else {
        const float h = (float)c;
        return Coef<AR>{h, (float)(c - (double)h)};
    }
}
// c x
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> cmul(Coef<AR> c, lv<AR, K> x)
{
    if constexpr (sizeof(AR) == 8) return c.hi * x;
    else return fmav(c.lo, x, c.hi * x);
}
// c x + acc
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> cfma(Coef<AR> c, lv<AR, K> x, lv<AR, K> acc)
{
    if constexpr (sizeof(AR) == 8) return fmav(c.hi, x, acc);
    else return fmav(c.lo, x, fmav(c.hi, x, acc));
}

// FP32 storage read in lane pairs (one float part per lane, 32 columns per wave, as FP64 storage is read):
// the layout of the FP32C near-axis tiles, whose FP64 arithmetic on a whole complex value per lane would
// need twice the registers.
struct f2pair {};

template <typename V> struct scal;
template <> struct scal<double2> { using R = double; };
template <> struct scal<float2> { using R = float; };
template <> struct scal<f2pair> { using R = float; };
// storage element type of a layout (what pointers into the planes point at)
template <typename V> struct stor { using T = V; };
template <> struct stor<f2pair> { using T = float2; };

// Global-memory access through address-space-1 pointers.  The kernels' pointers come from a descriptor
// table and the kernel arguments, so without the cast the compiler emits flat instructions, which also
// count against the LDS/scalar wait counter and make every LDS wait drain the prefetched loads.
#define FDETD_GLOBAL __attribute__((address_space(1)))
template <typename T> struct ibits;  // an integer of the same size, to move T through global memory
template <> struct ibits<double> { using I = unsigned long long; };
template <> struct ibits<float2> { using I = unsigned long long; };
template <> struct ibits<float> { using I = unsigned int; };
// Element i of the array at p.  Callers pass a wave-uniform p (a row start, kept in scalar registers) and a
// small per-lane i, so the loads use the scalar-base + 32-bit-vector-offset addressing form.
// The byte offset is formed in 32 bits (a row of a plane is far below 4 GiB), which is what that addressing
// form adds to the scalar base.
// They go through a buffer resource whose base is that row start (four scalar registers built by scalar
// instructions) and take the lane's byte offset as the vector offset: no per-load vector address
// arithmetic.  Word 3 of the resource is the gfx9-family value for raw (untyped) buffer access; the
// record count is left at its maximum, every offset being a lane's position within its row.
constexpr int kBufWord3 = 0x00020000;
template <typename T>
__device__ __forceinline__ T gld(const void *p, unsigned i)
{
    using I = typename ibits<T>::I;
    const unsigned off = i * (unsigned)sizeof(I);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, 0x7fffffff, kBufWord3);
    if constexpr (sizeof(I) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
template <typename T, int POL = 0>
__device__ __forceinline__ void gst(void *p, unsigned i, T v)
{
    using I = typename ibits<T>::I;
    const unsigned off = i * (unsigned)sizeof(I);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(p, (short)0, 0x7fffffff, kBufWord3);
    if constexpr (sizeof(I) == 8) {
        using V2 = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0u, 0, 0));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V2, v), r, off, 0, POL);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, POL);
    }
}
// Store of a stage output: non-temporal (bit 1 of the cache-policy operand on this target family) in the
// kernel variants the plan picks when it measured them faster for a batch -- on grids far larger than the
// caches, outputs that the L2 keeps only evict the rows other wavefronts read again -- else the default.
template <typename T, bool NT>
__device__ __forceinline__ void gst_out(void *p, unsigned i, T v)
{
    gst<T, NT ? 2 : 0>(p, i, v);
}
// Start of row q of component c of a vector of planes of P elements each (row length nz S elements).
template <typename E>
__device__ __forceinline__ const E *row_ptr(const void *base, int c, size_t P, int nz, int S, int q)
{
    return (const E *)base + (size_t)c * P * S + (size_t)q * nz * S;
}
// The descriptor table and the per-row tables are written by the host before the launch and only read
// here: through the constant address space they become scalar loads the compiler may hoist, instead of
// vector loads whose in-order wait counter would also wait for the prefetched rows.
#define FDETD_CONST __attribute__((address_space(4)))
using CDesc = const FDETD_CONST ProbDesc;
__device__ __forceinline__ double cld(const double *p, int i) { return ((const FDETD_CONST double *)p)[i]; }
// Stencil coefficient j of a table in the arithmetic type: the float copy for float arithmetic (no
// conversion per tap), the double table otherwise.
template <typename AR>
__device__ __forceinline__ AR tap(const FDETD_CONST double *d, const FDETD_CONST float *f, int j)
{
    if constexpr (sizeof(AR) == 4) return f[j];
    else return d[j];
}

// Storage access.  FP64 (double2 storage, K = 1): element = one double, index 2*(row*nz + col) + part.
// FP32 (float2 storage, K = 2): element = one float2, index row*nz + col.
template <typename V> struct elem;
// Lo = the element of the FP32C compensation words in the same layout (unused with FP64 storage).
template <> struct elem<double2> {
    using E = double;
    using Lo = float2;
    static constexpr int S = 2;  // lanes per column
    static constexpr int K = 1;
};
template <> struct elem<float2> {
    using E = float2;
    using Lo = float2;
    static constexpr int S = 1;
    static constexpr int K = 2;
};
template <> struct elem<f2pair> {  // used only by the translation units of wide stencils
    using E = float;
    using Lo = float;
    [[maybe_unused]] static constexpr int S = 2;
    [[maybe_unused]] static constexpr int K = 1;
};

template <typename AR>
__device__ __forceinline__ lv<AR, 1> to_lv(double e) { return lv<AR, 1>{{(AR)e}}; }
template <typename AR>
__device__ __forceinline__ lv<AR, 2> to_lv(float2 e) { return lv<AR, 2>{{(AR)e.x, (AR)e.y}}; }
template <typename AR>
__device__ __forceinline__ lv<AR, 1> to_lv(float e) { return lv<AR, 1>{{(AR)e}}; }

__device__ __forceinline__ void two_sum(float a, float b, float &s, float &e)
{
    s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// The E part of w_N = psi + beta_in Jbar (the argument of the highest power of H in the Horner form of
// the midpoint solution, section 2.1) for one loaded element: FP64 arithmetic, one rounding to the
// storage precision, the same operation as the separate w_N pass, so that both give the same bits.
__device__ __forceinline__ double wn_elem(double p, double j, double b) { return __builtin_fma(b, j, p); }
__device__ __forceinline__ float wn_elem(float p, float j, double b) { return (float)__builtin_fma(b, (double)j, (double)p); }
__device__ __forceinline__ float2 wn_elem(float2 p, float2 j, double b) { return float2{wn_elem(p.x, j.x, b), wn_elem(p.y, j.y, b)}; }

// x if c, else +0.  The mask goes through an empty asm so that the compiler cannot see it is all-ones or
// zero: a select between a freshly loaded value and zero under a wave-uniform condition would otherwise
// become a branch around the load, and the wave would wait at its join for every load in flight.
template <typename AR, int K>
__device__ __forceinline__ lv<AR, K> keep_if(bool c, lv<AR, K> x)
{
    unsigned m = c ? ~0u : 0u;
    asm volatile("" : "+v"(m));
    lv<AR, K> r;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        if constexpr (sizeof(AR) == 8) {
            const unsigned long long mm = ((unsigned long long)m << 32) | m;
            r.p[i] = __builtin_bit_cast(AR, __builtin_bit_cast(unsigned long long, x.p[i]) & mm);
        } else {
            r.p[i] = __builtin_bit_cast(AR, __builtin_bit_cast(unsigned, x.p[i]) & m);
        }
    }
    return r;
}

}  // namespace
}  // namespace fdetd
