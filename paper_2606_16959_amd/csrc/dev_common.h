// Device helpers shared by the kernels: complex values, fixed-order complex
// multiply-adds, 16-byte loads and stores, wave sums.
#pragma once

#include <hip/hip_runtime.h>

namespace hs {

template <typename R>
struct alignas(2 * sizeof(R)) C2 {
    R re, im;
};

// acc += c * x, in a fixed order of fused multiply-adds (the same in every
// kernel, so results do not depend on which kernel or batch size ran).
__device__ __forceinline__ void cfma(C2<float> &acc, C2<float> c, C2<float> x) {
    acc.re = __builtin_fmaf(c.re, x.re, acc.re);
    acc.re = __builtin_fmaf(-c.im, x.im, acc.re);
    acc.im = __builtin_fmaf(c.re, x.im, acc.im);
    acc.im = __builtin_fmaf(c.im, x.re, acc.im);
}
__device__ __forceinline__ void cfma(C2<double> &acc, C2<double> c, C2<double> x) {
    acc.re = __builtin_fma(c.re, x.re, acc.re);
    acc.re = __builtin_fma(-c.im, x.im, acc.re);
    acc.im = __builtin_fma(c.re, x.im, acc.im);
    acc.im = __builtin_fma(c.im, x.re, acc.im);
}

// (vr + i vi)(pr + i pi) in FP64: the product of an entry with D.  Spelled out,
// so that every kernel that forms a coefficient rounds it the same way.
__device__ __forceinline__ C2<double> cmul_d(double vr, double vi, double pr, double pi) {
    return C2<double>{__builtin_fma(vr, pr, -(vi * pi)), __builtin_fma(vi, pr, vr * pi)};
}

template <typename R>
__device__ __forceinline__ C2<R> cscale(C2<R> v, R s) {
    return C2<R>{v.re * s, v.im * s};
}

template <typename R>
__device__ __forceinline__ bool finite(C2<R> v) { return __builtin_isfinite(v.re) && __builtin_isfinite(v.im); }

// nrm2 points at the squared norm of state 0 inside [batch][4] reduction
// records (state b at nrm2[4 b]); null means no rescaling.
template <typename R>
__device__ __forceinline__ R inv_norm(const double *nrm2, int b) {
    return nrm2 ? (R)(1.0 / sqrt(nrm2[4 * b])) : (R)1;
}

__device__ __forceinline__ float rfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double rfma(double a, double b, double c) { return __builtin_fma(a, b, c); }

typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) f2v g_f2;
typedef const __attribute__((address_space(1))) f4v g_f4;
typedef const __attribute__((address_space(1))) d2v g_d2;

#ifndef HS_TILE_NT
#define HS_TILE_NT 1          // streaming (non-temporal) hint on coefficient and state loads
#endif
#if HS_TILE_NT
#define HS_LOAD(ptr) __builtin_nontemporal_load(ptr)
#else
#define HS_LOAD(ptr) (*(ptr))
#endif

// Single entries (odd offsets: the two rows of a pair read halves of the
// same 16-byte granule, so these loads keep the default cache policy and the
// second one hits in L2).
__device__ __forceinline__ C2<float> ld1(const C2<float> *p, int i) {
    const f2v v = *((g_f2 *)(p) + i);
    return C2<float>{v.x, v.y};
}
__device__ __forceinline__ C2<double> ld1(const C2<double> *p, int i) {
    const d2v v = HS_LOAD((g_d2 *)(p) + i);
    return C2<double>{v.x, v.y};
}
// entries i and i+1 (i even)
__device__ __forceinline__ void ld2(const C2<float> *p, int i, C2<float> &a, C2<float> &b) {
    const f4v v = HS_LOAD((g_f4 *)(p) + (i >> 1));
    a = C2<float>{v.x, v.y};
    b = C2<float>{v.z, v.w};
}
__device__ __forceinline__ void ld2(const C2<double> *p, int i, C2<double> &a, C2<double> &b) {
    a = ld1(p, i);
    b = ld1(p, i + 1);
}

typedef __attribute__((address_space(1))) f4v g_f4w;
typedef __attribute__((address_space(1))) d2v g_d2w;
// one complex128 row of an output state (STREAM: non-temporal)
template <bool STREAM>
__device__ __forceinline__ void st1(C2<double> *p, int i, C2<double> a) {
    const d2v u = {a.re, a.im};
    if (STREAM) __builtin_nontemporal_store(u, (g_d2w *)(p) + i);
    else *((g_d2w *)(p) + i) = u;
}
// rows i and i + 1 (i even) of an output state: one 16-byte store for
// complex64, two for complex128; STREAM streams them past the caches (a
// compile-time choice: with a run-time branch the compiler merges the two
// stores and drops the hint)
template <bool STREAM>
__device__ __forceinline__ void st2(C2<float> *p, int i, C2<float> a, C2<float> b) {
    const f4v v = {a.re, a.im, b.re, b.im};
    if (STREAM) __builtin_nontemporal_store(v, (g_f4w *)(p) + (i >> 1));
    else *((g_f4w *)(p) + (i >> 1)) = v;
}
template <bool STREAM>
__device__ __forceinline__ void st2(C2<double> *p, int i, C2<double> a, C2<double> b) {
    const d2v u = {a.re, a.im}, v = {b.re, b.im};
    if (STREAM) {
        __builtin_nontemporal_store(u, (g_d2w *)(p) + i);
        __builtin_nontemporal_store(v, (g_d2w *)(p) + i + 1);
    } else {
        *((g_d2w *)(p) + i) = u;
        *((g_d2w *)(p) + i + 1) = v;
    }
}

// State rows staged by open launches keep the default cache policy: other
// tiles read them again as out-of-tile partners, and those reads should hit.
__device__ __forceinline__ void ld2_cached(const C2<float> *p, int i, C2<float> &a, C2<float> &b) {
    const f4v v = *((g_f4 *)(p) + (i >> 1));
    a = C2<float>{v.x, v.y};
    b = C2<float>{v.z, v.w};
}
__device__ __forceinline__ C2<float> ld1_cached(const C2<float> *p, int i) { return ld1(p, i); }
__device__ __forceinline__ C2<double> ld1_cached(const C2<double> *p, int i) {
    const d2v u = *((g_d2 *)(p) + i);
    return C2<double>{u.x, u.y};
}
__device__ __forceinline__ void ld2_cached(const C2<double> *p, int i, C2<double> &a, C2<double> &b) {
    const d2v u = *((g_d2 *)(p) + i);
    const d2v v = *((g_d2 *)(p) + i + 1);
    a = C2<double>{u.x, u.y};
    b = C2<double>{v.x, v.y};
}

// A value of a table at a uniform address that the kernel does not write:
// constant memory as far as it goes, so the load is a scalar one.
template <typename V>
__device__ __forceinline__ V uload(const V &p) {
    return *(const __attribute__((address_space(4))) V *)&p;
}

// Where GateBlock::diag keeps the exponential of row x: entry j * (N >> rho) + c
// is element j (its pivot bits) of the coset of the reduced masks `basis`
// whose first row, the pivot bits taken out, is c.
__device__ __forceinline__ int64_t coset_index(uint32_t x, int rho, const uint32_t *basis, int64_t N) {
    uint32_t c = x, j = 0;
    for (int k = 0; k < rho; ++k)
        if ((x >> (31 - __builtin_clz(basis[k]))) & 1u) {
            j |= 1u << k;
            c ^= basis[k];
        }
    for (int k = rho - 1; k >= 0; --k) {
        const int q = 31 - __builtin_clz(basis[k]);
        c = ((c >> q >> 1) << q) | (c & ((1u << q) - 1));
    }
    return (int64_t)j * (N >> rho) + c;
}

// wave64 butterfly sum (fixed order)
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

}  // namespace hs
