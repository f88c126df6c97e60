// HIP kernels for gfx950 (MI355X): factor construction, the DIA tile kernel of
// general operators, the single-diagonal kernel and the FP64 reductions.  A
// product with stored diagonals is bandwidth-bound (about one complex FMA per
// stored coefficient), so nothing here uses MFMA; the kernels are built around
// coalesced 8/16-byte streams along each diagonal, LDS staging of the state
// tile and wave64 shuffle reductions.
#include <hip/hip_runtime.h>

#include <atomic>
#include <mutex>

#include "dev_common.h"
#include "hs_internal.h"
#include "storage_order.h"

namespace hs {

// ------------------------------------------------------------ construction

// E(x) = sum_k c_k (-1)^{popcount(x & z_k)};  out[coset_index(x)] = exp(-i dt E(x)), FP64.
struct PhaseArgs {
    int64_t N;
    int nz, rho;
    const uint64_t *zm;
    const double *cf;
    double dt;
    double *out;
    uint32_t basis[HS_MAX_SUPPORT];
};
__global__ void phase_table_kernel(PhaseArgs a) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < a.N;
         x += (int64_t)gridDim.x * blockDim.x) {
        double E = 0.0;
        for (int k = 0; k < a.nz; ++k) E += a.cf[k] * ((__popcll((uint64_t)x & a.zm[k]) & 1) ? -1.0 : 1.0);
        double s, c;
        sincos(-a.dt * E, &s, &c);
        const int64_t at = coset_index((uint32_t)x, a.rho, a.basis, a.N);
        a.out[2 * at] = c;
        a.out[2 * at + 1] = s;
    }
}

// One diagonal per blockIdx.y.  Entry i of diagonal d sits at row r = i - min(d, 0),
// column p = r + d.  Value: L[loc(r), loc(p)] (times D[p]) when r and p agree
// outside the support, else exactly 0; computed in FP64, stored as R at the
// entry's position in the factor's storage order (perm_pos).
template <typename R>
__global__ void construct_kernel(ConstructArgs a) {
    const int j = blockIdx.y;
    const int64_t d = a.offs[j];
    const int64_t len = (int64_t)a.N - (d < 0 ? -d : d);
    const int64_t neg = d < 0 ? d : 0;
    const int64_t clr = (len >> a.perm_s) << a.perm_c;
    C2<R> *out = reinterpret_cast<C2<R> *>(a.base) + a.elem_off[j];
    const uint64_t outside = ~(uint64_t)a.smask;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < len;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i - neg, p = r + d;
        double vr = 0.0, vi = 0.0;
        if (a.L == nullptr) {
            if (r == p) vr = 1.0;
        } else if ((((uint64_t)(r ^ p)) & outside) == 0) {
            uint32_t la = 0, lb = 0;
            if (a.contiguous) {
                la = (uint32_t)(r >> a.lb) & (uint32_t)(a.K - 1);
                lb = (uint32_t)(p >> a.lb) & (uint32_t)(a.K - 1);
            } else {
                for (int q = 0; q < a.nbits; ++q) {
                    la |= (uint32_t)((r >> a.bits[q]) & 1) << q;
                    lb |= (uint32_t)((p >> a.bits[q]) & 1) << q;
                }
            }
            const int64_t e = (int64_t)la * a.K + lb;
            vr = a.L[2 * e];
            vi = a.L[2 * e + 1];
        }
        if (a.phase && (vr != 0.0 || vi != 0.0)) {
            const int64_t at = coset_index((uint32_t)p, a.rho, a.basis, a.N);
            const C2<double> t = cmul_d(vr, vi, a.phase[2 * at], a.phase[2 * at + 1]);
            vr = t.re;
            vi = t.im;
        }
        out[perm_pos(i, a.perm_s, a.perm_c, clr)] = C2<R>{(R)vr, (R)vi};
    }
}

// dst[k] = entry start + k of a diagonal stored in the order (s, c)
template <typename R>
__global__ void perm_gather_kernel(const C2<R> *__restrict__ src, C2<R> *__restrict__ dst, int64_t start,
                                   int64_t count, int64_t len, int s, int c) {
    const int64_t clr = (len >> s) << c;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * blockDim.x)
        dst[k] = src[perm_pos(start + k, s, c, clr)];
}

// ------------------------------------------------------------ DIA tile kernel
//
// y = A x for an operator given by its stored diagonals, out of place.  A
// workgroup owns one tile of T = 2^kb * W rows:
//   row(i) = hi * 2^(qb+kb) + (i >> logW) * 2^qb + lw * W + (i & (W-1)),
// i.e. all 2^kb "levels" of the bits [qb, qb+kb) times a window of W
// consecutive low rows (contiguous tiles: qb = 0, W = 1, T = 2^kb).
// The state rows of the tile (all B states) are staged once into LDS with
// coalesced loads.  Every row then sums, in ascending-offset order, the stored
// coefficient of each diagonal times the partner amplitude x[r + d]: from LDS
// when the partner row lies in the tile, else from global memory if the
// coefficient is nonzero.  Every stored coefficient is read exactly once, by
// the thread that owns its row, along the diagonal in consecutive addresses.
//
// A thread owns pairs of adjacent rows (local indices i, i+1 with i even;
// a strided tile has an even W and a contiguous one W = 1 with qb = 0, so
// the two rows are adjacent in the state too).  For an
// even offset the two coefficients are adjacent and 16-byte aligned
// (diagonals start on 16-byte boundaries), so complex64 pairs are fetched
// with one 16-byte load; odd offsets use two 8-byte loads.  Loads are issued
// for all pairs of a diagonal before any is consumed, with clamped indices and
// masks instead of branches, so a wave keeps many loads in flight.

template <typename R>
__device__ __forceinline__ C2<R> cmask(C2<R> c, bool keep) {
    return keep ? c : C2<R>{(R)0, (R)0};
}

// Coefficients of one diagonal for every row pair a thread owns (masked
// loads: invalid rows read entry 0 and are zeroed when consumed).
template <typename R, int P, int NT, bool SINGLE = false>
__device__ __forceinline__ void load_diag(C2<R> (&c)[P][2], const DiagDesc &dd, int tid, int T,
                                          int base, int qb, int logW) {
    const C2<R> *cp = reinterpret_cast<const C2<R> *>(dd.ptr);
    const int neg = dd.off < 0 ? dd.off : 0;
    const int len = dd.hi - dd.lo;            // N - |d| entries
    const int W = 1 << logW;
    if constexpr (sizeof(R) == 8) {
        // complex128: the rows of pair p are (2p + k) NT + tid (tile_lidx), one
        // 16-byte load each
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = (2 * p + k) * NT + tid;
                int e = base + ((i >> logW) << qb) + (i & (W - 1)) + neg;
                e = (e >= 0 && e < len && i < T) ? e : 0;
                c[p][k] = ld1(cp, e);
            }
        return;
    }
    // SINGLE: entry-wise loads (a diagonal of odd length ends inside a pair)
    if (!SINGLE && (dd.off & 1) == 0) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int i0 = 2 * tid + 2 * NT * p;
            const int r0 = base + ((i0 >> logW) << qb) + (i0 & (W - 1));
            int e = r0 + neg;
            e = (e >= 0 && e < len && i0 < T) ? e : 0;   // even d: pairs never straddle lo/hi
            ld2(cp, e, c[p][0], c[p][1]);
        }
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int i0 = 2 * tid + 2 * NT * p;
            const int r0 = base + ((i0 >> logW) << qb) + (i0 & (W - 1));
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                int e = r0 + k + neg;
                e = (e >= 0 && e < len && i0 < T) ? e : 0;
                c[p][k] = ld1(cp, e);
            }
        }
    }
}

// HORNER: the output row is x0[r] + alpha * (A x)[r], one Horner stage of a
// polynomial in A applied to a state.
// RAG (contiguous launches only): N need not be a multiple of the tile;
// rows at or past N are neither loaded nor stored.
// STREAM (not with RAG): the output is written with non-temporal stores.
template <typename R, int B, int RPT, bool HORNER, int NT, bool RAG = false, bool STREAM = false>
__global__ __launch_bounds__(NT) void dia_tile_kernel(TileArgs a) {
    static_assert(RPT % 2 == 0, "rows come in pairs");
    constexpr int P = RPT / 2;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C2<R> *lds = reinterpret_cast<C2<R> *>(smem_raw);
    const int T = a.T;
    const int tid = threadIdx.x;
    const int qb = a.qb, kb = a.kb, logW = a.logW;
    const int W = 1 << logW;
    const int L = 1 << kb;
    const int blk = blockIdx.x;
    const int hi = blk >> a.nlw_log;
    const int lw = blk & ((1 << a.nlw_log) - 1);
    const int base = (hi << (qb + kb)) | (lw << logW);
    const C2<R> *x = reinterpret_cast<const C2<R> *>(a.x);
    C2<R> *y = reinterpret_cast<C2<R> *>(a.y);

    // Local index of row k (0 or 1) of the thread's pair p.  complex64: two
    // adjacent rows, i0 = 2 tid + 2 NT p and i0 + 1 (one 16-byte load or store
    // for both); complex128: rows (2p + k) NT + tid, so that each 16-byte
    // load, store and LDS access of a wave covers consecutive addresses
    // (adjacent rows would give every instruction half of each cache line).
    constexpr bool SPLIT = sizeof(R) == 8;
    auto lidx = [&](int p, int k) { return SPLIT ? (2 * p + k) * NT + tid : 2 * tid + 2 * NT * p + k; };
    auto row_of = [&](int i) { return base + ((i >> logW) << qb) + (i & (W - 1)); };

    // stage the tile: issue every load, then write LDS
    {
        C2<R> u[P][2][B];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if constexpr (SPLIT) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int i = lidx(p, k);
                    const int r = i < T ? row_of(i) : base;
#pragma unroll
                    for (int b = 0; b < B; ++b) {
                        if (RAG) u[p][k][b] = r < a.N ? x[b * a.stride + r] : C2<R>{(R)0, (R)0};
                        else u[p][k][b] = ld1_cached(x + b * a.stride, r);
                    }
                }
                continue;
            }
            const int i0 = lidx(p, 0);
            const int r0 = i0 < T ? row_of(i0) : base;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (RAG) {
                    const C2<R> z{(R)0, (R)0};
                    u[p][0][b] = r0 < a.N ? x[b * a.stride + r0] : z;
                    u[p][1][b] = r0 + 1 < a.N ? x[b * a.stride + r0 + 1] : z;
                } else {
                    ld2_cached(x + b * a.stride, r0, u[p][0][b], u[p][1][b]);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = lidx(p, k);
                if (i < T)
#pragma unroll
                    for (int b = 0; b < B; ++b) lds[b * T + i] = u[p][k][b];
            }
    }

    const int total = a.nd;
    C2<R> acc[P][2][B];
    // A row whose partner lies outside the tile gathers it from global memory.  For complex64 launches of one or two states the
    // gathers of G row pairs are issued before any is used (the gathered
    // values take 8 registers), so their latencies overlap; each row still
    // adds its LDS term first and its gathered term second, as the
    // one-row-at-a-time order would.  Other open launches have no registers
    // to spare (open complex128 and larger batches run at the 128-register
    // limit of 1024-thread workgroups) and gather row by row in the loop below.
    constexpr int kGather = sizeof(R) == 8 ? 0 : 8 / (2 * B * 2);
    constexpr int G = kGather >= P ? P : (kGather >= 1 ? kGather : 1);
    auto apply_open = [&](const C2<R> (&cc)[P][2], const DiagDesc &dd) {
#pragma unroll
        for (int g0 = 0; g0 < P; g0 += G) {
            C2<R> gv[G][2][B];
            C2<R> gc[G][2];
            bool gn[G][2];
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const int p = g0 + q;
                const int r0 = row_of(lidx(p, 0));
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int i = lidx(p, k);
                    const int r = SPLIT ? row_of(i) : r0 + k;
                    const bool valid = i < T && r >= dd.lo && r < dd.hi;
                    const C2<R> cv = cmask(cc[p][k], valid);
                    bool in;
                    int loc;
                    if (dd.regular) {
                        const int lvl = (i >> logW) + dd.m;
                        in = (unsigned)lvl < (unsigned)L;
                        loc = i + dd.m * W;
                    } else {
                        const int pr = r + dd.off;
                        in = (pr >> (qb + kb)) == hi && ((pr & ((1 << qb) - 1)) >> logW) == lw;
                        loc = (((pr >> qb) & (L - 1)) << logW) | (pr & (W - 1));
                    }
                    const bool nz = cv.re != (R)0 || cv.im != (R)0;
                    const int sl = in ? loc : (i < T ? i : 0);
                    const C2<R> ce = cmask(cv, in);
#pragma unroll
                    for (int b = 0; b < B; ++b) cfma(acc[p][k][b], ce, lds[b * T + sl]);
                    gn[q][k] = !in && nz;
                    gc[q][k] = cv;
                    if (gn[q][k]) {
                        const int pr = r + dd.off;
#pragma unroll
                        for (int b = 0; b < B; ++b) gv[q][k][b] = x[b * a.stride + pr];
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (gn[q][k])
#pragma unroll
                        for (int b = 0; b < B; ++b)
                            cfma(acc[g0 + q][k][b], gc[q][k], gv[q][k][b]);
        }
    };

    // the next diagonal's coefficients are loaded once this one's are used
    C2<R> c[P][2];
    load_diag<R, P, NT, RAG>(c, a.desc[0], tid, T, base, qb, logW);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int b = 0; b < B; ++b) acc[p][k][b] = C2<R>{(R)0, (R)0};
    for (int dj = 0; dj < total; ++dj) {
        const DiagDesc dd = a.desc[dj];
        if constexpr (kGather > 0) {
            apply_open(c, dd);
        } else {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int r0 = row_of(lidx(p, 0));
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int i = lidx(p, k);
                    const int r = SPLIT ? row_of(i) : r0 + k;
                    const bool valid = i < T && r >= dd.lo && r < dd.hi;
                    const C2<R> cv = cmask(c[p][k], valid);
                    bool in;
                    int loc;
                    if (dd.regular) {
                        const int lvl = (i >> logW) + dd.m;
                        in = (unsigned)lvl < (unsigned)L;
                        loc = i + dd.m * W;
                    } else {
                        const int pr = r + dd.off;
                        in = (pr >> (qb + kb)) == hi && ((pr & ((1 << qb) - 1)) >> logW) == lw;
                        loc = (((pr >> qb) & (L - 1)) << logW) | (pr & (W - 1));
                    }
                    const bool nz = cv.re != (R)0 || cv.im != (R)0;
                    const int sl = in ? loc : (i < T ? i : 0);
                    const C2<R> ce = cmask(cv, in);
#pragma unroll
                    for (int b = 0; b < B; ++b) cfma(acc[p][k][b], ce, lds[b * T + sl]);
                    if (!in && nz) {
                        const int pr = r + dd.off;
#pragma unroll
                        for (int b = 0; b < B; ++b) cfma(acc[p][k][b], cv, x[b * a.stride + pr]);
                    }
                }
            }
        }
        if (dj + 1 < total) load_diag<R, P, NT, RAG>(c, a.desc[dj + 1], tid, T, base, qb, logW);
    }

    if (HORNER) {
        const C2<R> *x0 = reinterpret_cast<const C2<R> *>(a.x0);
        const C2<R> al{(R)a.alpha_re, (R)a.alpha_im};
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int i0 = lidx(p, 0), i1 = lidx(p, 1);
            const int r0 = i0 < T ? row_of(i0) : base;
            const int r1 = SPLIT ? (i1 < T ? row_of(i1) : base) : r0 + 1;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                C2<R> v0, v1;
                if (RAG) {
                    const C2<R> z{(R)0, (R)0};
                    v0 = r0 < a.N ? x0[b * a.stride + r0] : z;
                    v1 = r1 < a.N ? x0[b * a.stride + r1] : z;
                } else if (SPLIT) {
                    v0 = ld1(x0 + b * a.stride, r0);
                    v1 = ld1(x0 + b * a.stride, r1);
                } else {
                    ld2(x0 + b * a.stride, r0, v0, v1);
                }
                cfma(v0, al, acc[p][0][b]);
                cfma(v1, al, acc[p][1][b]);
                acc[p][0][b] = v0;
                acc[p][1][b] = v1;
            }
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if constexpr (SPLIT) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = lidx(p, k);
                if (i < T) {
                    const int r = row_of(i);
#pragma unroll
                    for (int b = 0; b < B; ++b) {
                        if (!RAG) st1<STREAM>(y + b * a.stride, r, acc[p][k][b]);
                        else if (r < a.N) y[b * a.stride + r] = acc[p][k][b];
                    }
                }
            }
            continue;
        }
        const int i0 = lidx(p, 0);
        if (i0 < T) {
            const int r0 = row_of(i0);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (!RAG) {
                    st2<STREAM>(y + b * a.stride, r0, acc[p][0][b], acc[p][1][b]);
                } else {
                    if (r0 < a.N) y[b * a.stride + r0] = acc[p][0][b];
                    if (r0 + 1 < a.N) y[b * a.stride + r0 + 1] = acc[p][1][b];
                }
            }
        }
    }
}

// ------------------------------------------------------------ DIA row kernel
//
// The same product for operators too small to give every compute unit a tile:
// one thread per row and state, partners read from cache, the coefficients and
// partners of kRowsAhead diagonals loaded before any is used.  The sum runs in
// the same order with the same multiply-adds, so the values are the same.  A
// sum that is not finite is taken again without its zero coefficients
// (nonzero_row), so that an infinite amplitude reaches the rows coupled to it
// and no others.
//
// What bounds it: a handful of waves issuing one after the other, so the inner
// loop is kept to two loads and the multiply-adds per diagonal: buffer loads
// give the range checks, descriptors come through scalar loads a round ahead.
// N = 1024 complex128: 21 diagonals 4.1 us, 61 diagonals 5.5 us per product
// (8 ahead: 3.8 and 6.0 us; with masks and 64-bit addresses 5.9 and 12.7 us;
// one workgroup's tile walking the diagonals: 14.7 us for 21).
constexpr int kRowsAhead = 16;
constexpr int kRowsThreads = 64;
// rows x states up to which it is the faster: 65536 rows of 4 complex64 states
// 10 against 25 us, 2^18 rows of one 13 against 25 us, 2^18 rows of 3
// complex128 states 99 against 65 us (every state reads the coefficients again)
constexpr int64_t kRowsMax = int64_t(1) << 18;

// Buffer loads of entry i of a diagonal or state of `n` entries: an index
// outside [0, n) reads zero, so a row without a partner needs no mask.
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
typedef unsigned int u2v __attribute__((ext_vector_type(2)));
constexpr int kRawBuffer = 0x00020000;           // data format of a raw buffer
template <typename R>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, int n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, n * (int)sizeof(C2<R>), kRawBuffer);
}
__device__ __forceinline__ void buffer_get(__amdgpu_buffer_rsrc_t b, int i, C2<double> &v) {
    const u4v w = __builtin_amdgcn_raw_buffer_load_b128(b, i * 16, 0, 0);
    __builtin_memcpy(&v, &w, 16);
}
__device__ __forceinline__ void buffer_get(__amdgpu_buffer_rsrc_t b, int i, C2<float> &v) {
    const u2v w = __builtin_amdgcn_raw_buffer_load_b64(b, i * 8, 0, 0);
    __builtin_memcpy(&v, &w, 8);
}

// Row r of A x over the nonzero coefficients alone: diagonal j has the offset
// off(j) and the entries ptr(j), x(p) is amplitude p.
template <typename R, typename FO, typename FP, typename FX>
__device__ __forceinline__ C2<R> nonzero_row(int r, int N, int nd, FO off, FP ptr, FX x) {
    C2<R> acc{(R)0, (R)0};
#pragma unroll 1
    for (int j = 0; j < nd; ++j) {
        const int d = off(j);
        if (r + d < 0 || r + d >= N) continue;
        const C2<R> c = ld1_cached(reinterpret_cast<const C2<R> *>(ptr(j)), r + (d < 0 ? d : 0));
        if (c.re != (R)0 || c.im != (R)0) cfma(acc, c, x(r + d));
    }
    return acc;
}

template <typename R, bool HORNER>
__global__ __launch_bounds__(kRowsThreads) void dia_rows_kernel(TileArgs a) {
    const int r = blockIdx.x * kRowsThreads + threadIdx.x;
    const C2<R> *x = reinterpret_cast<const C2<R> *>(a.x) + (int64_t)blockIdx.y * a.stride;
    const int N = a.N, nd = a.nd;
    const __amdgpu_buffer_rsrc_t xb = buffer_of<R>(x, N);
    // descriptors, read through scalar loads one round ahead
    const void *ptr[kRowsAhead];
    int off[kRowsAhead];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int u = 0; u < kRowsAhead; ++u) {
            const DiagDesc &dd = a.desc[j0 + u < nd ? j0 + u : nd - 1];
            ptr[u] = uload(dd.ptr);
            off[u] = uload(dd.off);
        }
    };
    C2<R> acc{(R)0, (R)0};
    fetch(0);
    for (int j0 = 0; j0 < nd; j0 += kRowsAhead) {
        C2<R> c[kRowsAhead], v[kRowsAhead];
#pragma unroll
        for (int u = 0; u < kRowsAhead; ++u) {
            const int d = off[u];
            // past the last diagonal: no entries
            const int len = j0 + u < nd ? N - (d < 0 ? -d : d) : 0;
            buffer_get(buffer_of<R>(ptr[u], len), r + (d < 0 ? d : 0), c[u]);
            buffer_get(xb, r + d, v[u]);
        }
        if (j0 + kRowsAhead < nd) fetch(j0 + kRowsAhead);
#pragma unroll
        for (int u = 0; u < kRowsAhead; ++u) cfma(acc, c[u], v[u]);
    }
    if (r >= N) return;
    if (!finite(acc))
        acc = nonzero_row<R>(
            r, N, nd, [&](int j) { return uload(a.desc[j].off); }, [&](int j) { return uload(a.desc[j].ptr); },
            [&](int p) { return ld1_cached(x, p); });
    if (HORNER) {
        C2<R> y = reinterpret_cast<const C2<R> *>(a.x0)[(int64_t)blockIdx.y * a.stride + r];
        cfma(y, C2<R>{(R)a.alpha_re, (R)a.alpha_im}, acc);
        acc = y;
    }
    reinterpret_cast<C2<R> *>(a.y)[(int64_t)blockIdx.y * a.stride + r] = acc;
}

// ------------------------------------------------------------ DIA loop kernel
//
// All steps x <- A x of a small operator in one launch: a workgroup per state
// keeps the state in LDS and every coefficient of its rows in registers (24
// complex128 diagonals are 96 of the 128 VGPRs of one of 1024 threads, 48 are
// 192 of 256 of one of 512), so a step is one LDS read and the multiply-adds
// per diagonal and two barriers.  Zeros on both sides of the state stand for
// partners outside it.  The sum runs in the order and with the multiply-adds
// of the row kernel, and the steps are taken again as there when a sum is not
// finite, so the values are the same.
//
// What bounds it: the LDS reads, 16 KiB per diagonal and step of 1024 complex128
// rows.  A step of 21 diagonals there takes 1.17 us where a launch of the row
// kernel per step takes 4.1 (17 diagonals at N = 256: 0.59 us; 600 states 3.7
// us); 48 diagonals at N = 512 take 1.29 against 4.1 us.  512 threads of twice
// the rows for 21 diagonals: 1.30 us.
template <typename R>
constexpr int kLoopRowsPer = sizeof(R) == 8 ? 1 : 2;         // rows of a thread
template <typename R>
constexpr int kLoopRows = 1024 * kLoopRowsPer<R>;            // 48 KiB of LDS with the zeros

template <typename R, int ND, int NT>
__global__ __launch_bounds__(NT) void dia_loop_kernel(LoopArgs a) {
    constexpr int E = kLoopRowsPer<R>;
    __shared__ C2<R> lds[3 * E * NT];                        // zeros, the state, zeros
    __shared__ int again;                                    // some sum is not finite
    const int N = a.N, nt = blockDim.x, tid = threadIdx.x;
    if (tid == 0) again = 0;
    C2<R> *x = reinterpret_cast<C2<R> *>(a.x) + (int64_t)blockIdx.x * N;
    for (int i = tid; i < 3 * N; i += nt) lds[i] = i >= N && i < 2 * N ? x[i - N] : C2<R>{(R)0, (R)0};
    C2<R> c[ND][E];
#pragma unroll
    for (int j = 0; j < ND; ++j) {
        const int d = a.off[j];                              // past the last diagonal: 0, no entries
        const int len = j < a.nd ? N - (d < 0 ? -d : d) : 0;
        const __amdgpu_buffer_rsrc_t cb = buffer_of<R>(a.ptr[j], len);
#pragma unroll
        for (int e = 0; e < E; ++e) buffer_get(cb, tid + e * nt + (d < 0 ? d : 0), c[j][e]);
    }
    // a thread past the last row reads row N - 1's partners and writes nothing
    int row[E];
#pragma unroll
    for (int e = 0; e < E; ++e) row[e] = N + (tid + e * nt < N ? tid + e * nt : N - 1);
    __syncthreads();
    for (int s = 0; s < a.steps; ++s) {
        C2<R> acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            acc[e] = C2<R>{(R)0, (R)0};
            asm volatile("" : "+v"(row[e]));                 // keeps ND * E addresses out of the registers
        }
#pragma unroll
        for (int j = 0; j < ND; ++j) {
#pragma unroll
            for (int e = 0; e < E; ++e) cfma(acc[e], c[j][e], lds[row[e] + a.off[j]]);
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // four diagonals' partners in flight
        }
#pragma unroll
        for (int e = 0; e < E; ++e) asm volatile("" : "+v"(acc[e].re), "+v"(acc[e].im));   // sums end here, not below
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (tid + e * nt < N) lds[row[e]] = acc[e];
        __syncthreads();
    }
    // an amplitude that is not finite makes every row whose diagonals reach it
    // so, down to the last step: the steps again, from x, if any is left
    bool bad = false;
#pragma unroll
    for (int e = 0; e < E; ++e) bad = bad || !finite(lds[row[e]]);
    if (bad) again = 1;
    __syncthreads();
    if (again) {
        for (int i = tid; i < N; i += nt) lds[N + i] = x[i];
        __syncthreads();
#pragma unroll 1
        for (int s = 0; s < a.steps; ++s) {
            C2<R> acc[E];
#pragma unroll
            for (int e = 0; e < E; ++e)
                acc[e] = nonzero_row<R>(
                    row[e] - N, N, a.nd, [&](int j) { return a.off[j]; }, [&](int j) { return a.ptr[j]; },
                    [&](int p) { return lds[N + p]; });
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (tid + e * nt < N) lds[row[e]] = acc[e];
            __syncthreads();
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (tid + e * nt < N) x[tid + e * nt] = lds[row[e]];
}

// Single main-diagonal factor applied `steps` times: y[i] = v[i]^steps x[i]
// for N even, each thread two adjacent entries (one 16-byte load of the
// coefficients and of each state for complex64), the powers taken as
// `steps` successive complex multiplications in registers in the order of
// one step at a time, so the result equals `steps` single-step passes bit
// for bit while the diagonal and the states cross HBM once.  In place
// allowed.  STREAM: non-temporal output stores.  nrm2 is null in every present
// call; the product by 1 that it leaves holds the coefficients' load back until
// the state has arrived, without which a pass over 2^26 complex64 rows takes
// 0.287 instead of 0.263 ms.
template <typename R, int B, bool STREAM>
__global__ __launch_bounds__(256) void diag_steps_kernel(C2<R> *y, const C2<R> *x, const C2<R> *__restrict__ v,
                                                         int64_t N, int steps, const double *nrm2) {
    R scale[B];
#pragma unroll
    for (int b = 0; b < B; ++b) scale[b] = inv_norm<R>(nrm2, b);
    const int64_t npairs = N >> 1;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < npairs;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(2 * q);
        C2<R> c0, c1;
        ld2(v, i, c0, c1);
        C2<R> u[B][2];
#pragma unroll
        for (int b = 0; b < B; ++b) ld2(x + b * N, i, u[b][0], u[b][1]);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            C2<R> a0 = cscale(u[b][0], scale[b]), a1 = cscale(u[b][1], scale[b]);
            for (int s = 0; s < steps; ++s) {
                C2<R> t0{(R)0, (R)0}, t1{(R)0, (R)0};
                cfma(t0, c0, a0);
                cfma(t1, c1, a1);
                a0 = t0;
                a1 = t1;
            }
            st2<STREAM>(y + b * N, i, a0, a1);
        }
    }
}

template <typename R>
__global__ void scale_kernel(C2<R> *psi, int64_t N, const double *nrm2) {
    const int b = blockIdx.y;
    const R s = inv_norm<R>(nrm2, b);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x)
        psi[b * N + i] = cscale(psi[b * N + i], s);
}

// ------------------------------------------------------------ reductions
// Pass 1: block g of state b sums elements g*256+t, stepping by G*256, in
// FP64; wave64 butterfly, then the four waves in fixed order.  Pass 2: one
// block per state sums the G partials in a fixed tree.  No atomics, so the
// result is bit-reproducible.
//
// What bounds it: HBM for states beyond the last-level cache, which are read
// with streaming loads (n = 24, a complex64 against a complex128 pair of
// states, 768 MiB: 120 us = 6.7 TB/s in the kernel, 167 us a call; through the
// caches 186 us a call).  A norm of complex64 states has one stream of 8-byte
// loads per thread and few waves for a lone state, so it keeps four in flight
// (n = 26 181 -> 124 us a call); with 16-byte loads four are slower (n = 25,
// two complex128 states 233 against 200 us), as are the overlap's two streams
// (182 against 190).

// One amplitude through a streaming load (STREAM) or the caches; callers' states
// are aligned to their real type only.
template <bool STREAM>
__device__ __forceinline__ C2<float> ld_state(const C2<float> *p) {
    typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
    typedef const __attribute__((address_space(1))) f2u g_f2u;
    const f2u v = STREAM ? __builtin_nontemporal_load((g_f2u *)p) : *(g_f2u *)p;
    return C2<float>{v.x, v.y};
}
template <bool STREAM>
__device__ __forceinline__ C2<double> ld_state(const C2<double> *p) {
    typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
    typedef const __attribute__((address_space(1))) d2u g_d2u;
    const d2u v = STREAM ? __builtin_nontemporal_load((g_d2u *)p) : *(g_d2u *)p;
    return C2<double>{v.x, v.y};
}

template <typename TA, typename TB, bool DOT, bool STREAM>
__global__ __launch_bounds__(256) void reduce_partial_kernel(const void *A, const void *Bv, int64_t N,
                                                             int G, double *partial) {
    const int b = blockIdx.y;
    const C2<TA> *pa = reinterpret_cast<const C2<TA> *>(A) + b * N;
    const C2<TB> *pb = reinterpret_cast<const C2<TB> *>(Bv) + b * N;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t step = (int64_t)G * 256;
    int64_t i = blockIdx.x * 256 + threadIdx.x;
    if (!DOT && sizeof(TA) == 4)                             // complex64 norms: four loads in flight
        for (; i + 3 * step < N; i += 4 * step) {
            C2<TA> u[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = ld_state<STREAM>(pa + i + k * step);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double ar = (double)u[k].re, ai = (double)u[k].im;
                s[2] += ar * ar + ai * ai;
            }
        }
    for (; i < N; i += step) {
        const C2<TA> u = ld_state<STREAM>(pa + i);
        const double ar = (double)u.re, ai = (double)u.im;
        s[2] += ar * ar + ai * ai;
        if (DOT) {
            const C2<TB> w = ld_state<STREAM>(pb + i);
            const double br = (double)w.re, bi = (double)w.im;
            s[0] += ar * br + ai * bi;
            s[1] += ar * bi - ai * br;
            s[3] += br * br + bi * bi;
        }
    }
    __shared__ double red[4][4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double v = wave_sum(s[k]);
        if (lane == 0) red[wave][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        partial[((int64_t)b * G + blockIdx.x) * 4 + k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
}

__global__ __launch_bounds__(256) void reduce_final_kernel(const double *partial, int G, double *out) {
    const int b = blockIdx.x;
    __shared__ double red[256][4];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int g = threadIdx.x; g < G; g += 256)
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] += partial[((int64_t)b * G + g) * 4 + k];
#pragma unroll
    for (int k = 0; k < 4; ++k) red[threadIdx.x][k] = s[k];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int k = 0; k < 4; ++k) red[threadIdx.x][k] += red[threadIdx.x + w][k];
        __syncthreads();
    }
    if (threadIdx.x < 4) out[b * 4 + threadIdx.x] = red[0][threadIdx.x];
}

// Fidelity records: out[b] = (Re, Im <phi|psi>, <phi|phi>, <psi|psi>, F) from
// the reduction records, F = (Re^2 + Im^2) / (<phi|phi> <psi|psi>) evaluated
// as separate roundings (no fused multiply-add), as the host evaluates it.
__global__ void fidelity_records_kernel(const double *rec, int batch, double *out) {
#pragma clang fp contract(off)
    const int b = threadIdx.x;
    if (b < batch) {
        const double re = rec[4 * b], im = rec[4 * b + 1], np = rec[4 * b + 2], nq = rec[4 * b + 3];
        out[5 * b + 0] = re;
        out[5 * b + 1] = im;
        out[5 * b + 2] = np;
        out[5 * b + 3] = nq;
        out[5 * b + 4] = (re * re + im * im) / (np * nq);
    }
}

// ------------------------------------------------------------ launchers

static inline hipStream_t S(void *s) { return reinterpret_cast<hipStream_t>(s); }

static inline int grid_for(int64_t n, int per_block, int cap) {
    int64_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

int launch_phase_table(int64_t N, int nz, const uint64_t *zm, const double *cf, double dt,
                       const std::vector<uint64_t> &basis, double *out, void *stream) {
    if (basis.size() > HS_MAX_SUPPORT) return (int)hipErrorInvalidValue;
    PhaseArgs a{};
    a.N = N;
    a.nz = nz;
    a.rho = (int)basis.size();
    a.zm = zm;
    a.cf = cf;
    a.dt = dt;
    a.out = out;
    for (size_t k = 0; k < basis.size(); ++k) a.basis[k] = (uint32_t)basis[k];
    hipLaunchKernelGGL(phase_table_kernel, dim3(grid_for(N, 256, 1 << 20)), dim3(256), 0, S(stream), a);
    return (int)hipGetLastError();
}

int launch_construct(const ConstructArgs &a, int nd, int64_t max_len, bool c128, void *stream) {
    dim3 grid(grid_for(max_len, 256, 1 << 16), nd);
    if (c128)
        hipLaunchKernelGGL(construct_kernel<double>, grid, dim3(256), 0, S(stream), a);
    else
        hipLaunchKernelGGL(construct_kernel<float>, grid, dim3(256), 0, S(stream), a);
    return (int)hipGetLastError();
}

int launch_perm_gather(const void *src, void *dst, int64_t start, int64_t count, int64_t len, int s, int c,
                       bool c128, void *stream) {
    if (count <= 0) return 0;
    if (start < 0 || start + count > len || s < c || c < 0 || s > 30) return (int)hipErrorInvalidValue;
    const int g = grid_for(count, 256, 1 << 16);
    if (c128)
        hipLaunchKernelGGL(perm_gather_kernel<double>, dim3(g), dim3(256), 0, S(stream),
                           static_cast<const C2<double> *>(src), static_cast<C2<double> *>(dst), start, count, len,
                           s, c);
    else
        hipLaunchKernelGGL(perm_gather_kernel<float>, dim3(g), dim3(256), 0, S(stream),
                           static_cast<const C2<float> *>(src), static_cast<C2<float> *>(dst), start, count, len, s,
                           c);
    return (int)hipGetLastError();
}

static std::mutex &lds_attr_mutex() {
    static std::mutex m;
    return m;
}

// Launch with the smallest rows-per-thread instantiation (power of two, down
// to one row pair) that still gives every tile row a thread: a tile smaller
// than the kernel's capacity would otherwise issue masked loads and FMAs.
template <typename R, int B, int RPT, bool HORNER, int NT, bool RAG = false, bool STREAM = false>
static int tile_launch(const TileArgs &a, int rows_per_thread, size_t lds, int grid, void *stream) {
    if constexpr (RPT > 2) {
        if (rows_per_thread <= RPT / 2)
            return tile_launch<R, B, RPT / 2, HORNER, NT, RAG, STREAM>(a, rows_per_thread, lds, grid, stream);
    }
    auto kern = dia_tile_kernel<R, B, RPT, HORNER, NT, RAG, STREAM>;
    if (lds > 65536) {
        // allow this instantiation the dynamic LDS the launch needs (raised
        // only when a larger launch arrives; the planner keeps lds within the
        // device's per-workgroup limit)
        static std::atomic<int> allowed{65536};
        int cur = allowed.load();
        while ((int)lds > cur) {
            std::lock_guard<std::mutex> lock(lds_attr_mutex());
            cur = allowed.load();
            if ((int)lds <= cur) break;
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return (int)e;
            allowed.store((int)lds);
            cur = (int)lds;
        }
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, S(stream), a);
    return (int)hipGetLastError();
}

template <typename R, int B>
static int tile_dispatch_b(const TileArgs &a, bool horner, void *stream) {
    constexpr bool c128 = sizeof(R) == 8;
    constexpr int RPT = tile_rpt(c128, B, true);
    constexpr int NT = tile_threads(c128, B, true);
    const size_t lds = (size_t)a.T * B * sizeof(C2<R>);
    // every tile row must belong to a thread, and the tile must fit the LDS
    // budget; only contiguous launches may end in a partial tile
    if (a.T < 2 || a.T > NT * RPT || lds > (size_t)tile_lds_bytes(c128, B, true)) return (int)hipErrorInvalidValue;
    // a thread's row pair must be adjacent state rows: strided tiles need W >= 2
    if (a.qb != 0 && a.logW < 1) return (int)hipErrorInvalidValue;
    const bool rag = a.ragged != 0;
    if ((a.N % a.T != 0) != rag) return (int)hipErrorInvalidValue;
    if (rag && (a.qb != 0 || a.logW != 0 || a.nlw_log != 0)) return (int)hipErrorInvalidValue;
    const int grid = (int)((a.N + a.T - 1) / a.T);
    const int need = (a.T + NT - 1) / NT;
    const bool st = a.stream_out != 0;         // ragged launches keep plain stores
    if (!horner)
        return rag  ? tile_launch<R, B, RPT, false, NT, true>(a, need, lds, grid, stream)
               : st ? tile_launch<R, B, RPT, false, NT, false, true>(a, need, lds, grid, stream)
                    : tile_launch<R, B, RPT, false, NT>(a, need, lds, grid, stream);
    return rag  ? tile_launch<R, B, RPT, true, NT, true>(a, need, lds, grid, stream)
           : st ? tile_launch<R, B, RPT, true, NT, false, true>(a, need, lds, grid, stream)
                : tile_launch<R, B, RPT, true, NT>(a, need, lds, grid, stream);
}

template <typename R>
static int tile_dispatch(const TileArgs &a, int batch, bool horner, void *stream) {
    switch (batch) {
        case 1: return tile_dispatch_b<R, 1>(a, horner, stream);
        case 2: return tile_dispatch_b<R, 2>(a, horner, stream);
        case 3: return tile_dispatch_b<R, 3>(a, horner, stream);
        case 4: return tile_dispatch_b<R, 4>(a, horner, stream);
        case 5: return tile_dispatch_b<R, 5>(a, horner, stream);
        case 6: return tile_dispatch_b<R, 6>(a, horner, stream);
        case 7: return tile_dispatch_b<R, 7>(a, horner, stream);
        case 8: return tile_dispatch_b<R, 8>(a, horner, stream);
        default: return (int)hipErrorInvalidValue;
    }
}

template <typename R>
static int rows_launch(const TileArgs &a, int batch, bool horner, void *stream) {
    const dim3 g((a.N + kRowsThreads - 1) / kRowsThreads, batch);
    if (horner) hipLaunchKernelGGL((dia_rows_kernel<R, true>), g, dim3(kRowsThreads), 0, S(stream), a);
    else hipLaunchKernelGGL((dia_rows_kernel<R, false>), g, dim3(kRowsThreads), 0, S(stream), a);
    return (int)hipGetLastError();
}

template <typename R>
static int product_launch(const TileArgs &a, int batch, bool horner, void *stream) {
    if (a.nd < 1) return (int)hipErrorInvalidValue;      // both kernels read a first descriptor
    if ((int64_t)a.N * batch <= kRowsMax) return rows_launch<R>(a, batch, horner, stream);
    return tile_dispatch<R>(a, batch, horner, stream);
}

int launch_tile(const TileArgs &a, int batch, bool c128, void *stream) {
    return c128 ? product_launch<double>(a, batch, false, stream) : product_launch<float>(a, batch, false, stream);
}

bool loop_fits(int64_t N, int nd, bool c128) {
    const int64_t rows = c128 ? kLoopRows<double> : kLoopRows<float>;
    return nd >= 1 && (nd <= kLoopDiags / 2 ? N <= rows : nd <= kLoopDiags && N <= rows / 2);
}

template <typename R>
static int loop_launch(const LoopArgs &a, int batch, void *stream) {
    const int nt = ((a.N + kLoopRowsPer<R> - 1) / kLoopRowsPer<R> + 63) / 64 * 64;
    auto k = a.nd <= 8                ? dia_loop_kernel<R, 8, 1024>
             : a.nd <= 16             ? dia_loop_kernel<R, 16, 1024>
             : a.nd <= kLoopDiags / 2 ? dia_loop_kernel<R, kLoopDiags / 2, 1024>
                                      : dia_loop_kernel<R, kLoopDiags, 512>;
    hipLaunchKernelGGL(k, dim3(batch), dim3(nt), 0, S(stream), a);
    return (int)hipGetLastError();
}

int launch_loop(const LoopArgs &a, int batch, bool c128, void *stream) {
    if (!loop_fits(a.N, a.nd, c128) || a.N < 1 || batch < 1) return (int)hipErrorInvalidValue;
    return c128 ? loop_launch<double>(a, batch, stream) : loop_launch<float>(a, batch, stream);
}

int launch_tile_horner(const TileArgs &a, int batch, bool c128, void *stream) {
    if (!a.x0) return (int)hipErrorInvalidValue;
    return c128 ? product_launch<double>(a, batch, true, stream) : product_launch<float>(a, batch, true, stream);
}

template <typename R, bool STREAM>
static int diag_steps_dispatch(void *y, const void *x, const void *v, int64_t N, int batch, int steps,
                               const double *nrm2, void *stream) {
    C2<R> *py = reinterpret_cast<C2<R> *>(y);
    const C2<R> *px = reinterpret_cast<const C2<R> *>(x);
    const C2<R> *pv = reinterpret_cast<const C2<R> *>(v);
    const dim3 g(grid_for(N >> 1, 256, 1 << 20)), blk(256);
    switch (batch) {
#define HS_DSTEP_CASE(BB) \
    case BB: hipLaunchKernelGGL((diag_steps_kernel<R, BB, STREAM>), g, blk, 0, S(stream), py, px, pv, N, steps, nrm2); break;
        HS_DSTEP_CASE(1) HS_DSTEP_CASE(2) HS_DSTEP_CASE(3) HS_DSTEP_CASE(4)
        HS_DSTEP_CASE(5) HS_DSTEP_CASE(6) HS_DSTEP_CASE(7) HS_DSTEP_CASE(8)
#undef HS_DSTEP_CASE
        default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

int launch_diag_steps(void *y, const void *x, const void *diag, int64_t N, int batch, int steps,
                      const double *nrm2, bool c128, bool stream_out, void *stream) {
    if (N < 2 || (N & 1) || steps < 1) return (int)hipErrorInvalidValue;
    if (c128)
        return stream_out ? diag_steps_dispatch<double, true>(y, x, diag, N, batch, steps, nrm2, stream)
                          : diag_steps_dispatch<double, false>(y, x, diag, N, batch, steps, nrm2, stream);
    return stream_out ? diag_steps_dispatch<float, true>(y, x, diag, N, batch, steps, nrm2, stream)
                      : diag_steps_dispatch<float, false>(y, x, diag, N, batch, steps, nrm2, stream);
}

int launch_scale(void *psi, int64_t N, int batch, const double *nrm2, bool c128, void *stream) {
    dim3 g(grid_for(N, 256, 1 << 14), batch);
    if (c128)
        hipLaunchKernelGGL(scale_kernel<double>, g, dim3(256), 0, S(stream),
                           reinterpret_cast<C2<double> *>(psi), N, nrm2);
    else
        hipLaunchKernelGGL(scale_kernel<float>, g, dim3(256), 0, S(stream),
                           reinterpret_cast<C2<float> *>(psi), N, nrm2);
    return (int)hipGetLastError();
}

// Bytes of a reduction's states above which they are read past the caches: at
// 256 MiB (the last-level cache) streaming is slower, 92 against 84 us a call
// for two complex64 states of 2^24 rows, at 384 MiB faster, 107 against 116 us.
static constexpr size_t kReduceStream = size_t(256) << 20;

template <typename TA, typename TB, bool DOT>
static void reduce_partials(const void *A, const void *Bv, int batch, int64_t N, int G, double *partial, void *stream) {
    const size_t bytes = (size_t)batch * N * 2 * (sizeof(TA) + (DOT ? sizeof(TB) : 0));
    auto k = bytes > kReduceStream ? reduce_partial_kernel<TA, TB, DOT, true> : reduce_partial_kernel<TA, TB, DOT, false>;
    hipLaunchKernelGGL(k, dim3(G, batch), dim3(256), 0, S(stream), A, Bv, N, G, partial);
}

int launch_reduce(const void *A, int ta, const void *Bv, int tb, int batch, int64_t N,
                  double *partial, int G, double *out, bool dot, void *stream) {
    if (!dot) {
        if (ta == HS_C128) reduce_partials<double, double, false>(A, A, batch, N, G, partial, stream);
        else reduce_partials<float, float, false>(A, A, batch, N, G, partial, stream);
    } else {
        if (ta == HS_C128 && tb == HS_C128) reduce_partials<double, double, true>(A, Bv, batch, N, G, partial, stream);
        else if (ta == HS_C128) reduce_partials<double, float, true>(A, Bv, batch, N, G, partial, stream);
        else if (tb == HS_C128) reduce_partials<float, double, true>(A, Bv, batch, N, G, partial, stream);
        else reduce_partials<float, float, true>(A, Bv, batch, N, G, partial, stream);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL(reduce_final_kernel, dim3(batch), dim3(256), 0, S(stream), partial, G, out);
    return (int)hipGetLastError();
}

int launch_fidelity_records(const double *rec, int batch, double *out, void *stream) {
    hipLaunchKernelGGL(fidelity_records_kernel, dim3(1), dim3(64), 0, S(stream), rec, batch, out);
    return (int)hipGetLastError();
}

int launch_reduce_partials(const double *partial, int G, int batch, double *out, void *stream) {
    hipLaunchKernelGGL(reduce_final_kernel, dim3(batch), dim3(256), 0, S(stream), partial, G, out);
    return (int)hipGetLastError();
}

}  // namespace hs
