// One Horner stage y = x0 + alpha (H x) of an operator known as a Pauli sum,
// without its stored off-diagonals.
//
// Strings that flip the same bits m couple row r with the one row r ^ m, by a
// coefficient that a few parities of r select from a table (pauli_form.h), so
// a stage reads the state, the main diagonal and x0 and writes y.  The stored
// form (Eq. 6) has two diagonals per flipped qubit, each N - 2^q entries, half
// of them zero.
//
// A workgroup owns a tile of consecutive rows in LDS.  Partners inside the
// tile come from LDS; a mask with higher bits pairs the tile with another
// whole tile, whose rows are read from cache in 16-byte accesses, one mask
// ahead of their use.
//
// What bounds it: those partner reads.  At n = 23 (complex64 chain) a stage
// takes 104 us: 268 MB that it cannot do without and 12 partner tiles per
// tile, 0.8 GB, from the caches; the stored diagonals took 545 us.  Measured
// there: 8192-row tiles 237 us (113 registers spilled), 4096 rows 111 us,
// 1024-thread workgroups 110 us; contiguous eighths of the tiles per XCD 116
// us (the hardware's order keeps partners 8, 16, 32 tiles away on one XCD).
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "hs_internal.h"
#include "pauli_form.h"

namespace hs {

// A mask's record in scalar registers; add() is acc += coefficient(row r) v.
template <typename R>
struct MaskRec {
    uint32_t m, z0;
    int rank, tab;
    C2<R> c0, c1;
    __device__ __forceinline__ MaskRec() {}
    __device__ __forceinline__ explicit MaskRec(const PauliMask &k) {
        m = uload(k.m);
        rank = uload(k.rank);
        tab = uload(k.tab);
        z0 = uload(k.z0);
        const R *c = reinterpret_cast<const R *>(k.c);
        c0 = C2<R>{uload(c[0]), uload(c[1])};
        c1 = C2<R>{uload(c[2]), uload(c[3])};
    }
    // ROW: the row index of element e, VAL: its partner's amplitude
    template <int E, typename FR, typename FV>
    __device__ __forceinline__ void add(C2<R> (&acc)[E], const PauliMask &k, const C2<R> *table, FR row, FV val) const {
        if (rank == 0 && c0.im == (R)0) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const C2<R> v = val(e);
                acc[e].re = rfma(c0.re, v.re, acc[e].re);
                acc[e].im = rfma(c0.re, v.im, acc[e].im);
            }
        } else if (rank <= 1) {
            const uint32_t z = rank ? z0 : 0;
            if (c0.im == (R)0 && c1.im == (R)0) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const C2<R> v = val(e);
                    const R c = __popc(row(e) & z) & 1 ? c1.re : c0.re;
                    acc[e].re = rfma(c, v.re, acc[e].re);
                    acc[e].im = rfma(c, v.im, acc[e].im);
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const bool odd = __popc(row(e) & z) & 1;
                    cfma(acc[e], C2<R>{odd ? c1.re : c0.re, odd ? c1.im : c0.im}, val(e));
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                int q = 0;
                for (int t = 0; t < rank; ++t) q |= (__popc(row(e) & uload(k.z[t])) & 1) << t;
                cfma(acc[e], table[tab + q], val(e));
            }
        }
    }
};

// Row r of H x over the nonzero coefficients alone, for sums that are not
// finite: an infinite amplitude reaches the rows coupled to it and no others.
template <typename R>
__device__ __forceinline__ C2<R> pauli_nonzero_row(const PauliArgs &a, const C2<R> *x, uint32_t r) {
    C2<R> acc{(R)0, (R)0};
    if (a.diag) {
        const C2<R> d = ld1_cached(reinterpret_cast<const C2<R> *>(a.diag), (int)r);
        if (d.re != (R)0 || d.im != (R)0) cfma(acc, d, ld1_cached(x, (int)r));
    }
#pragma unroll 1
    for (int k = 0; k < a.nmask; ++k) {
        const PauliMask &m = a.masks[k];
        int q = 0;
        for (int t = 0; t < m.rank; ++t) q |= (__popc(r & m.z[t]) & 1) << t;
        const C2<R> c = reinterpret_cast<const C2<R> *>(a.tab)[m.tab + q], v = ld1_cached(x, (int)(r ^ m.m));
        if (c.im != (R)0) {
            cfma(acc, c, v);
        } else if (c.re != (R)0) {
            acc.re = rfma(c.re, v.re, acc.re);
            acc.im = rfma(c.re, v.im, acc.im);
        }
    }
    return acc;
}

// 16 bytes at a byte offset from a uniform base
__device__ __forceinline__ void get16(const char *base, uint32_t off, C2<float> (&v)[2]) {
    const f4v w = *(g_f4 *)((const __attribute__((address_space(1))) char *)base + off);
    v[0] = C2<float>{w.x, w.y};
    v[1] = C2<float>{w.z, w.w};
}
__device__ __forceinline__ void get16(const char *base, uint32_t off, C2<double> (&v)[1]) {
    const d2v w = *(g_d2 *)((const __attribute__((address_space(1))) char *)base + off);
    v[0] = C2<double>{w.x, w.y};
}

constexpr int kPauliThreads = 512;
constexpr int kPauliAccess = 2;      // 16-byte accesses per thread: 2048 complex64 or 1024 complex128 rows a tile

template <typename R, bool STREAM>
__global__ __launch_bounds__(kPauliThreads) __attribute__((amdgpu_waves_per_eu(4)))
void pauli_tile_kernel(PauliArgs a) {
    constexpr bool PAIR = sizeof(R) == 4;
    constexpr int H = PAIR ? 2 : 1, G = kPauliAccess, NT = kPauliThreads, T = G * H * NT;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C2<R> *lds = reinterpret_cast<C2<R> *>(smem_raw);
    const int tid = threadIdx.x;
    const int tiles = (int)(a.N / T);
    const int tile = blockIdx.x % tiles;
    const int b = blockIdx.x / tiles;

    const uint32_t base = (uint32_t)tile * T;
    const C2<R> *x = reinterpret_cast<const C2<R> *>(a.x) + (int64_t)b * a.N;
    auto at = [&](int p) { return H * (tid + p * NT); };
    // access p of the tile XOR m, its rows in memory order (m odd: a pair's
    // partners are each other's); uniform base and 32-bit offsets
    auto partner = [&](uint32_t m, C2<R> (&v)[G][H]) {
        const char *xp = reinterpret_cast<const char *>(x + (base ^ (m & ~(uint32_t)(T - 1))));
        const uint32_t lo = (m & (T - 1)) & ~(uint32_t)(H - 1);
#pragma unroll
        for (int p = 0; p < G; ++p) get16(xp, ((uint32_t)at(p) ^ lo) * (uint32_t)sizeof(C2<R>), v[p]);
    };
    C2<R> acc[G * H], cur[G][H];
    MaskRec<R> rec(a.masks[0]);
    partner(0, cur);
#pragma unroll
    for (int p = 0; p < G; ++p)
#pragma unroll
        for (int h = 0; h < H; ++h) {
            lds[at(p) + h] = cur[p][h];
            acc[p * H + h] = C2<R>{(R)0, (R)0};
        }
    if (a.diag) {
        const C2<R> *dg = reinterpret_cast<const C2<R> *>(a.diag) + base;
#pragma unroll
        for (int p = 0; p < G; ++p) {
            C2<R> d[2];
            if constexpr (PAIR) ld2(dg, at(p), d[0], d[1]);
            else d[0] = ld1(dg, at(p));
#pragma unroll
            for (int h = 0; h < H; ++h) cfma(acc[p * H + h], d[h], cur[p][h]);
        }
    }
    const C2<R> *table = reinterpret_cast<const C2<R> *>(a.tab);
    auto row = [&](int e) { return base + (uint32_t)(at(e / H) + e % H); };
    auto use = [&](const MaskRec<R> &rec, int k) {
        if (PAIR && (rec.m & 1)) rec.add(acc, a.masks[k], table, row, [&](int e) { return cur[e / H][H - 1 - e % H]; });
        else rec.add(acc, a.masks[k], table, row, [&](int e) { return cur[e / H][e % H]; });
    };
    // masks with bits above the tile come first (descending masks); the next
    // mask's record and partner rows are on their way while one is used
    int k = 0;
    if (a.nfar > 0) partner(rec.m, cur);
    for (; k < a.nfar; ++k) {
        const MaskRec<R> now = rec;
        rec = MaskRec<R>(a.masks[k + 1 < a.nmask ? k + 1 : k]);
        C2<R> nxt[G][H];
        if (k + 1 < a.nfar) partner(rec.m, nxt);
        use(now, k);
#pragma unroll
        for (int p = 0; p < G; ++p)
#pragma unroll
            for (int h = 0; h < H; ++h) cur[p][h] = nxt[p][h];
    }
    __syncthreads();
    for (; k < a.nmask; ++k) {
        const MaskRec<R> now = rec;
        rec = MaskRec<R>(a.masks[k + 1 < a.nmask ? k + 1 : k]);
        const int lo = (int)now.m & ~(H - 1);
#pragma unroll
        for (int p = 0; p < G; ++p) {
            const C2<R> *q = &lds[at(p) ^ lo];
            if constexpr (PAIR) {
                const f4v w = *reinterpret_cast<const f4v *>(q);
                cur[p][0] = C2<R>{w.x, w.y};
                cur[p][H - 1] = C2<R>{w.z, w.w};
            } else {
                cur[p][0] = *q;
            }
        }
        use(now, k);
    }
    const C2<R> *x0 = reinterpret_cast<const C2<R> *>(a.x0) + (int64_t)b * a.N + base;
    C2<R> *y = reinterpret_cast<C2<R> *>(a.y) + (int64_t)b * a.N + base;
    const C2<R> al{(R)a.alpha_re, (R)a.alpha_im};
#pragma unroll
    for (int e = 0; e < G * H; ++e)
        if (!finite(acc[e])) acc[e] = pauli_nonzero_row(a, x, row(e));
#pragma unroll
    for (int p = 0; p < G; ++p) {
        C2<R> v[2];
        if constexpr (PAIR) ld2(x0, at(p), v[0], v[1]);
        else v[0] = ld1(x0, at(p));
#pragma unroll
        for (int h = 0; h < H; ++h) cfma(v[h], al, acc[p * H + h]);
        if constexpr (PAIR) st2<STREAM>(y, at(p), v[0], v[1]);
        else st1<STREAM>(y, at(p), v[0]);
    }
}

// The same for small states: one thread per row, the partners of kPauliAhead
// masks in flight (8 in flight spill scalar registers: 5.3 against 4.2 us a
// stage at n = 10).  Same order of sums, same bits.
constexpr int kPauliAhead = 4;
constexpr int kPauliRowThreads = 64;

template <typename R>
__global__ __launch_bounds__(kPauliRowThreads) void pauli_rows_kernel(PauliArgs a) {
    const int r = blockIdx.x * kPauliRowThreads + threadIdx.x;
    if (r >= a.N) return;
    const C2<R> *x = reinterpret_cast<const C2<R> *>(a.x) + (int64_t)blockIdx.y * a.N;
    const C2<R> *table = reinterpret_cast<const C2<R> *>(a.tab);
    C2<R> acc[1] = {C2<R>{(R)0, (R)0}};
    const C2<R> v0 = reinterpret_cast<const C2<R> *>(a.x0)[(int64_t)blockIdx.y * a.N + r];
    if (a.diag) cfma(acc[0], ld1_cached(reinterpret_cast<const C2<R> *>(a.diag), r), ld1_cached(x, r));
    for (int k0 = 0; k0 < a.nmask; k0 += kPauliAhead) {
        C2<R> v[kPauliAhead];
        MaskRec<R> rec[kPauliAhead];
#pragma unroll
        for (int u = 0; u < kPauliAhead; ++u) rec[u] = MaskRec<R>(a.masks[k0 + u < a.nmask ? k0 + u : a.nmask - 1]);
#pragma unroll
        for (int u = 0; u < kPauliAhead; ++u) v[u] = ld1_cached(x, r ^ (int)rec[u].m);
#pragma unroll
        for (int u = 0; u < kPauliAhead; ++u)
            if (k0 + u < a.nmask)
                rec[u].add(acc, a.masks[k0 + u], table, [&](int) { return (uint32_t)r; }, [&](int) { return v[u]; });
    }
    if (!finite(acc[0])) acc[0] = pauli_nonzero_row(a, x, (uint32_t)r);
    C2<R> y = v0;
    cfma(y, C2<R>{(R)a.alpha_re, (R)a.alpha_im}, acc[0]);
    reinterpret_cast<C2<R> *>(a.y)[(int64_t)blockIdx.y * a.N + r] = y;
}

template <typename R>
static int pauli_launch(PauliArgs &a, int batch, bool stream_out, void *stream) {
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    constexpr int T = kPauliAccess * kPauliThreads * (sizeof(R) == 4 ? 2 : 1);
    if (a.N * batch <= kPauliRowsMax || a.N < T) {
        const dim3 g((unsigned)((a.N + kPauliRowThreads - 1) / kPauliRowThreads), batch);
        hipLaunchKernelGGL(pauli_rows_kernel<R>, g, dim3(kPauliRowThreads), 0, st, a);
        return (int)hipGetLastError();
    }
    a.nfar = 0;
    while (a.nfar < a.nmask && a.host_masks[a.nfar] >= (uint32_t)T) ++a.nfar;
    const dim3 g((unsigned)(a.N / T) * batch);
    constexpr size_t lds = T * sizeof(C2<R>);
    if (stream_out) hipLaunchKernelGGL((pauli_tile_kernel<R, true>), g, dim3(kPauliThreads), lds, st, a);
    else hipLaunchKernelGGL((pauli_tile_kernel<R, false>), g, dim3(kPauliThreads), lds, st, a);
    return (int)hipGetLastError();
}

int launch_pauli_horner(PauliArgs a, int batch, bool c128, bool stream_out, void *stream) {
    if (!a.x0 || a.x == a.y || a.N < 2 || (a.N & (a.N - 1)) || a.N > (int64_t(1) << HS_MAX_QUBITS))
        return (int)hipErrorInvalidValue;
    return c128 ? pauli_launch<double>(a, batch, stream_out, stream) : pauli_launch<float>(a, batch, stream_out, stream);
}

}  // namespace hs
