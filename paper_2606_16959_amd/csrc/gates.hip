// The coset kernel: a launch's tile program (gate_plan.h) applied to the
// state, one tile of one state per workgroup.
//
// A tile is every setting of the row bits in the launch's tile mask; all of a
// launch's factors couple rows inside one tile.  The workgroup loads the tile
// once (16 bytes per lane, runs of at least 256 bytes), keeps it in LDS and
// applies block after block: a thread holds a coset of 2^LC rows in registers
// and multiplies it by the factor's small dense matrix, so a factor costs one
// LDS read and one write of the tile and one barrier.  The matrix entries are
// read through scalar loads, or from cache where they depend on further row
// bits.
//
// What bounds it: HBM for large states (state read and written once per
// launch, and 16 bytes of D per row where a factor carries it).  A factor
// that flips three bits costs 16 FMAs per row, the one that carries D about
// 80 operations, which take less time than the bytes.  Four 32 KiB tiles (two
// of 64 KiB where the larger tile saves a launch) fit a CU's LDS, so one
// tile's loads and stores overlap the others' arithmetic.  States that stay in
// cache are bound by the chain inside a workgroup: per block a scalar-load
// round trip, an LDS round trip and a barrier, 17-24 us a launch of a
// complex128 state of 2^20 rows.
// Measured against one DIA SpMV per factor over the stored diagonals, a step:
// n = 26 lattice complex64 10.3 -> 0.81 ms (4.3 GB moved in three launches),
// n = 24 MaxCut with 8 states 4.5 -> 1.46 ms, n = 20 chain complex128
// 232 -> 58 us, n = 17 second order 82 -> 37 us.
#include <hip/hip_runtime.h>

#include <atomic>
#include <mutex>
#include <type_traits>

#include "dev_common.h"
#include "gate_plan.h"

namespace hs {

struct GateArgs {
    void *psi;
    int64_t N;                     // rows of a state, and elements between states
    int32_t batch;
    int32_t kt;                    // log2 of the tile's rows
    int32_t tiles;                 // of a state
    int32_t nin, nout;
    GateSeg in[kGateSegs], out[kGateSegs];     // the rest zero: deposits nothing
    uint32_t access_row[8];        // row bits of the linear phases' access p (local rows H p nt)
    const GateBlock *blocks;
    const uint32_t *words;
    const void *coef;
    const double *coef64;
    const void *stage_diag;        // or null: multiplies the tile as it is loaded
    const double *nrm2;            // per-state squared norms to divide out, or null
    double *norm_out;              // or null: partials of state b, tile t at [(b * tiles + t) * 4]
    int32_t by_rows;               // a block sums row by row (twice the LDS)
    int32_t steps;                 // > 1 only when the tile is the whole state
    int32_t first[4], last[4];     // step part q applies blocks [first[q], last[q])
};

template <typename R>
__device__ __forceinline__ constexpr int lds_pos(int i) {
    return gate_lds_pos(i, sizeof(R) == 8);
}

__device__ __forceinline__ uint32_t seg_deposit(const GateSeg *s, int n, uint32_t i) {
    uint32_t r = 0;
    for (int k = 0; k < n; k += 2)              // two segments per round of scalar loads
#pragma unroll
        for (int u = 0; u < 2; ++u) r |= ((i >> s[k + u].sh) & s[k + u].mask) << s[k + u].dst;
    return r;
}

// i x and -i y: the turned rows of kGateReal
template <typename R>
__device__ __forceinline__ C2<R> turn(C2<R> x) { return C2<R>{-x.im, x.re}; }
template <typename R>
__device__ __forceinline__ C2<R> unturn(C2<R> y) { return C2<R>{y.im, -y.re}; }

// A coset times the factor's matrix, kGateReal: x the coset's rows, out(i, y)
// takes row i of the result.  ODD: kmask has every bit, so the turns are
// register names and signs.  LANE: the matrix depends on the lane.
template <typename R, int RHO, bool ODD, bool LANE, typename FO>
__device__ __forceinline__ void apply_real(C2<R> (&x)[1 << RHO], const R *m, int kmask, FO out) {
    constexpr int D = 1 << RHO;
#pragma unroll
    for (int j = 1; j < D; ++j)
        if (ODD ? (__builtin_popcount(j) & 1) : (__builtin_popcount(j & kmask) & 1)) x[j] = turn(x[j]);
#pragma unroll
    for (int i = 0; i < D; ++i) {
        R row[D];
#pragma unroll
        for (int j = 0; j < D; ++j) row[j] = LANE ? m[i * D + j] : uload(m[i * D + j]);
        C2<R> y{(R)0, (R)0};
#pragma unroll
        for (int j = 0; j < D; ++j) {
            y.re = rfma(row[j], x[j].re, y.re);
            y.im = rfma(row[j], x[j].im, y.im);
        }
        if (ODD ? (__builtin_popcount(i) & 1) : (__builtin_popcount(i & kmask) & 1)) y = unturn(y);
        out(i, y);
    }
}

// The coefficient v D of one entry, multiplied and rounded to the state's dtype
// as the stored diagonals are (cmul_d).
template <typename R>
__device__ __forceinline__ C2<R> d_entry(double vr, double vi, d2v D) {
    const C2<double> t = cmul_d(vr, vi, D.x, D.y);
    return C2<R>{(R)t.re, (R)t.im};
}
// v real, or imaginary (imag): i v D
template <typename R>
__device__ __forceinline__ C2<R> d_entry_typed(double v, bool imag, d2v D) {
    const C2<R> g{(R)(v * D.x), (R)(v * D.y)};
    return imag ? C2<R>{-g.im, g.re} : g;
}

// The same for kGateRealD, partners j outermost (each D[j] is used by every
// row of the coset): entries table[j][i], d(j) is D of element j.
template <typename R, int RHO, bool ODD, bool LANE, typename FD, typename FO>
__device__ __forceinline__ void apply_real_d(const C2<R> (&x)[1 << RHO], const double *m, int kmask, FD d, FO out) {
    constexpr int D = 1 << RHO;
    C2<R> y[D];
#pragma unroll
    for (int i = 0; i < D; ++i) y[i] = C2<R>{(R)0, (R)0};
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const d2v dj = d(j);
        double e[D];
#pragma unroll
        for (int i = 0; i < D; ++i) e[i] = LANE ? m[j * D + i] : uload(m[j * D + i]);
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const bool imag = ODD ? (__builtin_popcount(i ^ j) & 1) : (__builtin_popcount((i ^ j) & kmask) & 1);
            cfma(y[i], d_entry_typed<R>(e[i], imag, dj), x[j]);
        }
    }
#pragma unroll
    for (int i = 0; i < D; ++i) out(i, y[i]);
}

constexpr int kGateThreads = 512;

// One kGateCosets block of rank RHO on the tile in LDS.  Spreading a coset's
// number over the index bits, LDS positions and rows of D are all linear over
// XOR, and a thread's cosets t, t + nt, ... differ in bits that t leaves 0: the
// thread's part is computed once, the rest in scalar registers.
// GENERAL: some kmask lacks a bit.
template <typename R, int RHO, bool GENERAL>
__device__ __forceinline__ void apply_cosets(const GateArgs &a, const GateBlock &B, C2<R> *lds, uint32_t base, int first,
                                             int nt) {
    constexpr int D = 1 << RHO;
    const int cosets = (1 << a.kt) >> RHO;
    const int ntype = B.ntype(), tshift = B.tshift(), nhole = B.nhole(), kmask = B.kmask();
    // the coset's first row: its number's bits around the holes
    auto spread = [&](int cs) {
        int rep = ntype ? cs & ((1 << tshift) - 1) : cs;
        for (int h = 0; h < nhole; ++h) {
            const int low = (1 << B.hole(h)) - 1;
            rep = ((rep & ~low) << 1) | (rep & low);
        }
        for (int t = 0; t < ntype; ++t) rep |= ((cs >> (tshift + t)) & 1) << ((B.tpos >> (8 * t)) & 31);
        return rep;
    };
    // the row's bits without the pivots (base's included)
    auto squeeze = [&](uint32_t r) {
#pragma unroll
        for (int c = RHO - 1; c >= 0; --c) {
            const int rp = B.rpiv(c);
            r = ((r >> rp >> 1) << rp) | (r & ((1u << rp) - 1));
        }
        return r;
    };
    const bool with_d = B.form() != kGateReal, lane = B.lane();
    int step[RHO];
#pragma unroll
    for (int q = 0; q < RHO; ++q) step[q] = lds_pos<R>((int)B.basis[q]);
    const int rep_t = spread(first), pos_t = lds_pos<R>(rep_t);
    const uint32_t row_t = with_d ? squeeze(base | seg_deposit(a.in, a.nin, (uint32_t)rep_t)) : 0;
    if (first >= cosets) return;
#pragma unroll 1
    for (int c0 = 0; c0 < cosets; c0 += nt) {
        const int rep_s = spread(c0), pos0 = pos_t ^ lds_pos<R>(rep_s);
        int type = 0;
        if (B.direct()) {
            type = (first + c0) >> tshift;
        } else if (B.inside()) {
            const int rep = rep_t ^ rep_s;
            for (int t = 0; t < B.nz(); ++t) type |= ((rep >> (B.tpos >> (8 * t) & 31)) & 1) << t;
        } else {
            const int rep = rep_t ^ rep_s;
            for (int t = 0; t < B.nz(); ++t)
                type |= (int)(((rep & uload(a.words[B.ztab + 2 * t])) | (base & uload(a.words[B.ztab + 2 * t + 1]))) != 0)
                        << t;
        }
        // the matrix of the lane, and of the wave where it has but one
        const int64_t kl = B.coef + ((int64_t)type << (2 * RHO));
        const int64_t ku = B.coef + ((int64_t)__builtin_amdgcn_readfirstlane(type) << (2 * RHO));
        auto at = [&](int j) -> C2<R> & {
            int m = 0;
#pragma unroll
            for (int q = 0; q < RHO; ++q)
                if ((j >> q) & 1) m ^= step[q];
            return lds[pos0 ^ m];
        };
        C2<R> x[D];
        auto out = [&](int i, C2<R> y) { at(i) = y; };
        if (!with_d) {
            const R *ml = reinterpret_cast<const R *>(a.coef) + kl, *mu = reinterpret_cast<const R *>(a.coef) + ku;
#pragma unroll
            for (int j = 0; j < D; ++j) x[j] = at(j);
            if (!GENERAL || kmask == D - 1) {
                if (lane) apply_real<R, RHO, true, true>(x, ml, kmask, out);
                else apply_real<R, RHO, true, false>(x, mu, kmask, out);
            } else {
                if (lane) apply_real<R, RHO, false, true>(x, ml, kmask, out);
                else apply_real<R, RHO, false, false>(x, mu, kmask, out);
            }
        } else {
            const double *ml = a.coef64 + kl, *mu = a.coef64 + ku;
            const uint32_t row_s = squeeze(seg_deposit(a.in, a.nin, (uint32_t)rep_s));
            g_d2 *dp = (g_d2 *)B.diag + (row_t ^ row_s);
            const int64_t len = a.N >> RHO;
            // complex64 holds every D of the coset, loaded before the rows;
            // complex128 has no registers for that
            constexpr bool ALL = sizeof(R) == 4;
            d2v dj[ALL ? D : 1];
            if constexpr (ALL)
#pragma unroll
                for (int j = 0; j < D; ++j) dj[j] = dp[j * len];
            auto d = [&](int j) -> d2v {
                if constexpr (ALL) return dj[j];
                else return dp[j * len];
            };
#pragma unroll
            for (int j = 0; j < D; ++j) x[j] = at(j);
            if (!GENERAL || kmask == D - 1) {
                if (lane) apply_real_d<R, RHO, true, true>(x, ml, kmask, d, out);
                else apply_real_d<R, RHO, true, false>(x, mu, kmask, d, out);
            } else {
                if (lane) apply_real_d<R, RHO, false, true>(x, ml, kmask, d, out);
                else apply_real_d<R, RHO, false, false>(x, mu, kmask, d, out);
            }
        }
    }
}

// A kGateRows block of rank up to kGateMaxCoset (general entries): every row's
// sum over its coset goes to the second half of LDS, then replaces the row.
template <typename R>
__device__ __forceinline__ void apply_rows(const GateArgs &a, const GateBlock &B, C2<R> *lds, uint32_t base, int tid,
                                           int nt) {
    const int T = 1 << a.kt;
    const uint32_t *w = a.words + B.wtab;
    const int rho = B.rho(), form = B.form(), kmask = B.kmask(), nz = B.nz(), dim = 1 << rho;
    g_d2 *dtab = (g_d2 *)B.diag;
    const C2<R> *mc = reinterpret_cast<const C2<R> *>(a.coef);
    const R *mr = reinterpret_cast<const R *>(a.coef);
#pragma unroll 1
    for (int i = tid; i < T; i += nt) {
        int own = 0, e = i;             // own coordinate, the coset's element 0
        for (int c = 0; c < rho; ++c)
            if ((i >> (int)uload(w[c])) & 1) {
                own |= 1 << c;
                e ^= (int)uload(w[rho + c]);
            }
        int64_t tab = 0;
        for (int t = 0; t < nz; ++t)
            tab |= (int64_t)(((e & uload(a.words[B.ztab + 2 * t])) | (base & uload(a.words[B.ztab + 2 * t + 1]))) != 0)
                   << t;
        tab = B.coef + tab * dim * dim;
        int64_t dc = 0;
        if (dtab) {
            dc = (int64_t)(base | seg_deposit(a.in, a.nin, (uint32_t)e));
            for (int c = rho - 1; c >= 0; --c) {
                const int rp = (int)uload(w[2 * rho + c]);
                dc = ((dc >> (rp + 1)) << rp) | (dc & ((int64_t(1) << rp) - 1));
            }
        }
        C2<R> y{(R)0, (R)0};
#pragma unroll 1
        for (int j = 0; j < dim; ++j) {
            int at = e;
            for (int c = 0; c < rho; ++c)
                if ((j >> c) & 1) at ^= (int)uload(w[rho + c]);
            const C2<R> x = lds[lds_pos<R>(at)];
            if (form == kGateReal) {
                const C2<R> xt = (__builtin_popcount(j & kmask) & 1) ? turn(x) : x;
                const R k = mr[tab + (int64_t)own * dim + j];
                y.re = rfma(k, xt.re, y.re);
                y.im = rfma(k, xt.im, y.im);
            } else if (form == kGateComplex) {
                cfma(y, mc[tab + (int64_t)own * dim + j], x);
            } else {
                const d2v D = dtab[(int64_t)j * (a.N >> rho) + dc];
                const int64_t k = tab + (int64_t)j * dim + own;
                if (form == kGateRealD)
                    cfma(y, d_entry_typed<R>(a.coef64[k], __builtin_popcount((own ^ j) & kmask) & 1, D), x);
                else
                    cfma(y, d_entry<R>(a.coef64[2 * k], a.coef64[2 * k + 1], D), x);
            }
        }
        if (form == kGateReal && (__builtin_popcount(own & kmask) & 1)) y = unturn(y);
        lds[T + i] = y;
    }
    __syncthreads();
#pragma unroll 1
    for (int i = tid; i < T; i += nt) lds[lds_pos<R>(i)] = lds[T + i];
}

// Sums of one unit (gate_plan.h), rows i0 .. i0 + C - 1 of the coset whose
// element 0 sits at LDS position pos0: y[i] = sum_j M[i0 + i][j] x[j], j
// ascending.  tab: the matrix's first entry; dp: D of the coset's element 0,
// the elements `len` entries apart.  LANE: the entries depend on the lane.
template <typename R, int C, int FORM, bool LANE>
__device__ __forceinline__ void unit_sums(const GateArgs &a, const GateBlock &B, const C2<R> *lds, int pos0, int64_t tab, int i0,
                                          g_d2 *dp, int64_t len, C2<R> (&y)[C]) {
    constexpr bool PAIRS = FORM == kGateComplex || FORM == kGateComplexD, WITH_D = FORM == kGateRealD || FORM == kGateComplexD;
    constexpr int E = PAIRS ? 2 : 1;                // reals of an entry
    using M = typename std::conditional<WITH_D, double, R>::type;
    // partners per round, whose entries are loaded at once: 64 scalar
    // registers, or 32 vector registers where they differ between lanes
    constexpr int FIT = (LANE ? 32 : 64) / (C * E * ((int)sizeof(M) / 4)), JB = FIT > 4 ? 4 : FIT < 1 ? 1 : FIT;
    const int rho = B.rho(), dim = 1 << rho, kmask = B.kmask();
    const uint32_t *w = a.words + B.wtab, *jm = w + 3 * rho + B.nhole() + B.ntype();
    const int s0 = lds_pos<R>((int)uload(w[rho])), s1 = lds_pos<R>((int)uload(w[rho + 1]));
    const M *m = reinterpret_cast<const M *>(WITH_D ? (const void *)a.coef64 : a.coef) + E * tab;
#pragma unroll
    for (int i = 0; i < C; ++i) y[i] = C2<R>{(R)0, (R)0};
#pragma unroll 1
    for (int j = 0; j < dim; j += JB) {
        int pj = pos0 ^ lds_pos<R>((int)uload(jm[j >> 2]));
        if (JB < 2) pj ^= (j & 1) ? s0 : 0;
        if (JB < 4) pj ^= (j & 2) ? s1 : 0;
        C2<R> x[JB];
        d2v D[JB];
        M e[C][JB][E];
#pragma unroll
        for (int q = 0; q < JB; ++q) {
            x[q] = lds[pj ^ ((q & 1) ? s0 : 0) ^ ((q & 2) ? s1 : 0)];
            if constexpr (WITH_D) D[q] = dp[(j + q) * len];
        }
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
            for (int q = 0; q < JB; ++q)
#pragma unroll
                for (int c = 0; c < E; ++c) {
                    const M &v = m[E * (WITH_D ? (j + q) * dim + i0 + i : (i0 + i) * dim + j + q) + c];
                    e[i][q][c] = LANE ? v : uload(v);
                }
#pragma unroll
        for (int q = 0; q < JB; ++q) {
            const bool odd = __builtin_popcount((j + q) & kmask) & 1;
            if constexpr (FORM == kGateReal) {
                const C2<R> xt = odd ? turn(x[q]) : x[q];
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    y[i].re = rfma(e[i][q][0], xt.re, y[i].re);
                    y[i].im = rfma(e[i][q][0], xt.im, y[i].im);
                }
            } else {
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    C2<R> k;
                    if constexpr (FORM == kGateComplex) k = C2<R>{e[i][q][0], e[i][q][1]};
                    else if constexpr (FORM == kGateRealD)
                        k = d_entry_typed<R>(e[i][q][0], ((__builtin_popcount((i0 + i) & kmask) & 1) != 0) != odd, D[q]);
                    else k = d_entry<R>(e[i][q][0], e[i][q][1], D[q]);
                    cfma(y[i], k, x[q]);
                }
            }
        }
    }
    if constexpr (FORM == kGateReal)
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (__builtin_popcount((i0 + i) & kmask) & 1) y[i] = unturn(y[i]);
}

// A kGateRows block of rank above kGateMaxCoset.  A thread has one unit: it
// reads every element of its coset once from LDS for C rows and keeps the sums
// in registers until all threads have read.
//
// What bounds it: the multiply-adds, 2^(rank + 1) per row, and at few tiles the
// chain of partners (a scalar load of entries, an LDS read) of each wave.  C is
// the rows a thread of the launch has, so that a unit needs no loop and a
// partner's LDS read and its entries' scalar loads serve C rows.  Two steps of
// a transverse-field chain, us: stored diagonals streamed / every row summed
// alone / units: n = 12 complex64 budget 32 (rank 4) 97 / 310 / 57, budget 128
// (rank 6) 267 / 910 / 114, budget 1024 (rank 9) 1490 / 5130 / 555; n = 18
// complex128, 8 states, budget 128 740 / 3090 / 397; n = 22 complex64 budget
// 128 4250 / 6050 / 637.
template <typename R, int C>
__device__ __forceinline__ void apply_units(const GateArgs &a, const GateBlock &B, C2<R> *lds, uint32_t base, int tid) {
    constexpr int LC = C == 16 ? 4 : C == 8 ? 3 : 2;
    const int rho = B.rho(), nhole = B.nhole(), ntype = B.ntype(), tshift = B.tshift(), nz = B.nz();
    const uint32_t *w = a.words + B.wtab, *jm = w + 3 * rho + nhole + ntype;
    const bool active = tid < (1 << a.kt) / C, lane = B.lane();
    C2<R> y[C];
    int pos = 0;
    if (active) {
        int rep = tid & ((1 << tshift) - 1);
        for (int h = 0; h < nhole; ++h) {
            const int low = (1 << uload(w[3 * rho + h])) - 1;
            rep = ((rep & ~low) << 1) | (rep & low);
        }
        for (int t = 0; t < ntype; ++t)
            rep |= ((tid >> (tshift + rho - LC + t)) & 1) << uload(w[3 * rho + nhole + t]);
        int i0 = ((tid >> tshift) & ((1 << (rho - LC)) - 1)) << LC, type = 0;
        for (int t = 0; t < nz; ++t)
            type |= (int)(((rep & uload(a.words[B.ztab + 2 * t])) | (base & uload(a.words[B.ztab + 2 * t + 1]))) != 0) << t;
        if (!lane) {
            i0 = __builtin_amdgcn_readfirstlane(i0);
            type = __builtin_amdgcn_readfirstlane(type);
        }
        const int64_t tab = B.coef + ((int64_t)type << (2 * rho));
        g_d2 *dp = (g_d2 *)B.diag;
        if (dp) {
            uint32_t row = base | seg_deposit(a.in, a.nin, (uint32_t)rep);
            for (int c = rho - 1; c >= 0; --c) {
                const int rp = (int)uload(w[2 * rho + c]);
                row = ((row >> rp >> 1) << rp) | (row & ((1u << rp) - 1));
            }
            dp += row;
        }
        const int64_t len = a.N >> rho;
        const int pos0 = lds_pos<R>(rep);
        pos = pos0 ^ lds_pos<R>((int)jm[i0 >> 2]);
        const int form = B.form();
        if (form == kGateReal) {
            if (lane) unit_sums<R, C, kGateReal, true>(a, B, lds, pos0, tab, i0, dp, len, y);
            else unit_sums<R, C, kGateReal, false>(a, B, lds, pos0, tab, i0, dp, len, y);
        } else if (form == kGateRealD) {
            if (lane) unit_sums<R, C, kGateRealD, true>(a, B, lds, pos0, tab, i0, dp, len, y);
            else unit_sums<R, C, kGateRealD, false>(a, B, lds, pos0, tab, i0, dp, len, y);
        } else if (form == kGateComplex) {
            unit_sums<R, C, kGateComplex, true>(a, B, lds, pos0, tab, i0, dp, len, y);
        } else {
            unit_sums<R, C, kGateComplexD, true>(a, B, lds, pos0, tab, i0, dp, len, y);
        }
    }
    __syncthreads();
    if (active) {
        int s[LC];
#pragma unroll
        for (int c = 0; c < LC; ++c) s[c] = lds_pos<R>((int)uload(w[rho + c]));
#pragma unroll
        for (int i = 0; i < C; ++i) {
            int p = pos;
#pragma unroll
            for (int c = 0; c < LC; ++c)
                if ((i >> c) & 1) p ^= s[c];
            lds[p] = y[i];
        }
    }
}

__device__ __forceinline__ GateBlock uload_block(const GateBlock &p) {
    GateBlock r;
    r.diag = uload(p.diag);
    r.holes = uload(p.holes);
    r.tpos = uload(p.tpos);
#pragma unroll
    for (int c = 0; c < kGateMaxCoset; ++c) r.basis[c] = uload(p.basis[c]);
    r.coef = uload(p.coef);
    r.ztab = uload(p.ztab);
    r.wtab = uload(p.wtab);
    r.what = uload(p.what);
    r.number = uload(p.number);
    r.rpivots = uload(p.rpivots);
    return r;
}

// LEVEL 0 is for programs of cosets up to kGateMaxCoset whose entries are
// imaginary for every single flip (transverse fields, XX + YY bonds: most
// programs), a third of the code; 1 adds other real and general entries, 2
// larger cosets.
template <typename R, bool STREAM, int LEVEL>
__global__ __launch_bounds__(kGateThreads) __attribute__((amdgpu_waves_per_eu(4))) void gate_kernel(GateArgs a) {
    constexpr bool PAIR = sizeof(R) == 4;           // linear phases: two adjacent rows per 16-byte access
    constexpr int H = PAIR ? 2 : 1;
    constexpr int G = 8;                            // 16-byte accesses of a thread's linear rows
    constexpr bool GENERAL = LEVEL > 0;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C2<R> *lds = reinterpret_cast<C2<R> *>(smem_raw);
    const int tid = threadIdx.x;
    const int nt = blockDim.x;
    const int T = 1 << a.kt;

    // Workgroups (8 tiles, states, eighths) are dealt to the 8 XCDs
    // round-robin, so the states of one tile follow 8 apart on one XCD and
    // find its D in that XCD's L2.
    const int tile = (int)(blockIdx.z * gridDim.x + blockIdx.x), b = (int)blockIdx.y;
    // Linear phases: access p of thread t covers local row(s) H (t + p nt) (and
    // + 1 for complex64).  Rows and LDS positions are linear over the bits of
    // the thread and of the access, as in apply_cosets.
    auto row_part = [&](int p) { return a.access_row[p]; };
    // The thread's number, opaque to the compiler: each phase computes its
    // rows and LDS positions afresh instead of holding them in registers
    // through the blocks.
    auto fresh = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));
        return t;
    };
    const uint32_t base = seg_deposit(a.out, a.nout, (uint32_t)tile);
    C2<R> *psi = reinterpret_cast<C2<R> *>(a.psi) + (int64_t)b * a.N + base;
    {
        C2<R> u[G][H];
        const int t = fresh();
        const uint32_t row_t = seg_deposit(a.in, a.nin, (uint32_t)(H * t));
        const C2<R> *src = psi + row_t;
#pragma unroll
        for (int p = 0; p < G; ++p)
            if (H * p * nt < T) {
                if constexpr (PAIR) ld2(src + row_part(p), 0, u[p][0], u[p][1]);
                else u[p][0] = ld1(src + row_part(p), 0);
            }
        if (a.nrm2) {
            const R scale = inv_norm<R>(a.nrm2, b);
#pragma unroll
            for (int p = 0; p < G; ++p)
#pragma unroll
                for (int h = 0; h < H; ++h) u[p][h] = cscale(u[p][h], scale);
        }
        if (a.stage_diag) {
            const C2<R> *dg = reinterpret_cast<const C2<R> *>(a.stage_diag) + base + row_t;
#pragma unroll
            for (int p = 0; p < G; ++p)
                if (H * p * nt < T) {
                    C2<R> k[2];
                    if constexpr (PAIR) ld2_cached(dg + row_part(p), 0, k[0], k[1]);
                    else k[0] = ld1_cached(dg + row_part(p), 0);
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        C2<R> y{(R)0, (R)0};
                        cfma(y, k[h], u[p][h]);
                        u[p][h] = y;
                    }
                }
        }
        const int pos_t = lds_pos<R>(H * t);
        if (H * t < T)
#pragma unroll
            for (int p = 0; p < G; ++p)
                if (H * p * nt < T)
#pragma unroll
                    for (int h = 0; h < H; ++h) lds[pos_t ^ lds_pos<R>(H * p * nt + h)] = u[p][h];
    }

    {
        for (int s = 0; s < a.steps; ++s) {
            const int part = a.steps == 1 ? 0 : s == 0 ? 1 : s == a.steps - 1 ? 3 : 2;
            const int k1 = a.last[part];
            for (int k = a.first[part]; k < k1; ++k) {
                const GateBlock B = uload_block(a.blocks[k]);
                __syncthreads();
                if (B.kind() == kGateCosets) {
                    if (B.rho() == 3) apply_cosets<R, 3, GENERAL>(a, B, lds, base, fresh(), nt);
                    else if (B.rho() == 2) apply_cosets<R, 2, GENERAL>(a, B, lds, base, fresh(), nt);
                    else apply_cosets<R, 1, GENERAL>(a, B, lds, base, fresh(), nt);
                } else if (B.kind() == kGateDiag) {
                    const C2<R> *dg = reinterpret_cast<const C2<R> *>(B.diag);
#pragma unroll 1
                    for (int i = H * fresh(); i < T; i += H * nt) {
                        const int r = (int)(base | seg_deposit(a.in, a.nin, (uint32_t)i));
                        C2<R> d[2];
                        if constexpr (PAIR) ld2_cached(dg, r, d[0], d[1]);
                        else d[0] = ld1_cached(dg, r);
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            C2<R> y{(R)0, (R)0};
                            cfma(y, d[h], lds[lds_pos<R>(i + h)]);
                            lds[lds_pos<R>(i + h)] = y;
                        }
                    }
                } else if constexpr (GENERAL) {
                    // rows per thread: 16 or 8 of a full tile, at least 4
                    if (B.rho() <= kGateMaxCoset) {
                        apply_rows<R>(a, B, lds, base, fresh(), nt);
                    } else if constexpr (LEVEL == 2) {
                        if (PAIR && T >= 16 * nt) apply_units<R, PAIR ? 16 : 8>(a, B, lds, base, fresh());
                        else if (T >= 8 * nt) apply_units<R, 8>(a, B, lds, base, fresh());
                        else apply_units<R, 4>(a, B, lds, base, fresh());
                    }
                }
            }
        }
        __syncthreads();

        {
            const int t = fresh();
            C2<R> *dst = psi + seg_deposit(a.in, a.nin, (uint32_t)(H * t));
            const int pos_t = lds_pos<R>(H * t);
            double ss = 0.0;
            if (H * t < T)
#pragma unroll
                for (int p = 0; p < G; ++p)
                    if (H * p * nt < T) {
                        C2<R> y[2];
#pragma unroll
                        for (int h = 0; h < H; ++h) y[h] = lds[pos_t ^ lds_pos<R>(H * p * nt + h)];
                        if (a.norm_out)
#pragma unroll
                            for (int h = 0; h < H; ++h) {
                                const double re = (double)y[h].re, im = (double)y[h].im;
                                ss += re * re + im * im;
                            }
                        if constexpr (PAIR) st2<STREAM>(dst + row_part(p), 0, y[0], y[1]);
                        else st1<STREAM>(dst + row_part(p), 0, y[0]);
                    }
            if (a.norm_out) {
                // FP64 sum of |y|^2 over the tile's rows in a fixed order:
                // rows per thread, a wave butterfly, then the waves in order
                __syncthreads();
                double *red = reinterpret_cast<double *>(smem_raw);
                const double w = wave_sum(ss);
                if ((tid & 63) == 0) red[tid >> 6] = w;
                __syncthreads();
                if (tid == 0) {
                    double sum = 0.0;
                    for (int q = 0; q < (nt >> 6); ++q) sum += red[q];
                    double *o = a.norm_out + ((size_t)b * a.tiles + tile) * 4;
                    o[0] = 0.0;
                    o[1] = 0.0;
                    o[2] = sum;
                    o[3] = 0.0;
                }
            }
        }
    }
}

// ------------------------------------------------------------ launcher

static std::mutex &gate_attr_mutex() {
    static std::mutex m;
    return m;
}

template <typename R, bool STREAM, int LEVEL>
static int gate_launch(GateArgs &a, void *stream) {
    auto kern = gate_kernel<R, STREAM, LEVEL>;
    const int T = 1 << a.kt;
    const size_t tile = (size_t)T * sizeof(C2<R>) * (a.by_rows ? 2 : 1), lds = tile < 256 ? 256 : tile;
    // every linear row has a thread (8 accesses of 16 bytes each); launches of
    // few tiles get up to one thread per two rows
    constexpr int RPT = 8 * 16 / (int)sizeof(C2<R>);
    int nt = (int64_t)a.tiles * a.batch < 1024 ? T / 2 : T / RPT;
    if (nt < 64) nt = 64;
    if (nt > kGateThreads) nt = kGateThreads;
    if (nt * RPT < T) return (int)hipErrorInvalidValue;
    if (lds > 65536) {
        static std::atomic<int> allowed{65536};
        if ((int)lds > allowed.load()) {
            std::lock_guard<std::mutex> lock(gate_attr_mutex());
            if ((int)lds > allowed.load()) {
                const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                if (e != hipSuccess) return (int)e;
                allowed.store((int)lds);
            }
        }
    }
    constexpr int H = sizeof(R) == 4 ? 2 : 1;
    for (int p = 0; p < 8; ++p) {
        const uint32_t i = (uint32_t)(H * p * nt);
        a.access_row[p] = 0;
        if (i < (uint32_t)T)
            for (int k = 0; k < a.nin; ++k) a.access_row[p] |= ((i >> a.in[k].sh) & a.in[k].mask) << a.in[k].dst;
    }
    unsigned gx = a.tiles < 8 ? a.tiles : 8;
    while ((unsigned)a.tiles / gx > 32768) gx *= 2;
    hipLaunchKernelGGL(kern, dim3(gx, (unsigned)a.batch, (unsigned)a.tiles / gx), dim3(nt), lds,
                       reinterpret_cast<hipStream_t>(stream), a);
    return (int)hipGetLastError();
}

template <typename R>
static int gate_level(GateArgs &a, int level, bool stream_out, void *stream) {
    if (level == 0) return stream_out ? gate_launch<R, true, 0>(a, stream) : gate_launch<R, false, 0>(a, stream);
    if (level == 1) return stream_out ? gate_launch<R, true, 1>(a, stream) : gate_launch<R, false, 1>(a, stream);
    return stream_out ? gate_launch<R, true, 2>(a, stream) : gate_launch<R, false, 2>(a, stream);
}

int launch_gates(const GateLaunch &L, const GateTables &t, const GateRun &r, bool c128, bool stream_out, void *stream) {
    GateArgs a{};
    if (L.in.size() > (size_t)kGateSegs || L.out.size() > (size_t)kGateSegs) return (int)hipErrorInvalidValue;
    // row pairs of the linear phases are adjacent in the state
    if (!(L.tile & 1) || L.kt < 1 || L.rows != (int64_t(1) << L.kt)) return (int)hipErrorInvalidValue;
    const int64_t tiles = r.N / L.rows;            // a power of two
    if (tiles < 1 || tiles > (1 << 24) || r.batch > 65535 || (r.steps > 1 && tiles != 1)) return (int)hipErrorInvalidValue;
    a.psi = r.psi;
    a.N = r.N;
    a.batch = r.batch;
    a.kt = L.kt;
    a.tiles = (int32_t)tiles;
    a.nin = (int32_t)L.in.size();
    a.nout = (int32_t)L.out.size();
    for (int k = 0; k < a.nin; ++k) a.in[k] = L.in[k];
    for (int k = 0; k < a.nout; ++k) a.out[k] = L.out[k];
    a.blocks = t.blocks;
    a.words = t.words;
    a.coef = t.coef;
    a.coef64 = t.coef64;
    a.stage_diag = r.stage_diag;
    a.nrm2 = r.nrm2;
    a.norm_out = r.norm_out;
    a.by_rows = r.by_rows;
    a.steps = r.steps;
    for (int q = 0; q < 4; ++q) {
        a.first[q] = r.first[q];
        a.last[q] = r.last[q];
    }
    if (r.by_rows && r.level < 1) return (int)hipErrorInvalidValue;
    return c128 ? gate_level<double>(a, r.level, stream_out, stream) : gate_level<float>(a, r.level, stream_out, stream);
}

}  // namespace hs
