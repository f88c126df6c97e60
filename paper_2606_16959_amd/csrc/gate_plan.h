// The factors as programs of small dense products (host planning and the
// records the kernels read).
//
// A factor's exponential couples a row only with the rows its group's X-masks
// reach: the masks span 2^rho flips, and the factor is one 2^rho x 2^rho
// product on every coset r ^ span, with entries of the factor's local unitary
// (L[loc(r), loc(r')], times D[r'] for the factor that carries the diagonal
// terms).  The stored diagonals (Eq. 6) hold the same entries once per row and
// diagonal, about half of them structural zeros.  A launch that applies the
// products needs no coefficient stream: it moves the state, and D where the
// factor carries it.  Entries are rounded to the state's dtype exactly as the
// stored ones are, and every row sums its products in the order of ascending
// offsets, so the results are those of the stored diagonals bit for bit.
#pragma once

#include <cstdint>
#include <map>
#include <memory>
#include <vector>

#include "hs_internal.h"

namespace hs {

constexpr int kGateMaxCoset = 3;     // rank of the largest coset a thread holds in registers
constexpr int kGateMaxType = 4;      // type bits that a block's coset numbering keeps apart
constexpr int kGateSegs = 16;        // bit segments of a tile or of its complement

// LDS position of tile-local row i: XOR of the low bits with higher ones, so
// that the rows a wave reads for one coset element fall on distinct banks
// whichever bits the coset spans.  It is linear over XOR: the position of
// row i ^ m is that of i XOR that of m.
constexpr int gate_lds_pos(int i, bool c128) {
    const int lb = c128 ? 4 : 5;       // rows of one 256-byte bank line
    return i ^ (((i >> lb) & ((1 << (lb - 1)) - 1)) << 1) ^ ((i >> (2 * lb - 2)) & 1);
}

// How a factor's entries are kept (R: the state's real type).
//   kGateReal     entries real or imaginary by one parity of the flip; stored
//                 as R values of the product between rows turned by i^kappa
//                 (kappa_j = parity(j & kmask)): M'[i][j] = i^(kappa_i -
//                 kappa_j) M[i][j], all real, so an entry is two FMAs
//   kGateComplex  general entries, (re, im) pairs of R
//   kGateRealD    the factor carries D: FP64 moduli v, M = v or i v by
//                 parity((i ^ j) & kmask); the coefficient is the rounded v D[j]
//   kGateComplexD general FP64 entries with D
enum GateForm { kGateReal = 0, kGateComplex = 1, kGateRealD = 2, kGateComplexD = 3 };

// kGateCosets: a thread holds whole cosets (rank up to kGateMaxCoset, forms
// Real and RealD).  kGateRows: above that rank a thread sums a piece of a
// coset's rows (below: units), up to it, for general entries, its rows one by
// one.  kGateDiag: the product with a diagonal.
enum GateKind { kGateCosets = 0, kGateDiag = 1, kGateRows = 2 };

// One factor on the tile.
//
// A coset's number is spread over the tile-local index bits that are no
// holes (the pivots, 0 in a coset's first row, and the type bits).  The top
// ntype bits of the number are the type bits' values: with at least 64 cosets
// per type they are the same for all lanes of a wave, whose matrix then comes
// through scalar loads.  With fewer cosets ntype is 0, type bits are no
// holes, and each lane loads its own matrix.
//
// Units of a kGateRows block of rank above kGateMaxCoset: C consecutive rows of
// one coset (C a power of two, the launch's choice).  A unit's number is, from
// the low end, the coset's number without the types (tshift bits), which piece
// of the coset, and the ntype type bits.  With at least 64 cosets per type the
// types and pieces are the same for all lanes of a wave (the types are holes);
// with fewer each lane loads its own entries and ntype is 0.
struct alignas(64) GateBlock {     // one scalar load
    const void *diag;              // kGateDiag: N entries; forms with D: FP64 [2^rho][N >> rho],
                                   // element j of coset c (coset_index)
    uint64_t holes;                // ascending local positions, one byte each
    uint32_t tpos;                 // local position of type bit t: byte t
    uint32_t basis[kGateMaxCoset]; // reduced masks of the coset, in tile-local index space
    int32_t coef;                  // first entry: table[type][i][j], or [type][j][i] with D
    int32_t ztab;                  // in `words`, nz type bits: pairs (local bit, row bit outside the tile)
    int32_t wtab;                  // kGateRows: in `words`, rho local pivots, masks, row pivots; with units
                                   // also nhole holes, ntype type positions and the masks of elements 0, 4, ..
    uint32_t what;                 // kind, rho, form, nz: 4 bits each; kmask: 16
    uint32_t number;               // nhole, ntype, tshift: 8 bits each; lane, inside, direct: flags
    uint32_t rpivots;              // row bits of the pivots, ascending, one byte each
    uint32_t pad[2];

    constexpr int kind() const { return (int)(what & 15); }
    constexpr int rho() const { return (int)(what >> 4 & 15); }
    constexpr int form() const { return (int)(what >> 8 & 15); }
    constexpr int nz() const { return (int)(what >> 12 & 15); }
    constexpr int kmask() const { return (int)(what >> 16); }
    constexpr int nhole() const { return (int)(number & 255); }
    constexpr int ntype() const { return (int)(number >> 8 & 255); }
    constexpr int tshift() const { return (int)(number >> 16 & 255); }   // log2(cosets) - ntype
    constexpr bool lane() const { return number >> 24 & 1; }             // each lane loads its own matrix
    constexpr bool inside() const { return number >> 25 & 1; }           // every type bit is in the tile, at tpos
    constexpr bool direct() const { return number >> 28; }               // the type is the coset number's top bits
    constexpr int hole(int h) const { return (int)(holes >> (8 * h) & 63); }
    constexpr int rpiv(int c) const { return (int)(rpivots >> (8 * c) & 31); }
};
static_assert(sizeof(GateBlock) == 64, "one scalar load");

// dst bits of a segment: ((i >> sh) & mask) << dst
struct GateSeg {
    int32_t sh;
    uint32_t mask;
    int32_t dst;
};

// ------------------------------------------------------------ host planning

// One factor of a step as a coset product (or a diagonal alone).
struct GateStep {
    int factor = 0;                // stored factor
    int pos = 0;                   // its position in the part's sequence
    bool diag_only = false;        // D and nothing else
    bool carries_d = false;
    uint64_t flips = 0;            // union of the masks
    std::vector<uint64_t> basis;   // reduced masks by ascending highest bit (the pivots): ascending
                                   // coset coordinates are ascending rows
    std::vector<int> type_bits;    // support bits that are no pivots: they select the product
    bool closed = true;            // the cosets hold every nonzero entry of the local unitary
    int form = kGateReal;
    int kmask = 0;
    std::shared_ptr<const std::vector<double>> entries;   // [type][i][j] ([type][j][i] with D) as `form` keeps them, in FP64
    uint64_t pivots() const {
        uint64_t p = 0;
        for (uint64_t v : basis) p |= 1ull << (63 - __builtin_clzll(v));
        return p;
    }
};

struct GateLaunch {
    int first = 0, count = 0;      // positions of its steps
    uint64_t tile = 0;             // row bits of the tile
    int kt = 0;                    // log2 of its rows
    int64_t rows = 0;
    int block0 = 0, block1 = 0;
    int stage_diag = -1;           // factor whose diagonal multiplies the tile as it is loaded
    std::vector<GateSeg> in, out;  // tile-local bits -> row bits; tile number -> row bits
};

struct GateProgram {
    bool by_rows = false;               // some block sums row by row (twice the LDS)
    int level = 0;                      // kernel instance: 2 for units, 1 for other kGateRows blocks or a kmask
                                        // that lacks a bit
    bool closed = true;                 // no entry couples rows of different cosets or tiles
    std::vector<GateLaunch> launches;
    std::vector<GateBlock> blocks;      // diag filled at upload from dfactor
    std::vector<int> dfactor;           // factor whose D the block reads, or -1
    std::vector<uint32_t> words;
    std::vector<double> coef;           // forms Real and Complex (rounded to the dtype at upload)
    std::vector<double> coef64;         // forms RealD and ComplexD
    std::map<int, int> coef_of;         // factor -> first entry
};

std::vector<uint64_t> gate_basis(const Plan &P, int factor);
GateStep gate_step(const Plan &P, int factor, int pos);
// `made`: steps by factor that are at hand, completed
std::vector<GateStep> gate_steps(const Plan &P, const std::vector<int> &seq, std::map<int, GateStep> *made = nullptr);

// Launches for `steps`: consecutive steps share a launch while a tile of
// 2^kt rows that holds the low wlog bits (rows in one run) holds every bit
// they flip; at most max_factors factors per launch (0: any number).
// `loop`: one launch of the whole state whose blocks are applied again and
// again (no diagonal folded into the load), whatever max_factors says.
// Appends to `out`.
void gate_launches(const Plan &P, const std::vector<GateStep> &steps, int kt, int wlog, int max_factors, bool loop,
                   GateProgram &out);

// Device tables of a program and one launch's run-time arguments (gates.hip).
struct GateTables {
    const GateBlock *blocks = nullptr;
    const uint32_t *words = nullptr;
    const void *coef = nullptr;
    const double *coef64 = nullptr;
};
struct GateRun {
    void *psi = nullptr;
    int64_t N = 0;
    int batch = 1;
    bool by_rows = false;          // as GateProgram's
    int level = 0;
    const void *stage_diag = nullptr;
    const double *nrm2 = nullptr;
    double *norm_out = nullptr;    // partials of state b, tile t at [(b * tiles + t) * 4]
    int steps = 1;
    int32_t first[4] = {0, 0, 0, 0}, last[4] = {0, 0, 0, 0};   // step part q applies blocks [first[q], last[q])
};
int launch_gates(const GateLaunch &L, const GateTables &t, const GateRun &r, bool c128, bool stream_out, void *stream);

// Segments that deposit consecutive index bits into the set bits of `mask`.
std::vector<GateSeg> gate_segments(uint64_t mask);

}  // namespace hs
