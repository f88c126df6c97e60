// A Pauli sum by X-masks: row r couples with r ^ m by one coefficient per
// mask m, selected by parities of r.
#pragma once

#include <complex>
#include <cstdint>
#include <vector>

#include "hs_internal.h"

namespace hs {

constexpr int kPauliMaxRank = 4;     // parities of a mask's table
constexpr int kPauliMaxMasks = 4096;
// rows x states up to which a stage goes row by row: n = 18 8.4 us (tiles 10.0),
// n = 18 with 4 states 19.9 us (tiles 17.4)
constexpr int64_t kPauliRowsMax = int64_t(1) << 19;

// One mask as the kernels read it (64 bytes, one scalar load): its first two
// coefficients in the state's dtype, the whole table beside it.
struct PauliMask {
    uint32_t m;
    int32_t rank;
    int32_t tab;                     // first of its 2^rank coefficients (complex)
    uint32_t z0;                     // parity mask of table index bit 0
    double c[4];                     // coefficients 0 and 1, in complex64 as floats in the first 16 bytes
    uint32_t z[4];                   // parity masks of all index bits
};

struct PauliForm {
    std::vector<PauliMask> masks;    // m != 0, descending
    std::vector<uint32_t> m;         // their masks alone
    std::vector<std::complex<double>> tab;
};

// The form of a sum of `terms`, or false when a mask has more independent
// parities than a table holds or there are too many masks.  A coefficient sums
// its strings in term order, as a stored entry does.  A row sums the main diagonal
// and then the masks in descending order, where stored diagonals go by ascending
// offset: the one product that can differ from them in rounding.
bool pauli_form(const std::vector<Term> &terms, PauliForm &out);

struct PauliArgs {
    void *y;                         // y = x0 + alpha (H x); y may alias x0, not x
    const void *x, *x0;
    const void *diag;                // main diagonal, N entries of the dtype, or null
    int64_t N;
    int32_t nmask, nfar;
    const PauliMask *masks;
    const void *tab;                 // complex of the dtype
    double alpha_re, alpha_im;
    const uint32_t *host_masks;      // host copy of the masks
};
int launch_pauli_horner(PauliArgs a, int batch, bool c128, bool stream_out, void *stream);

}  // namespace hs
