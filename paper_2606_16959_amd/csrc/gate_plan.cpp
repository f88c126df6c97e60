// Host planning of the coset programs (gate_plan.h): plain C++, no device.

#include "gate_plan.h"

#include <algorithm>
#include <cmath>

namespace hs {
namespace {

int popc64(uint64_t v) { return __builtin_popcountll(v); }
uint64_t top_bit(uint64_t v) { return 1ull << (63 - __builtin_clzll(v)); }

// bits of v at the positions of `mask`, packed
uint64_t pack_bits(uint64_t v, uint64_t mask) {
    uint64_t o = 0;
    int j = 0;
    for (uint64_t m = mask; m; m &= m - 1, ++j) o |= ((v >> __builtin_ctzll(m)) & 1ull) << j;
    return o;
}
// the packed bits of v spread to the positions of `mask`
uint64_t spread_bits(uint64_t v, uint64_t mask) {
    uint64_t o = 0;
    for (uint64_t m = mask; m; m &= m - 1, v >>= 1)
        if (v & 1) o |= m & -m;
    return o;
}

// Fully reduced masks of the span of `masks`, by ascending highest bit.
std::vector<uint64_t> reduced_span(const std::vector<uint64_t> &masks) {
    std::vector<uint64_t> red;
    for (uint64_t v : masks) {
        for (uint64_t r : red)
            if (v & top_bit(r)) v ^= r;
        if (!v) continue;
        for (uint64_t &r : red)
            if (r & top_bit(v)) r ^= v;
        red.push_back(v);
    }
    std::sort(red.begin(), red.end());
    return red;
}

uint64_t combine(const std::vector<uint64_t> &basis, uint64_t j) {
    uint64_t v = 0;
    for (size_t c = 0; c < basis.size(); ++c)
        if ((j >> c) & 1) v ^= basis[c];
    return v;
}

}  // namespace

std::vector<GateSeg> gate_segments(uint64_t mask) {
    std::vector<GateSeg> out;
    int sh = 0;
    for (int q = 0; q < 64;) {
        if (!((mask >> q) & 1)) {
            ++q;
            continue;
        }
        int e = q;
        while (e < 64 && ((mask >> e) & 1)) ++e;
        const int len = e - q;
        out.push_back({sh, (uint32_t)((1ull << len) - 1), q});
        sh += len;
        q = e;
    }
    return out;
}

std::vector<uint64_t> gate_basis(const Plan &P, int factor) {
    std::vector<uint64_t> masks;
    for (int k : P.factors[factor].terms) masks.push_back(P.terms[k].x);
    return reduced_span(masks);
}

GateStep gate_step(const Plan &P, int factor, int pos) {
    const Factor &F = P.factors[factor];
    GateStep g;
    g.factor = factor;
    g.pos = pos;
    g.carries_d = F.has_diag;
    g.diag_only = F.terms.empty();
    if (g.diag_only) return g;
    for (int k : F.terms) g.flips |= P.terms[k].x;
    g.basis = gate_basis(P, factor);
    const int rho = (int)g.basis.size(), R = 1 << rho, K = 1 << F.bits.size();
    uint64_t support = 0;
    for (int q : F.bits) support |= 1ull << q;
    const uint64_t free_bits = support & ~g.pivots();
    for (int q : F.bits)
        if ((free_bits >> q) & 1) g.type_bits.push_back(q);
    // every nonzero entry couples rows of one coset
    std::vector<char> span(K, 0);
    for (int j = 0; j < R; ++j) span[pack_bits(combine(g.basis, j), support)] = 1;
    for (int a = 0; a < K; ++a)
        for (int b = 0; b < K; ++b)
            if (!span[a ^ b] && F.L[(size_t)a * K + b] != 0.0) g.closed = false;
    // the products, one per setting of the free support bits; local indices are
    // linear over XOR
    const int types = 1 << g.type_bits.size();
    std::vector<int> el(R), ty(types);
    for (int j = 0; j < R; ++j) el[j] = (int)pack_bits(combine(g.basis, j), support);
    for (int t = 0; t < types; ++t) ty[t] = (int)pack_bits(spread_bits((uint64_t)t, free_bits), support);
    auto at = [&](int t, int i, int j) { return F.L[(size_t)(ty[t] ^ el[i]) * K + (ty[t] ^ el[j])]; };
    // one parity of the flip that decides between real and imaginary entries
    // (unit flips first; every entry must agree)
    std::vector<int> kd(R, 0);       // by flip: 1 real, 2 imaginary entries
    for (int t = 0; t < types; ++t)
        for (int i = 0; i < R; ++i)
            for (int j = 0; j < R; ++j) {
                const std::complex<double> v = at(t, i, j);
                kd[i ^ j] |= (v.real() != 0.0 ? 1 : 0) | (v.imag() != 0.0 ? 2 : 0);
            }
    bool typed = false;
    for (int km = R - 1; km >= 0 && !typed; --km) {      // R <= 1024; R - 1 (every flip imaginary) fits most
        bool ok = true;
        for (int m = 0; m < R && ok; ++m) ok = (kd[m] & ~((popc64(m & km) & 1) ? 2 : 1)) == 0;
        if (ok) {
            typed = true;
            g.kmask = km;
        }
    }
    g.form = typed ? (g.carries_d ? kGateRealD : kGateReal) : (g.carries_d ? kGateComplexD : kGateComplex);
    std::vector<char> kap(R);
    for (int j = 0; j < R; ++j) kap[j] = (char)(popc64(j & g.kmask) & 1);
    auto out = std::make_shared<std::vector<double>>();
    out->reserve((size_t)types * R * R * (typed ? 1 : 2));
    for (int t = 0; t < types; ++t)
        for (int p = 0; p < R; ++p)
            for (int q = 0; q < R; ++q) {
                const int i = g.carries_d ? q : p, j = g.carries_d ? p : q;
                const std::complex<double> v = at(t, i, j);
                if (!typed) {
                    out->push_back(v.real());
                    out->push_back(v.imag());
                } else if (kap[i] == kap[j]) {
                    out->push_back(v.real());
                } else {
                    out->push_back(!g.carries_d && kap[i] ? -v.imag() : v.imag());
                }
            }
    g.entries = out;
    return g;
}

std::vector<GateStep> gate_steps(const Plan &P, const std::vector<int> &seq, std::map<int, GateStep> *made) {
    std::map<int, GateStep> own;
    if (!made) made = &own;
    std::vector<GateStep> out;
    for (size_t pos = 0; pos < seq.size(); ++pos) {
        auto it = made->find(seq[pos]);
        if (it == made->end()) it = made->emplace(seq[pos], gate_step(P, seq[pos], 0)).first;
        out.push_back(it->second);
        out.back().pos = (int)pos;
    }
    return out;
}

void gate_launches(const Plan &P, const std::vector<GateStep> &steps, int kt, int wlog, int max_factors, bool loop,
                   GateProgram &out) {
    const uint64_t all = (1ull << P.n) - 1;
    kt = loop ? P.n : std::min(kt, P.n);
    wlog = std::min(wlog, kt);
    size_t i = 0;
    while (i < steps.size()) {
        // the run of steps one tile holds
        uint64_t need = 0;
        size_t j = i;
        int w = wlog;
        while (j < steps.size()) {
            const uint64_t nx = need | steps[j].flips;
            if (!loop && max_factors > 0 && (int)(j - i) >= max_factors) break;
            if (popc64(nx | ((1ull << w) - 1)) > kt) {
                if (j > i) break;
                // a single wide factor: shorten the runs, down to row pairs
                while (w > 1 && popc64(nx | ((1ull << w) - 1)) > kt) --w;
            }
            need = nx;
            ++j;
        }
        GateLaunch L;
        L.first = (int)i;
        L.count = (int)(j - i);
        uint64_t tile = (need | ((1ull << w) - 1)) & all;
        for (int q = 0; q < P.n && popc64(tile) < kt; ++q) tile |= 1ull << q;
        L.tile = tile;
        L.kt = popc64(tile);
        L.rows = int64_t(1) << L.kt;
        L.in = gate_segments(tile);
        L.out = gate_segments(all & ~tile);
        L.block0 = (int)out.blocks.size();
        for (size_t q = i; q < j; ++q) {
            const GateStep &g = steps[q];
            out.closed = out.closed && g.closed && (g.flips & ~tile) == 0;
            if (g.diag_only && q == i && !loop) {
                L.stage_diag = g.factor;
                continue;
            }
            GateBlock b{};
            out.dfactor.push_back(g.carries_d ? g.factor : -1);
            if (g.diag_only) {
                b.what = kGateDiag;
                out.blocks.push_back(b);
                continue;
            }
            std::vector<uint64_t> loc;
            uint64_t piv = 0, types = 0;
            for (uint64_t v : g.basis) {
                loc.push_back(pack_bits(v, tile));
                piv |= top_bit(loc.back());
            }
            const uint32_t rho = (uint32_t)loc.size(), nz = (uint32_t)g.type_bits.size();
            b.ztab = (int)out.words.size();
            for (int zb : g.type_bits) {
                const uint64_t z = 1ull << zb, zl = pack_bits(z & tile, tile);
                types |= zl;
                out.words.push_back((uint32_t)zl);
                out.words.push_back((uint32_t)(z & ~tile));
            }
            std::vector<double> &dst = g.carries_d ? out.coef64 : out.coef;
            const bool pairs = g.form == kGateComplex || g.form == kGateComplexD;
            auto tab = out.coef_of.find(g.factor);        // a factor's entries are held once
            if (tab == out.coef_of.end()) {
                while (dst.size() % 4) dst.push_back(0.0);
                tab = out.coef_of.emplace(g.factor, (int)(dst.size() / (pairs ? 2 : 1))).first;
                dst.insert(dst.end(), g.entries->begin(), g.entries->end());
            }
            b.coef = tab->second;
            const bool rows = rho > (uint32_t)kGateMaxCoset || pairs;
            if (rows || g.kmask != (1 << rho) - 1) out.level = std::max(out.level, rho > (uint32_t)kGateMaxCoset ? 2 : 1);
            b.what = (rows ? kGateRows : kGateCosets) | rho << 4 | (uint32_t)g.form << 8 | nz << 12 |
                     (uint32_t)g.kmask << 16;
            if (rows) {
                b.wtab = (int)out.words.size();
                for (uint64_t v : loc) out.words.push_back((uint32_t)(63 - __builtin_clzll(v)));
                for (uint64_t v : loc) out.words.push_back((uint32_t)v);
                for (uint64_t v : g.basis) out.words.push_back((uint32_t)(63 - __builtin_clzll(v)));
                if (rho <= (uint32_t)kGateMaxCoset) {
                    out.by_rows = true;
                } else {
                    // 64 cosets per type: one type and one piece of the matrix per wave
                    const uint32_t free_bits = (uint32_t)L.kt - rho, nt = (uint32_t)popc64(types);
                    const bool lane = free_bits < nt + 6;
                    const uint64_t held = lane ? 0 : types, holes = piv | held;
                    b.number = (uint32_t)popc64(holes) | (uint32_t)popc64(held) << 8 |
                               (free_bits - (uint32_t)popc64(held)) << 16 | (lane ? 1u << 24 : 0u);
                    for (uint64_t p = holes; p; p &= p - 1) out.words.push_back((uint32_t)__builtin_ctzll(p));
                    for (uint64_t p = held; p; p &= p - 1) out.words.push_back((uint32_t)__builtin_ctzll(p));
                    for (uint64_t j = 0; j < 1ull << rho; j += 4) out.words.push_back((uint32_t)combine(loc, j));
                }
                out.blocks.push_back(b);
                continue;
            }
            const uint32_t nt = (uint32_t)popc64(types);
            uint64_t holes = piv;
            uint32_t ntype = 0, nhole = 0;
            // 64 cosets per type: one type per wave (type bits outside the
            // tile are one for the workgroup)
            if (nt && nt <= (uint32_t)kGateMaxType && L.kt >= (int)(rho + nt) + 6) {
                holes |= types;
                ntype = nt;
            }
            const bool inside = nt == nz && nz <= 4;
            if (nt <= 4) {
                int k = 0;
                for (uint64_t p = types; p; p &= p - 1) b.tpos |= (uint32_t)__builtin_ctzll(p) << (8 * k++);
            }
            for (uint64_t p = holes; p; p &= p - 1) b.holes |= (uint64_t)__builtin_ctzll(p) << (8 * nhole++);
            b.number = nhole | ntype << 8 | ((uint32_t)L.kt - rho - ntype) << 16 | (nt && !ntype ? 1u << 24 : 0u) |
                       (inside ? 1u << 25 : 0u) |
                       (ntype && ntype == nz ? 1u << 28 : 0u);
            for (uint32_t c = 0; c < rho; ++c) {
                b.basis[c] = (uint32_t)loc[c];
                b.rpivots |= (uint32_t)(63 - __builtin_clzll(g.basis[c])) << (8 * c);
            }
            out.blocks.push_back(b);
        }
        L.block1 = (int)out.blocks.size();
        out.launches.push_back(L);
        i = j;
    }
}

}  // namespace hs
