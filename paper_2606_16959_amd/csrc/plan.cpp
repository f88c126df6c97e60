// Host planning: Pauli parsing, first-fit grouping under the diagonal budget,
// local unitaries and the structural dry run that fixes each factor's
// diagonal set before any storage exists (paper: Eq. 4 and Eq. 5 applied per
// factor, Section 3.1; Eq. 6 and the "structural dry run", Section 3.2).
//
// Reading of the grouping (the paper does not describe how the H_j of Eq. 4
// are formed): Z-only terms form the diagonal factor; every other term joins
// the first existing group whose members it all commutes with and whose exact
// exponential stays within the budget, else it opens a new group.  Because a
// group's members commute and each Pauli squares to I, the group exponential
// is exactly prod_k (cos(c_k dt) I - i sin(c_k dt) P_k).

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <map>
#include <set>

#include "hs_internal.h"
#include "pauli_form.h"

namespace hs {
namespace {

int popc(uint64_t v) { return __builtin_popcountll(v); }

bool commute(const Term &a, const Term &b) {
    return ((popc(a.x & b.z) + popc(a.z & b.x)) & 1) == 0;
}

uint64_t pext_bits(uint64_t v, const std::vector<int> &bits) {
    uint64_t o = 0;
    for (size_t j = 0; j < bits.size(); ++j) o |= ((v >> bits[j]) & 1ull) << j;
    return o;
}

int64_t spread_bits(uint64_t a, const std::vector<int> &bits) {
    int64_t o = 0;
    for (size_t j = 0; j < bits.size(); ++j) o |= (int64_t)((a >> j) & 1ull) << bits[j];
    return o;
}

// The product over members (first member applied first) of
// cos(th) I - i sin(th) P, restricted to the support bits, with
// P[y, y^m] = i^ny (-1)^{popcount((y^m) & z)}.  Row y has entries only at
// y ^ s for s in the span of the members' flips, so the product is kept as
// those: masks in ascending order, entry (y, y ^ masks[j]) at v[y * S + j].
struct LocalUnitary {
    std::vector<int> bits;
    std::vector<uint64_t> masks;
    std::vector<std::complex<double>> v;
};

void local_unitary(const std::vector<Term> &terms, const std::vector<int> &members, double dt, LocalUnitary &u) {
    uint64_t s = 0;
    for (int k : members) s |= terms[k].x | terms[k].z;
    u.bits.clear();
    for (int q = 0; q < 64; ++q)
        if ((s >> q) & 1ull) u.bits.push_back(q);
    const uint64_t K = 1ull << u.bits.size();
    u.masks.assign(1, 0);
    u.v.assign(K, 1.0);
    std::vector<std::complex<double>> nv;
    std::vector<uint64_t> nm;
    std::vector<int> own, other;                // index of a new mask, and of it ^ m, among the old; -1 none
    static const std::complex<double> ipow[4] = {{1, 0}, {0, 1}, {-1, 0}, {0, -1}};
    auto find = [&](uint64_t m) {
        auto it = std::lower_bound(u.masks.begin(), u.masks.end(), m);
        return it != u.masks.end() && *it == m ? (int)(it - u.masks.begin()) : -1;
    };
    for (int k : members) {
        const Term &t = terms[k];
        const uint64_t m = pext_bits(t.x, u.bits), z = pext_bits(t.z, u.bits);
        const double th = t.c * dt;
        const double c = std::cos(th), sn = std::sin(th);
        const std::complex<double> ph = ipow[t.ny & 3];
        nm = u.masks;
        if (find(m) < 0)
            for (uint64_t q : u.masks) nm.push_back(q ^ m);
        std::sort(nm.begin(), nm.end());
        const size_t S = u.masks.size(), NS = nm.size();
        own.assign(NS, -1);
        other.assign(NS, -1);
        for (size_t j = 0; j < NS; ++j) {
            own[j] = find(nm[j]);
            other[j] = find(nm[j] ^ m);
        }
        nv.assign(K * NS, 0.0);
        for (uint64_t y = 0; y < K; ++y) {
            const uint64_t src = y ^ m;
            const double sg = (popc(src & z) & 1) ? -1.0 : 1.0;
            // -i sin(th) * (i^ny * sg)
            const std::complex<double> w = std::complex<double>(0.0, -sn) * (ph * sg);
            for (size_t j = 0; j < NS; ++j) {
                const std::complex<double> a = own[j] < 0 ? 0.0 : u.v[y * S + own[j]];
                const std::complex<double> b = other[j] < 0 ? 0.0 : u.v[src * S + other[j]];
                nv[y * NS + j] = c * a + w * b;
            }
        }
        u.masks.swap(nm);
        u.v.swap(nv);
    }
}

// Offsets spr(y ^ s) - spr(y) of the entries above the threshold, ascending;
// zeroes the rest.
std::vector<int64_t> offsets_of(LocalUnitary &u) {
    const size_t K = (size_t)1 << u.bits.size(), S = u.masks.size();
    std::vector<int64_t> spr(K), offs;
    for (size_t a = 0; a < K; ++a) spr[a] = spread_bits((uint64_t)a, u.bits);
    offs.reserve(K * S);
    for (size_t y = 0; y < K; ++y)
        for (size_t j = 0; j < S; ++j) {
            std::complex<double> &v = u.v[y * S + j];
            if (std::abs(v) > kTau)
                offs.push_back(spr[y ^ u.masks[j]] - spr[y]);
            else
                v = 0.0;
        }
    std::sort(offs.begin(), offs.end());
    offs.erase(std::unique(offs.begin(), offs.end()), offs.end());
    return offs;
}

// K x K row-major matrix
std::vector<std::complex<double>> dense(const LocalUnitary &u) {
    const size_t K = (size_t)1 << u.bits.size(), S = u.masks.size();
    std::vector<std::complex<double>> L(K * K, 0.0);
    for (size_t y = 0; y < K; ++y)
        for (size_t j = 0; j < S; ++j) L[y * K + (y ^ u.masks[j])] = u.v[y * S + j];
    return L;
}

bool support_ok(const std::vector<Term> &terms, const std::vector<int> &members) {
    uint64_t s = 0;
    for (int k : members) s |= terms[k].x | terms[k].z;
    return popc(s) <= HS_MAX_SUPPORT;
}

int count_diags(const std::vector<Term> &terms, const std::vector<int> &members, double dt) {
    LocalUnitary u;
    local_unitary(terms, members, dt, u);
    return (int)offsets_of(u).size();
}

}  // namespace

hs_status parse_terms(int n, int n_terms, const char *const *strings, const double *coeffs,
                      std::vector<Term> &terms, std::string &msg) {
    char buf[256];
    terms.clear();
    double cmax = 0.0;
    for (int k = 0; k < n_terms; ++k) {
        const double re = coeffs[2 * k], im = coeffs[2 * k + 1];
        if (!std::isfinite(re) || !std::isfinite(im)) { msg = "non-finite coefficient"; return HS_EINVAL; }
        cmax = std::max(cmax, std::hypot(re, im));
    }
    for (int k = 0; k < n_terms; ++k) {
        if (std::fabs(coeffs[2 * k + 1]) > 1e-12 * cmax) {
            snprintf(buf, sizeof buf, "term %d has imaginary coefficient %.3g: H is not Hermitian", k,
                     coeffs[2 * k + 1]);
            msg = buf;
            return HS_ENONHERMITIAN;
        }
        const char *s = strings[k];
        if (!s) { msg = "null Pauli string"; return HS_EINVAL; }
        Term tm;
        int len = 0;
        for (; s[len]; ++len) {
            if (len >= n) break;
            const uint64_t bit = 1ull << len;
            switch (s[len]) {
                case 'I': break;
                case 'X': tm.x |= bit; break;
                case 'Z': tm.z |= bit; break;
                case 'Y': tm.x |= bit; tm.z |= bit; ++tm.ny; break;
                default:
                    snprintf(buf, sizeof buf, "term %d: bad Pauli character '%c'", k, s[len]);
                    msg = buf;
                    return HS_EINVAL;
            }
        }
        if (len != n || s[len] != '\0') {
            snprintf(buf, sizeof buf, "term %d: string length differs from n_qubits=%d", k, n);
            msg = buf;
            return HS_EINVAL;
        }
        tm.c = coeffs[2 * k];
        terms.push_back(tm);
    }

    return HS_OK;
}

bool pauli_form(const std::vector<Term> &terms, PauliForm &out) {
    static const std::complex<double> ipow[4] = {{1, 0}, {0, 1}, {-1, 0}, {0, -1}};
    out = PauliForm();
    std::map<uint64_t, std::vector<const Term *>> by_mask;
    for (const Term &t : terms)
        if (t.x) by_mask[t.x].push_back(&t);
    if (by_mask.size() > (size_t)kPauliMaxMasks) return false;
    for (auto it = by_mask.rbegin(); it != by_mask.rend(); ++it) {
        const uint64_t m = it->first;
        PauliMask k{};
        k.m = (uint32_t)m;
        k.tab = (int32_t)out.tab.size();
        // independent parity masks, and the sums of them that give each term's
        std::vector<uint64_t> basis;
        auto pattern = [&](uint64_t z) {
            for (uint32_t q = 0; q < (1u << basis.size()); ++q) {
                uint64_t v = 0;
                for (size_t j = 0; j < basis.size(); ++j)
                    if ((q >> j) & 1) v ^= basis[j];
                if (v == z) return (int)q;
            }
            return -1;
        };
        for (const Term *t : it->second)
            if (pattern(t->z) < 0) {
                if (basis.size() == (size_t)kPauliMaxRank) return false;
                basis.push_back(t->z);
            }
        k.rank = (int32_t)basis.size();
        for (size_t j = 0; j < basis.size(); ++j) k.z[j] = (uint32_t)basis[j];
        k.z0 = k.z[0];
        bool any = false;
        for (uint32_t q = 0; q < (1u << basis.size()); ++q) {
            std::complex<double> h = 0.0;
            for (const Term *t : it->second) {
                // parity of (r ^ m) & z, r's own parities being q
                const int odd = (popc((uint64_t)(q & (uint32_t)pattern(t->z))) + popc(m & t->z)) & 1;
                h += ipow[t->ny & 3] * (odd ? -t->c : t->c);
            }
            any = any || h != 0.0;
            out.tab.push_back(h);
        }
        if (!any) {                  // cancelling strings
            out.tab.resize(k.tab);
            continue;
        }
        const std::complex<double> c0 = out.tab[k.tab], c1 = out.tab[k.tab + (k.rank ? 1 : 0)];
        k.c[0] = c0.real();
        k.c[1] = c0.imag();
        k.c[2] = c1.real();
        k.c[3] = c1.imag();
        out.masks.push_back(k);
        out.m.push_back(k.m);
    }
    return true;
}

void layout_factor(Factor &f, int64_t N, size_t elem_bytes) {
    const size_t align = kDiagAlignBytes / elem_bytes;
    size_t pos = 0;
    f.elem_off.clear();
    for (int64_t d : f.offs) {
        f.elem_off.push_back(pos);
        const size_t len = (size_t)(N - (d < 0 ? -d : d));
        pos += (len + align - 1) / align * align;
    }
    f.elems_total = pos;
}

hs_status make_plan(int n, int n_terms, const char *const *strings, const double *coeffs,
                    double t, int steps, int budget, unsigned flags, Plan &P, std::string &msg) {
    char buf[256];
    if (n < 1 || n > HS_MAX_QUBITS) {
        snprintf(buf, sizeof buf, "n_qubits=%d outside [1, %d]", n, HS_MAX_QUBITS);
        msg = buf;
        return n > HS_MAX_QUBITS ? HS_ETOOLARGE : HS_EINVAL;
    }
    if (n_terms < 1 || !strings || !coeffs) { msg = "need n_terms >= 1, strings and coeffs"; return HS_EINVAL; }
    if (steps < 1) { msg = "steps must be >= 1"; return HS_EINVAL; }
    if (budget < 1) { msg = "budget must be >= 1"; return HS_EINVAL; }
    if (!std::isfinite(t)) { msg = "t must be finite"; return HS_EINVAL; }
    if (flags & ~(unsigned)(HS_MERGE_DIAG | HS_ORDER2 | HS_ORDER4)) { msg = "unknown build flag"; return HS_EINVAL; }
    if ((flags & HS_ORDER2) && (flags & HS_ORDER4)) { msg = "choose one product order"; return HS_EINVAL; }

    P = Plan();
    P.n = n;
    P.N = (int64_t)1 << n;
    P.t = t;
    P.steps = steps;
    P.dt = t / steps;
    P.budget = budget;
    P.flags = flags;

    if (hs_status st = parse_terms(n, n_terms, strings, coeffs, P.terms, msg)) return st;

    // first-fit grouping
    std::vector<std::vector<int>> groups;
    for (int i = 0; i < n_terms; ++i) {
        const Term &t = P.terms[i];
        if (t.x == 0) { P.diag.push_back(i); continue; }
        bool placed = false;
        for (auto &g : groups) {
            bool ok = true;
            for (int j : g)
                if (!commute(t, P.terms[j])) { ok = false; break; }
            if (!ok) continue;
            std::vector<int> cand = g;
            cand.push_back(i);
            if (!support_ok(P.terms, cand)) continue;
            if (count_diags(P.terms, cand, P.dt) <= budget) {
                g.push_back(i);
                placed = true;
                break;
            }
        }
        if (!placed) {
            std::vector<int> one{i};
            if (!support_ok(P.terms, one)) {
                snprintf(buf, sizeof buf, "term %d acts on more than %d qubits", i, HS_MAX_SUPPORT);
                msg = buf;
                return HS_ETOOLARGE;
            }
            const int nd = count_diags(P.terms, one, P.dt);
            if (nd > budget) {
                snprintf(buf, sizeof buf, "term %d alone needs %d diagonals > budget %d", i, nd, budget);
                msg = buf;
                return HS_EBUDGET;
            }
            groups.push_back(one);
        }
    }

    auto diag_factor = [&](double h) {
        Factor d;
        d.has_diag = true;
        d.dt = h;
        d.offs = {0};
        for (int k : P.diag) d.smask |= P.terms[k].z;
        return d;
    };
    auto group_factor = [&](const std::vector<int> &g, double h, bool with_diag) {
        Factor f;
        f.has_diag = with_diag;
        f.dt = h;
        f.terms = g;
        LocalUnitary u;
        local_unitary(P.terms, f.terms, h, u);
        f.offs = offsets_of(u);
        f.bits = u.bits;
        f.L = dense(u);
        for (int q : f.bits) f.smask |= 1ull << q;
        for (int k : f.terms) f.xmask_union |= P.terms[k].x;
        return f;
    };
    P.order = (flags & HS_ORDER4) ? 4 : (flags & HS_ORDER2) ? 2 : 1;
    if (P.order == 1) {
        const bool merge = (flags & HS_MERGE_DIAG) != 0;
        if (!P.diag.empty() && (!merge || groups.empty())) P.factors.push_back(diag_factor(P.dt));
        for (size_t j = 0; j < groups.size(); ++j)
            P.factors.push_back(group_factor(groups[j], P.dt, merge && j == 0 && !P.diag.empty()));
        for (size_t k = 0; k < P.factors.size(); ++k) P.seq.push_back((int)k);
    } else {
        // Symmetric products over F = (D, G_1, ..., G_m): S2(h) applies
        // F_1..F_{L-1} with h/2, F_L with h, then F_{L-1}..F_1 with h/2;
        // S4(dt) = S2(p dt) S2(p dt) S2((1-4p) dt) S2(p dt) S2(p dt),
        // p = 1/(4 - 4^(1/3)).  D stays a factor of its own; every distinct
        // (factor, time step) pair is stored once.
        const int L = (P.diag.empty() ? 0 : 1) + (int)groups.size();
        std::vector<std::pair<int, double>> seq;     // (F index, h); F index 0 = D when present
        auto s2 = [&](double h) {
            if (L == 1) { seq.push_back({0, h}); return; }
            for (int j = 0; j < L - 1; ++j) seq.push_back({j, h / 2});
            seq.push_back({L - 1, h});
            for (int j = L - 2; j >= 0; --j) seq.push_back({j, h / 2});
        };
        if (P.order == 2) {
            s2(P.dt);
        } else {
            const double p = 1.0 / (4.0 - std::pow(4.0, 1.0 / 3.0));
            s2(p * P.dt);
            s2(p * P.dt);
            s2((1 - 4 * p) * P.dt);
            s2(p * P.dt);
            s2(p * P.dt);
        }
        // Neighbours with the same generator combine, exp(-i a G) exp(-i b G) =
        // exp(-i (a + b) G): S4's junctions F_1(p dt/2) F_1(p dt/2) and the
        // like.  Sums are taken left to right.
        std::vector<std::pair<int, double>> merged;
        for (auto &e : seq) {
            if (!merged.empty() && merged.back().first == e.first) merged.back().second += e.second;
            else merged.push_back(e);
        }
        std::map<std::pair<int, double>, int> made;
        auto stored = [&](const std::pair<int, double> &e) {
            auto it = made.find(e);
            if (it == made.end()) {
                const bool is_diag = !P.diag.empty() && e.first == 0;
                const int g = e.first - (P.diag.empty() ? 0 : 1);
                P.factors.push_back(is_diag ? diag_factor(e.second) : group_factor(groups[g], e.second, false));
                it = made.emplace(e, (int)P.factors.size() - 1).first;
            }
            return it->second;
        };
        for (auto &e : merged) P.seq.push_back(stored(e));
        // A symmetric step starts and ends with F_1, so consecutive steps meet
        // in F_1(last h) F_1(first h): stored once as the joint factor.
        if (merged.size() > 1 && merged.front().first == merged.back().first)
            P.joint = stored({merged.front().first, merged.back().second + merged.front().second});
    }
    for (auto &f : P.factors) {
        if (f.xmask_union) {
            f.xlb = __builtin_ctzll(f.xmask_union);
            f.xhb = 64 - __builtin_clzll(f.xmask_union);
        }
    }
    return HS_OK;
}

}  // namespace hs
