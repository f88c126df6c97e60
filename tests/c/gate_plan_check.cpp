// The coset programs of the evolution (gate_plan.h), walked on the host
// the way the kernel walks them and compared with exact Pauli rotations:
// seeded random Pauli sums (1..12 qubits, supports anywhere, every product
// order, merged or separate diagonal factor), tiles from 4 rows to the whole
// state, both coset sizes, capped factor counts and the looped whole-state
// form.  Also: tiles and cosets cover every row once, and LDS positions are a
// permutation.  Built with g++ and the sanitizers by the CPU tests.
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <string>
#include <vector>

#include "../../paper_2606_16959_amd/csrc/gate_plan.h"

typedef std::complex<double> cd;

static uint32_t deposit(const std::vector<hs::GateSeg> &s, uint32_t i) {
    uint32_t r = 0;
    for (auto &g : s) r |= ((i >> g.sh) & g.mask) << g.dst;
    return r;
}

// the product as exact rotations, one term at a time
static void direct(const hs::Plan &P, const std::vector<int> &seq, std::vector<cd> &psi) {
    static const cd ip[4] = {{1, 0}, {0, 1}, {-1, 0}, {0, -1}};
    for (int f : seq) {
        const hs::Factor &F = P.factors[f];
        if (F.has_diag)
            for (int64_t x = 0; x < P.N; ++x) {
                double E = 0;
                for (int k : P.diag) E += P.terms[k].c * (__builtin_popcountll(x & P.terms[k].z) & 1 ? -1.0 : 1.0);
                psi[x] *= std::polar(1.0, -F.dt * E);
            }
        for (int k : F.terms) {
            const hs::Term &t = P.terms[k];
            std::vector<cd> y(psi.size());
            for (int64_t r = 0; r < P.N; ++r) {
                const int64_t x = r ^ (int64_t)t.x;
                const cd p = ip[t.ny & 3] * (__builtin_popcountll(x & t.z) & 1 ? -1.0 : 1.0);
                y[r] = std::cos(t.c * F.dt) * psi[r] - cd(0, 1) * std::sin(t.c * F.dt) * p * psi[x];
            }
            psi.swap(y);
        }
    }
}

static int pop(uint64_t v) { return __builtin_popcountll(v) & 1; }

// entry M[i][j] of an operation, as the kernel reads its table (D excluded)
static cd entry(const hs::GateProgram &G, const hs::GateBlock &op, int64_t type, int i, int j) {
    const int R = 1 << op.rho();
    const int ki = pop(i & op.kmask()), kj = pop(j & op.kmask());
    const int64_t tab = op.coef + type * R * R;
    switch (op.form()) {
        case hs::kGateReal: {          // M = i^(kappa_j - kappa_i) M'
            const double m = G.coef[tab + i * R + j];
            return ki == kj ? cd(m, 0) : (ki ? cd(0, -m) : cd(0, m));
        }
        case hs::kGateComplex: return cd(G.coef[2 * (tab + i * R + j)], G.coef[2 * (tab + i * R + j) + 1]);
        case hs::kGateRealD: return ki == kj ? cd(G.coef64[tab + j * R + i], 0) : cd(0, G.coef64[tab + j * R + i]);
        default: return cd(G.coef64[2 * (tab + j * R + i)], G.coef64[2 * (tab + j * R + i) + 1]);
    }
}

static int walk(const hs::Plan &P, const hs::GateProgram &G, const hs::GateLaunch &L, std::vector<cd> &psi) {
    auto diag = [&](int factor, int64_t x) {
        double E = 0;
        for (int k : P.diag) E += P.terms[k].c * (__builtin_popcountll(x & P.terms[k].z) & 1 ? -1.0 : 1.0);
        return std::polar(1.0, -P.factors[factor].dt * E);
    };
    const int T = 1 << L.kt;
    std::vector<char> seen(P.N, 0);
    for (int64_t tile = 0; tile < P.N / L.rows; ++tile) {
        const uint32_t base = deposit(L.out, (uint32_t)tile);
        std::vector<cd> lds(T, 0.0);
        for (int i = 0; i < T; ++i) {
            const int64_t r = base | deposit(L.in, i);
            if (r >= P.N || seen[r]++) return 1;
            if ((i & 1) && r != (int64_t)(base | deposit(L.in, i - 1)) + 1) return 2;   // pairs adjacent
            lds[i] = psi[r];
            if (L.stage_diag >= 0) lds[i] *= diag(L.stage_diag, r);
        }
        for (int k = L.block0; k < L.block1; ++k) {
            const hs::GateBlock &B = G.blocks[k];
            const int df = G.dfactor[k], R = 1 << B.rho();
            if (B.kind() == hs::kGateDiag) {
                for (int i = 0; i < T; ++i) lds[i] *= diag(df, base | deposit(L.in, i));
                continue;
            }
            const bool rows = B.kind() == hs::kGateRows;
            if (!rows && (B.rho() > hs::kGateMaxCoset || B.form() == hs::kGateComplex || B.form() == hs::kGateComplexD)) return 5;
            const uint32_t *w = rows ? &G.words[B.wtab] : nullptr;
            std::vector<char> hit(T, 0);
            int64_t wave_type = 0;
            for (int t = 0; t < (T >> B.rho()); ++t) {
                int rep = t;
                if (rows) {                            // the t-th row with its pivot bits 0
                    for (int c = 0; c < B.rho(); ++c) {
                        const int low = (1 << w[c]) - 1;
                        rep = ((rep & ~low) << 1) | (rep & low);
                    }
                } else {
                    if (B.nhole() != B.rho() + B.ntype() || B.tshift() != L.kt - B.rho() - B.ntype()) return 3;
                    rep = B.ntype() ? t & ((1 << B.tshift()) - 1) : t;
                    for (int h = 0; h < B.nhole(); ++h) {
                        const int low = (1 << B.hole(h)) - 1;
                        rep = ((rep & ~low) << 1) | (rep & low);
                    }
                    for (int q = 0; q < B.ntype(); ++q)
                        rep |= ((t >> (B.tshift() + q)) & 1) << ((B.tpos >> (8 * q)) & 31);
                }
                int64_t type = 0;
                for (int z = 0; z < B.nz(); ++z)
                    type |= (int64_t)(((rep & G.words[B.ztab + 2 * z]) | (base & G.words[B.ztab + 2 * z + 1])) != 0) << z;
                if (!rows && B.direct() && type != (t >> B.tshift())) return 12;
                if (!rows && B.inside()) {
                    int64_t at_pos = 0;
                    for (int z = 0; z < B.nz(); ++z) at_pos |= (int64_t)((rep >> (B.tpos >> (8 * z) & 31)) & 1) << z;
                    if (at_pos != type) return 13;
                }
                if ((t & 63) == 0) wave_type = type;
                if (!rows && !B.lane() && type != wave_type) return 11;    // one matrix per wave
                std::vector<cd> y(R, 0.0);
                std::vector<int> at(R);
                for (int j = 0; j < R; ++j) {
                    at[j] = rep;
                    for (int q = 0; q < B.rho(); ++q)
                        if ((j >> q) & 1) at[j] ^= (int)(rows ? w[B.rho() + q] : B.basis[q]);
                    if (at[j] < 0 || at[j] >= T || hit[at[j]]++ || (j && at[j] <= at[j - 1])) return 4;
                    const int64_t row = base | deposit(L.in, at[j]);
                    int own = 0;                       // a row's coordinate is its pivot bits
                    for (int c = 0; c < B.rho(); ++c) own |= (int)((row >> (rows ? w[2 * B.rho() + c] : B.rpiv(c))) & 1) << c;
                    if (own != j) return 7;
                    cd x = lds[at[j]];
                    if (df >= 0) x *= diag(df, row);
                    for (int i = 0; i < R; ++i) y[i] += entry(G, B, type, i, j) * x;
                }
                for (int i = 0; i < R; ++i) lds[at[i]] = y[i];
            }
        }
        for (int i = 0; i < T; ++i) psi[base | deposit(L.in, i)] = lds[i];
    }
    for (int64_t r = 0; r < P.N; ++r)
        if (!seen[r]) return 6;
    return 0;
}

int main() {
    for (int c128 = 0; c128 < 2; ++c128)
        for (int T = 2; T <= 16384; T *= 2) {
            std::vector<char> hit(T, 0);
            for (int i = 0; i < T; ++i) {
                const int p = hs::gate_lds_pos(i, c128), m = (i * 2654435761u) % T;
                if (p < 0 || p >= T || hit[p]++) { std::printf("lds position T=%d i=%d\n", T, i); return 1; }
                if (hs::gate_lds_pos(i ^ m, c128) != (p ^ hs::gate_lds_pos(m, c128))) { std::printf("not linear\n"); return 1; }
            }
        }
    std::mt19937_64 rng(7);
    int checked = 0;
    for (int it = 0; it < 120; ++it) {
        const int n = 1 + (int)(rng() % 12);
        const int nt = 1 + (int)(rng() % 18);
        const char *paulis = it % 3 == 0 ? "XYYX" : "IXYZ";
        std::vector<std::string> s(nt, std::string(n, 'I'));
        std::vector<double> c(2 * nt, 0.0);
        for (int k = 0; k < nt; ++k) {
            const int w = 1 + (int)(rng() % 4);
            for (int j = 0; j < w; ++j) s[k][rng() % n] = paulis[rng() % 4];
            if (k && rng() % 4 == 0) {        // a neighbour that flips the same bits
                s[k] = s[k - 1];
                for (int q = 0; q < n; ++q) {
                    if (s[k][q] == 'X' && rng() % 2) s[k][q] = 'Y';
                    else if (s[k][q] == 'I' && rng() % 4 == 0) s[k][q] = 'Z';
                }
            }
            c[2 * k] = std::uniform_real_distribution<double>(-2.0, 2.0)(rng);
        }
        std::vector<const char *> sp(nt);
        for (int k = 0; k < nt; ++k) sp[k] = s[k].c_str();
        const unsigned flags = (rng() % 2 ? HS_MERGE_DIAG : 0u) | (unsigned[]){0u, HS_ORDER2, HS_ORDER4}[rng() % 3];
        hs::Plan P;
        std::string msg;
        if (hs::make_plan(n, nt, sp.data(), c.data(), 1.3, 3, 81, flags, P, msg) != HS_OK) continue;
        std::vector<cd> psi0(P.N);
        for (auto &v : psi0) v = cd(std::normal_distribution<double>()(rng), std::normal_distribution<double>()(rng));
        std::vector<cd> ref = psi0;
        direct(P, P.seq, ref);
        const std::vector<hs::GateStep> steps = hs::gate_steps(P, P.seq);
        for (int form = 0; form < 6; ++form) {
            const bool loop = form == 2;
            const int kt = 2 + (int)(rng() % 11), wlog = 1 + (int)(rng() % 5);
            hs::GateProgram G;
            hs::gate_launches(P, steps, kt, wlog, form == 1 ? 1 : 0, loop, G);
            std::vector<cd> got = psi0;
            if (loop && G.launches.size() != 1) { std::printf("loop: %zu launches\n", G.launches.size()); return 1; }
            if (form == 1 && G.launches.size() < P.seq.size()) { std::printf("unfused: too few launches\n"); return 1; }
            for (auto &L : G.launches)
                if (int e = walk(P, G, L, got)) {
                    std::printf("case %d n=%d kt=%d form=%d: walk error %d\n", it, n, kt, form, e);
                    return 1;
                }
            double err = 0, nrm = 0;
            for (int64_t r = 0; r < P.N; ++r) {
                err = std::max(err, std::abs(got[r] - ref[r]));
                nrm = std::max(nrm, std::abs(ref[r]));
            }
            // at most 18 rotations x 90 factors of a few roundings each, entries below 1e-15 dropped
            if (!(err <= 1e-12 * nrm)) {
                std::printf("case %d n=%d kt=%d wlog=%d form=%d: error %.3e of %.3e\n", it, n, kt, wlog, form, err, nrm);
                return 1;
            }
            ++checked;
        }
    }
    std::printf("%d programs checked\n", checked);
    return checked > 300 ? 0 : 1;
}
