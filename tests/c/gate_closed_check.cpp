// The closure check of the coset programs: a program of a plan's own factors
// is closed; a nonzero entry between rows of different cosets, put into a
// factor's local unitary, is found whatever the tile.
#include <cstdio>
#include <string>
#include <vector>

#include "../../paper_2606_16959_amd/csrc/gate_plan.h"

int main() {
    const std::vector<const char *> s = {"XXIIII", "YYIIII", "IZXIII", "IIIXXI", "IIIYYI", "ZZZZZZ"};
    std::vector<double> c;
    for (size_t k = 0; k < s.size(); ++k) {
        c.push_back(0.3 + 0.1 * k);
        c.push_back(0.0);
    }
    int planted = 0;
    for (unsigned flags : {0u, HS_MERGE_DIAG, HS_ORDER2}) {
        hs::Plan P;
        std::string msg;
        if (hs::make_plan(6, (int)s.size(), s.data(), c.data(), 1.0, 2, 64, flags, P, msg) != HS_OK) return 1;
        for (size_t f = 0; f <= P.factors.size(); ++f)
            for (int kt : {2, 4, 6}) {
                hs::Plan Q = P;
                bool broken = false;
                if (f < P.factors.size() && !P.factors[f].terms.empty()) {
                    // masks of rank below the support leave entries outside the cosets
                    const int K = 1 << P.factors[f].bits.size();
                    for (int b = 1; b < K && !broken; ++b) {
                        bool zero = true;
                        for (int a = 0; a < K; ++a) zero = zero && P.factors[f].L[(size_t)a * K + (a ^ b)] == 0.0;
                        const hs::GateStep g = hs::gate_step(P, (int)f, 0);
                        if (!zero || ((size_t)1 << g.basis.size()) == (size_t)K) continue;
                        // a flip that no product of the members' flips makes
                        uint64_t full = 0;
                        for (size_t q = 0; q < P.factors[f].bits.size(); ++q)
                            if ((b >> q) & 1) full |= 1ull << P.factors[f].bits[q];
                        for (uint64_t v : g.basis)
                            if ((full >> (63 - __builtin_clzll(v))) & 1) full ^= v;
                        if (!full) continue;
                        Q.factors[f].L[(size_t)1 * K + (1 ^ b)] = 1e-3;
                        broken = true;
                        ++planted;
                    }
                }
                hs::GateProgram G;
                hs::gate_launches(Q, hs::gate_steps(Q, Q.seq), kt, 2, 0, kt == 6, G);
                bool used = false;
                for (int k : Q.seq) used = used || k == (int)f;
                if (G.closed == (broken && used)) {
                    std::printf("flags %u factor %zu kt %d: planted %d, closed %d\n", flags, f, kt, (int)broken, (int)G.closed);
                    return 1;
                }
                int at = 0;
                for (auto &L : G.launches) {
                    if (L.first != at || L.count < 1) return 2;
                    at += L.count;
                }
                if (at != (int)Q.seq.size()) return 3;
            }
    }
    std::printf("%d planted entries checked\n", planted);
    return planted > 10 ? 0 : 4;
}
