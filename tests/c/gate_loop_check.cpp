// The looped whole-state form of a step's coset program is one launch and the
// same blocks whatever the cap on factors per launch; without the loop the cap
// holds.  TFIM and Heisenberg chains of 2..12 qubits, every product order.
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../paper_2606_16959_amd/csrc/gate_plan.h"

int main() {
    int checked = 0;
    for (int n = 2; n <= 12; ++n)
        for (int heis = 0; heis < 2; ++heis)
            for (unsigned flags : {0u, HS_MERGE_DIAG, HS_ORDER2, HS_ORDER4}) {
                std::vector<std::string> s;
                for (int q = 0; q + 1 < n; ++q)
                    for (char c : std::string(heis ? "XYZ" : "Z")) {
                        s.push_back(std::string(n, 'I'));
                        s.back()[q] = s.back()[q + 1] = c;
                    }
                for (int q = 0; q < n; ++q) {
                    s.push_back(std::string(n, 'I'));
                    s.back()[q] = 'X';
                }
                std::vector<const char *> sp;
                for (auto &v : s) sp.push_back(v.c_str());
                std::vector<double> c(2 * s.size(), 0.0);
                for (size_t k = 0; k < s.size(); ++k) c[2 * k] = 0.3 + 0.1 * k;
                hs::Plan P;
                std::string msg;
                if (hs::make_plan(n, (int)s.size(), sp.data(), c.data(), 1.0, 10, 16, flags, P, msg) != HS_OK) return 1;
                const std::vector<hs::GateStep> steps = hs::gate_steps(P, P.seq);
                hs::GateProgram ref;
                hs::gate_launches(P, steps, 10, 5, 0, true, ref);
                for (int cap = 1; cap <= 7; ++cap) {
                    hs::GateProgram G;
                    hs::gate_launches(P, steps, 10, 5, cap, true, G);
                    if (G.launches.size() != 1 || G.launches[0].block0 != 0 || G.launches[0].block1 != (int)P.seq.size() ||
                        G.blocks.size() != ref.blocks.size() ||
                        std::memcmp(G.blocks.data(), ref.blocks.data(), G.blocks.size() * sizeof(hs::GateBlock)) ||
                        G.words != ref.words || G.coef != ref.coef || G.coef64 != ref.coef64 || G.dfactor != ref.dfactor) {
                        std::printf("n=%d heis=%d flags=%u cap=%d: %zu launches, blocks of the first [%d, %d) of %zu\n", n, heis,
                                    flags, cap, G.launches.size(), G.launches[0].block0, G.launches[0].block1, P.seq.size());
                        return 1;
                    }
                    hs::GateProgram U;
                    hs::gate_launches(P, steps, 10, 5, cap, false, U);
                    if (U.launches.size() < (P.seq.size() + cap - 1) / cap) return 2;
                    ++checked;
                }
            }
    std::printf("%d looped programs checked\n", checked);
    return 0;
}
