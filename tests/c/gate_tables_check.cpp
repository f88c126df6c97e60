// A coset program holds each factor's matrices once, however often the step
// parts apply it: first-, second- and fourth-order products of a Heisenberg
// chain, all four parts of a step appended to one program.
#include <cstdio>
#include <set>
#include <string>
#include <vector>

#include "../../paper_2606_16959_amd/csrc/gate_plan.h"

int main() {
    for (int budget : {16, 128, 1024})
        for (unsigned flags : {HS_MERGE_DIAG, HS_ORDER2, HS_ORDER4}) {
            const int n = 10;
            std::vector<std::string> s;
            for (int q = 0; q + 1 < n; ++q)
                for (char c : std::string("XYZ")) {
                    s.push_back(std::string(n, 'I'));
                    s.back()[q] = s.back()[q + 1] = c;
                }
            std::vector<const char *> sp;
            for (auto &v : s) sp.push_back(v.c_str());
            std::vector<double> c(2 * s.size(), 0.0);
            for (size_t k = 0; k < s.size(); ++k) c[2 * k] = 0.3 + 0.1 * k;
            hs::Plan P;
            std::string msg;
            if (hs::make_plan(n, (int)s.size(), sp.data(), c.data(), 1.0, 10, budget, flags, P, msg) != HS_OK) return 1;
            const std::vector<hs::GateStep> steps = hs::gate_steps(P, P.seq);
            hs::GateProgram G;
            size_t room = 0;
            std::set<int> seen;
            for (auto &g : steps)
                if (!g.diag_only && seen.insert(g.factor).second) room += g.entries->size() + 3;   // 4-entry alignment
            for (int part = 0; part < 4; ++part) hs::gate_launches(P, steps, 8, 3, 0, false, G);
            if (G.coef.size() + G.coef64.size() > room) {
                std::printf("budget %d flags %u: %zu entries, %zu in all factors\n", budget, flags,
                            G.coef.size() + G.coef64.size(), room);
                return 1;
            }
        }
    std::printf("tables checked\n");
    return 0;
}
