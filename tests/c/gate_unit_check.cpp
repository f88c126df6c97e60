// Units of the coset programs (gate_plan.h: factors of rank above the coset a
// thread holds), walked on the host as the kernel walks them for 4, 8 and 16
// rows per thread: every row of the tile is summed once, a wave that shares one
// matrix has one type and one piece of it, no table is read past its end, and
// the result equals exact Pauli rotations.  Ranks 4 to 10, supports spread over
// the tile and outside it, real and general entries, with and without D.
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
static int par(uint64_t v) { return __builtin_popcountll(v) & 1; }

static void rotate(const hs::Plan &P, const hs::Factor &F, std::vector<cd> &psi) {
    static const cd ip[4] = {{1, 0}, {0, 1}, {-1, 0}, {0, -1}};
    if (F.has_diag)
        for (int64_t x = 0; x < P.N; ++x) {
            double E = 0;
            for (int k : P.diag) E += P.terms[k].c * (par(x & P.terms[k].z) ? -1.0 : 1.0);
            psi[x] *= std::polar(1.0, -F.dt * E);
        }
    for (int k : F.terms) {
        const hs::Term &t = P.terms[k];
        std::vector<cd> y(psi.size());
        for (int64_t r = 0; r < P.N; ++r) {
            const int64_t x = r ^ (int64_t)t.x;
            y[r] = std::cos(t.c * F.dt) * psi[r] -
                   cd(0, 1) * std::sin(t.c * F.dt) * (ip[t.ny & 3] * (par(x & t.z) ? -1.0 : 1.0)) * psi[x];
        }
        psi.swap(y);
    }
}

static int units(const hs::Plan &P, const hs::GateProgram &G, const hs::GateLaunch &L, const hs::GateBlock &B, int df, int LC,
                 std::vector<cd> &psi) {
    const int T = 1 << L.kt, C = 1 << LC, rho = B.rho(), dim = 1 << rho;
    auto w = [&](int k) { return G.words.at(B.wtab + k); };
    const int nhole = B.nhole(), ntype = B.ntype(), jm = 3 * rho + nhole + ntype;
    std::vector<cd> out(P.N);
    for (int64_t tile = 0; tile < P.N / L.rows; ++tile) {
        const uint32_t base = deposit(L.out, (uint32_t)tile);
        std::vector<int> done(T, 0);
        int wave_type = 0, wave_i0 = 0;
        for (int tid = 0; tid < T / C; ++tid) {
            int rep = tid & ((1 << B.tshift()) - 1);
            for (int h = 0; h < nhole; ++h) {
                const int low = (1 << w(3 * rho + h)) - 1;
                rep = ((rep & ~low) << 1) | (rep & low);
            }
            for (int t = 0; t < ntype; ++t) rep |= ((tid >> (B.tshift() + rho - LC + t)) & 1) << w(3 * rho + nhole + t);
            const int i0 = ((tid >> B.tshift()) & ((1 << (rho - LC)) - 1)) << LC;
            int type = 0;
            for (int z = 0; z < B.nz(); ++z)
                type |= (((rep & G.words.at(B.ztab + 2 * z)) | (base & G.words.at(B.ztab + 2 * z + 1))) != 0) << z;
            if (tid % 64 == 0) wave_type = type, wave_i0 = i0;
            if (!B.lane() && (type != wave_type || i0 != wave_i0)) return 1;
            if (rep >= T) return 2;
            auto at = [&](int j) {
                int m = (int)w(jm + (j >> 2));
                if (j & 1) m ^= (int)w(rho);
                if (j & 2) m ^= (int)w(rho + 1);
                return rep ^ m;
            };
            for (int i = i0; i < i0 + C; ++i) {
                cd y = 0;
                for (int j = 0; j < dim; ++j) {
                    const int64_t row = base | deposit(L.in, at(j));
                    cd x = psi[row];
                    if (df >= 0) {
                        double E = 0;
                        for (int k : P.diag) E += P.terms[k].c * (par(row & P.terms[k].z) ? -1.0 : 1.0);
                        x *= std::polar(1.0, -P.factors[df].dt * E);
                    }
                    const int ki = par(i & B.kmask()), kj = par(j & B.kmask());
                    const int64_t tab = B.coef + (int64_t)type * dim * dim, e = df >= 0 ? tab + j * dim + i : tab + i * dim + j;
                    const std::vector<double> &c = df >= 0 ? G.coef64 : G.coef;
                    cd m;
                    if (B.form() == hs::kGateReal) m = ki == kj ? cd(c.at(e), 0) : ki ? cd(0, -c.at(e)) : cd(0, c.at(e));
                    else if (B.form() == hs::kGateRealD) m = ki == kj ? cd(c.at(e), 0) : cd(0, c.at(e));
                    else m = cd(c.at(2 * e), c.at(2 * e + 1));
                    y += m * x;
                }
                if (at(i) < 0 || at(i) >= T || done[at(i)]++) return 3;
                out[base | deposit(L.in, at(i))] = y;
            }
        }
        for (int i = 0; i < T; ++i)
            if (done[i] != 1) return 4;
    }
    psi.swap(out);
    return 0;
}

int main() {
    std::mt19937_64 rng(11);
    int checked = 0, general = 0, shared = 0, with_d = 0, top = 0;
    for (int it = 0; it < 400; ++it) {
        const int n = 4 + (int)(rng() % 9), nt = 4 + (int)(rng() % 10), kind = (int)(rng() % 4);
        std::vector<std::string> s(nt, std::string(n, 'I'));
        std::vector<double> c(2 * nt, 0.0);
        for (int k = 0; k < nt; ++k) {
            // single flips with a Z beside, XX and YY pairs, or anything
            const int q = (int)(rng() % n), p = (int)(rng() % n);
            if (kind == 0) s[k][k % n] = 'X';
            else if (kind == 1) s[k][p] = 'Z', s[k][q] = rng() % 2 ? 'X' : 'Y';
            else if (kind == 2) s[k][q] = s[k][p] = rng() % 2 ? 'X' : 'Y';
            else
                for (int j = 0; j < 3; ++j) s[k][rng() % n] = "XYZX"[rng() % 4];
            if (k == 0 && it % 2) s[k] = std::string(n, 'Z');
            c[2 * k] = std::uniform_real_distribution<double>(-2.0, 2.0)(rng);
        }
        std::vector<const char *> sp(nt);
        for (int k = 0; k < nt; ++k) sp[k] = s[k].c_str();
        hs::Plan P;
        std::string msg;
        if (hs::make_plan(n, nt, sp.data(), c.data(), 1.3, 3, 1 << 16, it % 4 < 3 ? HS_MERGE_DIAG : 0u, P, msg) != HS_OK) continue;
        const std::vector<hs::GateStep> steps = hs::gate_steps(P, P.seq);
        hs::GateProgram G;
        const int kt = 4 + (int)(rng() % 10), wlog = 1 + (int)(rng() % 5);
        hs::gate_launches(P, steps, kt, wlog, 0, it % 5 == 0, G);
        for (auto &L : G.launches)
            for (int b = L.block0; b < L.block1; ++b) {
                const hs::GateBlock &B = G.blocks[b];
                if (B.kind() != hs::kGateRows || B.rho() <= hs::kGateMaxCoset) continue;
                int seq = L.stage_diag >= 0 ? 1 : 0;
                for (auto &M : G.launches) {
                    if (&M == &L) break;
                    seq += M.block1 - M.block0 + (M.stage_diag >= 0);
                }
                const hs::Factor &F = P.factors[P.seq[seq + b - L.block0]];
                std::vector<cd> psi(P.N), ref;
                for (auto &v : psi) v = cd(std::normal_distribution<double>()(rng), std::normal_distribution<double>()(rng));
                for (int LC = 2; LC <= 4; ++LC) {
                    ref = psi;
                    rotate(P, F, ref);
                    if (int e = units(P, G, L, B, G.dfactor[b], LC, psi)) {
                        std::printf("case %d n=%d kt=%d rank %d, %d rows: error %d\n", it, n, L.kt, B.rho(), 1 << LC, e);
                        return 1;
                    }
                    double err = 0, nrm = 0;
                    for (int64_t r = 0; r < P.N; ++r) {
                        err = std::max(err, std::abs(psi[r] - ref[r]));
                        nrm = std::max(nrm, std::abs(ref[r]));
                    }
                    // a row sums up to 1024 products, entries below 1e-15 dropped
                    if (!(err <= 4e-12 * nrm)) {
                        std::printf("case %d n=%d kt=%d rank %d: error %.3e of %.3e\n", it, n, L.kt, B.rho(), err, nrm);
                        return 1;
                    }
                }
                ++checked;
                general += B.form() == hs::kGateComplex || B.form() == hs::kGateComplexD;
                shared += !B.lane();
                with_d += G.dfactor[b] >= 0;
                top = std::max(top, B.rho());
            }
    }
    std::printf("%d blocks of units checked: %d general, %d with one matrix per wave, %d with D, ranks to %d\n", checked, general,
                shared, with_d, top);
    return checked > 100 && general > 5 && shared > 5 && with_d > 10 && top == 10 ? 0 : 1;
}
