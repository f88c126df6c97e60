// C ABI of the hamsim library (declared in include/hamsim.h): handle
// lifetime, device construction of the factor diagonals, the evolve loop
// (launch planning: tile geometry and fusion of consecutive factors), the
// generic DIA SpMV and the FP64 reductions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "gate_plan.h"
#include "hs_internal.h"
#include "tile_plan.h"

using hs::DiagDesc;
using hs::Factor;
using hs::Plan;
using hs::TileArgs;
using namespace hs::plan;

namespace {

thread_local std::string g_err;

hs_status fail(hs_status s, const std::string &m) {
    g_err = m;
    return s;
}

}  // namespace

namespace hs {
void set_last_error(const std::string &m) { g_err = m; }

bool device_range_ok(const void *p, size_t bytes, const char *what, std::string &msg) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        msg = std::string(what) + ": no current device";
        return false;
    }
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        msg = std::string(what) + " is not device memory (a host address?)";
        return false;
    }
    if (at.type != hipMemoryTypeDevice && at.type != hipMemoryTypeManaged) {
        msg = std::string(what) + " is not device memory (a host address?)";
        return false;
    }
    if (at.type == hipMemoryTypeDevice && at.device != dev) {
        msg = std::string(what) + " lives on device " + std::to_string(at.device) + ", the current device is " +
              std::to_string(dev);
        return false;
    }
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) == hipSuccess && base && size) {
        const char *lo = static_cast<const char *>(base);
        if (static_cast<const char *>(p) + bytes > lo + size) {
            msg = std::string(what) + " extends past the end of its allocation";
            return false;
        }
    } else {
        (void)hipGetLastError();      // pool allocations may not report a range
    }
    return true;
}
}  // namespace hs

namespace {

hs_status hip_fail(hipError_t e, const char *what) {
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return e == hipErrorOutOfMemory ? HS_ENOMEM : HS_EDEVICE;
}

#define HS_HIP(call, what)                                  \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return hip_fail(e_, what);    \
    } while (0)

// One entry of the fusion list (hs_step_launches): consecutive factors whose
// coupling hulls one closed tile of the batch's rows holds.
struct Run {
    int first = 0;              // position of the first factor in the step sequence
    std::vector<int> factors;   // factor indices at consecutive sequence positions
    Geo geo;
    bool elementwise = false;   // a single main-diagonal factor
    bool open = false;          // no closed tile holds the factor's coupling range
};

// The factor sequence of each part of an evolution of several steps.  With a
// joint factor J the steps of a symmetric product run s_0 .. s_{L-2} J, then
// (s_1 .. s_{L-2} J) for the middle steps, then s_1 .. s_{L-1}; part 0 is a
// lone step.  Without a joint every part is the plain step.
enum { kPartLone = 0, kPartFirst = 1, kPartMiddle = 2, kPartLast = 3, kParts = 4 };

std::vector<int> part_sequence(const Plan &P, int part) {
    const auto &q = P.seq;
    if (P.joint < 0 || part == kPartLone) return q;
    std::vector<int> out;
    const size_t L = q.size();
    const size_t a = part == kPartFirst ? 0 : 1;
    const size_t b = part == kPartLast ? L : L - 1;
    for (size_t i = a; i < b; ++i) out.push_back(q[i]);
    if (part != kPartLast) out.push_back(P.joint);
    return out;
}

// The coset program of every step part on the device, with its launches
// (gate_plan.h).
struct GatePlan {
    hs::GateProgram prog;
    int launch0[kParts] = {0}, launch1[kParts] = {0};   // part q makes launches [launch0[q], launch1[q])
    std::vector<hs::GateBlock> blocks;           // prog.blocks with their diagonals' addresses
    std::vector<float> coef32;
    std::vector<char> host;                      // the tables as uploaded; alive as long as the plan
    void *dev = nullptr;
    hs::GateTables tab;
};

}  // namespace

struct hs_factors_s {
    Plan plan;
    bool built = false;
    int dtype = HS_C64;
    int device = 0;
    double *work_dev = nullptr;      // [8][G][4] partials, then [8][4] records
    double *norm_dev = nullptr;      // per-tile norm partials of the step's last launch, on demand
    size_t norm_bytes = 0;
    hipStream_t alloc_stream = nullptr;   // device memory is stream-ordered on this stream
    std::map<PlanKey, std::unique_ptr<GatePlan>> plans;
    std::unique_ptr<GatePlan> whole;      // whole evolutions of small states
    std::mutex mu;
    // D = exp(-i h E) of every factor that carries it: N entries of the
    // handle's dtype in natural order when the factor is nothing else (its
    // own diagonal, or one of diag_own), else FP64 entries in the order the
    // factor's coset product reads them
    std::vector<const void *> diag_of;
    std::vector<void *> owned;       // device allocations of the build

    double *partials() { return work_dev; }
    double *records() { return work_dev + (size_t)HS_MAX_BATCH * hs::kReduceBlocks * 4; }

    // Stream-ordered frees (hipFree would wait for the whole device, stalling
    // other handles' work on other streams).
    ~hs_factors_s() {
        for (void *p : owned) (void)hipFreeAsync(p, alloc_stream);
        for (auto &kv : plans)
            if (kv.second->dev) (void)hipFreeAsync(kv.second->dev, alloc_stream);
        if (whole && whole->dev) (void)hipFreeAsync(whole->dev, alloc_stream);
        if (norm_dev) (void)hipFreeAsync(norm_dev, alloc_stream);
    }
};

namespace {

// The fusion list of every step part (host only): greedy fusion extends a run
// while the union of coupling hulls still fits one closed tile of the batch's
// rows with row runs of at least w_min elements.  hs_step_launches reports it
// and choose_storage_order reads it; hs_evolve launches coset programs
// (form_gate_plan).
void form_runs(const Plan &P, int dtype, const PlanKey &key, std::vector<Run> (&all)[kParts]) {
    const int n = P.n;
    const int batch = key.chunk;
    const bool fuse = key.fuse != 0;
    const int Tmax = tile_rows_max(dtype, batch, P.N);
    const int Wmin = w_min(dtype, key);
    const int max_fuse = key.max_fuse;
    for (int part = 0; part < (P.joint < 0 ? 1 : kParts); ++part) {
        // runs are consecutive positions of the part's factor sequence
        const std::vector<int> seq = part_sequence(P, part);
        std::vector<Run> &runs = all[part];
        runs.clear();
        const int F = (int)seq.size();
        int f = 0;
        while (f < F) {
            Run run;
            run.first = f;
            run.factors.push_back(seq[f]);
            const Factor &F0 = P.factors[seq[f]];
            int lb = F0.xlb, hb = F0.xhb;
            bool empty = F0.xmask_union == 0;
            if (F0.offs.size() == 1 && F0.offs[0] == 0 && empty) {
                run.elementwise = true;
            }
            int ndiag = (int)F0.offs.size();
            int g = f + 1;
            while (fuse && g < F && (int)run.factors.size() < max_fuse) {
                const Factor &G = P.factors[seq[g]];
                int nlb = lb, nhb = hb;
                if (G.xmask_union) {
                    if (empty) { nlb = G.xlb; nhb = G.xhb; }
                    else { nlb = std::min(lb, G.xlb); nhb = std::max(hb, G.xhb); }
                }
                const Geo geo = geometry(nlb, nhb, n, Tmax);
                const bool good = geo.ok && (geo.qb == 0 || (1 << geo.logW) >= Wmin);
                if (!good || ndiag + (int)G.offs.size() > hs::kMaxDiagsPerLaunch) break;
                run.factors.push_back(seq[g]);
                run.elementwise = false;
                ndiag += (int)G.offs.size();
                lb = nlb; hb = nhb;
                if (G.xmask_union) empty = false;
                ++g;
            }
            run.geo = geometry(empty ? 0 : lb, empty ? 0 : hb, n, Tmax);
            if (!run.geo.ok) run.geo = geometry(lb, hb, n, tile_rows_max(dtype, 1, P.N));
            run.open = !run.geo.ok;
            runs.push_back(run);
            f = g;
        }
    }
    for (int part = 1; P.joint < 0 && part < kParts; ++part) all[part] = all[0];
}

// Storage order of every factor (perm_pos): a factor that the one-state plan
// (default fusion) applies only in closed strided launches, whose level
// stride 2^qb rows spans at least HAMSIM_PERM_MIN_BYTES (default 1 MiB, where
// every level of a tile lies on its own 2 MB page; 0: never), is stored with
// s = qb of the launch with the smallest qb.  Its chunks hold
// HAMSIM_PERM_CHUNK_WINDOWS (default 4) of that launch's windows of W
// consecutive rows, or HAMSIM_PERM_CHUNK_BYTES when that is set (nonzero):
// neighbouring tiles, which run at the same time on other compute units, then
// read each level's chunk together.  The order serves a launch that streams the
// stored diagonals; hs_evolve reads none of them, so here it costs a natural-
// order copy of a permuted lone diagonal and a gather in host copies.
void choose_storage_order(Plan &P, int dtype) {
    for (auto &f : P.factors) f.perm_s = f.perm_c = 0;
    const int min_bytes = env_int("HAMSIM_PERM_MIN_BYTES", 1 << 20, 0, 1 << 30);
    if (min_bytes == 0) return;
    const size_t sc = elem_bytes(dtype);
    const int chunk_bytes = env_int("HAMSIM_PERM_CHUNK_BYTES", 0, 0, 1 << 24);
    const int chunk_windows = env_int("HAMSIM_PERM_CHUNK_WINDOWS", 4, 1, 1 << 12);
    std::vector<Run> runs[kParts];
    form_runs(P, dtype, plan_key(1, true), runs);
    std::vector<int> smin(P.factors.size(), -1), wlog(P.factors.size(), 0);
    for (int part = 0; part < kParts; ++part)
        for (const Run &run : runs[part]) {
            const bool strided = !run.open && !run.elementwise && run.geo.qb > 0;
            for (int k : run.factors) {
                const int q = strided ? run.geo.qb : 0;
                if (smin[k] < 0 || q < smin[k]) {
                    smin[k] = q;
                    wlog[k] = run.geo.logW;
                }
            }
        }
    for (size_t k = 0; k < P.factors.size(); ++k) {
        Factor &F = P.factors[k];
        const int q = smin[k];
        if (q <= 0 || q > 30 || ((size_t)1 << q) * sc < (size_t)min_bytes) continue;
        bool multiple = true;
        for (int64_t d : F.offs) multiple = multiple && ((d < 0 ? -d : d) & ((int64_t(1) << q) - 1)) == 0;
        if (!multiple) continue;
        // chunk entries: a power of two, at least 2 (pairs stay adjacent), at most 2^q
        const int64_t want = chunk_bytes ? (int64_t)chunk_bytes / (int64_t)sc
                                         : ((int64_t)chunk_windows << wlog[k]);
        const int c = std::min(q, std::max(1, ilog2(std::max<int64_t>(2, want))));
        F.perm_s = q;
        F.perm_c = c;
    }
}

// log2 rows of an evolution's largest tiles: 64 KiB of LDS, so that two
// workgroups share a CU, halved (down to 1024 rows) while the launch would
// have fewer than 256 of them, one per compute unit.  form_gate_plan takes
// half of it where that needs no more launches.
int gate_tile_bits(int dtype, int64_t N, int batch) {
    int kt = dtype == HS_C128 ? 12 : 13;
    while (kt > 10 && ((N * batch) >> kt) < 256) --kt;
    return kt;
}

// Uploads a program's tables in one copy; the host copy lives as long as the
// plan, so the ordered copy is safe.
hs_status upload_gates(hs_factors_s *h, GatePlan &gp, hipStream_t st) {
    hs::GateProgram &p = gp.prog;
    gp.blocks = p.blocks;
    for (size_t k = 0; k < gp.blocks.size(); ++k)
        gp.blocks[k].diag = p.dfactor[k] >= 0 ? h->diag_of[p.dfactor[k]] : nullptr;
    const bool c128 = h->dtype == HS_C128;
    if (!c128) gp.coef32.assign(p.coef.begin(), p.coef.end());
    constexpr int kTabs = 4;
    const struct {
        const void *src;
        size_t bytes;
    } part[kTabs] = {{gp.blocks.data(), gp.blocks.size() * sizeof(hs::GateBlock)},
                     {p.words.data(), p.words.size() * sizeof(uint32_t)},
                     {c128 ? (const void *)p.coef.data() : (const void *)gp.coef32.data(),
                      p.coef.size() * (c128 ? 8 : 4)},
                     {p.coef64.data(), p.coef64.size() * 8}};
    size_t off[kTabs];
    gp.host.clear();
    for (int k = 0; k < kTabs; ++k) {
        off[k] = gp.host.size();
        gp.host.resize(off[k] + (part[k].bytes + 255) / 256 * 256);
        if (part[k].bytes) std::memcpy(gp.host.data() + off[k], part[k].src, part[k].bytes);
    }
    HS_HIP(hipMallocAsync(&gp.dev, gp.host.size(), st), "hipMallocAsync(coset tables)");
    char *base = static_cast<char *>(gp.dev);
    HS_HIP(hipMemcpyAsync(base, gp.host.data(), gp.host.size(), hipMemcpyHostToDevice, st), "coset tables");
    gp.tab.blocks = reinterpret_cast<const hs::GateBlock *>(base + off[0]);
    gp.tab.words = reinterpret_cast<const uint32_t *>(base + off[1]);
    gp.tab.coef = base + off[2];
    gp.tab.coef64 = reinterpret_cast<const double *>(base + off[3]);
    // what a launch needs stays: the launches, and `host` for the ordered copy
    std::vector<double>().swap(gp.prog.coef);
    std::vector<double>().swap(gp.prog.coef64);
    std::vector<float>().swap(gp.coef32);
    return HS_OK;
}

// The coset programs of every step part for one plan key, or (loop) of a
// whole small state, on the host.
std::unique_ptr<GatePlan> form_gate_plan(const Plan &P, int dtype, const PlanKey &key, bool loop) {
    std::unique_ptr<GatePlan> gp(new GatePlan());
    const int wlog = ilog2(std::max<int64_t>(2, w_min(dtype, key)));
    const int max_factors = !key.fuse ? 1 : key.max_fuse < hs::kMaxRun ? key.max_fuse : 0;
    const int parts = P.joint < 0 ? 1 : kParts;     // without a joint factor every part is the plain step
    std::map<int, hs::GateStep> made;
    std::vector<hs::GateStep> steps[kParts];
    for (int q = 0; q < parts; ++q) steps[q] = hs::gate_steps(P, part_sequence(P, q), &made);
    auto form = [&](int kt, GatePlan &g) {
        g.prog = hs::GateProgram();
        for (int q = 0; q < kParts; ++q) {
            g.launch0[q] = q < parts ? (int)g.prog.launches.size() : g.launch0[0];
            if (q < parts) hs::gate_launches(P, steps[q], kt, wlog, max_factors, loop, g.prog);
            g.launch1[q] = q < parts ? (int)g.prog.launches.size() : g.launch1[0];
        }
    };
    const int kt = gate_tile_bits(dtype, P.N, key.chunk);
    form(kt, *gp);
    if (!loop && kt > (dtype == HS_C128 ? 11 : 12)) {
        // half the tile where it needs no more launches: four workgroups share
        // a CU instead of two and overlap each other's phases better (n = 25
        // lattice 508 -> 457 us, MaxCut n = 24 with 8 states 1715 -> 1579 us a
        // step; a quarter of the tile gains nothing more)
        GatePlan half;
        form(kt - 1, half);
        if (half.prog.launches.size() <= gp->prog.launches.size()) std::swap(*gp, half);
    }
    return gp;
}

// The same on the device.
hs_status make_gate_plan(hs_factors_s *h, const PlanKey &key, bool loop, std::unique_ptr<GatePlan> &out, void *stream) {
    std::unique_ptr<GatePlan> gp = form_gate_plan(h->plan, h->dtype, key, loop);
    // the looped form applies a part's blocks from one launch
    for (int q = 0; loop && q < kParts; ++q)
        if (gp->launch1[q] != gp->launch0[q] + 1) return fail(HS_EDEVICE, "looped coset program of several launches");
    if (hs_status s = upload_gates(h, *gp, reinterpret_cast<hipStream_t>(stream))) {
        if (gp->dev) (void)hipFreeAsync(gp->dev, reinterpret_cast<hipStream_t>(stream));
        return s;
    }
    out = std::move(gp);
    return HS_OK;
}

// Rows up to which hs_evolve runs a whole evolution in one launch
// (HAMSIM_WHOLE_MAX_ROWS, capped by the tile one workgroup holds; 0 never).
// The default is where one workgroup per state stops beating a launch per run
// and step: n = 12 11.8 against 13.5 us a step (complex128 13.1 against 14.4),
// n = 13 18.5 against 14.1 us.
int64_t whole_max_rows(int dtype) {
    const int lim = dtype == HS_C128 ? hs::kWholeRowsC128 : hs::kWholeRowsC64;
    return env_int("HAMSIM_WHOLE_MAX_ROWS", 4096, 0, lim);
}

bool evolves_whole(const Plan &P, int dtype, bool renorm, bool fuse) {
    return !renorm && fuse && P.N <= whole_max_rows(dtype);
}

// A step that is one diagonal factor, without renormalisation: one pass.
bool evolves_lone_diagonal(const Plan &P, bool renorm) {
    return P.joint < 0 && !renorm && P.seq.size() == 1 && P.factors[P.seq[0]].terms.empty();
}

hs_status check_handle(hs_factors f) {
    if (!f) return fail(HS_EINVAL, "null handle");
    return HS_OK;
}

}  // namespace

extern "C" {

const char *hs_last_error(void) { return g_err.c_str(); }
int hs_abi_version(void) { return 1; }

hs_status hs_plan(int n_qubits, int n_terms, const char *const *pauli_terms, const double *coeffs,
                  double t, int steps, int budget, unsigned flags, hs_factors *out) {
    if (!out) return fail(HS_EINVAL, "null output handle");
    *out = nullptr;
    hs_factors_s *h = new (std::nothrow) hs_factors_s();
    if (!h) return fail(HS_ENOMEM, "host allocation failed");
    std::string msg;
    hs_status s = hs::make_plan(n_qubits, n_terms, pauli_terms, coeffs, t, steps, budget, flags,
                                h->plan, msg);
    if (s != HS_OK) {
        delete h;
        return fail(s, msg);
    }
    for (auto &f : h->plan.factors) hs::layout_factor(f, h->plan.N, 8);
    *out = h;
    g_err.clear();
    return HS_OK;
}

// Handles up to this size live in one allocation.
constexpr size_t kOneAllocation = size_t(256) << 20;

static hs_status build_device(hs_factors_s *h, void *stream) {
    Plan &P = h->plan;
    const size_t sc = elem_bytes(h->dtype);
    const bool c128 = h->dtype == HS_C128;
    HS_HIP(hipGetDevice(&h->device), "hipGetDevice");
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    h->alloc_stream = st;
    choose_storage_order(P, h->dtype);
    // Device memory.  A small handle is one allocation (an allocation costs
    // more host time than building its diagonals takes); a large one has an
    // allocation per factor.
    struct Piece {
        size_t bytes;
        void **where;
    };
    std::vector<Piece> pieces;
    std::vector<void *> dtab(P.factors.size(), nullptr);
    for (size_t k = 0; k < P.factors.size(); ++k) {
        hs::Factor &f = P.factors[k];
        hs::layout_factor(f, P.N, sc);
        pieces.push_back({f.elems_total * sc, &f.dev});
        // D beside the factor's diagonals, unless it is the factor in natural order
        if (f.has_diag && !(f.terms.empty() && f.perm_s == 0))
            pieces.push_back({(size_t)P.N * (f.terms.empty() ? sc : 16), &dtab[k]});
    }
    pieces.push_back({sizeof(double) * ((size_t)HS_MAX_BATCH * hs::kReduceBlocks * 4 + HS_MAX_BATCH * 4),
                      reinterpret_cast<void **>(&h->work_dev)});
    size_t sum = 0;
    for (const Piece &q : pieces) sum += (q.bytes + 255) / 256 * 256;
    if (sum <= kOneAllocation) {
        void *slab = nullptr;
        HS_HIP(hipMallocAsync(&slab, sum, st), "hipMallocAsync(factors)");
        h->owned.push_back(slab);
        char *at = static_cast<char *>(slab);
        for (const Piece &q : pieces) {
            *q.where = at;
            at += (q.bytes + 255) / 256 * 256;
        }
    } else {
        for (const Piece &q : pieces) {
            HS_HIP(hipMallocAsync(q.where, q.bytes, st), "hipMallocAsync(factor diagonals)");
            h->owned.push_back(*q.where);
        }
    }

    // every host table in one upload: Z masks and coefficients of the diagonal
    // terms, then per factor offsets, element offsets and the local unitary
    std::vector<char> host;
    auto put = [&](const void *src, size_t bytes) {
        const size_t at = host.size();
        host.resize(at + (bytes + 15) / 16 * 16);
        if (bytes) std::memcpy(host.data() + at, src, bytes);
        return at;
    };
    std::vector<uint64_t> zm;
    std::vector<double> cf;
    for (int k : P.diag) {
        zm.push_back(P.terms[k].z);
        cf.push_back(P.terms[k].c);
    }
    const size_t at_zm = put(zm.data(), zm.size() * 8), at_cf = put(cf.data(), cf.size() * 8);
    const int64_t zero_off = 0;
    const size_t at_zero = put(&zero_off, 8);
    struct At {
        size_t offs, eo, L;
    };
    std::vector<At> at;
    for (auto &f : P.factors) {
        const std::vector<uint64_t> eo(f.elem_off.begin(), f.elem_off.end());
        At x{};
        x.offs = put(f.offs.data(), f.offs.size() * 8);
        x.eo = put(eo.data(), eo.size() * 8);
        x.L = put(f.L.data(), f.terms.empty() ? 0 : f.L.size() * 16);
        at.push_back(x);
    }
    std::vector<void *> temps;          // freed once the stream is synchronised
    auto cleanup = [&]() {
        for (void *p : temps) (void)hipFreeAsync(p, st);
    };
    hipError_t e = hipSuccess;
    void *tab = nullptr;
    if ((e = hipMallocAsync(&tab, host.size(), st)) != hipSuccess) return hip_fail(e, "hipMallocAsync(tables)");
    temps.push_back(tab);
    if ((e = hipMemcpyAsync(tab, host.data(), host.size(), hipMemcpyHostToDevice, st)) != hipSuccess) {
        cleanup();
        return hip_fail(e, "table upload");
    }
    char *dt = static_cast<char *>(tab);
    // D of a factor with further terms stays with the handle, in the order its
    // coset product reads; a factor that is D alone is rounded from a temporary
    // FP64 table in natural order, one per distinct time step
    std::map<double, double *> phases;
    for (size_t k = 0; k < P.factors.size(); ++k) {
        const hs::Factor &f = P.factors[k];
        if (!f.has_diag || (f.terms.empty() && phases.count(f.dt))) continue;
        double *phase = static_cast<double *>(dtab[k]);
        if (f.terms.empty()) {
            if ((e = hipMallocAsync(reinterpret_cast<void **>(&phase), (size_t)P.N * 16, st)) != hipSuccess) {
                cleanup();
                return hip_fail(e, "phase table setup");
            }
            temps.push_back(phase);
            phases[f.dt] = phase;
        }
        int le = hs::launch_phase_table(P.N, (int)P.diag.size(), reinterpret_cast<uint64_t *>(dt + at_zm),
                                        reinterpret_cast<double *>(dt + at_cf), f.dt,
                                        f.terms.empty() ? std::vector<uint64_t>() : hs::gate_basis(P, (int)k), phase, stream);
        if (le) { cleanup(); return hip_fail((hipError_t)le, "phase table kernel"); }
    }
    for (size_t k = 0; k < P.factors.size(); ++k) {
        const hs::Factor &f = P.factors[k];
        hs::ConstructArgs a{};
        a.base = f.dev;
        a.N = (int32_t)P.N;
        a.smask = (uint32_t)f.smask;
        a.offs = reinterpret_cast<int64_t *>(dt + at[k].offs);
        a.elem_off = reinterpret_cast<uint64_t *>(dt + at[k].eo);
        a.K = 1;
        if (!f.terms.empty()) {
            a.L = reinterpret_cast<double *>(dt + at[k].L);
            a.K = 1 << f.bits.size();
            a.nbits = (int)f.bits.size();
            for (int q = 0; q < a.nbits; ++q) a.bits[q] = (int8_t)f.bits[q];
            a.lb = f.bits.empty() ? 0 : f.bits[0];
            a.contiguous = f.bits.empty() || f.bits.back() - f.bits.front() + 1 == (int)f.bits.size();
        }
        if (f.has_diag) a.phase = f.terms.empty() ? phases[f.dt] : static_cast<double *>(dtab[k]);
        if (f.has_diag && !f.terms.empty())
            for (uint64_t m : hs::gate_basis(P, (int)k)) a.basis[a.rho++] = (uint32_t)m;
        a.perm_s = f.perm_s;
        a.perm_c = f.perm_c;
        int le = hs::launch_construct(a, (int)f.offs.size(), P.N, c128, stream);
        if (le) { cleanup(); return hip_fail((hipError_t)le, "construct kernel"); }
        if (dtab[k] && f.terms.empty()) {       // stored out of natural order: once more in order
            a.base = dtab[k];
            a.offs = reinterpret_cast<int64_t *>(dt + at_zero);
            a.elem_off = reinterpret_cast<uint64_t *>(dt + at_zero);
            a.perm_s = a.perm_c = 0;
            le = hs::launch_construct(a, 1, P.N, c128, stream);
            if (le) { cleanup(); return hip_fail((hipError_t)le, "diagonal kernel"); }
        }
        h->diag_of.push_back(dtab[k] ? dtab[k] : f.has_diag ? f.dev : nullptr);
    }
    e = hipStreamSynchronize(st);
    cleanup();
    if (e != hipSuccess) return hip_fail(e, "construction");
    h->built = true;
    return HS_OK;
}

hs_status hs_build_factors(int n_qubits, int n_terms, const char *const *pauli_terms,
                           const double *coeffs, double t, int steps, int budget, hs_dtype dtype,
                           unsigned flags, void *stream, hs_factors *out) {
    if (!out) return fail(HS_EINVAL, "null output handle");
    *out = nullptr;
    if (dtype != HS_C64 && dtype != HS_C128) return fail(HS_EINVAL, "dtype must be HS_C64 or HS_C128");
    hs_factors h = nullptr;
    hs_status s = hs_plan(n_qubits, n_terms, pauli_terms, coeffs, t, steps, budget, flags, &h);
    if (s != HS_OK) return s;
    h->dtype = dtype;
    s = build_device(h, stream);
    if (s != HS_OK) {
        std::string keep = g_err;
        delete h;
        g_err = keep;
        return s;
    }
    *out = h;
    g_err.clear();
    return HS_OK;
}

hs_status hs_evolve(hs_factors f, void *psi, int batch, int steps, void *stream, unsigned flags) {
    if (hs_status s = check_handle(f)) return s;
    if (!f->built) return fail(HS_EINVAL, "handle was planned, not built");
    if (!psi) return fail(HS_EINVAL, "null state pointer");
    if (batch < 1) return fail(HS_EINVAL, "batch must be >= 1");
    if (steps < 0) return fail(HS_EINVAL, "steps must be >= 0");
    if (flags & ~(unsigned)(HS_RENORM | HS_NO_FUSE)) return fail(HS_EINVAL, "unknown evolve flag");
    if (reinterpret_cast<uintptr_t>(psi) % 16) return fail(HS_EINVAL, "state pointer must be 16-byte aligned");
    const Plan &P = f->plan;
    const size_t sc = elem_bytes(f->dtype);
    {
        // checked before the zero-step return, so a caller can validate a
        // state without enqueuing work
        std::string msg;
        if (!hs::device_range_ok(psi, (size_t)batch * P.N * sc, "state", msg)) return fail(HS_EINVAL, msg);
    }
    if (steps == 0) return HS_OK;
    std::lock_guard<std::mutex> lock(f->mu);
    int cur_dev = 0;
    HS_HIP(hipGetDevice(&cur_dev), "hipGetDevice");
    if (cur_dev != f->device) return fail(HS_EINVAL, "current device differs from the build device");
    const bool c128 = f->dtype == HS_C128;
    const bool fuse = !(flags & HS_NO_FUSE);
    const bool renorm = (flags & HS_RENORM) != 0;
    if (evolves_lone_diagonal(P, renorm)) {
        // a step that is one diagonal factor: all steps in one pass (the
        // same multiplications, one step after the other, per entry)
        for (int c0 = 0; c0 < batch; c0 += HS_MAX_BATCH) {
            const int chunk = std::min(HS_MAX_BATCH, batch - c0);
            void *p = static_cast<char *>(psi) + (size_t)c0 * P.N * sc;
            int e = hs::launch_diag_steps(p, p, f->diag_of[P.seq[0]], P.N, chunk, steps, nullptr, c128,
                                          stream_out(chunk, P.N, f->dtype), stream);
            if (e) return hip_fail((hipError_t)e, "diag kernel launch");
        }
        return HS_OK;
    }
    if (evolves_whole(P, f->dtype, renorm, fuse)) {
        // a small state: the whole evolution of every state in one launch
        if (!f->whole)
            if (hs_status s = make_gate_plan(f, plan_key(1, true), true, f->whole, stream)) return s;
        const GatePlan &gp = *f->whole;
        for (int64_t c0 = 0; c0 < batch; c0 += 32768) {
            hs::GateRun r;
            r.psi = static_cast<char *>(psi) + (size_t)c0 * P.N * sc;
            r.N = P.N;
            r.batch = (int)std::min<int64_t>(32768, batch - c0);
            r.by_rows = gp.prog.by_rows;
            r.level = gp.prog.level;
            r.steps = steps;
            for (int q = 0; q < kParts; ++q) {
                r.first[q] = gp.prog.launches[gp.launch0[q]].block0;
                r.last[q] = gp.prog.launches[gp.launch0[q]].block1;
            }
            int e = hs::launch_gates(gp.prog.launches[0], gp.tab, r, c128, false, stream);
            if (e) return hip_fail((hipError_t)e, "whole-evolution kernel launch");
        }
        return HS_OK;
    }
    for (int c0 = 0; c0 < batch; c0 += HS_MAX_BATCH) {
        const int chunk = std::min(HS_MAX_BATCH, batch - c0);
        const PlanKey key = plan_key(chunk, fuse);
        auto it = f->plans.find(key);
        if (it == f->plans.end()) {
            std::unique_ptr<GatePlan> gp;
            if (hs_status s = make_gate_plan(f, key, false, gp, stream)) return s;
            it = f->plans.emplace(key, std::move(gp)).first;
        }
        const GatePlan &gp = *it->second;
        if (renorm) {
            // the step's last launch sums |y|^2 per tile: room for its partials
            size_t need = 0;
            for (int q = 0; q < kParts; ++q) {
                const hs::GateLaunch &L = gp.prog.launches[gp.launch1[q] - 1];
                need = std::max(need, (size_t)chunk * (P.N / L.rows) * 4 * sizeof(double));
            }
            if (need > f->norm_bytes) {
                hipStream_t hst = reinterpret_cast<hipStream_t>(stream);
                if (f->norm_dev) HS_HIP(hipFreeAsync(f->norm_dev, hst), "hipFreeAsync(norm partials)");
                f->norm_dev = nullptr;
                f->norm_bytes = 0;
                HS_HIP(hipMallocAsync(reinterpret_cast<void **>(&f->norm_dev), need, hst),
                       "hipMallocAsync(norm partials)");
                f->norm_bytes = need;
            }
        }
        void *p = static_cast<char *>(psi) + (size_t)c0 * P.N * sc;
        const bool streamed = stream_out(chunk, P.N, f->dtype) != 0;
        const double *rec = f->records() + 2;    // squared norm of state b at rec[4 b]
        for (int s = 0; s < steps; ++s) {
            const int part = steps == 1 ? kPartLone
                             : s == 0 ? kPartFirst : s == steps - 1 ? kPartLast : kPartMiddle;
            const int l0 = gp.launch0[part], l1 = gp.launch1[part];
            for (int l = l0; l < l1; ++l) {
                const hs::GateLaunch &L = gp.prog.launches[l];
                hs::GateRun r;
                r.psi = p;
                r.N = P.N;
                r.batch = chunk;
                r.by_rows = gp.prog.by_rows;
                r.level = gp.prog.level;
                r.stage_diag = L.stage_diag >= 0 ? f->diag_of[L.stage_diag] : nullptr;
                r.nrm2 = (renorm && s > 0 && l == l0) ? rec : nullptr;
                r.norm_out = (renorm && l + 1 == l1) ? f->norm_dev : nullptr;
                r.first[0] = L.block0;
                r.last[0] = L.block1;
                int e = hs::launch_gates(L, gp.tab, r, c128, streamed, stream);
                if (e) return hip_fail((hipError_t)e, "coset kernel launch");
            }
            if (renorm) {
                const int tiles = (int)(P.N / gp.prog.launches[l1 - 1].rows);
                int e = hs::launch_reduce_partials(f->norm_dev, tiles, chunk, f->records(), stream);
                if (e) return hip_fail((hipError_t)e, "norm reduction");
            }
        }
        if (renorm) {
            int e = hs::launch_scale(p, P.N, chunk, rec, c128, stream);
            if (e) return hip_fail((hipError_t)e, "scale kernel");
        }
    }
    return HS_OK;
}

hs_status hs_factors_info(hs_factors f, int *n_qubits, int *n_factors, int *n_terms,
                          int *n_diag_terms, int *dtype, double *dt, int *steps) {
    if (hs_status s = check_handle(f)) return s;
    if (n_qubits) *n_qubits = f->plan.n;
    if (n_factors) *n_factors = (int)f->plan.factors.size();
    if (n_terms) *n_terms = (int)f->plan.terms.size();
    if (n_diag_terms) *n_diag_terms = (int)f->plan.diag.size();
    if (dtype) *dtype = f->dtype;
    if (dt) *dt = f->plan.dt;
    if (steps) *steps = f->plan.steps;
    return HS_OK;
}

hs_status hs_diag_terms(hs_factors f, int *term_idx, int cap) {
    if (hs_status s = check_handle(f)) return s;
    if (cap < (int)f->plan.diag.size() || (!term_idx && !f->plan.diag.empty()))
        return fail(HS_EINVAL, "output too small");
    std::copy(f->plan.diag.begin(), f->plan.diag.end(), term_idx);
    return HS_OK;
}

static hs_status get_factor(hs_factors f, int k, const Factor **out) {
    if (hs_status s = check_handle(f)) return s;
    if (k < 0 || k >= (int)f->plan.factors.size()) return fail(HS_EINVAL, "factor index out of range");
    *out = &f->plan.factors[k];
    return HS_OK;
}

hs_status hs_factor_info(hs_factors f, int k, int *has_diag, int *n_group_terms, int *n_diags,
                         unsigned long long *support_mask, size_t *bytes) {
    const Factor *F = nullptr;
    if (hs_status s = get_factor(f, k, &F)) return s;
    if (has_diag) *has_diag = F->has_diag ? 1 : 0;
    if (n_group_terms) *n_group_terms = (int)F->terms.size();
    if (n_diags) *n_diags = (int)F->offs.size();
    if (support_mask) *support_mask = F->smask;
    if (bytes) *bytes = F->elems_total * elem_bytes(f->dtype);
    return HS_OK;
}

hs_status hs_step_sequence(hs_factors f, int *seq, int cap, int *len) {
    if (hs_status s = check_handle(f)) return s;
    const auto &q = f->plan.seq;
    if (len) *len = (int)q.size();
    if (seq) {
        if (cap < (int)q.size()) return fail(HS_EINVAL, "output too small");
        std::copy(q.begin(), q.end(), seq);
    }
    return HS_OK;
}

hs_status hs_step_joint(hs_factors f, int *factor) {
    if (hs_status s = check_handle(f)) return s;
    if (!factor) return fail(HS_EINVAL, "null output");
    *factor = f->plan.joint;
    return HS_OK;
}

hs_status hs_factor_step(hs_factors f, int k, double *h) {
    const Factor *F = nullptr;
    if (hs_status s = get_factor(f, k, &F)) return s;
    if (!h) return fail(HS_EINVAL, "null output");
    *h = F->dt;
    return HS_OK;
}

hs_status hs_factor_terms(hs_factors f, int k, int *term_idx, int cap) {
    const Factor *F = nullptr;
    if (hs_status s = get_factor(f, k, &F)) return s;
    if (cap < (int)F->terms.size() || (!term_idx && !F->terms.empty())) return fail(HS_EINVAL, "output too small");
    std::copy(F->terms.begin(), F->terms.end(), term_idx);
    return HS_OK;
}

hs_status hs_factor_offsets(hs_factors f, int k, long long *offsets, int cap) {
    const Factor *F = nullptr;
    if (hs_status s = get_factor(f, k, &F)) return s;
    if (cap < (int)F->offs.size() || !offsets) return fail(HS_EINVAL, "output too small");
    for (size_t j = 0; j < F->offs.size(); ++j) offsets[j] = (long long)F->offs[j];
    return HS_OK;
}

hs_status hs_factor_copy_diagonal(hs_factors f, int k, int j, long long start, long long count,
                                  void *host_dst, void *stream) {
    const Factor *F = nullptr;
    if (hs_status s = get_factor(f, k, &F)) return s;
    if (!f->built) return fail(HS_EINVAL, "handle was planned, not built");
    if (j < 0 || j >= (int)F->offs.size()) return fail(HS_EINVAL, "diagonal index out of range");
    const int64_t d = F->offs[j];
    const long long len = f->plan.N - (d < 0 ? -d : d);
    if (start < 0 || count < 0 || start + count > len || !host_dst)
        return fail(HS_EINVAL, "range outside the diagonal's N - |d| entries");
    if (count == 0) return HS_OK;
    const size_t sc = elem_bytes(f->dtype);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const char *src = static_cast<const char *>(F->dev) + F->elem_off[j] * sc;
    if (F->perm_s == 0) {
        HS_HIP(hipMemcpyAsync(host_dst, src + (size_t)start * sc, (size_t)count * sc, hipMemcpyDeviceToHost, st),
               "hipMemcpyAsync(diagonal)");
        HS_HIP(hipStreamSynchronize(st), "hipStreamSynchronize");
        return HS_OK;
    }
    // stored out of natural order: gather the range in pieces of at most
    // 2^22 entries into a temporary, copying each piece to the host
    const long long piece = std::min<long long>(count, 1ll << 22);
    void *tmp = nullptr;
    HS_HIP(hipMallocAsync(&tmp, (size_t)piece * sc, st), "hipMallocAsync(diagonal copy)");
    hipError_t he = hipSuccess;
    for (long long k0 = 0; k0 < count && he == hipSuccess; k0 += piece) {
        const long long m = std::min(piece, count - k0);
        const int e = hs::launch_perm_gather(src, tmp, start + k0, m, len, F->perm_s, F->perm_c,
                                             f->dtype == HS_C128, stream);
        he = e ? (hipError_t)e
               : hipMemcpyAsync(static_cast<char *>(host_dst) + (size_t)k0 * sc, tmp, (size_t)m * sc,
                                hipMemcpyDeviceToHost, st);
        // the next piece reuses the temporary: wait for this copy first
        if (he == hipSuccess) he = hipStreamSynchronize(st);
    }
    const hipError_t fe = hipFreeAsync(tmp, st);
    const hipError_t se = hipStreamSynchronize(st);
    if (he != hipSuccess) return hip_fail(he, "diagonal gather");
    if (fe != hipSuccess) return hip_fail(fe, "hipFreeAsync(diagonal copy)");
    if (se != hipSuccess) return hip_fail(se, "hipStreamSynchronize");
    return HS_OK;
}

hs_status hs_factor_storage(hs_factors f, int k, int *split_bit, int *chunk_bits) {
    const Factor *F = nullptr;
    if (hs_status s = get_factor(f, k, &F)) return s;
    if (split_bit) *split_bit = F->perm_s;
    if (chunk_bits) *chunk_bits = F->perm_c;
    return HS_OK;
}

hs_status hs_step_launches(hs_factors f, int batch, unsigned flags, int part, int *n_launches,
                           int *first_factor, int *n_factors, int cap) {
    if (hs_status s = check_handle(f)) return s;
    if (!f->built) return fail(HS_EINVAL, "handle was planned, not built");
    if (batch < 1 || !n_launches) return fail(HS_EINVAL, "batch >= 1 and an output are required");
    if (part < 0 || part >= kParts) return fail(HS_EINVAL, "part must be 0..3");
    if (flags & ~(unsigned)(HS_RENORM | HS_NO_FUSE)) return fail(HS_EINVAL, "unknown evolve flag");
    const int chunk = std::min(HS_MAX_BATCH, batch);
    std::vector<Run> all[kParts];
    form_runs(f->plan, f->dtype, plan_key(chunk, !(flags & HS_NO_FUSE)), all);
    const auto &runs = all[part];
    *n_launches = (int)runs.size();
    if (first_factor && n_factors) {
        if (cap < (int)runs.size()) return fail(HS_EINVAL, "output too small");
        for (size_t i = 0; i < runs.size(); ++i) {
            first_factor[i] = runs[i].first;
            n_factors[i] = (int)runs[i].factors.size();
        }
    }
    return HS_OK;
}

hs_status hs_evolve_launches(hs_factors f, int batch, unsigned flags, int part, int *n_launches, int *first_factor,
                             int *n_factors, int cap) {
    if (hs_status s = check_handle(f)) return s;
    if (!f->built) return fail(HS_EINVAL, "handle was planned, not built");
    if (batch < 1 || !n_launches) return fail(HS_EINVAL, "batch >= 1 and an output are required");
    if (part < 0 || part >= kParts) return fail(HS_EINVAL, "part must be 0..3");
    if (flags & ~(unsigned)(HS_RENORM | HS_NO_FUSE)) return fail(HS_EINVAL, "unknown evolve flag");
    const Plan &P = f->plan;
    const bool fuse = !(flags & HS_NO_FUSE), renorm = (flags & HS_RENORM) != 0;
    std::vector<std::pair<int, int>> out;
    if (evolves_lone_diagonal(P, renorm) || evolves_whole(P, f->dtype, renorm, fuse)) {
        out.push_back({0, (int)part_sequence(P, part).size()});
    } else {
        std::lock_guard<std::mutex> lock(f->mu);
        const PlanKey key = plan_key(std::min(HS_MAX_BATCH, batch), fuse);
        auto it = f->plans.find(key);
        std::unique_ptr<GatePlan> formed;
        if (it == f->plans.end()) formed = form_gate_plan(P, f->dtype, key, false);
        const GatePlan &gp = formed ? *formed : *it->second;
        for (int l = gp.launch0[part]; l < gp.launch1[part]; ++l)
            out.push_back({gp.prog.launches[l].first, gp.prog.launches[l].count});
    }
    *n_launches = (int)out.size();
    if (first_factor && n_factors) {
        if (cap < (int)out.size()) return fail(HS_EINVAL, "output too small");
        for (size_t i = 0; i < out.size(); ++i) {
            first_factor[i] = out[i].first;
            n_factors[i] = out[i].second;
        }
    }
    return HS_OK;
}

static size_t footprint_bytes(const Plan &P, int dtype, int batch) {
    const size_t sc = elem_bytes(dtype);
    size_t total = 0;
    for (const auto &F : P.factors) {
        const size_t align = hs::kDiagAlignBytes / sc;
        for (int64_t d : F.offs) {
            const size_t len = (size_t)(P.N - (d < 0 ? -d : d));
            total += (len + align - 1) / align * align * sc;
        }
    }
    total += (size_t)batch * P.N * sc;                                // the states
    for (size_t k = 0; k < P.factors.size(); ++k) {
        const Factor &F = P.factors[k];
        // D in FP64 beside the factor's diagonals, or the table that a factor of
        // D alone is built from: 16 N (complex128 states have room for two)
        if (F.has_diag) total += (size_t)P.N * 2 * sc;
        // its matrices in the coset tables, at most a complex value per entry;
        // a batch with a remainder has a program of its own for it
        if (!F.terms.empty())
            total += ((size_t)2 << (F.bits.size() + hs::gate_basis(P, (int)k).size())) * (F.has_diag ? 8 : sc / 2) *
                     (batch > HS_MAX_BATCH && batch % HS_MAX_BATCH ? 2 : 1);
    }
    for (int k : P.seq)                                               // and its blocks, in every step part
        total += (P.joint < 0 ? 1 : kParts) * (sizeof(hs::GateBlock) + 4 * (64 + ((size_t)1 << hs::gate_basis(P, k).size()) / 4)) *
                 (batch > HS_MAX_BATCH && batch % HS_MAX_BATCH ? 2 : 1);
    bool open = false;                                                // a factor no closed tile holds
    for (const auto &F : P.factors)
        if (F.xmask_union && !geometry(F.xlb, F.xhb, P.n, tile_rows_max(dtype, 1, P.N)).ok) open = true;
    if (open) total += (size_t)std::min(batch, HS_MAX_BATCH) * P.N * sc;   // a reserve, as for a scratch state
    // per-tile norm partials when renormalising (tiles of at least 64 rows)
    total += (size_t)std::min(batch, HS_MAX_BATCH) * (size_t)(P.N / 64 + 1) * 4 * sizeof(double);
    total += sizeof(double) * ((size_t)HS_MAX_BATCH * hs::kReduceBlocks * 4 + HS_MAX_BATCH * 4);
    for (const auto &F : P.factors) total += F.L.size() * 16;         // local unitaries while building
    total += 64 * 1024;                                               // the build's other tables
    return total;
}

hs_status hs_footprint(hs_factors f, int batch, size_t *bytes) {
    if (hs_status s = check_handle(f)) return s;
    if (batch < 1 || !bytes) return fail(HS_EINVAL, "batch >= 1 and an output are required");
    *bytes = footprint_bytes(f->plan, f->dtype, batch);
    return HS_OK;
}

hs_status hs_footprint_dtype(hs_factors f, int batch, hs_dtype dtype, size_t *bytes) {
    if (hs_status s = check_handle(f)) return s;
    if (batch < 1 || !bytes) return fail(HS_EINVAL, "batch >= 1 and an output are required");
    if (dtype != HS_C64 && dtype != HS_C128) return fail(HS_EINVAL, "dtype must be HS_C64 or HS_C128");
    *bytes = footprint_bytes(f->plan, dtype, batch);
    return HS_OK;
}

hs_status hs_check(hs_factors f, void *stream, int *violated) {
    if (hs_status s = check_handle(f)) return s;
    if (!f->built || !violated) return fail(HS_EINVAL, "built handle and output required");
    HS_HIP(hipStreamSynchronize(reinterpret_cast<hipStream_t>(stream)), "hipStreamSynchronize");
    std::lock_guard<std::mutex> lock(f->mu);
    bool closed = !f->whole || f->whole->prog.closed;
    for (const auto &kv : f->plans) closed = closed && kv.second->prog.closed;
    *violated = closed ? 0 : 1;
    return HS_OK;
}

hs_status hs_free_factors(hs_factors f) {
    if (!f) return HS_OK;
    delete f;
    return HS_OK;
}

hs_status hs_dia_spmv(int n_diags, const long long *offsets, const void *const *diags, const void *x,
                      void *y, int batch, long long N, hs_dtype dtype, void *stream) {
    if (dtype != HS_C64 && dtype != HS_C128) return fail(HS_EINVAL, "bad dtype");
    if (n_diags < 1 || n_diags > 65535 || !offsets || !diags || !x || !y || batch < 1)
        return fail(HS_EINVAL, "bad arguments");
    if (N < 1 || N > (1ll << HS_MAX_QUBITS)) return fail(HS_EINVAL, "N must be in [1, 2^30]");
    const size_t sc = elem_bytes(dtype);
    const char *xb = static_cast<const char *>(x);
    char *yb = static_cast<char *>(y);
    const size_t span = (size_t)batch * N * sc;
    if (xb < yb + span && yb < xb + span) return fail(HS_EINVAL, "x and y overlap");
    if (reinterpret_cast<uintptr_t>(x) % 16 || reinterpret_cast<uintptr_t>(y) % 16)
        return fail(HS_EINVAL, "x and y must be 16-byte aligned");
    for (int j = 0; j < n_diags; ++j) {
        if (offsets[j] <= -N || offsets[j] >= N) return fail(HS_EINVAL, "offset out of range");
        if (j && offsets[j] <= offsets[j - 1]) return fail(HS_EINVAL, "offsets must ascend strictly");
        if (!diags[j]) return fail(HS_EINVAL, "null diagonal pointer");
        if (reinterpret_cast<uintptr_t>(diags[j]) % 16) return fail(HS_EINVAL, "diagonals must be 16-byte aligned");
        std::string msg;
        const size_t len = (size_t)(N - (offsets[j] < 0 ? -offsets[j] : offsets[j]));
        if (!hs::device_range_ok(diags[j], len * sc, "diagonal", msg)) return fail(HS_EINVAL, msg);
    }
    {
        std::string msg;
        if (!hs::device_range_ok(x, span, "x", msg) || !hs::device_range_ok(y, span, "y", msg))
            return fail(HS_EINVAL, msg);
    }
    std::vector<DiagDesc> hd;
    for (int c0 = 0; c0 < batch; c0 += HS_MAX_BATCH) {
        const int chunk = std::min(HS_MAX_BATCH, batch - c0);
        const Geo geo = generic_geometry(offsets, n_diags, N, dtype, chunk);
        fill_descs(offsets, diags, n_diags, N, geo, hd);
        DiagDesc *ddev = nullptr;
        hipStream_t st = reinterpret_cast<hipStream_t>(stream);
        HS_HIP(hipMallocAsync(reinterpret_cast<void **>(&ddev), sizeof(DiagDesc) * n_diags, st),
               "hipMallocAsync(descriptors)");
        hipError_t e = hipMemcpyAsync(ddev, hd.data(), sizeof(DiagDesc) * n_diags, hipMemcpyHostToDevice, st);
        TileArgs a = open_args(geo, ddev, n_diags, xb + (size_t)c0 * N * sc, yb + (size_t)c0 * N * sc, N);
        a.stream_out = stream_out(chunk, N, dtype);
        if (e == hipSuccess) e = (hipError_t)hs::launch_tile(a, chunk, dtype == HS_C128, stream);
        hipError_t e2 = hipStreamSynchronize(st);
        (void)hipFreeAsync(ddev, st);
        if (e != hipSuccess) return hip_fail(e, "dia_spmv launch");
        if (e2 != hipSuccess) return hip_fail(e2, "dia_spmv");
    }
    return HS_OK;
}

static hs_status reduce_call(const void *A, int ta, const void *B, int tb, int batch, long long N,
                             void *stream, bool dot, std::vector<double> &rec) {
    const int G = hs::kReduceBlocks;
    double *work = nullptr;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    HS_HIP(hipMallocAsync(reinterpret_cast<void **>(&work), sizeof(double) * ((size_t)batch * G * 4 + (size_t)batch * 4), st),
           "hipMallocAsync(reduce)");
    double *out = work + (size_t)batch * G * 4;
    int le = hs::launch_reduce(A, ta, B, tb, batch, N, work, G, out, dot, stream);
    rec.assign((size_t)batch * 4, 0.0);
    hipError_t e = (hipError_t)le;
    if (e == hipSuccess) e = hipMemcpyAsync(rec.data(), out, sizeof(double) * batch * 4, hipMemcpyDeviceToHost, st);
    hipError_t e2 = hipStreamSynchronize(st);
    (void)hipFreeAsync(work, st);
    if (e != hipSuccess) return hip_fail(e, "reduction");
    if (e2 != hipSuccess) return hip_fail(e2, "reduction");
    return HS_OK;
}

hs_status hs_norm2(const void *psi, int batch, long long N, hs_dtype dtype, void *stream, double *out) {
    if (!psi || !out || batch < 1 || N < 1) return fail(HS_EINVAL, "bad arguments");
    if (dtype != HS_C64 && dtype != HS_C128) return fail(HS_EINVAL, "bad dtype");
    {
        std::string msg;
        if (!hs::device_range_ok(psi, (size_t)batch * N * elem_bytes(dtype), "state", msg)) return fail(HS_EINVAL, msg);
    }
    std::vector<double> rec;
    if (hs_status s = reduce_call(psi, dtype, psi, dtype, batch, N, stream, false, rec)) return s;
    for (int b = 0; b < batch; ++b) out[b] = rec[4 * b + 2];
    return HS_OK;
}

hs_status hs_fidelity(const void *phi, int phi_dtype, const void *psi, int psi_dtype, int batch,
                      long long N, void *stream, double *out) {
    if (!phi || !psi || !out || batch < 1 || N < 1) return fail(HS_EINVAL, "bad arguments");
    for (int t : {phi_dtype, psi_dtype})
        if (t != HS_C64 && t != HS_C128) return fail(HS_EINVAL, "bad dtype");
    {
        std::string msg;
        if (!hs::device_range_ok(phi, (size_t)batch * N * elem_bytes(phi_dtype), "phi", msg) ||
            !hs::device_range_ok(psi, (size_t)batch * N * elem_bytes(psi_dtype), "psi", msg))
            return fail(HS_EINVAL, msg);
    }
    std::vector<double> rec;
    if (hs_status s = reduce_call(phi, phi_dtype, psi, psi_dtype, batch, N, stream, true, rec)) return s;
    for (int b = 0; b < batch; ++b) {
        const double re = rec[4 * b], im = rec[4 * b + 1], np = rec[4 * b + 2], nq = rec[4 * b + 3];
        out[5 * b + 0] = re;
        out[5 * b + 1] = im;
        out[5 * b + 2] = np;
        out[5 * b + 3] = nq;
        out[5 * b + 4] = (re * re + im * im) / (np * nq);
    }
    return HS_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- no allocation
//
// Scratch of hs_fidelity_noalloc: the FP64 reduction partials of up to
// HS_MAX_BATCH states ([8][kReduceBlocks][4]) and their records ([8][4]),
// 256.25 KiB in every GPU the library runs on, held until the process ends.
// Host code never uses the array's name as an address: each device's copy is
// found once with hipGetSymbolAddress and its pointer kept per device.
namespace {
constexpr size_t kNoAllocPartials = (size_t)HS_MAX_BATCH * hs::kReduceBlocks * 4;
constexpr size_t kNoAllocDoubles = kNoAllocPartials + (size_t)HS_MAX_BATCH * 4;
constexpr int kNoAllocDevices = 64;
}  // namespace

static __device__ __align__(256) double scratch[kNoAllocDoubles];

static double *noalloc_scratch(std::string &msg) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        msg = std::string("hipGetDevice: ") + hipGetErrorString(e);
        return nullptr;
    }
    if (dev < 0 || dev >= kNoAllocDevices) {
        msg = "device index beyond the 64 devices the scratch table covers";
        return nullptr;
    }
    static std::mutex mu;
    static double *ptr[kNoAllocDevices] = {};
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            msg = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
            return nullptr;
        }
        ptr[dev] = static_cast<double *>(p);
    }
    return ptr[dev];
}

extern "C" hs_status hs_fidelity_noalloc(const void *phi, int phi_dtype, const void *psi, int psi_dtype, int batch,
                                         long long N, void *stream, double *out_dev) {
    if (!phi || !psi || !out_dev || N < 1) return fail(HS_EINVAL, "bad arguments");
    if (batch < 1 || batch > HS_MAX_BATCH)
        return fail(HS_EINVAL, "batch must be 1.." + std::to_string(HS_MAX_BATCH) +
                                   ": the static scratch holds the partial sums of that many states");
    for (int t : {phi_dtype, psi_dtype})
        if (t != HS_C64 && t != HS_C128) return fail(HS_EINVAL, "bad dtype");
    std::string msg;
    if (!hs::device_range_ok(phi, (size_t)batch * N * elem_bytes(phi_dtype), "phi", msg) ||
        !hs::device_range_ok(psi, (size_t)batch * N * elem_bytes(psi_dtype), "psi", msg) ||
        !hs::device_range_ok(out_dev, (size_t)batch * 5 * sizeof(double), "out", msg))
        return fail(HS_EINVAL, msg);
    double *s = noalloc_scratch(msg);
    if (!s) return fail(HS_EDEVICE, msg);
    double *rec = s + kNoAllocPartials;
    // every partial and record the kernels read is written by this call first
    int e = hs::launch_reduce(phi, phi_dtype, psi, psi_dtype, batch, N, s, hs::kReduceBlocks, rec, true, stream);
    if (e) return hip_fail((hipError_t)e, "reduction");
    e = hs::launch_fidelity_records(rec, batch, out_dev, stream);
    if (e) return hip_fail((hipError_t)e, "fidelity records");
    return HS_OK;
}
