"""The work that users of this framework have it do, as timed cases.

Every case goes through the package's public calls: Trotter evolution of one
or many states, whole small jobs from Pauli strings, diagonal Hamiltonians,
the Taylor update, the single-propagator pipeline, DIA products with a
caller's own diagonals, and state overlaps.  `exact` gives the same results
in 64 bits from plain torch and numpy, by Pauli rotations on the state, dense
matrices or row-by-row sums.
"""
import math

import numpy as np
import torch

import paper_2606_16959_amd as hs
from paper_2606_16959_amd import dia

BUDGET = 16            # diagonals per Trotter factor
TOL = 1e-6             # Taylor tolerance of the propagator pipelines
LARGEST = 1 << 27      # rows x states x steps of the largest listed case


def listed():
    return [
        # the smallest job: an 8-qubit chain, ten steps; latency is all of it
        {"name": "evolve_tfim_n8", "kind": "evolve", "model": "tfim", "n": 8, "batch": 1, "dtype": "c128",
         "t": 1.0, "r": 10, "steps": 10, "order": 1, "renorm": False},
        # a served request, whole: factors from the strings, evolution, norms
        {"name": "job_heis_n13", "kind": "job", "model": "heis", "n": 13, "batch": 3, "dtype": "c64",
         "t": 1.0, "r": 40, "steps": 40, "order": 1, "renorm": False},
        # a mid-size chain in double precision, from a state that fits the caches
        {"name": "evolve_heis_n20", "kind": "evolve", "model": "heis", "n": 20, "batch": 1, "dtype": "c128",
         "t": 2.0, "r": 100, "steps": 10, "order": 1, "renorm": False},
        # second-order product, an odd number of states, renormalised each step
        {"name": "evolve_order2_n17", "kind": "evolve", "model": "heis", "n": 17, "batch": 3, "dtype": "c64",
         "t": 1.0, "r": 50, "steps": 8, "order": 2, "renorm": True},
        # eight states at once under a MaxCut Hamiltonian with a mixer
        {"name": "evolve_maxcut_n24_b8", "kind": "evolve", "model": "maxcut", "n": 24, "batch": 8, "dtype": "c64",
         "t": 1.0, "r": 200, "steps": 1, "order": 1, "renorm": False},
        # the largest: a 5x5 lattice and an idle qubit, 512 MiB of state
        {"name": "evolve_lattice_n26", "kind": "evolve", "model": "lattice", "n": 26, "batch": 1, "dtype": "c64",
         "t": 1.0, "r": 50, "steps": 2, "order": 1, "renorm": False},
        # a cost function alone: one diagonal, many steps
        {"name": "diagonal_n22_b2", "kind": "evolve", "model": "cost", "n": 22, "batch": 2, "dtype": "c64",
         "t": 1.0, "r": 200, "steps": 25, "order": 1, "renorm": False},
        # the Taylor update on a chain, H kept in hand
        {"name": "taylor_tfim_n23", "kind": "taylor", "model": "tfim", "n": 23, "batch": 1, "dtype": "c64",
         "theta": 0.9, "terms": 9, "steps": 1},
        # the Taylor update from the strings on, at a small size
        {"name": "taylor_job_heis_n12", "kind": "taylor_job", "model": "heis", "n": 12, "batch": 1, "dtype": "c128",
         "t": 0.5},
        # Algorithm 3 from the strings on: step search, propagator, U^r psi
        {"name": "alg3_tfim_n10", "kind": "alg3", "model": "tfim", "n": 10, "batch": 1, "dtype": "c128",
         "t": 0.25, "budget": 61},
        # DIA product with the caller's own diagonals, a size that is no power of two
        {"name": "spmv_ragged_b3", "kind": "spmv", "N": 1000003, "diags": 21, "batch": 3, "dtype": "c64"},
        # overlap and norms of states in two precisions
        {"name": "overlap_n24_b2", "kind": "overlap", "N": 1 << 24, "batch": 2, "dtype": "c64", "other": "c128"},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["evolve"] * 6 + ["job"] * 2 + ["taylor"] * 2 + ["taylor_job", "alg3", "spmv", "spmv", "overlap"])
    dtype = rng.choice(["c64", "c64", "c128"])
    if kind == "evolve":
        model = rng.choice(["tfim", "heis", "maxcut", "lattice", "cost"])
        n = rng.randint(4, 24 if dtype == "c64" else 23)
        if model == "maxcut" or model == "cost":
            n = max(4, n - n % 2)
        batch = rng.randint(1, 8)
        while (batch << n) > LARGEST // 2:
            batch -= 1
        steps = max(1, min(_log_int(rng, 1, 60), LARGEST // 2 // (batch << n)))
        order = 1 if model == "cost" else rng.choice([1, 1, 2])
        renorm = model != "cost" and rng.random() < 0.25
        return {"kind": kind, "model": model, "n": n, "batch": batch, "dtype": dtype, "t": 1.0,
                "r": max(steps, rng.randint(20, 200)), "steps": steps, "order": order, "renorm": renorm}
    if kind == "job":
        n = rng.randint(6, 18)
        model = rng.choice(["tfim", "heis", "maxcut"])
        if model == "maxcut":
            n -= n % 2
        steps = rng.randint(5, 60)
        return {"kind": kind, "model": model, "n": n, "batch": rng.randint(1, 8), "dtype": dtype, "t": 1.0,
                "r": steps, "steps": steps, "order": 1, "renorm": rng.random() < 0.25}
    if kind == "taylor":
        n = rng.randint(10, 22)
        model = rng.choice(["tfim", "heis", "lattice"])
        batch = rng.randint(1, 4)
        while (batch << n) > (1 << 22):
            batch -= 1
        return {"kind": kind, "model": model, "n": n, "batch": max(1, batch), "dtype": dtype,
                "theta": round(rng.uniform(0.3, 1.0), 3), "terms": rng.randint(3, 11),
                "steps": max(1, min(rng.randint(1, 6), (1 << 22) // (max(1, batch) << n)))}
    if kind == "taylor_job":
        return {"kind": kind, "model": rng.choice(["tfim", "heis"]), "n": rng.randint(6, 14), "batch": rng.randint(1, 4),
                "dtype": dtype, "t": round(rng.uniform(0.1, 0.6), 3)}
    if kind == "alg3":
        n = rng.randint(5, 10)
        return {"kind": kind, "model": "tfim", "n": n, "batch": rng.randint(1, 3), "dtype": dtype,
                "t": round(rng.uniform(0.05, 0.25), 3), "budget": 2 * n + 1 + rng.randint(10, 60)}
    if kind == "spmv":
        N = _log_int(rng, 1000, 1 << 22)
        batch = rng.randint(1, 8)
        while batch > 1 and batch * N > (1 << 23):
            batch -= 1
        return {"kind": kind, "N": N, "diags": rng.randint(3, 41), "batch": batch, "dtype": dtype}
    return {"kind": kind, "N": _log_int(rng, 1000, 1 << 24), "batch": rng.randint(1, 4), "dtype": dtype,
            "other": rng.choice(["c64", "c128"])}


# ------------------------------------------------------------------ inputs

def _rng(seed, salt):
    return np.random.default_rng([int(seed), salt])


def _cubic_graph(n, rng):
    while True:
        pairs = rng.permutation(np.repeat(np.arange(n), 3)).reshape(-1, 2)
        edges = {tuple(sorted((int(a), int(b)))) for a, b in pairs}
        if np.all(pairs[:, 0] != pairs[:, 1]) and len(edges) == len(pairs):
            return sorted(edges)


def _hamiltonian(model, n, seed):
    """Ordered terms [({qubit: Pauli}, coefficient)] of a model of `n` qubits."""
    rng = _rng(seed, 1)
    if model in ("tfim", "lattice"):
        h = rng.uniform(0.5, 3.1)
        if model == "tfim":
            sites, bonds = n, [(q, q + 1) for q in range(n - 1)]
        else:                      # rows x cols sites, the remaining qubits idle
            cols = max(2, math.isqrt(n))
            rows = n // cols
            sites = rows * cols
            bonds = [(cols * r + c, cols * r + c + 1) for r in range(rows) for c in range(cols - 1)]
            bonds += [(cols * r + c, cols * r + c + cols) for r in range(rows - 1) for c in range(cols)]
        return [({i: "Z", j: "Z"}, -1.0) for i, j in bonds] + [({q: "X"}, -h) for q in range(sites)]
    if model == "heis":
        terms = [({q: p, q + 1: p}, 1.0) for q in range(n - 1) for p in "XYZ"]
        return terms + [({q: "Z"}, float(v)) for q, v in enumerate(rng.uniform(-1.0, 1.0, n))]
    edges = _cubic_graph(n, rng)   # weighted MaxCut cost, with or without a mixer
    w = rng.uniform(1.0, 10.0, len(edges))
    terms = [({}, 0.5 * float(w.sum()))] + [({i: "Z", j: "Z"}, -0.5 * float(x)) for (i, j), x in zip(edges, w)]
    return terms + ([({q: "X"}, 0.7) for q in range(n)] if model == "maxcut" else [])


def _strings(terms, n):
    return ["".join(ops.get(q, "I") for q in range(n)) for ops, _ in terms], [c for _, c in terms]


def _states(N, batch, dtype, seed):
    """Random-phase states of unit norm, [batch, N] on the device."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) % (1 << 62))
    real = torch.float32 if dtype == "c64" else torch.float64
    u = torch.rand((batch, N), generator=g, device="cuda", dtype=real) * (2.0 * math.pi)
    return torch.polar(torch.full_like(u, 1.0 / math.sqrt(N)), u)


def _taylor_dt(case, seed):
    """dt with dt * (sum of all coefficients) = theta."""
    terms = _hamiltonian(case["model"], case["n"], seed)
    return case["theta"] / sum(2 ** len([p for p in ops.values() if p in "XY"]) * abs(c) for ops, c in terms)


def _spmv_inputs(case, seed):
    N, rng = case["N"], _rng(seed, 2)
    near = rng.integers(-64, 65, size=case["diags"])
    far = (rng.uniform(-0.9, 0.9, size=case["diags"]) * N).astype(np.int64)
    offs = sorted({int(o) for o in np.where(rng.random(case["diags"]) < 0.5, near, far)} | {0})
    real = torch.float32 if case["dtype"] == "c64" else torch.float64
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) % (1 << 62) + 1)
    diags = [torch.view_as_complex(torch.randn((N - abs(o), 2), generator=g, device="cuda", dtype=real) * 0.2)
             for o in offs]
    return offs, diags, _states(N, case["batch"], case["dtype"], seed)


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "spmv":
        st["offsets"], st["diags"], st["x"] = _spmv_inputs(case, seed)
        st["y"] = torch.empty_like(st["x"])
        return st
    if kind == "overlap":
        st["phi"] = _states(case["N"], case["batch"], case["dtype"], seed)
        st["psi"] = _states(case["N"], case["batch"], case["other"], seed + 1)
        return st
    st["strings"], st["coeffs"] = _strings(_hamiltonian(case["model"], case["n"], seed), case["n"])
    st["psi"] = _states(1 << case["n"], case["batch"], case["dtype"], seed)
    if kind == "evolve":
        st["factors"] = hs.build_factors(st["strings"], st["coeffs"], case["n"], case["t"], case["r"], BUDGET,
                                         dtype=case["dtype"], order=case["order"])
    if kind == "taylor":
        H = dia.from_pauli(st["strings"], st["coeffs"], case["n"])
        st["H"] = H if case["dtype"] == "c128" else H.to_c64()
        st["dt"] = _taylor_dt(case, seed)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "evolve":
        return hs.evolve(st["factors"], st["psi"], case["steps"], renorm=case["renorm"])
    if kind == "job":
        f = hs.build_factors(st["strings"], st["coeffs"], case["n"], case["t"], case["r"], BUDGET,
                             dtype=case["dtype"], order=case["order"])
        hs.evolve(f, st["psi"], case["steps"], renorm=case["renorm"])
        norms = hs.norm2(st["psi"])
        f.close()
        return st["psi"], norms
    if kind == "taylor":
        return dia.taylor_evolve(st["H"], st["psi"], st["dt"], case["terms"], case["steps"])
    if kind == "taylor_job":
        r, K = dia.taylor_simulate(st["strings"], st["coeffs"], case["n"], case["t"], st["psi"], tol=TOL,
                                   dtype=case["dtype"])
        return st["psi"], r, K
    if kind == "alg3":
        r, K, nd = dia.simulate(st["strings"], st["coeffs"], case["n"], case["t"], st["psi"],
                                budget=case["budget"], tol=TOL, dtype=case["dtype"])
        return st["psi"], r, K, nd
    if kind == "spmv":
        return hs.dia_spmv(st["offsets"], st["diags"], st["x"], y=st["y"])
    return hs.fidelity(st["phi"], st["psi"])


# -------------------------------------------------------------------- work

def work(case):
    """Bytes and operations that a pass cannot do without: each state read
    once and written once, a caller's diagonals read once; six operations
    per row for every Pauli rotation and for the diagonal phase, eight for
    every complex multiply-add."""
    kind = case["kind"]
    sc = 8 if case["dtype"] == "c64" else 16
    if kind == "overlap":
        so = 8 if case["other"] == "c64" else 16
        rows = case["batch"] * case["N"]
        return {"bytes": rows * (sc + so), "flops": rows * 16}
    if kind == "spmv":
        offs = case["N"] * case["diags"] * 0.75      # half of the offsets are near 0, half reach far
        return {"bytes": int(offs * sc + 2 * case["batch"] * case["N"] * sc), "flops": int(8 * offs * case["batch"])}
    terms = _hamiltonian(case["model"], case["n"], 0)
    flips = len([1 for ops, _ in terms if any(p in "XY" for p in ops.values())])
    rows = case["batch"] << case["n"]
    if kind == "alg3":
        applications = 16 * flips
    elif kind == "taylor_job":
        applications = 100 * flips
    elif kind == "taylor":
        applications = case["steps"] * case["terms"] * (flips + 1)
    else:
        applications = case["steps"] * (flips + 1) * (2 if case["order"] == 2 and flips else 1)
    return {"bytes": 2 * rows * sc, "flops": rows * 6 * applications}


# ------------------------------------------------------------------- exact

def _masks(ops):
    x = sum(1 << q for q, p in ops.items() if p in "XY")
    z = sum(1 << q for q, p in ops.items() if p in "YZ")
    return x, z, sum(1 for p in ops.values() if p == "Y")


def _sign(idx, z):
    """(-1)^popcount(idx & z) as float64."""
    par = torch.zeros_like(idx)
    q = 0
    while z >> q:
        if (z >> q) & 1:
            par ^= (idx >> q) & 1
        q += 1
    return 1.0 - 2.0 * par.to(torch.float64)


def _pauli(psi, idx, ops):
    """P psi for [batch, N] states: (P psi)[x ^ m] = i^ny (-1)^popcount(x & z) psi[x]."""
    x, z, ny = _masks(ops)
    out = psi if z == 0 else psi * _sign(idx, z)
    if x:
        n = idx.numel().bit_length() - 1
        out = out.reshape([psi.shape[0]] + [2] * n)
        out = out.flip([n - q for q in range(n) if (x >> q) & 1]).reshape(psi.shape)
    return out * (1j ** ny)


def _energies(terms, idx):
    E = torch.zeros(idx.numel(), dtype=torch.float64, device=idx.device)
    for ops, c in terms:
        x, z, _ = _masks(ops)
        if x == 0:
            E += c * _sign(idx, z)
    return E


def _diag_count(terms, group, dt):
    """Nonzero diagonals of the product of a commuting group's rotations."""
    qs = sorted({q for k in group for q in terms[k][0]})
    pauli = {"I": np.eye(2), "X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]), "Z": np.diag([1, -1])}
    U = np.eye(1 << len(qs), dtype=np.complex128)
    for k in group:
        ops, c = terms[k]
        P = np.eye(1)
        for q in qs:                       # first qubit = least significant bit
            P = np.kron(pauli[ops.get(q, "I")], P)
        U = (math.cos(c * dt) * np.eye(len(P)) - 1j * math.sin(c * dt) * P) @ U
    val = [sum(1 << q for j, q in enumerate(qs) if (a >> j) & 1) for a in range(len(U))]
    a, b = np.nonzero(np.abs(U) > 1e-15)
    return len({val[j] - val[i] for i, j in zip(a, b)})


def _groups(terms, dt):
    """First-fit groups of commuting terms whose exponential keeps the budget."""
    groups, known = [], {}
    for k, (ops, _) in enumerate(terms):
        x, z, _ny = _masks(ops)
        if x == 0:
            continue
        for g in groups:
            if any((bin(x & _masks(terms[j][0])[1]).count("1") + bin(z & _masks(terms[j][0])[0]).count("1")) & 1
                   for j in g):
                continue
            if len({q for j in g + [k] for q in terms[j][0]}) > 10:
                continue
            if known.setdefault(tuple(g + [k]), None) is None:
                known[tuple(g + [k])] = _diag_count(terms, g + [k], dt)
            if known[tuple(g + [k])] <= BUDGET:
                g.append(k)
                break
        else:
            groups.append([k])
    return groups


def _exact_evolve(case, seed):
    terms = _hamiltonian(case["model"], case["n"], seed)
    psi = _states(1 << case["n"], case["batch"], case["dtype"], seed).to(torch.complex128)
    idx = torch.arange(1 << case["n"], device=psi.device)
    dt = case["t"] / case["r"]
    E = _energies(terms, idx)
    gens = [None] + _groups(terms, dt)     # None: the diagonal factor
    if case["order"] == 2 and len(gens) > 1:
        seq = [(g, dt / 2) for g in gens[:-1]] + [(gens[-1], dt)] + [(g, dt / 2) for g in gens[-2::-1]]
    else:
        seq = [(g, dt) for g in gens]
    if case["renorm"]:
        psi /= torch.linalg.vector_norm(psi, dim=1, keepdim=True)
    for _ in range(case["steps"]):
        for g, h in seq:
            if g is None:
                psi *= torch.polar(torch.ones_like(E), -h * E)
                continue
            for k in g:
                ops, c = terms[k]
                psi = math.cos(c * h) * psi - 1j * math.sin(c * h) * _pauli(psi, idx, ops)
        if case["renorm"]:
            psi /= torch.linalg.vector_norm(psi, dim=1, keepdim=True)
    return psi


def _apply_h(terms, E, idx, psi):
    out = psi * E
    for ops, c in terms:
        if any(p in "XY" for p in ops.values()):
            out += c * _pauli(psi, idx, ops)
    return out


def _exact_taylor(case, seed, dt, K, steps):
    terms = _hamiltonian(case["model"], case["n"], seed)
    psi = _states(1 << case["n"], case["batch"], case["dtype"], seed).to(torch.complex128)
    idx = torch.arange(1 << case["n"], device=psi.device)
    E = _energies(terms, idx)
    for _ in range(steps):
        t, acc = psi, psi.clone()
        for k in range(1, K + 1):
            t = _apply_h(terms, E, idx, t) * (-1j * dt / k)
            acc += t
        psi = acc
    return psi


def _dense_h(terms, n):
    idx = torch.arange(1 << n, device="cuda")
    eye = torch.eye(1 << n, dtype=torch.complex128, device="cuda")
    return _apply_h(terms, _energies(terms, idx), idx, eye).T.contiguous()   # rows of eye are the unit states


def _offset_maxima(H):
    """Largest modulus on each nonzero diagonal, by ascending offset."""
    N = len(H)
    col = torch.arange(N, device=H.device)
    off = (col[None, :] - col[:, None] + N - 1).reshape(-1)
    mx = torch.zeros(2 * N - 1, dtype=torch.float64, device=H.device)
    mx.scatter_reduce_(0, off, H.abs().reshape(-1), "amax")
    mx = mx.cpu().numpy()
    return {int(d) - (N - 1): float(mx[d]) for d in np.nonzero(mx)[0]}


def _sums(a, b, N):
    return {x + y for x in a for y in b if -N < x + y < N}


def _exact_alg3(case, seed):
    n, N, t, budget = case["n"], 1 << case["n"], case["t"], case["budget"]
    H = _dense_h(_hamiltonian(case["model"], n, seed), n)
    mx = _offset_maxima(H)
    nu = sum(mx[d] for d in sorted(mx))
    powers, maxima, upto, last = [H], [float(H.abs().max())], [{0} | set(mx)], set(mx)

    def term(k):                                  # max |H^k| and the offsets of H^0 .. H^k
        nonlocal last
        while len(powers) < k:
            powers.append(powers[-1] @ H)
            maxima.append(float(powers[-1].abs().max()))
            last = _sums(last, set(mx), N)
            upto.append(upto[-1] | last)
        return maxima[k - 1], upto[k - 1]

    def propagator(r):                            # squarings, terms and offsets at step t / r
        s = 0
        while t / r * nu > 0.5 * 2.0 ** s:
            s += 1
        c, K = 1.0, 0
        for k in range(1, 31):
            c *= t / r / 2 ** s / k
            m, _ = term(k)
            if c * m < TOL:
                break
            K = k
        offs = upto[K - 1] if K else {0}
        for _ in range(s):
            if len(offs) > budget:
                break
            offs = _sums(offs, offs, N)
        return s, K, offs

    r = 1
    if len(propagator(1)[2]) > budget:
        lo, r = 1, 2
        while len(propagator(r)[2]) > budget:
            lo, r = r, 2 * r
        while r - lo > 1:
            mid = (lo + r) // 2
            if len(propagator(mid)[2]) > budget:
                lo = mid
            else:
                r = mid
    s, K, offs = propagator(r)
    U = torch.eye(N, dtype=torch.complex128, device="cuda")
    T = U.clone()
    for k in range(1, K + 1):
        T = T @ H * (-1j * t / r / 2 ** s / k)
        U = U + T
    U = torch.linalg.matrix_power(U, 2 ** s)
    psi = _states(N, case["batch"], case["dtype"], seed).to(torch.complex128)
    return psi @ torch.linalg.matrix_power(U, r).T.contiguous(), r, K, len(offs)


def _exact_taylor_job(case, seed):
    # r and K from nu(H) alone: |t / r| nu <= 1, and (|t / r| nu)^(K+1) / (K+1)! < TOL
    terms = _hamiltonian(case["model"], case["n"], seed)
    idx = torch.arange(1 << case["n"], device="cuda")
    nu = float(_energies(terms, idx).abs().max())
    for ops, c in terms:                          # every chain term flips one qubit or a bond
        if set(ops.values()) == {"X"}:
            nu += 2 * abs(c) * len(ops)           # a bond's XX + YY: 2 |c| on two diagonals
    r = max(1, math.ceil(case["t"] * nu))
    x = case["t"] / r * nu
    K, b = 0, x
    while K == 0 or b >= TOL:
        K += 1
        b *= x / (K + 1)
    return _exact_taylor(case, seed, case["t"] / r, K, r), r, K


def exact(case, seed):
    kind = case["kind"]
    if kind == "evolve":
        return _exact_evolve(case, seed)
    if kind == "job":
        psi = _exact_evolve(case, seed)
        return psi, (psi.abs() ** 2).sum(dim=1).cpu().numpy()
    if kind == "taylor":
        return _exact_taylor(case, seed, _taylor_dt(case, seed), case["terms"], case["steps"])
    if kind == "taylor_job":
        return _exact_taylor_job(case, seed)
    if kind == "alg3":
        return _exact_alg3(case, seed)
    if kind == "spmv":
        offs, diags, x = _spmv_inputs(case, seed)
        x = x.to(torch.complex128)
        y = torch.zeros_like(x)
        for o, v in zip(offs, diags):             # row r meets column r + o; entry min(r, r + o)
            lo, hi = max(0, -o), min(case["N"], case["N"] - o)
            y[:, lo:hi] += v.to(torch.complex128) * x[:, lo + o:hi + o]
        return y
    phi = _states(case["N"], case["batch"], case["dtype"], seed).to(torch.complex128)
    psi = _states(case["N"], case["batch"], case["other"], seed + 1).to(torch.complex128)
    dot = (phi.conj() * psi).sum(dim=1).cpu().numpy()
    p2, q2 = ((v.abs() ** 2).sum(dim=1).cpu().numpy() for v in (phi, psi))
    return np.stack([dot.real, dot.imag, p2, q2, np.abs(dot) ** 2 / (p2 * q2)], axis=1)
