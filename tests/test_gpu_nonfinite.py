"""Infinite and NaN amplitudes in products with operators: a row is affected
only through a nonzero coefficient, whatever else the kernels load (structural
zeros of stored diagonals, diagonals they pad to, coefficients that cancel),
and its value is that of the sum over its nonzero coefficients in ascending
offset order."""
import numpy as np
import pytest

from gpu_common import hs_gpu, note, tol_c64

pytestmark = pytest.mark.gpu


def _reference(diags, x):
    """The sum over nonzero coefficients, real products one after the other."""
    N = x.shape[-1]
    re, im = np.zeros(x.shape), np.zeros(x.shape)
    with np.errstate(invalid="ignore"):
        for o in sorted(diags):
            lo, hi = max(0, -o), min(N, N - o)
            c, v = diags[o], x[..., lo + o:hi + o]
            keep = np.broadcast_to(c != 0, v.shape)
            r, i = re[..., lo:hi], im[..., lo:hi]
            re[..., lo:hi] = np.where(keep, r + c.real * v.real - c.imag * v.imag, r)
            im[..., lo:hi] = np.where(keep, i + c.real * v.imag + c.imag * v.real, i)
    return re, im


def _check(got, re, im, dtype, mag):
    for g, w in ((got.real, re), (got.imag, im)):
        assert np.array_equal(np.isnan(g), np.isnan(w))
        inf = np.isinf(w)
        assert np.array_equal(g[inf], w[inf].astype(g.dtype)) and np.array_equal(np.isinf(g), inf)
        ok = np.isfinite(w)
        assert np.all(np.abs(g[ok] - w[ok]) <= (1e-14 if dtype == "c128" else tol_c64()) * mag)


def _sparse(N, nd, dtype, seed):
    """Diagonals half of whose entries are zero, the main one absent."""
    rng = np.random.default_rng(seed)
    pool = [1, -1, N - 1, 1 - N] + [int(o) for o in rng.permutation(2 * N - 1) - (N - 1)]
    offs = list(dict.fromkeys(o for o in pool if o and abs(o) < N))[:nd]
    out = {}
    for o in offs:
        v = rng.normal(size=N - abs(o)) + 1j * rng.normal(size=N - abs(o))
        out[o] = (v * (rng.random(N - abs(o)) < 0.5)).astype(np.complex128 if dtype == "c128" else np.complex64)
    return out


@pytest.mark.parametrize("N,nd,dtype", [(64, 3, "c64"), (300, 9, "c128"), (1000, 17, "c64"), (1024, 21, "c128"),
                                        (512, 40, "c128"), (1024, 33, "c64"), (5000, 7, "c128"), (70000, 33, "c64")])
def test_products_reach_only_coupled_rows(N, nd, dtype):
    hs, torch = hs_gpu()
    from paper_2606_16959_amd import dia
    note(f"non-finite amplitudes N={N} diagonals={nd} {dtype}")
    npd = np.complex128 if dtype == "c128" else np.complex64
    diags = _sparse(N, nd, dtype, N + nd)
    rng = np.random.default_rng(N)
    x = (rng.normal(size=(2, N)) + 1j * rng.normal(size=(2, N))).astype(npd)
    x[0, N // 2] = np.inf
    x[1, N // 3] = complex(-np.inf, 1.0)
    x[1, 5] = complex(0.0, np.nan)
    re, im = _reference({o: v.astype(np.complex128) for o, v in diags.items()}, x.astype(np.complex128))
    assert np.isfinite(re).mean() > 0.3 and not np.isfinite(re).all()
    offs = sorted(diags)
    dev = [torch.from_numpy(diags[o]).cuda() for o in offs]
    mag = nd * max(np.abs(v).max() for v in diags.values()) * 6.0
    _check(hs.dia_spmv(offs, dev, torch.from_numpy(x).cuda()).cpu().numpy(), re, im, dtype, mag)
    U = dia.from_dict({o: v.astype(np.complex128) for o, v in diags.items()}, N)
    if dtype == "c64":
        U = U.to_c64()
    psi = torch.from_numpy(x.copy()).cuda()
    dia.evolve(U, psi, 1)
    _check(psi.cpu().numpy(), re, im, dtype, mag)


@pytest.mark.parametrize("n,batch,dtype", [(6, 1, "c128"), (12, 2, "c64"), (19, 2, "c64"), (19, 1, "c128"), (20, 1, "c64")])
def test_taylor_stage_reaches_only_coupled_rows(n, batch, dtype):
    """XX + YY bonds: a row is coupled through a bond only where its two bits
    differ; elsewhere the coefficient cancels."""
    hs, torch = hs_gpu()
    from paper_2606_16959_amd import dia
    note(f"non-finite amplitudes in a Taylor stage n={n} batch={batch} {dtype}")
    bonds = [(q, q + 1) for q in range(n - 1)]
    strings = ["".join(p if q in b else "I" for q in range(n)) for b in bonds for p in "XY"]
    H = dia.from_pauli(strings, [0.5] * len(strings), n)
    if dtype == "c64":
        H = H.to_c64()
    N = 1 << n
    psi = torch.ones((batch, N), dtype=torch.complex128 if dtype == "c128" else torch.complex64, device="cuda")
    at = (N // 3) & ~1 | (N >> 1)
    psi[:, at] = float("inf")
    dia.taylor_evolve(H, psi, 0.1, 1, 1)
    bad = ~torch.isfinite(torch.view_as_real(psi)).all(-1)
    # string index 0 is the highest or the lowest bit: bonds are the same pairs
    want = {at} | {at ^ (3 << q) for q in range(n - 1) if ((at >> q) & 1) != ((at >> (q + 1)) & 1)}
    for b in range(batch):
        assert set(bad[b].nonzero().flatten().tolist()) == want


@pytest.mark.parametrize("N,dtype", [(300, "c64"), (512, "c128"), (1500, "c64")])
def test_an_amplitude_that_leaves_the_state_is_forgotten(N, dtype):
    """U with one superdiagonal shifts the state down: after 5 steps an infinite
    amplitude of the first five rows is gone, one further up has moved by 5."""
    hs, torch = hs_gpu()
    from paper_2606_16959_amd import dia
    note(f"shift of an infinite amplitude N={N} {dtype}")
    U = dia.from_dict({1: np.full(N - 1, 0.5)}, N)
    if dtype == "c64":
        U = U.to_c64()
    x = np.random.default_rng(N).normal(size=(2, N)).astype(np.complex128 if dtype == "c128" else np.complex64)
    x[0, 3] = np.inf
    x[1, 100] = np.inf
    psi = torch.from_numpy(x.copy()).cuda()
    dia.evolve(U, psi, 5)
    got = psi.cpu().numpy()
    want = np.zeros_like(x)
    with np.errstate(invalid="ignore"):
        want[:, :N - 5] = x[:, 5:] * 0.5 ** 5
    want[1, 95] = got[1, 95]
    assert not np.isfinite(got[1, 95]) and np.array_equal(got, want, equal_nan=True)
