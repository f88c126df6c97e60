"""Products with stored diagonals at the size where the row kernel hands over
to the tile kernel: one state of N rows (row kernel) gives the bits of the
same state in a batch large enough for the tiles, and both the definition
y[r] = sum_d A[r, r + d] x[r + d].  Also the row kernel's edges: fewer
diagonals than it loads ahead, one row, the Horner form."""
import numpy as np
import pytest

from gpu_common import hs_gpu, note, tol_c64

pytestmark = pytest.mark.gpu
ROWS_MAX = 1 << 18            # rows x states of the row kernel


def _operator(N, nd, seed):
    rng = np.random.default_rng(seed)
    offs = sorted({0, N - 1, 1 - N} | {int(o) for o in rng.integers(1 - N, N, size=nd)} | {-1, 1, 2} & set(range(1 - N, N)))
    return {o: rng.normal(size=N - abs(o)) + 1j * rng.normal(size=N - abs(o)) for o in offs}


def _reference(diags, x):
    y, mag = np.zeros_like(x), np.zeros(x.shape)
    N = x.shape[-1]
    for o, v in diags.items():
        lo, hi = max(0, -o), min(N, N - o)
        y[..., lo:hi] += v * x[..., lo + o:hi + o]
        mag[..., lo:hi] += np.abs(v) * np.abs(x[..., lo + o:hi + o])
    return y, mag


@pytest.mark.parametrize("N,nd,dtype", [(1, 1, "c64"), (2, 2, "c128"), (63, 13, "c64"), (1025, 30, "c128"),
                                        (ROWS_MAX, 17, "c64"), (ROWS_MAX - 1, 5, "c128"), (ROWS_MAX // 3, 16, "c128")])
def test_row_kernel_equals_tiles_and_definition(N, nd, dtype):
    hs, torch = hs_gpu()
    npd = np.complex128 if dtype == "c128" else np.complex64
    diags = {o: v.astype(npd) for o, v in _operator(N, nd, N + nd).items()}
    batch = ROWS_MAX // N + 1 if N > 60000 else 3
    note(f"row kernel N={N} diagonals={len(diags)} {dtype} batch={batch}")
    rng = np.random.default_rng(N)
    x = (rng.normal(size=(batch, N)) + 1j * rng.normal(size=(batch, N))).astype(npd)
    offs = sorted(diags)
    dev = [torch.from_numpy(diags[o]).cuda() for o in offs]
    dev = [torch.cat([v, v.new_zeros(2)])[:v.numel()] for v in dev]
    many = hs.dia_spmv(offs, dev, torch.from_numpy(x).cuda()).cpu().numpy()
    one = hs.dia_spmv(offs, dev, torch.from_numpy(x[:1].copy()).cuda()).cpu().numpy()
    assert np.array_equal(one[0].view(np.uint8), many[0].view(np.uint8))
    ref, mag = _reference({o: v.astype(np.complex128) for o, v in diags.items()}, x.astype(np.complex128))
    fac = 1e-14 if dtype == "c128" else tol_c64()
    assert np.all(np.abs(many - ref) <= fac * mag + 1e-300)


@pytest.mark.parametrize("n,dtype", [(1, "c128"), (6, "c64"), (11, "c128"), (12, "c64"), (17, "c128"), (18, "c64")])
def test_taylor_by_masks(n, dtype):
    """A Taylor update of an operator from Pauli strings, applied by its
    X-masks, against the same operator from its stored diagonals (which has no
    masks); one state gives the bits it has in a batch (n = 17 and 18: the row
    kernel and the tile kernel).  Strings of one, two and four parities per
    mask, real and imaginary entries, and a pair that cancels in half the rows."""
    hs, torch = hs_gpu()
    from paper_2606_16959_amd import dia
    note(f"taylor by masks n={n} {dtype}")
    rng = np.random.default_rng(n)
    strings = ["I" * q + "X" + "I" * (n - q - 1) for q in range(n)] + ["Z" * n]
    if n >= 6:
        tail = "I" * (n - 6)
        strings += ["XXIIII" + tail, "YYIIII" + tail, "XYZIII" + tail, "IXZIII" + tail, "IXIZII" + tail,
                    "IXIIZI" + tail, "IXIIIZ" + tail, "ZIIIIY" + tail]
        if n > 6:
            strings += ["I" * (n - 2) + "YX", "X" + "I" * (n - 2) + "X", "Y" + "Z" * (n - 2) + "Y"]
    coeffs = rng.uniform(0.2, 1.0, len(strings))
    coeffs[len(strings) - 1] = coeffs[len(strings) - 2]
    H = dia.from_pauli(strings, coeffs, n)
    plain = dia.from_dict(H.to_dict(), 1 << n)
    if dtype == "c64":
        H, plain = H.to_c64(), plain.to_c64()
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    real = torch.float64 if dtype == "c128" else torch.float32
    x = torch.view_as_complex(torch.randn((5, 1 << n, 2), generator=g, device="cuda", dtype=real))
    dt = 0.5 / dia.norm_bound(dia.from_dict(H.to_dict(), 1 << n))
    many, one, ref = x.clone(), x[3:4].clone(), x.clone()
    dia.taylor_evolve(H, many, dt, 4, 2)
    dia.taylor_evolve(H, one, dt, 4, 2)
    dia.taylor_evolve(plain, ref, dt, 4, 2)
    assert torch.equal(many[3], one[0])
    # |dt| nu = 1/2: 8 stages of at most 2 n + 20 multiply-adds, each of the
    # step's scale; rounding of the coefficients included
    eps = 2.0 ** -52 if dtype == "c128" else 2.0 ** -23
    assert (many - ref).abs().max().item() <= 8 * (2 * n + 20) * eps * x.abs().max().item()
