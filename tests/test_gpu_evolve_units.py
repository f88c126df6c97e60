"""Factors of rank 4 and above (budgets beyond 16) give the bits of one DIA
SpMV per factor over the diagonals copied back: ranks 4 to 10, tiles from one
coset to 8192 rows (4, 8 and 16 rows of a coset per thread), one matrix per wave
and one per lane, real and general entries, with and without D."""
import numpy as np
import pytest

from gpu_common import env, hs_gpu, note
from test_gpu_evolve_knobs import _products
from workloads import hamiltonians as wh

pytestmark = pytest.mark.gpu

GENERAL_D = ["ZZIIIIIIII", "IIXXIIIIZI", "IIYZIIIIII", "IIIIXIIXII", "ZZIIIIIIIY", "IIZYIIIIII"]
GENERAL = ["IIXIIIIIII", "IIIIIIIIXI", "XIIIIIZIII", "IIIIZIIIIY", "IIIIYZIIII", "XZIIIIIIXI"]


@pytest.mark.parametrize("family,n,dtype,budget,batch,whole", [
    ("tfim", 4, "c128", 31, 1, True), ("tfim", 5, "c64", 63, 2, True), ("tfim", 10, "c64", 2047, 1, True),
    ("tfim", 10, "c128", 1023, 2, False), ("heis", 10, "c128", 128, 3, True), ("tfim", 12, "c64", 32, 1, True),
    ("tfim", 12, "c128", 128, 2, False), ("tfim", 13, "c64", 64, 3, True), ("heis", 13, "c64", 1024, 1, False),
    ("tfim", 14, "c128", 512, 8, False), ("heis", 16, "c64", 128, 8, False), ("tfim", 17, "c128", 32, 8, False),
    ("tfim", 18, "c64", 128, 8, False), ("tfim", 19, "c128", 31, 8, False), ("tfim", 20, "c64", 32, 8, False),
    ("general", 10, "c64", 1024, 1, True), ("general", 10, "c128", 1024, 3, False), ("general", 18, "c64", 1024, 8, False),
    ("general_d", 10, "c128", 1024, 1, True), ("general_d", 10, "c64", 1024, 3, False),
    ("general_d", 17, "c128", 1024, 8, False)])
def test_large_cosets_give_the_bits_of_products(family, n, dtype, budget, batch, whole):
    hs, torch = hs_gpu()
    note(f"units {family} n={n} {dtype} budget={budget} batch={batch}")
    if family == "tfim":
        H = wh.tfim_1d(n, 1.0, 0.7)
        strings, coeffs = H.strings, H.coeffs
    elif family == "heis":
        H = wh.heisenberg_1d(n, 1.0, fields=np.linspace(-1, 1, n))
        strings, coeffs = H.strings, H.coeffs
    else:                                    # the last qubits idle, or the factors' types outside the tile
        strings = [s + "I" * (n - 10) for s in (GENERAL if family == "general" else GENERAL_D)]
        coeffs = np.array([0.3, 0.4, 0.5, 0.6, 0.7, 0.8])
    f = hs.build_factors(strings, coeffs, n, 1.0, 5, budget, dtype=dtype)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    real = torch.float64 if dtype == "c128" else torch.float32
    psi0 = torch.view_as_complex(torch.randn((batch, 1 << n, 2), generator=g, device="cuda", dtype=real)) / 2 ** (n / 2)
    want = _products(hs, torch, f, psi0.clone(), 2)
    with env(HAMSIM_WHOLE_MAX_ROWS=8192 if whole else 0):
        got = hs.evolve(f, psi0.clone(), 2).cpu().numpy()
    assert np.array_equal(got, want)
    f.close()
