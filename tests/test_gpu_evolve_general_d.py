"""Factors with general complex entries that carry the diagonal terms: the
coefficients hs_evolve forms are those stored, so a step gives the bits of one
DIA SpMV per factor over the diagonals copied back, in complex128 too."""
import numpy as np
import pytest

from gpu_common import hs_gpu, note
from test_gpu_evolve_knobs import _products

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strings", [
    ["ZZIIIIIIII", "IIIIIIIIIX", "IIIIIIIIXX", "IIIIIIZIXI"],       # rank 2
    ["ZZIIIIIIII", "YIZIIIIIII", "IIIZIIIIYI", "YIIIIIIIYZ"],
    ["ZZIIIIIIII", "IIXXIIIIZI", "IIYZIIIIII", "IIIIXIIXII", "ZZIIIIIIIY", "IIZYIIIIII"]])       # rank 4
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_general_entries_with_d(strings, dtype):
    hs, torch = hs_gpu()
    note(f"general entries with D {strings[1]} {dtype}")
    f = hs.build_factors(strings, [0.3 + 0.1 * k for k in range(len(strings))], 10, 1.0, 5, 1024, dtype=dtype)
    rng = np.random.default_rng(3)
    x = rng.normal(size=(2, 1024)) + 1j * rng.normal(size=(2, 1024))
    psi = torch.from_numpy(x.astype(np.complex64 if dtype == "c64" else np.complex128)).cuda()
    want = _products(hs, torch, f, psi.clone(), 2)
    for fuse in (True, False):
        assert np.array_equal(hs.evolve(f, psi.clone(), 2, fuse=fuse).cpu().numpy(), want)
    f.close()
