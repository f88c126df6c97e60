"""hs_footprint covers what building a handle and evolving with it take from
the device at their peak (the high-water mark of the stream-ordered pool, which
serves every allocation of the library)."""
import ctypes

import numpy as np
import pytest

from gpu_common import hs_gpu, note
from workloads import hamiltonians as wh

pytestmark = pytest.mark.gpu

USED_MEM_CURRENT, USED_MEM_HIGH = 7, 8          # hipMemPoolAttr


def _pool():
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    pool = ctypes.c_void_p()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0

    def get(attr):
        v = ctypes.c_uint64()
        assert hip.hipMemPoolGetAttribute(pool, attr, ctypes.byref(v)) == 0
        return v.value

    def reset():
        v = ctypes.c_uint64(0)
        assert hip.hipMemPoolSetAttribute(pool, USED_MEM_HIGH, ctypes.byref(v)) == 0
    return get, reset


@pytest.mark.parametrize("family,n,dtype,budget,order,merge,batch", [
    ("heis", 20, "c64", 16, 1, True, 1), ("heis", 20, "c128", 16, 1, True, 1), ("tfim", 20, "c64", 16, 1, False, 3),
    ("heis", 18, "c64", 16, 2, True, 1), ("heis", 18, "c128", 16, 4, True, 2), ("tfim", 12, "c64", 1023, 1, True, 9),
    ("heis", 11, "c128", 1024, 4, True, 11), ("heis", 8, "c64", 16, 4, True, 1)])
def test_peak_is_within_the_footprint(family, n, dtype, budget, order, merge, batch):
    hs, torch = hs_gpu()
    note(f"footprint {family} n={n} {dtype} budget={budget} order={order} merge={merge} batch={batch}")
    H = wh.tfim_1d(n, 1.0, 0.7) if family == "tfim" else wh.heisenberg_1d(n, 1.0, fields=np.linspace(-1, 1, n))
    elem = 16 if dtype == "c128" else 8
    psi = torch.zeros((batch, 1 << n), dtype=torch.complex128 if dtype == "c128" else torch.complex64, device="cuda")
    psi[:, 0] = 1
    torch.cuda.synchronize()
    get, reset = _pool()
    before = get(USED_MEM_CURRENT)
    reset()
    f = hs.build_factors(H.strings, H.coeffs, n, 1.0, 10, budget, dtype=dtype, order=order, merge_diag=merge)
    torch.cuda.synchronize()
    built = get(USED_MEM_HIGH) - before
    hs.evolve(f, psi, 2, renorm=True)
    torch.cuda.synchronize()
    peak = get(USED_MEM_HIGH) - before
    print(f"built {built} peak {peak} footprint {f.footprint(batch) - psi.numel() * elem}")
    assert 0 < built <= peak <= f.footprint(batch) - psi.numel() * elem
    f.close()
