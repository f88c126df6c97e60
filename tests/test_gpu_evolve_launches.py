"""evolve_launches names the launches of a step: every position of the part's
sequence once and in order, one entry where one launch applies all steps, one
per factor without fusion, and fewer than the fusion list where tiles of single
states hold more factors than tiles of a batch."""
import numpy as np
import pytest

from gpu_common import env, hs_gpu, note
from workloads import hamiltonians as wh, workload_hamiltonian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,order,dtype", [(8, 1, "c64"), (13, 1, "c128"), (14, 2, "c64"), (16, 4, "c128")])
def test_launches_cover_the_sequence(n, order, dtype):
    hs, torch = hs_gpu()
    note(f"evolve launches n={n} order={order} {dtype}")
    H = wh.heisenberg_1d(n, 1.0, fields=np.linspace(-1, 1, n))
    f = hs.build_factors(H.strings, H.coeffs, n, 1.0, 10, 16, dtype=dtype, order=order)
    d = f.describe()
    psi = torch.zeros((3, 1 << n), dtype=torch.complex64 if dtype == "c64" else torch.complex128, device="cuda")
    for part in range(4):
        seq = f.part_sequence(part, d)
        for fuse in (True, False):
            for renorm in (True, False):
                for called in (False, True):              # before and after the plan is on the device
                    got = f.evolve_launches(3, fuse=fuse, part=part, renorm=renorm)
                    assert [p for a, c in got for p in range(a, a + c)] == list(range(len(seq)))
                    if n <= 12 and fuse and not renorm:
                        assert got == [(0, len(seq))]
                    elif not fuse:
                        assert len(got) == len(seq)
                    hs.evolve(f, psi, 1, fuse=fuse, renorm=renorm)
    with env(HAMSIM_MAX_FUSE=2):
        assert all(c <= 2 for _, c in f.evolve_launches(3, renorm=True))
    assert f.check_closure()
    f.close()


def test_eight_maxcut_states_take_three_launches():
    hs, torch = hs_gpu()
    note("evolve launches maxcut_3reg_n24 8 states")
    H = workload_hamiltonian("maxcut_3reg_n24")
    f = hs.build_factors(H.strings, H.coeffs, 24, 1.0, 200, 16, dtype="c64")
    assert len(f.evolve_launches(8)) == 3 and len(f.step_launches(8)) == 4
    f.close()
    cost = wh.maxcut(6, [(0, 1), (2, 5)], [1.0, 2.0], mixer=0.0)
    f = hs.build_factors(cost.strings, cost.coeffs, 6, 1.0, 4, 16)
    assert f.evolve_launches(1) == f.evolve_launches(1, renorm=True) == [(0, 1)]
    f.close()
