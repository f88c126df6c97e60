"""Evolutions under every launch setting that changes the plan (factors per
launch, row runs, one factor per launch, whole evolutions on or off) give the
bits of one DIA SpMV per factor over the diagonals copied back from the
handle, and a setting leaves nothing behind in the handle."""
import numpy as np
import pytest

from gpu_common import env, hs_gpu, note
from workloads import hamiltonians as wh

pytestmark = pytest.mark.gpu


def _products(hs, torch, f, psi, steps):
    """psi after `steps` steps, one product per factor."""
    d = f.describe()
    mats = []
    for k, fac in enumerate(d["factors"]):
        mats.append((fac["offsets"], [torch.from_numpy(f.copy_diagonal(k, j, o)).cuda()
                                      for j, o in enumerate(fac["offsets"])]))
    for s in range(steps):
        part = 0 if steps == 1 else 1 if s == 0 else 3 if s == steps - 1 else 2
        for k in f.part_sequence(part, d):
            psi = hs.dia_spmv(*mats[k], psi)
    return psi.cpu().numpy()


@pytest.mark.parametrize("family,n,dtype,order,steps", [
    ("tfim", 8, "c128", 1, 1), ("tfim", 8, "c64", 1, 3), ("heis", 8, "c64", 2, 1), ("heis", 12, "c128", 1, 3),
    ("tfim", 12, "c64", 2, 3), ("heis", 12, "c64", 4, 2), ("tfim", 13, "c64", 1, 2), ("heis", 14, "c128", 2, 2)])
def test_every_launch_setting_gives_the_same_bits(family, n, dtype, order, steps):
    hs, torch = hs_gpu()
    note(f"evolve settings {family} n={n} {dtype} order={order} steps={steps}")
    H = wh.tfim_1d(n, 1.0, 0.7) if family == "tfim" else wh.heisenberg_1d(n, 1.0, fields=np.linspace(-1, 1, n))
    f = hs.build_factors(H.strings, H.coeffs, n, 1.0, 10, 16, dtype=dtype, order=order)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(3, 1 << n)) + 1j * rng.normal(size=(3, 1 << n))
    psi0 = torch.from_numpy((x / np.linalg.norm(x, axis=1, keepdims=True)).astype(
        np.complex128 if dtype == "c128" else np.complex64)).cuda()
    want = _products(hs, torch, f, psi0.clone(), steps)
    settings = [{}] + [{"HAMSIM_MAX_FUSE": k} for k in (1, 2, 3, 7)]
    settings += [{"HAMSIM_MAX_FUSE": 2, "HAMSIM_WHOLE_MAX_ROWS": 0}, {"HAMSIM_WHOLE_MAX_ROWS": 8192},
                 {"HAMSIM_WHOLE_MAX_ROWS": 0}, {"HAMSIM_WMIN_BYTES": 2048, "HAMSIM_WHOLE_MAX_ROWS": 0}, {}]
    for kw in settings:
        for fuse in (True, False):
            with env(**kw):
                got = hs.evolve(f, psi0.clone(), steps, fuse=fuse).cpu().numpy()
            assert np.array_equal(got, want), (kw, fuse)
    f.close()
    # a fresh handle whose first call has the setting
    f = hs.build_factors(H.strings, H.coeffs, n, 1.0, 10, 16, dtype=dtype, order=order)
    with env(HAMSIM_MAX_FUSE=2):
        got = hs.evolve(f, psi0.clone(), steps).cpu().numpy()
    assert np.array_equal(got, want)
    assert np.array_equal(hs.evolve(f, psi0.clone(), steps).cpu().numpy(), want)
    f.close()
