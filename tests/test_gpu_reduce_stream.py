"""Norms and overlaps on both sides of the size at which the reductions stream
their states past the caches, with a remainder of the loads a thread keeps in
flight, against FP64 sums on the host."""
import numpy as np
import pytest

from gpu_common import hs_gpu, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,batch,a,b", [(1, 1, "c64", None), (4 * 262144 + 1, 1, "c128", None),
                                         (3 * 262144 + 7, 2, "c64", "c128"), (1 << 24, 1, "c128", None),
                                         ((1 << 24) + 5, 1, "c128", None), ((1 << 23) + 3, 3, "c64", "c64"),
                                         (7000001, 2, "c128", "c64")])
def test_reductions_across_the_streaming_size(N, batch, a, b):
    hs, torch = hs_gpu()
    note(f"reductions N={N} batch={batch} {a} {b}")
    rng = np.random.default_rng(N)

    def states(d):
        x = rng.standard_normal((batch, 2 * N), dtype=np.float32)
        return x.view(np.complex64) if d == "c64" else x.astype(np.float64).view(np.complex128)
    x = states(a)
    x64 = x.astype(np.complex128)
    # FP64 sums of N terms in another order: each at most N 2^-53 of the terms' sum
    tol = 2 * N * 2.0**-53
    nx = np.sum(np.abs(x64)**2, axis=1)
    if b is None:
        got = np.asarray(hs.norm2(torch.from_numpy(x).cuda()))
        assert np.all(np.abs(got - nx) <= (tol + 4 * 2.0**-53) * nx)
        return
    y = states(b)
    y64 = y.astype(np.complex128)
    rec = hs.fidelity(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    dot, mag = np.sum(np.conj(x64) * y64, axis=1), np.sum(np.abs(x64) * np.abs(y64), axis=1)
    ny = np.sum(np.abs(y64)**2, axis=1)
    assert np.all(np.abs(rec[:, 0] + 1j * rec[:, 1] - dot) <= (2 * tol + 8 * 2.0**-53) * mag)
    assert np.all(np.abs(rec[:, 2] - nx) <= (tol + 4 * 2.0**-53) * nx)
    assert np.all(np.abs(rec[:, 3] - ny) <= (tol + 4 * 2.0**-53) * ny)
