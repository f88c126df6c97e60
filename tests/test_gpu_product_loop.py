"""Alg. 3's loop in one launch (operators of up to 1024 complex128 or 2048
complex64 rows and 24 diagonals, or half the rows and 48 diagonals) gives the
bits of one product after the other through the general entry, at the edges of
its sizes and just beyond them."""
import numpy as np
import pytest

from gpu_common import hs_gpu, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nd,dtype,batch,steps", [
    (1, 1, "c128", 3, 4), (2, 3, "c64", 1, 1), (63, 8, "c128", 1, 2), (64, 9, "c64", 3, 5), (65, 16, "c128", 2, 3),
    (129, 17, "c64", 9, 2), (1000, 24, "c128", 2, 3), (1023, 24, "c64", 1, 4), (1024, 21, "c128", 3, 7),
    (1024, 25, "c128", 1, 2), (1025, 24, "c128", 1, 2), (2047, 23, "c64", 2, 3), (2048, 24, "c64", 1, 5),
    (2049, 24, "c64", 1, 2), (512, 48, "c128", 2, 3), (511, 25, "c128", 1, 2), (512, 49, "c128", 1, 2),
    (513, 48, "c128", 1, 2), (1024, 48, "c64", 3, 2), (1023, 33, "c64", 1, 3), (1025, 48, "c64", 1, 2)])
def test_loop_equals_single_products(N, nd, dtype, batch, steps):
    hs, torch = hs_gpu()
    from paper_2606_16959_amd import dia
    note(f"product loop N={N} diagonals={nd} {dtype} batch={batch} steps={steps}")
    npd = np.complex128 if dtype == "c128" else np.complex64
    rng = np.random.default_rng(100 * N + nd)
    pool = [o for o in (N - 1, 1 - N, 1, -1) if abs(o) < N] + [int(o) for o in rng.permutation(2 * N - 1) - (N - 1)]
    offs = sorted(list(dict.fromkeys([0] + pool))[:nd])
    diags = {o: 0.3 * (rng.normal(size=N - abs(o)) + 1j * rng.normal(size=N - abs(o))) for o in offs}
    U = dia.from_dict(diags, N)
    if dtype == "c64":
        U = U.to_c64()
    x = (rng.normal(size=(batch, N)) + 1j * rng.normal(size=(batch, N))).astype(npd)
    if N > 64:
        x[0, N // 2] = np.inf             # a partner that is not finite stays with the rows it reaches
        x[-1, 3] = np.nan
    psi = torch.from_numpy(x.copy()).cuda()
    dia.evolve(U, psi, steps)
    dev = [torch.from_numpy(diags[o].astype(npd)).cuda() for o in offs]
    ref = torch.from_numpy(x.copy()).cuda()
    for _ in range(steps):
        ref = hs.dia_spmv(offs, dev, ref)
    got, want = psi.cpu().numpy(), ref.cpu().numpy()
    assert np.array_equal(got, want, equal_nan=True)
    if N > 64:
        assert np.isfinite(got).sum() < got.size
