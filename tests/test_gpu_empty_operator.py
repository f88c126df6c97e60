"""An operator whose Pauli strings all cancel stores no diagonals: as a
propagator it maps every state to zero, and its Taylor update is the identity."""
import numpy as np
import pytest

from gpu_common import hs_gpu, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(1, 1), (2, 3), (12, 1), (16, 8)])
def test_operator_without_diagonals(n, batch):
    hs, torch = hs_gpu()
    from paper_2606_16959_amd import dia
    note(f"operator without diagonals n={n} batch={batch}")
    string = "X" + "I" * (n - 1)
    H = dia.from_pauli([string, string], [0.5, -0.5], n)
    assert H.n_diags == 0
    psi = torch.ones((batch, 1 << n), dtype=torch.complex128, device="cuda")
    dia.taylor_evolve(H, psi, 0.1, 3, 2)
    assert torch.equal(psi, torch.ones_like(psi))
    assert dia.evolve(H, psi, 0) is psi and torch.equal(psi, torch.ones_like(psi))
    dia.evolve(H, psi, 2)
    assert not psi.cpu().numpy().any()
