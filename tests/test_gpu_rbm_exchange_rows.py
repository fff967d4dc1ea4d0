"""RBM local energies under exchanges on both sides of the line between eight and
sixteen table rows in flight, against the oracle."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import eloc, rbm as orbm
from gpu_common import dev_bits, dev_c128, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


# N_h float64 factors and logarithms per connected configuration: 1e-10 as in the other parity tests
@pytest.mark.parametrize("Nh", [1, 15, 16, 17, 240, 255, 256, 257, 272, 289, 1024])
@pytest.mark.parametrize("kind", ["heisenberg", "tfim"])
def test_rows_in_flight(Nh, kind):
    flush(f"rbm rows in flight Nh={Nh} {kind}")
    ctx = V.Context(0)
    N, B = 70, 3
    p = si.rbm_params(N, Nh, std=0.3 / np.sqrt(Nh), is_complex=True, seed=Nh)
    m = V.Model.rbm(ctx, N, Nh, True)
    m.set_params(dev_c128(p))
    bits = si.random_bits(B, N, seed=3)
    H = V.Hamiltonian.heisenberg(ctx, N, 1, True, 1.0) if kind == "heisenberg" else \
        V.Hamiltonian.tfim(ctx, N, 1, True, 1.0, 0.7)
    got = m.local_energy(H, dev_bits(si.pack_bits(bits))).cpu().numpy()
    ref = eloc.local_energy(lambda X: orbm.log_psi(p, X, Nh), kind, bits, N, 1, True, 1.0, 0.7)
    assert np.max(np.abs(got - ref)) <= 1e-10 * max(1.0, np.abs(ref).max())
