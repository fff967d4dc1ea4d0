"""CNN local energies where the window kernel's activations come within a few
bytes of the LDS: 8 channels on 89 x 7 (9 984 entries) leave room for its fixed
arrays only with the general kernel; one site less fits the window kernel."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import cnn as ocnn, eloc
from gpu_common import dev_bits, dev_c128, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


@pytest.mark.parametrize("Lx,Ly,C,k", [(89, 7, 8, 2), (13, 43, 4, 2), (29, 43, 4, 1), (83, 5, 12, 2), (69, 9, 8, 2)])
def test_local_energy_near_the_lds_limit(Lx, Ly, C, k):
    flush(f"cnn local energies near the LDS limit {Lx}x{Ly} C={C} k={k}")
    ctx = V.Context(0)
    N = Lx * Ly
    p = si._normal_params(ocnn.num_params(C, k), 0.3 / np.sqrt(C * k * k), True, seed=N)
    m = V.Model.cnn(ctx, Lx, Ly, C, k)
    m.set_params(dev_c128(p))
    bits = si.random_bits(1, N, seed=2)
    H = V.Hamiltonian.tfim(ctx, Lx, Ly, True, 1.0, 0.8)
    got = m.local_energy(H, dev_bits(si.pack_bits(bits))).cpu().numpy()
    f = lambda X: np.concatenate([ocnn.log_psi(p, X[i:i + 64], Lx, Ly, C, k) for i in range(0, len(X), 64)])
    ref = eloc.local_energy(f, "tfim", bits, Lx, Ly, True, 1.0, 0.8)
    assert np.max(np.abs(got - ref)) <= 1e-9 * np.abs(ref).max()
