"""RBM local energies whose factors 1 - sigma tanh(theta) tanh(2 W) are tiny: a
product of many of them stays in range.  Unit j has theta_j = 13 on the
configuration and W_j0 = 18, so a flip of site 0 multiplies psi by
cosh(23) / cosh(13) per unit while its factor is about 1e-11; 32 of them
underflow unless the product is rescaled on the way."""
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


# four samples per wavefront from 8 192 samples and 33 sites, otherwise one; 17, 32 and 48 units.
# 1 - t T with t T = 1 - 1e-11 carries 2^-53 / 1e-11 relative, over N_h units: 1.1e-5 N_h, doubled
@pytest.mark.parametrize("N,B", [(5, 3), (40, 8192)])
@pytest.mark.parametrize("Nh", [17, 32, 48])
@pytest.mark.parametrize("kind", ["tfim", "heisenberg"])
def test_products_of_tiny_factors(N, B, Nh, kind):
    flush(f"rbm tiny factors N={N} B={B} Nh={Nh} {kind}")
    ctx = V.Context(0)
    p = np.zeros(N + Nh + N * Nh, dtype=np.complex128)
    W = p[N + Nh:].reshape(Nh, N)
    W[:, 0] = 18.0
    p[N:N + Nh] = 13.0 - 18.0  # theta = 13 where site 0 is up
    m = V.Model.rbm(ctx, N, Nh, True)
    m.set_params(dev_c128(p))
    bits = np.zeros((min(B, 64), N), dtype=np.uint8)
    bits[:, 0] = 1
    H = V.Hamiltonian.tfim(ctx, N, 1, True, 1.0, 1.0) if kind == "tfim" else \
        V.Hamiltonian.heisenberg(ctx, N, 1, True, 1.0)
    got = m.local_energy(H, dev_bits(si.pack_bits(np.resize(bits, (B, N))))).cpu().numpy()
    ref = eloc.local_energy(lambda X: orbm.log_psi(p, X, Nh), kind, bits[:1], N, 1, True, 1.0, 1.0)[0]
    assert np.isfinite(ref) and abs(ref) > 1e60
    assert np.max(np.abs(got - ref)) <= 2.2e-5 * Nh * abs(ref)
