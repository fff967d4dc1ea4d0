"""Float64 CNN with an output bias of a large imaginary part: Re log psi is the sum
of log|cos| of the bias itself (zero weights in the second layer), whatever its size."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import cnn as ocnn
from gpu_common import dev_bits, dev_c128, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


# cosine to 2.5 2^-53 absolute, over the smallest |cos| of the four biases, N terms of each
@pytest.mark.parametrize("y", [3.0, 1e6, 1e15, 2.0 ** 54, 1e17, 1e22, 1e300])
def test_output_phase(y):
    flush(f"cnn output phase {y}")
    Lx = Ly = 5
    C, k, N = 4, 2, 25
    p = si._normal_params(ocnn.num_params(C, k), 0.3, True, seed=3)
    W1, b1, W2, b2 = ocnn.split(p, C, k)
    p[C * k * k + C:] = 0.0
    b = np.array([y, -1.25 * y, 1.5 * y, 1.75 * y])
    p[-C:] = 1j * b
    m = V.Model.cnn(V.Context(0), Lx, Ly, C, k)
    m.set_params(dev_c128(p))
    got = m.log_psi(dev_bits(si.pack_bits(si.random_bits(3, N, seed=1)))).cpu().numpy()
    c = np.abs(np.cos(b))
    assert np.max(np.abs(got.real - N * np.log(c).sum())) <= N * C * (2.5 * 2.0 ** -53 / c.min() + 8 * 2.0 ** -53)
