"""Float64 CNN log psi on both sides of the line between one thread per output and
matrix products: channels 1 to 16, samples of at most and more than 256 outputs, few
samples and more than three a compute unit."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import cnn as ocnn
from gpu_common import dev_bits, dev_c128, assert_logpsi_close, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


@pytest.mark.parametrize("Lx,Ly,C,k", [(1, 1, 1, 1), (16, 16, 1, 1), (64, 64, 1, 3), (43, 58, 2, 8), (5, 3, 2, 3), (17, 5, 3, 2),
                                       (43, 2, 3, 2), (16, 4, 4, 4), (13, 5, 4, 2), (7, 7, 5, 4), (13, 4, 5, 3), (5, 5, 8, 3),
                                       (5, 5, 9, 2), (7, 4, 9, 2), (29, 1, 9, 1), (4, 4, 16, 2)])
@pytest.mark.parametrize("B", [5, 768, 769])
def test_log_psi_at_the_line(Lx, Ly, C, k, B):
    if B > 5 and Lx * Ly > 300:
        B = 6
    flush(f"cnn log psi {Lx}x{Ly} C={C} k={k} B={B}")
    p = si._normal_params(ocnn.num_params(C, k), 0.4 / np.sqrt(C * k), True, seed=Lx + C)
    m = V.Model.cnn(V.Context(0), Lx, Ly, C, k)
    m.set_params(dev_c128(p))
    bits = si.random_bits(B, Lx * Ly, seed=8)
    got = m.log_psi(dev_bits(si.pack_bits(bits))).cpu().numpy()
    assert_logpsi_close(got, ocnn.log_psi(p, bits, Lx, Ly, C, k), 1e-10)


# two, four and eight waves a sample: up to 64, 128 and more positions per row tile; one channel
@pytest.mark.parametrize("Lx,Ly,C,k", [(3, 3, 3, 3), (8, 8, 5, 2), (13, 5, 4, 3), (16, 8, 3, 2), (43, 3, 4, 1), (5, 5, 17, 2),
                                       (13, 5, 17, 1), (16, 16, 1, 4), (64, 64, 1, 1), (17, 17, 2, 2)])
@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
def test_rows_of_many_samples(Lx, Ly, C, k, dtype):
    flush(f"cnn rows {Lx}x{Ly} C={C} k={k} {dtype}")
    p = si._normal_params(ocnn.num_params(C, k), 0.3 / np.sqrt(C * k), True, seed=Lx + C)
    m = V.Model.cnn(V.Context(0), Lx, Ly, C, k)
    m.set_params(dev_c128(p))
    few = si.random_bits(4, Lx * Ly, seed=8)
    s = dev_bits(si.pack_bits(np.resize(few, (900, Lx * Ly))))
    O = m.grad_log_psi(s, getattr(torch, dtype)).cpu().numpy()
    ref = ocnn.grad_log_psi(p, few, Lx, Ly, C, k)
    scale = max(1.0, np.abs(ref).max())
    assert np.max(np.abs(O - np.resize(ref, O.shape))) <= (1e-10 if dtype == "complex128" else 2.0 ** -23) * scale
    lp = m.log_psi(s).cpu().numpy()
    assert_logpsi_close(lp, np.resize(ocnn.log_psi(p, few, Lx, Ly, C, k), 900), 1e-10)
