"""GPU parity of the autoregressive state's 16-configuration kernels at the
edges of their blocks: hidden units below, at and above a tile and past the
number of degrees (several units per degree), sites that fill no whole tile or
word, batches that end inside a block, and a network too large for them."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_common import DEV, dev_bits, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import arnqs, eloc  # noqa: E402
from paper_2108_03409_amd import nqsvmc as V  # noqa: E402

# (Lx, Ly, hidden, configurations); 96 sites and 120 units: the general kernels
CASES = [(3, 1, 1, 1), (4, 4, 16, 16), (5, 1, 13, 17), (11, 3, 17, 33), (16, 4, 50, 50), (13, 5, 66, 7), (12, 8, 120, 5)]


@pytest.mark.parametrize("Lx,Ly,H,B", CASES)
def test_batch_kernels_match_oracle(Lx, Ly, H, B):
    N = Lx * Ly
    flush(f"ar batch kernels N={N} H={H} B={B}")
    ctx = V.Context(0)
    th = si.ar_params(N, H, seed=3 * N + H, std=0.4)
    m = V.Model.autoregressive(ctx, N, H)
    m.set_params(torch.from_numpy(th).to(DEV))
    x = si.random_bits(B, N, seed=N)
    s = dev_bits(si.pack_bits(x))
    ref = arnqs.log_psi(th, x, N, H)
    lp = m.log_psi(s).cpu().numpy()
    assert np.all(lp.imag == 0.0)
    assert np.max(np.abs(lp.real - ref)) < 1e-12 * max(1.0, np.abs(ref).max())
    O = m.grad_log_psi(s, torch.float64).cpu().numpy()
    assert np.max(np.abs(O - arnqs.grad_log_psi(th, x, N, H))) < 1e-12
    f = lambda X: arnqs.log_psi(th, X, N, H).astype(np.complex128)
    for kind, ham in (("tfim", V.Hamiltonian.tfim(ctx, Lx, Ly, True, 1.0, 0.9)),
                      ("heisenberg", V.Hamiltonian.heisenberg(ctx, Lx, Ly, True, 1.0))):
        got = m.local_energy(ham, s).cpu().numpy()
        er = eloc.local_energy(f, kind, x, Lx, Ly, True, 1.0, 0.9)
        assert np.all(got.imag == 0.0)
        assert np.max(np.abs(got - er) / np.maximum(1.0, np.abs(er))) < 1e-10, kind
