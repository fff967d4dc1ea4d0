"""RBM calls on both sides of the line between theta formed inside the kernels
(small calls) and by the matrix cores: log psi, local energies and O_k against
the oracle.  Both routes add at most N + 1 products of modulus |W|, so theta
differs by less than 2 (N + 1) 2^-52 (|b| + N max|W|); 1e-11 relative leaves the
elementary functions' and sums' rounding a factor of 100."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import rbm as orbm, eloc as oeloc
from gpu_common import dev_bits, dev_c128, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


# (N, N_h, B): the smallest; 64 | 65 rows of W; two slots per lane of 32 | 33 rows;
# two words of spins; B and B N N_h at and past their lines
@pytest.mark.parametrize("N,Nh,B", [(3, 1, 1), (10, 10, 33), (64, 64, 17), (65, 64, 17), (64, 65, 17), (32, 65, 40),
                                    (32, 128, 40), (33, 65, 40), (6, 6, 8192), (6, 6, 8193), (16, 64, 4096),
                                    (16, 64, 4097), (10, 300, 9)])
@pytest.mark.parametrize("kind", ["tfim", "heisenberg"])
def test_small_calls(N, Nh, B, kind):
    if kind == "heisenberg" and N % 2:
        N += 1
    flush(f"rbm small N={N} Nh={Nh} B={B} {kind}")
    ctx = V.Context(0)
    p = si.rbm_params(N, Nh, std=0.3 / np.sqrt(N), is_complex=True, seed=N + Nh)
    m = V.Model.rbm(ctx, N, Nh, True)
    m.set_params(dev_c128(p))
    H = V.Hamiltonian.tfim(ctx, N, 1, True, 1.0, 0.7) if kind == "tfim" else \
        V.Hamiltonian.heisenberg(ctx, N, 1, True, 1.0)
    bits = si.random_bits(B, N, seed=B)
    s = dev_bits(si.pack_bits(bits))
    idx = np.unique(np.r_[0, B // 2, B - 1])
    close = lambda got, ref: np.max(np.abs(got - ref)) <= 1e-11 * max(1.0, np.abs(ref).max())
    f = lambda x: orbm.log_psi(p, x, Nh)
    assert close(m.log_psi(s).cpu().numpy()[idx], f(bits[idx]))
    ref = oeloc.local_energy(f, kind, bits[idx], N, 1, True, 1.0, 0.7 if kind == "tfim" else 0.0)
    assert close(m.local_energy(H, s).cpu().numpy()[idx], ref)
    for dt, tol in ((torch.complex128, 1.0), (torch.complex64, None)):
        g = m.grad_log_psi(s, dtype=dt).cpu().numpy()[idx]
        r = orbm.grad_log_psi(p, bits[idx], Nh)
        assert close(g, r) if tol else np.max(np.abs(g - r)) <= 2.0 ** -23 * max(1.0, np.abs(r).max())
