"""Loads that rely on a buffer's range for what lies past the last sample or site:
the float32 Gram with a workspace full of other numbers behind its samples, and log
psi of many samples (weights of sites past the last) against log psi of few."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_common import DEV, dev_bits, dev_c128, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


# entries of S: float32 sums of N products of float32 entries, (N + 16) 2^-23 of the diagonals
@pytest.mark.parametrize("N,K", [(1, 129), (3, 385), (9, 127), (18, 257), (31, 1)])
@pytest.mark.parametrize("cplx", [False, True])
def test_gram_in_a_used_workspace(N, K, cplx):
    flush(f"gram in a used workspace N={N} K={K} cplx={cplx}")
    rng = np.random.default_rng(N + K)
    ctx = V.Context(0)
    mode = V.SR_COMPLEX if cplx else V.SR_REAL
    dt = np.complex64 if cplx else np.float32

    def problem(n):
        O = rng.normal(size=(n, K)) + (1j * rng.normal(size=(n, K)) if cplx else 0.0)
        return (O * 1e3).astype(dt), rng.normal(size=n) + 1j * rng.normal(size=n)

    O, e = problem(700)
    V.sr_fisher(ctx, torch.from_numpy(O).to(DEV), torch.from_numpy(e).to(DEV), mode=mode)
    O, e = problem(N)
    S, _, _ = V.sr_fisher(ctx, torch.from_numpy(O).to(DEV), torch.from_numpy(e).to(DEV), mode=mode)
    X = O.astype(np.complex128 if cplx else np.float64)
    X = X - X.mean(0)
    ref = X.conj().T @ X / N
    d = np.sqrt(np.diag(ref).real)
    assert np.all(np.abs(S.cpu().numpy() - ref) <= (N + 16) * 2.0 ** -23 * np.outer(d, d) + 1e-30)


# both kernels sum N + N_h float64 terms of order one in different orders
@pytest.mark.parametrize("N", [1, 4, 5, 33, 60, 61, 64, 65, 100, 124, 125])
@pytest.mark.parametrize("Nh", [1, 16, 50])
def test_log_psi_of_many_samples(N, Nh):
    flush(f"log psi of many samples N={N} Nh={Nh}")
    ctx = V.Context(0)
    p = si.rbm_params(N, Nh, std=0.2, is_complex=True, seed=N)
    m = V.Model.rbm(ctx, N, Nh, True)
    m.set_params(dev_c128(p))
    s = dev_bits(si.pack_bits(si.random_bits(8192, N, seed=5)))
    many = m.log_psi(s).cpu().numpy()
    few = np.concatenate([m.log_psi(s[i:i + 1024].contiguous()).cpu().numpy() for i in range(0, 8192, 1024)])
    assert np.max(np.abs(many - few)) <= (N + 50) * 2.0 ** -50 * max(1.0, np.abs(few).max())
