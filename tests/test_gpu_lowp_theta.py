"""float32 / bfloat16 log psi of the RBM at the edges of the theta product's
tiles (32 sites a step, words of 64 spins, 64 samples, 64 real columns) against
the oracle with the same rounded parameters: theta_j carries (N + 16) 2^-23
(|b_j| + sum_i |W_ji|) of float32 accumulation, log cosh (|slope| <= |tanh|,
below 2 here) and its float32 evaluation 2^-19 (1 + |theta_j|) a unit."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import rbm as orbm
from gpu_common import dev_bits, dev_c128, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


def _round(p, prec):
    t = torch.from_numpy(np.stack([p.real, p.imag]))
    r = t.to(torch.bfloat16 if prec == V.VMC_BF16 else torch.float32).to(torch.float64).numpy()
    return r[0] + 1j * r[1]


@pytest.mark.parametrize("N", [1, 31, 32, 33, 63, 64, 65, 96, 97, 100, 128, 129])
@pytest.mark.parametrize("Nh,B", [(1, 1), (31, 64), (32, 65), (33, 63), (70, 130)])
@pytest.mark.parametrize("prec", [V.VMC_F32, V.VMC_BF16])
def test_log_psi_lowp(N, Nh, B, prec):
    flush(f"lowp theta N={N} Nh={Nh} B={B} prec={prec}")
    ctx = V.Context(0)
    p = si.rbm_params(N, Nh, std=0.25 / np.sqrt(N), is_complex=True, seed=N + Nh)
    m = V.Model.rbm(ctx, N, Nh, True)
    m.set_params(dev_c128(p))
    m.set_precision(prec)
    pr = _round(p, prec)
    bits = si.random_bits(B, N, seed=B)
    got = m.log_psi(dev_bits(si.pack_bits(bits))).cpu().numpy()
    sg = 2.0 * bits - 1.0
    b, Wj = pr[N:N + Nh], pr[N + Nh:].reshape(Nh, N)
    th = b + sg @ Wj.T
    bound = 2 * (N + 16) * 2.0 ** -23 * (np.abs(b) + np.abs(Wj).sum(1)).sum() \
        + 2.0 ** -19 * (1 + np.abs(th)).sum(1) + 1e-12
    assert np.all(np.abs(got - orbm.log_psi(pr, bits, Nh)) <= bound)
