"""Log psi of the autoregressive state where its conditionals are saturated: the
sum of log(1 + e^{-|l|}) keeps its relative precision, whatever the magnitude."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import arnqs
from gpu_common import DEV, dev_bits, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


# Logits b2 only, bits agreeing with them: log psi = -(1/2) sum log1p(e^{-|l|}).  Bound: e^{-|l|}
# to 2 ulp, N additions of positive terms with one rounding each, the last logarithm: (N + 8) 2^-53
@pytest.mark.parametrize("N,H", [(50, 29), (65, 17), (3, 1), (96, 120)])
@pytest.mark.parametrize("l", [0.5, 10.0, 20.0, 30.0, 40.0, 300.0, 700.0])
@pytest.mark.parametrize("B", [16, 20000])  # few samples and many
def test_relative_precision(N, H, l, B):
    flush(f"ar saturated N={N} H={H} l={l} B={B}")
    ctx = V.Context(0)
    sign = np.where(np.arange(N) % 3 == 0, -1.0, 1.0)
    th = np.zeros(arnqs.num_params(N, H))
    mag = l * (1.0 + 0.01 * np.arange(N) / N)
    th[-N:] = sign * mag
    m = V.Model.autoregressive(ctx, N, H)
    m.set_params(torch.from_numpy(th).to(DEV))
    x = np.repeat((sign > 0).astype(np.uint8)[None], B, 0)
    got = m.log_psi(dev_bits(si.pack_bits(x))).cpu().numpy()
    ref = -0.5 * np.log1p(np.exp(-mag.astype(np.longdouble))).sum()
    assert np.all(got.imag == 0.0)
    assert np.max(np.abs(got.real - ref)) <= (N + 8) * 2.0 ** -53 * abs(ref)
