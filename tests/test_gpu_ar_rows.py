"""Autoregressive O_k on every route (a configuration per wave, 16 per work-group,
the general kernel) and type: few and many configurations, few parameters, more
sites than the padded weights take, long complex128 rows."""
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


# float64 sums of N + H terms of order one: 1e-12; float32 rows rounded once
@pytest.mark.parametrize("N,H,B", [(2, 1, 1), (3, 1, 700), (10, 10, 515), (10, 11, 513), (11, 10, 512), (30, 20, 513),
                                   (30, 20, 16387), (350, 3, 9), (600, 2, 6), (64, 50, 512), (64, 50, 515), (40, 130, 5)])
@pytest.mark.parametrize("dtype", ["float32", "float64", "complex64", "complex128"])
def test_rows(N, H, B, dtype):
    flush(f"ar rows N={N} H={H} B={B} {dtype}")
    ctx = V.Context(0)
    th = si.ar_params(N, H, seed=N + H, std=0.3 / np.sqrt(max(1, H / 16)))
    m = V.Model.autoregressive(ctx, N, H)
    m.set_params(torch.from_numpy(th).to(DEV))
    few = si.random_bits(min(B, 11), N, seed=N)
    O = m.grad_log_psi(dev_bits(si.pack_bits(np.resize(few, (B, N)))), getattr(torch, dtype))
    ref = torch.from_numpy(np.asarray(arnqs.grad_log_psi(th, few, N, H))).to(DEV)
    tol = 1e-12 if dtype in ("float64", "complex128") else 2.0 ** -23
    for b0 in range(0, B, len(few)):
        got = O[b0:b0 + len(few)].to(torch.complex128)
        assert torch.all((got - ref[:len(got)]).abs() <= tol * max(1.0, float(ref.abs().max()))), b0
