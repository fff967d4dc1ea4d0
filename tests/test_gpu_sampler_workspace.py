"""The RBM chains' second call takes theta of its first states from scratch
memory: inside the context's workspace, within its limit, and the chains are the
same where the limit leaves no room for it."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_common import dev_c128, host_bits, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


@pytest.mark.parametrize("prop", [V.PROP_FLIP, V.PROP_EXCHANGE])
def test_workspace_limit_and_memory(prop):
    flush(f"sampler workspace proposal={prop}")
    N, Nh, C = 64, 512, 4096
    p = si.rbm_params(N, Nh, std=0.02, is_complex=True, seed=4)
    out, used = [], []
    for limit in (0, 1 << 20):  # theta of 4 096 chains: 32 MiB
        ctx = V.Context(0)
        m = V.Model.rbm(ctx, N, Nh, True)
        m.set_params(dev_c128(p))
        H = V.Hamiltonian.heisenberg(ctx, 8, 8, True, 1.0) if prop == V.PROP_EXCHANGE else \
            V.Hamiltonian.tfim(ctx, 8, 8, True, 1.0, 1.0)
        S = V.Sampler(ctx, m, H, proposal=prop, n_chains=C, therm_sweeps=1, sweep_steps=8, seed=5)
        first, _, _ = S.sample(C)
        ctx.set_workspace_limit(limit)
        ctx.sync()
        free0 = torch.cuda.mem_get_info()[0]
        s, lp, acc = S.sample(2 * C)
        ctx.sync()
        used.append(free0 - torch.cuda.mem_get_info()[0])
        out.append((host_bits(first), host_bits(s), lp.cpu().numpy(), acc))
    a, b = out
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[3] == b[3]
    assert np.max(np.abs(a[2] - b[2])) < 1e-10 * max(1.0, np.abs(a[2]).max())
    # outside the limit only the call's outputs, a few MiB of torch's blocks
    assert used[1] < 24 << 20
