"""GPU parity of the float64 CNN kernels on the matrix cores at the edges of
their 16 x 16 x 4 operands: channels and taps below, at and above a tile,
positions that fill no whole tile."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import cnn as ocnn, lattice as olat
from oracle import metropolis as omet
from gpu_common import dev_bits, dev_c128, host_bits, assert_logpsi_close, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    return V.Context(0)


def _cnn(ctx, Lx, Ly, C, k, std, seed):
    p = si._normal_params(ocnn.num_params(C, k), std, True, seed=seed)
    m = V.Model.cnn(ctx, Lx, Ly, C, k)
    m.set_params(dev_c128(p))
    return m, p


# one channel and tap; two row tiles; 25 taps (two tap tiles); 33 channels on 9
# positions (partial sums of dW1 do not fit beside them); the largest sample
@pytest.mark.parametrize("Lx,Ly,C,k,B", [(5, 3, 1, 1, 7), (9, 7, 17, 2, 5), (11, 6, 5, 5, 4), (3, 3, 33, 3, 3),
                                         (64, 64, 1, 2, 2), (13, 6, 64, 2, 2)])
def test_net_tile_edges(ctx, Lx, Ly, C, k, B):
    flush(f"cnn float64 network {Lx}x{Ly} C={C} k={k} B={B}")
    m, p = _cnn(ctx, Lx, Ly, C, k, 0.3 / np.sqrt(C * k), seed=5 * Lx + C)
    bits = si.random_bits(B, Lx * Ly, seed=6)
    s = dev_bits(si.pack_bits(bits))
    assert_logpsi_close(m.log_psi(s).cpu().numpy(), ocnn.log_psi(p, bits, Lx, Ly, C, k), 1e-10)
    ref = ocnn.grad_log_psi(p, bits, Lx, Ly, C, k)
    scale = max(1.0, np.abs(ref).max())
    assert np.max(np.abs(m.grad_log_psi(s, torch.complex128).cpu().numpy() - ref)) <= 1e-10 * scale
    rng = np.random.default_rng(7)
    gv = rng.normal(size=B) + 1j * rng.normal(size=B)
    out = m.log_psi_vjp(s, dev_c128(gv)).cpu().numpy()
    assert np.max(np.abs(out - ref.conj().T @ gv)) <= 1e-10 * scale * np.abs(gv).sum()


# 5 and 17 channels (a partial k step, two row tiles); smallest tori of the window
# path; sites that fill no whole pass; 300 samples (a work-group takes two); one
# sample (its passes split over work-groups); 25 taps
@pytest.mark.parametrize("Lx,Ly,C,k,B", [(7, 5, 5, 3, 300), (9, 9, 17, 2, 3), (7, 7, 16, 4, 2), (16, 16, 4, 3, 1),
                                         (1, 1, 3, 1, 4), (11, 9, 3, 5, 2)])
def test_local_energy_window_products(ctx, Lx, Ly, C, k, B):
    flush(f"cnn float64 local energies {Lx}x{Ly} C={C} k={k} B={B}")
    m, p = _cnn(ctx, Lx, Ly, C, k, 0.4 / np.sqrt(C * k), seed=7 * Lx + C)
    N = Lx * Ly
    H = V.Hamiltonian.tfim(ctx, Lx, Ly, min(Lx, Ly) >= 3, 1.0, 3.0)
    bits = si.random_bits(B, N, seed=8)
    got = m.local_energy(H, dev_bits(si.pack_bits(bits))).cpu().numpy()
    f = lambda b: ocnn.log_psi(p, b, Lx, Ly, C, k)
    for b in list(range(min(B, 4))) + [B - 1]:
        sp, mel, cnt = olat.connected("tfim", bits[b], Lx, Ly, min(Lx, Ly) >= 3, 1.0, 3.0)
        terms = mel[:cnt] * np.exp(f(sp[:cnt]) - f(bits[b:b + 1])[0])
        assert abs(got[b] - terms.sum()) <= 1e-10 * np.abs(terms).sum(), b


def _sample(ctx, m, H, nc, per, limit=0):
    ctx.set_workspace_limit(limit)
    try:
        S = V.Sampler(ctx, m, H, proposal=V.PROP_FLIP, n_chains=nc, therm_sweeps=1, seed=11)
        parts = [S.sample(nc * per) for _ in range(2)]  # the second call restarts from the stored configurations
    finally:
        ctx.set_workspace_limit(0)
    return [torch.cat(x) for x in ([p[0] for p in parts], [p[1] for p in parts])]


# smallest torus of 4 x 4 taps; partial k step and row tile; one tap; 17 channels
# and 5 x 5 taps (the general kernel)
@pytest.mark.parametrize("Lx,Ly,C,k,nc", [(7, 7, 16, 4, 3), (9, 5, 5, 3, 5), (3, 5, 3, 1, 4), (11, 6, 12, 2, 3),
                                          (5, 4, 17, 2, 3), (9, 9, 2, 5, 2)])
def test_sampler_replays_oracle(ctx, Lx, Ly, C, k, nc):
    flush(f"cnn float64 sampler replay {Lx}x{Ly} C={C} k={k} chains={nc}")
    per = 2
    m, p = _cnn(ctx, Lx, Ly, C, k, 0.6 / np.sqrt(C * k), seed=9 * Lx + C)
    H = V.Hamiltonian.tfim(ctx, Lx, Ly, True, 1.0, 3.0)
    s, lp = _sample(ctx, m, H, nc, per)
    s = host_bits(s).reshape(2 * per, nc, -1)
    ch = omet.Chains(lambda b: ocnn.log_psi(p, b, Lx, Ly, C, k), Lx * Ly, "flip", seed=11, chain_ids=np.arange(nc),
                     therm_sweeps=1)
    os_, ol = ch.sample(2 * per)
    assert ch.near_ties == 0
    for q in range(2 * per):
        for c in range(nc):
            assert np.array_equal(s[q, c], si.pack_bits(os_[q, c])[0]), (q, c)
    assert_logpsi_close(lp.cpu().numpy(), ol.ravel(), 1e-9)


def test_sampler_workspace_limits(ctx):
    # chains in batches of three, and the general kernel below the state of one batch,
    # give the chains of the unlimited call
    flush("cnn float64 sampler under workspace limits")
    Lx, Ly, C, k, nc = 8, 7, 6, 3, 7
    m, _ = _cnn(ctx, Lx, Ly, C, k, 0.2, seed=77)
    H = V.Hamiltonian.tfim(ctx, Lx, Ly, True, 1.0, 3.0)
    s0, lp0 = _sample(ctx, m, H, nc, 2)
    per = 56 * C * Lx * Ly
    general = -(-16 * nc * C * Lx * Ly // 256) * 256
    for limit in (4 * per + 256, general):
        s1, lp1 = _sample(ctx, m, H, nc, 2, limit)
        assert torch.equal(s0, s1), limit
        assert_logpsi_close(lp1.cpu().numpy(), lp0.cpu().numpy(), 1e-10)
    with pytest.raises(V.VMCError) as e:
        _sample(ctx, m, H, nc, 2, general - 256)
    assert e.value.name == "WORKSPACE"
