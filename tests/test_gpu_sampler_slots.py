"""RBM chains at the edges of the sampler's split of the hidden units: slots of
64 per lane, one or two waves per chain, theta carried along (flips, exchanges)
or formed between sweeps (global proposals); the spins over several words.
Every configuration and acceptance equals the oracle's replay of the same
random stream; log psi of the records agrees within 1e-10."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import rbm as orbm, lattice as olat, metropolis as omet
from gpu_common import host_bits, dev_c128, assert_logpsi_close, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402

FEW, MANY = 16, 1100  # at most, and more than, one chain per SIMD (four per compute unit)


@pytest.mark.parametrize("Nh,n_chains", [
    (1, FEW), (64, FEW), (65, FEW), (128, FEW), (129, FEW), (256, FEW), (257, FEW), (512, FEW),
    (513, FEW), (769, FEW), (1024, FEW),
    (129, MANY), (256, MANY), (257, MANY), (384, MANY), (448, MANY), (512, MANY), (897, MANY)])
@pytest.mark.parametrize("prop,Lx,sweep", [("flip", 5, 3), ("exchange", 70, 130), ("made_mix", 7, 7)])
def test_replay_at_slot_edges(Nh, n_chains, prop, Lx, sweep):
    flush(f"sampler slots Nh={Nh} chains={n_chains} {prop}")
    ctx = V.Context(0)
    N, n_rec = Lx, 2
    p = si.rbm_params(N, Nh, std=0.3 / np.sqrt(Nh), is_complex=True, seed=N + Nh)
    m = V.Model.rbm(ctx, N, Nh, True)
    m.set_params(dev_c128(p))
    H = V.Hamiltonian.heisenberg(ctx, Lx, 1, True, 1.0) if prop == "exchange" else \
        V.Hamiltonian.tfim(ctx, Lx, 1, True, 1.0, 1.0)
    ids = [0, 1, n_chains - 1]
    kw = dict(n_chains=n_chains, therm_sweeps=1, sweep_steps=sweep, seed=11)
    okw = {}
    if prop == "made_mix":
        mp = si.made_params(N, 12, seed=5)
        q = V.MADE(ctx, N, 12)
        q.set_params(torch.from_numpy(mp).to("cuda:0"))
        kw.update(proposal=V.PROP_MADE_MIX, global_steps=1)
        okw = dict(made=(mp, N, 12), global_steps=1)
    else:
        kw.update(proposal=V.PROP_EXCHANGE if prop == "exchange" else V.PROP_FLIP)
    S = V.Sampler(ctx, m, H, **kw)
    if prop == "made_mix":
        S.set_proposal_made(q)
    ch = omet.Chains(lambda x: orbm.log_psi(p, x, Nh), N, prop, seed=11, chain_ids=ids,
                     bond_list=olat.bonds(Lx, 1, True), sweep_steps=sweep, therm_sweeps=1, **okw)
    for n in (n_rec, 1):  # the second call continues the same streams
        s, lp, _ = S.sample(n_chains * n)
        s = host_bits(s).reshape(n, n_chains, -1)
        lp = lp.cpu().numpy().reshape(n, n_chains)
        os_, ol = ch.sample(n)
        for r, c in enumerate(ids):
            for k in range(n):
                assert np.array_equal(s[k, c], si.pack_bits(os_[k, r])[0]), (k, c)
            assert_logpsi_close(lp[:, c], ol[:, r], 1e-10)
    assert ch.near_ties == 0
