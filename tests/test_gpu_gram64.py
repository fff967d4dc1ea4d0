"""Float64 Gram on the matrix cores (complex128 / float64 O): S and F against
numpy at the edges of the 64 x 64 tiles and of the sample splits, with and
without room for the split's partial tiles.  Every entry of S is a sum of N
products of centred values: |S - S_ref| <= (N + 64) 2^-52 (diag S)^(1/2) outer
(diag S)^(1/2) bounds both sides' rounding."""
import numpy as np
import pytest

from gpu_common import DEV, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


# one tile; tile edges; odd sample counts (a half-filled pair of real samples); many
# samples on few tiles (split ranges); three tile rows
@pytest.mark.parametrize("N,K", [(3, 2), (65, 64), (999, 65), (20001, 40), (7000, 130)])
@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("split", [True, False])
def test_fisher_f64(N, K, real, split):
    flush(f"float64 gram N={N} K={K} real={real} split={split}")
    rng = np.random.default_rng(N + K)
    O = rng.normal(size=(N, K)) + (0.0 if real else 1j * rng.normal(size=(N, K)))
    e = rng.normal(size=N) + 1j * rng.normal(size=N)
    d = torch.from_numpy(O).to(DEV), torch.from_numpy(e).to(DEV)
    ctx = V.Context(0)
    if not split:
        # the limit that just holds the solve without partial tiles: found by its refusal
        lo, hi = 0, 1 << 34
        while hi - lo > 512:
            mid = (lo + hi) // 2
            ctx.set_workspace_limit(max(mid, 1))
            try:
                V.sr_fisher(ctx, *d)
                hi = mid
            except V.VMCError as err:
                assert err.name == "WORKSPACE"
                lo = mid
        ctx.set_workspace_limit(hi)
    for mode in (V.SR_COMPLEX, V.SR_REAL):
        S, F, _ = V.sr_fisher(ctx, *d, nu_rel=0.5, mode=mode)
        X = (O - O.mean(0)) / np.sqrt(N)
        ref = X.conj().T @ X
        ref = ref.real.astype(complex) if mode == V.SR_REAL else ref.astype(complex)
        g = np.sqrt(np.abs(np.diag(ref)))
        ref[np.arange(K), np.arange(K)] *= 1.5
        tol = (N + 64) * 2.0 ** -52 * 1.5 * np.outer(g, g)
        assert np.all(np.abs(S.cpu().numpy() - ref) <= tol), mode
        Fr = (O - O.mean(0)).conj().T @ (e - e.mean()) / N
        assert np.all(np.abs(F.cpu().numpy() - Fr) <= (N + 64) * 2.0 ** -52 * 2 * g * np.abs(e - e.mean()).max())
