"""Centring and float32 Gram at their edges: 8- and 16-sample stages, 256-sample
chunks, sample splits, 128-wide tiles, odd parameter counts, weights, and the
energy sums beside the column sums (32 768 samples).  Xc is rounded to float32
(relative 2^-24 an entry) and every entry of S a float32 sum of n = min(N, one
split) products: |S - S_ref| <= (min(N, 4096) + 16) 2^-23 (diag S)^(1/2) outer
(diag S)^(1/2); F and the energy statistics are float64 sums: N 2^-52 relative
to the sums of moduli."""
import numpy as np
import pytest

from gpu_common import DEV, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


@pytest.mark.parametrize("N,K", [(2, 1), (7, 129), (8, 128), (9, 127), (17, 3), (255, 257), (256, 65), (257, 65),
                                 (263, 385), (2050, 130), (4097, 33), (32767, 5), (32768, 7), (40001, 131)])
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("weighted", [False, True])
def test_fisher_f32(N, K, cplx, weighted):
    flush(f"float32 gram N={N} K={K} cplx={cplx} weighted={weighted}")
    rng = np.random.default_rng(N * 1000 + K)
    O = rng.normal(size=(N, K)) + (1j * rng.normal(size=(N, K)) if cplx else 0.0)
    O = O.astype(np.complex64 if cplx else np.float32)
    e = rng.normal(size=N) + 1j * rng.normal(size=N)
    w = rng.uniform(0.5, 2.0, size=N) if weighted else None
    ctx = V.Context(0)
    S, F, info = V.sr_fisher(ctx, torch.from_numpy(O).to(DEV), torch.from_numpy(e).to(DEV),
                             weights=None if w is None else torch.from_numpy(w).to(DEV),
                             mode=V.SR_COMPLEX if cplx else V.SR_REAL)
    p = (np.ones(N) if w is None else w) / (N if w is None else w.sum())
    O64 = O.astype(np.complex128 if cplx else np.float64)
    Oc = O64 - p @ O64
    em = p @ e
    ref = (Oc.conj() * p[:, None]).T @ Oc
    d = np.sqrt(np.diag(ref).real)
    assert np.all(np.abs(S.cpu().numpy() - ref) <= (min(N, 4096) + 16) * 2.0 ** -23 * np.outer(d, d) + 1e-300)
    Fr = (Oc.conj() * p[:, None]).T @ (e - em)
    Fa = (np.abs(Oc) * p[:, None]).T @ np.abs(e - em)
    assert np.all(np.abs(F.cpu().numpy() - Fr) <= (N + 64) * 2.0 ** -50 * Fa + 1e-15)
    assert abs(info["e_mean"] - em) <= (N + 64) * 2.0 ** -52 * (p @ np.abs(e))
    assert abs(info["e_var"] - p @ np.abs(e - em) ** 2) <= (N + 64) * 2.0 ** -51 * (p @ np.abs(e) ** 2)
