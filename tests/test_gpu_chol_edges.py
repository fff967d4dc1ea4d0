"""Dense solve at the edges of the Cholesky blocks (16 x 16 register tiles of
the 64 x 64 diagonal block, 64-row blocks, 256-column panels): the solution is
backward stable, |S x + F|_2 <= 8 K 2^-52 (|S|_F |x|_2 + |F|_2) with the S and F
the library forms, the smallest pivot is the Cholesky's of the same S, and a
column of zeros is reported as the first non-positive pivot."""
import numpy as np
import pytest

from gpu_common import DEV, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 48, 63, 64, 65, 127, 129, 255, 257, 320, 513, 641, 1025])
@pytest.mark.parametrize("real", [False, True])
def test_solve_at_block_edges(K, real):
    flush(f"chol K={K} real={real}")
    ctx = V.Context(0)
    rng = np.random.default_rng(K)
    N = 2 * K + 8
    O = rng.normal(size=(N, K)) + (0.0 if real else 1j * rng.normal(size=(N, K)))
    e = rng.normal(size=N) + 1j * rng.normal(size=N)
    d, de = torch.from_numpy(O).to(DEV), torch.from_numpy(e).to(DEV)
    mode = V.SR_REAL if real else V.SR_COMPLEX
    S, F, _ = V.sr_fisher(ctx, d, de, nu_rel=1e-3, mode=mode)
    x, info = V.sr_solve(ctx, d, de, nu_rel=1e-3, mode=mode)
    S, F, x = S.cpu().numpy(), F.cpu().numpy(), x.cpu().numpy()
    if real:
        F = F.real
    r = np.linalg.norm(S @ x + F)
    assert r <= 8 * K * 2.0 ** -52 * (np.linalg.norm(S) * np.linalg.norm(x) + np.linalg.norm(F)), r
    piv = np.abs(np.diag(np.linalg.cholesky(S))).min() ** 2
    assert abs(info["min_pivot"] - piv) <= 8 * K * 2.0 ** -52 * np.linalg.norm(S)
    for k in sorted({0, K // 2, min(15, K - 1), min(16, K - 1), min(64, K - 1), K - 1}):
        O0 = O.copy()
        O0[:, k] = 0.0
        x0, info0 = V.sr_solve(ctx, torch.from_numpy(O0).to(DEV), de, nu_rel=0.0, mode=mode, raise_on_error=False)
        assert x0 is None and info0["status"] == "NOT_PD" and info0["fail_index"] == k


# the trailing update's squares of 4 x 4 and 8 x 8 tiles, with a ragged last square and row
@pytest.mark.parametrize("K", [3650, 6721])
def test_solve_large(K):
    flush(f"chol K={K}")
    ctx = V.Context(0)
    gen = torch.Generator(device=DEV).manual_seed(K)
    O = torch.randn(K + 8, K, dtype=torch.complex64, device=DEV, generator=gen)
    e = torch.randn(K + 8, dtype=torch.complex128, device=DEV, generator=gen)
    S, F, _ = V.sr_fisher(ctx, O, e, nu_rel=1e-1)
    x, _ = V.sr_solve(ctx, O, e, nu_rel=1e-1)
    r = torch.linalg.vector_norm(S @ x + F).item()
    scale = (torch.linalg.vector_norm(S) * torch.linalg.vector_norm(x) + torch.linalg.vector_norm(F)).item()
    assert r <= 8 * K * 2.0 ** -52 * scale, (r, scale)
