"""Eigensolver on matrices whose squares leave the float64 range: every result
scales with a power of two.  Rotations work on scaled pairs, so the bounds are
those of the unscaled matrix."""
import numpy as np
import pytest

from gpu_common import dev_c128, flush

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2108_03409_amd import nqsvmc as V  # noqa: E402


# 2^-498 ~ 1e-150 (squares below 1e-290), 2^465 ~ 1e140; the norms of the sweeps' stopping
# rule are sums of squares, so 2^-530 and 2^512 are not asked for
@pytest.mark.parametrize("K", [2, 64])
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("e2", [-498, 0, 465])
def test_eigh_scales_with_powers_of_two(K, cplx, e2):
    flush(f"eigh scaled K={K} complex={cplx} 2^{e2}")
    rng = np.random.default_rng(K)
    X = np.ones((1, 2)) if K == 2 else rng.normal(size=(K + 3, K)) + (1j * rng.normal(size=(K + 3, K)) if cplx else 0)
    if K == 2 and cplx:
        X = np.array([[1.0, 1.0j]])
    A = X.conj().T @ X
    s = 2.0 ** e2
    ev, Vm, sweeps = V.eigh(V.Context(0), dev_c128(A * s))
    ev, Vm = ev.cpu().numpy() / s, Vm.cpu().numpy()
    ref = np.linalg.eigvalsh(A)
    assert np.max(np.abs(np.sort(ev) - ref)) <= 1e-12 * np.abs(ref).max()
    assert np.linalg.norm((Vm * ev) @ Vm.conj().T - A) <= 1e-12 * np.linalg.norm(A)
    assert np.linalg.norm(Vm.conj().T @ Vm - np.eye(K)) <= 1e-11
    assert sweeps <= 20


@pytest.mark.parametrize("e2", [-498, 465])
def test_real_pseudo_inverse_scales(e2):
    """The solve's real path: O scaled by 2^(e2 / 2) scales S by 2^e2 and x by 2^(-e2 / 2)."""
    flush(f"real pseudo-inverse scaled 2^{e2}")
    e2 = e2 // 2 * 2
    rng = np.random.default_rng(3)
    O = rng.normal(size=(300, 40))
    e = dev_c128(rng.normal(size=300))
    ctx = V.Context(0)
    x = []
    for s in (1.0, 2.0 ** (e2 // 2)):
        r, info = V.sr_solve_eig(ctx, torch.from_numpy(O * s).to("cuda:0"), e, mode=V.SR_REAL, eps_pinv=1e-8)
        x.append(r.cpu().numpy() * s)
        assert info["sweeps"] <= 20
    assert np.max(np.abs(x[1] - x[0])) <= 1e-10 * np.abs(x[0]).max()
