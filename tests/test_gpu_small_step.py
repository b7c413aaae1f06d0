"""The short launch chains of small systems: f~ formed by the launch that orthonormalizes the next
direction (tiny FP64 handles; the smallest split ones and those with a dense K0), the two-launch
FP64 transforms, and the adaptive update's residual tests inside another launch.

The update against the same Krylov expansion in numpy, its responses from the handle's own
density_response_batch, which has none of these. FP64 within 1e-9: the two orders of the sums differ by
1e-13, times the condition of the Gram matrix (at most 1e4 here). Split forms 2e-6: their responses
are within 1e-6 of FP64 for any last bit of v. Sizes: one to 64 atoms, and on both sides of where the
dispatch leaves f~ to the next launch (split 20 / 30 atoms, dense K0 in FP64 30 / 37).
"""

import numpy as np
import pytest

from tests.gpu_helpers import rel, t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2303_03529_amd import krylov  # noqa: E402
from tests.test_gpu_window import IDS, PRECISIONS, arguments, make  # noqa: E402

TOL = {krylov.KK_FP64: 1e-9, krylov.KK_MIXED_F16: 2e-6, krylov.KK_MIXED_BF16: 2e-6}


def prepared(y, precision):
    h = krylov.Handle()
    h.prepare(*arguments(y, False), precision)
    return h


def case(atoms, dense):
    rng = np.random.default_rng(1000 + atoms)
    n2 = 2 * atoms
    K0 = -np.eye(n2) + 0.05 / np.sqrt(n2) * rng.standard_normal((n2, n2)) if dense else None
    return make(atoms, 500 + atoms), 0.01 * rng.standard_normal(n2), K0


def reference(h, delta, m, K0):
    """x = V (F^T F)^-1 F^T f~ over m directions, and the residual after each."""
    k0 = (lambda x: -x) if K0 is None else (lambda x: K0 @ x)
    ft, V, F, residuals = k0(delta), [], [], []
    src = ft
    for _ in range(m):
        w = src.copy()
        for v in V + V:
            w = w - (v @ w) * v
        v = w / np.linalg.norm(w)
        V.append(v)
        src = k0(h.density_response_batch(t(v[None])).cpu().numpy()[0] - v)
        F.append(src)
        c = np.linalg.solve(np.array(F) @ np.array(F).T, np.array(F) @ ft)
        residuals.append(np.linalg.norm(c @ np.array(F) - ft) / np.linalg.norm(ft))
    return c @ np.array(V), residuals


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("dense", [False, True], ids=["identity", "dense"])
@pytest.mark.parametrize("atoms", [1, 2, 16, 20, 30, 37, 64])
def test_update(atoms, dense, precision):
    y, delta, K0 = case(atoms, dense)
    m = min(4, 2 * atoms - 1)
    h = prepared(y, precision)
    try:
        got = [h.krylov_kernel_apply(t(delta), m, K0=None if K0 is None else t(K0))[0].cpu().numpy() for _ in range(2)]
        want, _ = reference(h, delta, m, K0)
    finally:
        h.close()
    print(atoms, dense, precision, rel(got[0], want), flush=True)
    assert np.array_equal(got[0], got[1])
    assert rel(got[0], want) < TOL[precision]


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("atoms", [12, 64, 100])
def test_adaptive_ranks(atoms, precision):
    """A handle's later adaptive updates enqueue as many directions at once as its last one took:
    more, fewer and as many as the next needs, each with the rank and the result of a fresh handle."""
    y, delta, _ = case(atoms, False)
    h = prepared(y, precision)
    try:
        _, residuals = reference(h, delta, 6, None)
        cuts = [0.5 * (residuals[r - 1] + residuals[r - 2]) for r in (5, 5, 2, 4, 3, 3)]
        got = [h.krylov_kernel_apply_adaptive(t(delta), 8, cut) for cut in cuts]
        short = h.krylov_kernel_apply_adaptive(t(delta), 2, cuts[0])  # m_max below the last rank
    finally:
        h.close()
    assert [g[1].rank_used for g in got] == [5, 5, 2, 4, 3, 3] and short[1].rank_used == 2
    for (x, info), cut, m_max in zip(got + [short], cuts + cuts[:1], [8] * 6 + [2]):
        h = prepared(y, precision)
        try:
            want, fresh = h.krylov_kernel_apply_adaptive(t(delta), m_max, cut)
        finally:
            h.close()
        assert info.rank_used == fresh.rank_used and info.status == fresh.status == 0
        assert abs(info.ls_residual - fresh.ls_residual) <= TOL[precision]
        assert rel(x.cpu().numpy(), want.cpu().numpy()) < TOL[precision]
