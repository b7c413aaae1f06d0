"""The reverse pass's Krylov part where its one block holds two (513-1024 atoms) and eight (above 1024)
entries a thread: L = |K delta|^2 of systems with one orbital per atom, gradients with respect to delta, gamma and W
against central differences (h = 1e-4 along a random direction) of the library's own forward, and the sweep with
dL/dH against the one without (1e-10). The difference's own error is O(h^2) ~ 1e-8 of the
value and the forward's rounding over h; bound 2e-6 as for the dense K0 in test_gpu_adjoint.
"""

import numpy as np
import pytest

from tests.gpu_helpers import rel, t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2303_03529_amd import krylov  # noqa: E402


@pytest.mark.parametrize("atoms", [600, 1040])
def test_gradients(atoms):
    rng = np.random.default_rng(atoms)
    m, h = 4, 1e-4
    eye = torch.eye(atoms, dtype=torch.float64, device="cuda")
    Q = [torch.linalg.qr(t(rng.standard_normal((atoms, atoms))))[0].contiguous() for _ in range(2)]
    eps = [t(np.sort(rng.uniform(-10.0, 10.0, atoms))) for _ in range(2)]
    d = np.abs(np.arange(atoms)[:, None] - np.arange(atoms)[None, :])
    x0 = dict(delta=0.01 * rng.standard_normal(2 * atoms), gamma=5.0 / (1.0 + d), W=-0.4)
    e = rng.standard_normal((atoms, atoms)) / atoms
    step = dict(delta=0.01 * rng.standard_normal(2 * atoms), gamma=0.5 * (e + e.T), W=0.3)
    handle = krylov.Handle()

    def prepare(p):
        handle.prepare(np.arange(atoms + 1, dtype=np.int32), eye, eye, *Q, *eps, t(p["gamma"]), p["W"], 0.25,
                       float(atoms), krylov.KK_FP64)
        return t(p["delta"])

    def loss(p):
        x = handle.krylov_kernel_apply(prepare(p), m)[0].cpu().numpy()
        return float(x @ x)

    try:
        delta = prepare(x0)
        x, info = handle.krylov_kernel_apply(delta, m)
        assert info.rank_used == m
        g = [handle.krylov_kernel_adjoint(delta, m, 2.0 * x, reuse_forward=True, want_H=H) for H in (False, True)]
        g = [{k: r[k].cpu().numpy() for k in x0} for r in g]
        fd = {k: (loss(dict(x0, **{k: x0[k] + h * step[k]})) - loss(dict(x0, **{k: x0[k] - h * step[k]}))) / (2 * h)
              for k in x0}
    finally:
        handle.close()
    an = {k: float(np.sum(g[0][k] * step[k])) for k in x0}
    print(atoms, {k: (an[k], fd[k]) for k in x0}, [rel(g[1][k], g[0][k]) for k in x0], flush=True)
    for k in x0:
        assert rel(g[1][k], g[0][k]) < 1e-10, k
        assert abs(an[k] - fd[k]) < 2e-6 * abs(fd[k]), k
