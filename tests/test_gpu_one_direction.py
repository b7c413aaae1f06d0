"""FP64 handles of both forms (114-120 atoms of 9 orbitals): single directions on K-split products or on
unsplit 64 x 64 tiles, by what the prepared spectrum leaves of them (ascending levels: unsplit;
shuffled levels, of which nothing is left out: split), launches of several directions always on
the latter. Bounds: FP64 1e-11, the sums' order; the same form again to the bit.
"""

import numpy as np
import pytest

from tests.gpu_helpers import rel, t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2303_03529_amd import krylov  # noqa: E402
from tests.test_gpu_window import arguments, make  # noqa: E402

TOL = 1e-11


def once(h, v, delta, K0):
    """Responses of one, two and three directions, the update by graph and without allocation, its gradient without H."""
    out = torch.empty_like(delta)
    x = h.krylov_kernel_apply(delta, 4, K0=K0)[0].clone()
    h.krylov_kernel_apply_noalloc(delta, 4, K0=K0, out=out)
    assert torch.equal(x, out)
    assert torch.equal(x, h.krylov_kernel_apply(delta, 4, K0=K0)[0])
    g = h.krylov_kernel_adjoint(delta, 4, 2.0 * x, K0=K0, reuse_forward=True, want_H=False)
    r = [h.density_response_batch(v[:k].contiguous()).clone() for k in (1, 2, 3)]
    return [y.cpu().numpy() for y in [x, g["delta"], g["gamma"], *r]]


@pytest.mark.parametrize("dense", [False, True], ids=["identity", "dense"])
@pytest.mark.parametrize("atoms", [113, 114, 120, 121])
def test_both_forms_in_turn(atoms, dense):
    y = make(atoms, 40 + atoms)
    rng = np.random.default_rng(atoms)
    n2 = 2 * atoms
    v, delta = t(rng.standard_normal((3, n2))), t(0.01 * rng.standard_normal(n2))
    K0 = t(-np.eye(n2) + 0.05 / np.sqrt(n2) * rng.standard_normal((n2, n2))) if dense else None
    orders = (True, False, False, True)
    h = krylov.Handle()
    try:
        got = []
        for shuffled in orders:
            h.prepare(*arguments(y, shuffled), krylov.KK_FP64)
            got.append(once(h, v, delta, K0))
    finally:
        h.close()
    for g, shuffled in zip(got, orders):
        f = krylov.Handle()
        try:
            f.prepare(*arguments(y, shuffled), krylov.KK_FP64)
            fresh = once(f, v, delta, K0)
        finally:
            f.close()
        assert all(np.array_equal(a, b) for a, b in zip(g, fresh))
    err = [rel(a, b) for a, b in zip(got[0], got[1])] + [rel(got[0][3][0], got[0][5][0])]
    print(atoms, dense, err, flush=True)
    assert max(err) < TOL, err
