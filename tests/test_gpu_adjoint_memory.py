"""The reverse pass where the device has little memory left: dL/dH takes as many directions at a time
as there is room for, down to one, and at last leaves its contractions uncut (12 padded
matrices in all), instead of returning KK_ENOMEM.

The rest of the device's memory is held by torch during the call. Against the same gradients with
memory for the whole group: the directions are summed in other groups and the contractions
in other pieces, 1e-9 (the commutators of dL/dH cancel, which costs digits).
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

KEYS = ("delta", "gamma", "W", "H_up", "H_dn")


def hold_all_but(nbytes):
    """Blocks that leave about nbytes free on the device."""
    torch.cuda.empty_cache()
    held = []
    while (free := torch.cuda.mem_get_info()[0] - nbytes) > 1 << 24:
        try:
            held.append(torch.empty(free // (1 << 21) << 21, dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            held.append(torch.empty(free // 2 // (1 << 21) << 21, dtype=torch.uint8, device="cuda"))
    return held


def gradients(h, delta, m):
    x, _ = h.krylov_kernel_apply(delta, m)
    g = h.krylov_kernel_adjoint(delta, m, 2.0 * x, reuse_forward=True)
    return [g[k].cpu().numpy() for k in KEYS]


# `left`: padded matrices free at the call. 250 atoms (padded 2304): room for a few directions of 8
# matrices each; 128 atoms (padded 1152): not for one beside the partial products of the K-split.
@pytest.mark.parametrize("atoms,padded,m,left", [(250, 2304, 6, 36), (128, 1152, 8, 24)])
def test_gradients_with_little_memory(atoms, padded, m, left):
    y = make(atoms, 800 + atoms)
    delta = t(0.01 * np.random.default_rng(atoms).standard_normal(2 * atoms))
    matrix = 8 * padded * padded
    other = make(171, 1)  # the kernels of the uncut contractions, loaded while memory is free
    h, warm = krylov.Handle(), krylov.Handle()
    try:
        h.prepare(*arguments(y, False), krylov.KK_FP64)
        warm.prepare(*arguments(other, False), krylov.KK_FP64)
        gradients(warm, t(np.ones(342)), 2)
        want = [gradients(h, delta, rank) for rank in (m, 1)]
        h.prepare(*arguments(other, False), krylov.KK_FP64)  # another shape: the workspace is given back
        h.prepare(*arguments(y, False), krylov.KK_FP64)
        h.krylov_kernel_apply(delta, m)
        torch.cuda.synchronize()
        held = hold_all_but(left * matrix)
        try:
            free = torch.cuda.mem_get_info()[0]
            assert free < 8 * m * matrix, "the whole group would fit"
            got = [gradients(h, delta, rank) for rank in (m, 1, m)]
        finally:
            del held
            torch.cuda.empty_cache()
    finally:
        h.close()
        warm.close()
    err = [rel(a, b) for g, w in zip(got, want + want[:1]) for a, b in zip(g, w)]
    print(atoms, left, free / matrix, err, flush=True)
    assert max(err) < 1e-9, err
    for a, b in zip(got[0], got[2]):
        assert np.array_equal(a, b)
