"""Tile lists of a batch: every tile of every system once, whatever the threshold between the tile
classes, the order of the levels (ascending: blocks left out; shuffled: none) and the number of
tiles per XCD, and the lists of another threshold in the same batch. Each system against its own
handle (FP64 1e-11, the sums' order; FP16 x 3 2e-6, each within 1e-6 of FP64); a system whose residual is zero
stops before its first direction and leaves the others as they are.
"""

import numpy as np
import pytest

from tests.gpu_helpers import rel, t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2303_03529_amd import krylov  # noqa: E402
from tests.test_gpu_window import IDS, PRECISIONS, TOL, arguments, make  # noqa: E402

NAMES = ("offsets", "S", "Z", "Q_up", "Q_dn", "eps_up", "eps_dn", "gamma", "W", "kT", "n_electrons")


# one atom (one tile of either class an item); a few; more tiles than the chip holds at once
@pytest.mark.parametrize("sizes", [[1], [3, 40, 15], [150, 7, 61, 118, 90, 33, 139, 100]], ids=["1", "3", "8"])
@pytest.mark.parametrize("precision", PRECISIONS[:2], ids=IDS[:2])
def test_thresholds(sizes, precision):
    rng = np.random.default_rng(len(sizes))
    args = [arguments(make(n, 900 + n), i % 2 == 1) for i, n in enumerate(sizes)]
    deltas = [t(0.01 * rng.standard_normal(2 * n)) for n in sizes]
    if len(sizes) > 1:
        deltas[1].zero_()
    m = min(4, 2 * min(sizes) - 1)
    b = krylov.Batch().prepare([dict(zip(NAMES, a)) for a in args], precision)
    got = {}
    try:
        for threshold, per_cu in ((0, 4), (512, 1), (1 << 30, 8), (512, 2), (0, 1)):
            b.set_tuning(threshold, per_cu)
            out, info = b.krylov_kernel_apply(deltas, m)
            out = [x.cpu().numpy() for x in out]
            assert [i.rank_used for i in info] == [0 if len(sizes) > 1 and k == 1 else m for k in range(len(sizes))]
            for x, y in zip(out, got.setdefault(threshold, out)):
                assert np.array_equal(x, y), threshold
    finally:
        b.close()
    for k, (a, delta) in enumerate(zip(args, deltas)):
        h = krylov.Handle()
        try:
            h.prepare(*a, precision)
            want = h.krylov_kernel_apply(delta, m)[0].cpu().numpy()
        finally:
            h.close()
        for threshold, out in got.items():
            if not want.any():
                assert not out[k].any()
            else:
                assert rel(out[k], want) < TOL[precision], (sizes[k], threshold)
