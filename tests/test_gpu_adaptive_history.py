"""The rank of an adaptive update depends on its inputs only. How many directions go out at once follows the
handle's last adaptive update, and a direction's residual is tested by the solve or by one block of
another launch accordingly (512, 256 or 1024 threads): the same bits either way, so that a tolerance
of exactly a reported residual, or of the next number below it, ends the expansion at the same
direction. Ranks on both sides of the last one that is tested in another launch (16), both
preconditioners.
"""

import numpy as np
import pytest

from tests.gpu_helpers import t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.test_gpu_small_step import case, prepared  # noqa: E402
from tests.test_gpu_window import IDS, PRECISIONS  # noqa: E402

M_MAX = 20


def update(h, delta, m_max, tol, K0):
    x, info = h.krylov_kernel_apply_adaptive(delta, m_max, tol, K0=K0)
    return x.cpu().numpy(), info


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("dense", [False, True], ids=["identity", "dense"])
@pytest.mark.parametrize("atoms", [12, 64, 140, 300])
def test_rank_does_not_depend_on_the_last_update(atoms, dense, precision):
    y, delta, K0 = case(atoms, dense)
    delta, K0 = t(delta), None if K0 is None else t(K0)
    h = prepared(y, precision)
    try:
        # one direction after another (the last rank was 1), and the residual that each reports
        reported = []
        for m in range(1, M_MAX + 1):
            update(h, delta, 1, 1e-300, K0)
            reported.append(update(h, delta, m, 1e-300, K0)[1].ls_residual)
        ranks = [r for r in range(2, M_MAX, 1 if atoms < 200 else 3) if reported[r - 1] > 1e-9 and reported[r - 1] < min(reported[:r - 1])]
        assert len(ranks) >= 5
        failed = []
        for r in ranks:
            for tol in (reported[r - 1], np.nextafter(reported[r - 1], 0.0)):
                update(h, delta, 1, 1e-300, K0)
                x, info = update(h, delta, M_MAX, tol, K0)
                assert info.ls_residual <= tol or info.rank_used == M_MAX
                for last in (r - 1, r + 1, M_MAX):
                    update(h, delta, last, 1e-300, K0)
                    x2, info2 = update(h, delta, M_MAX, tol, K0)
                    if info2 != info or not np.array_equal(x, x2):
                        failed.append((r, last, info.rank_used, info2.rank_used, info.ls_residual, info2.ls_residual))
    finally:
        h.close()
    print(atoms, dense, precision, len(ranks), ranks[-1], failed[:3], flush=True)
    assert not failed, failed
