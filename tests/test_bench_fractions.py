"""bench.py's count of the products that the window tables leave: whole products where the library
has no windows (cells of up to 128 atoms), else tile by tile, counted here from the factors themselves."""

import numpy as np
import pytest

import bench

KT, MU = 0.25, 8.0


def levels(nb):
    rng = np.random.default_rng(nb)
    return np.sort(rng.uniform(-30.0, 30.0, (2, nb)), axis=1)


@pytest.mark.parametrize("precision", ["fp64", "mixed", "bf16"])
@pytest.mark.parametrize("nb", [144, 486, 1152])
def test_no_windows_in_small_cells(nb, precision):
    assert bench.executed_fractions(levels(nb), MU, KT, precision) == {"forward_fermi": 1.0, "back_mulliken": 1.0}


@pytest.mark.parametrize("precision,nb,rows", [("fp64", 2250, 128), ("mixed", 2250, 128), ("bf16", 2250, 128),
                                               ("fp64", 3888, 128), ("mixed", 3888, 256), ("bf16", 3888, 256)])
def test_tiles_left(precision, nb, rows):
    e = levels(nb)
    got = bench.executed_fractions(e, MU, KT, precision)
    fwd = 0.0
    for x in e:
        f, fc = 1.0 / (1.0 + np.exp((x - MU) / KT)), 1.0 / (1.0 + np.exp((MU - x) / KT))
        lo, hi = np.minimum.outer(np.arange(nb), np.arange(nb)), np.maximum.outer(np.arange(nb), np.arange(nb))
        z = np.maximum((x[hi] - x[lo]) / KT, 1e-300)
        F = f[lo] * fc[hi] * -np.expm1(-z) / z          # |F| / beta
        np.fill_diagonal(F, f * fc)
        cut = 2.0 ** (-42 if precision == "mixed" else -60) * (1.0 if precision == "mixed" else F.max())
        for i in range(0, nb, rows):
            for j in range(0, nb, 128):
                tile = F[i:i + rows, j:j + 128]
                if (tile >= cut).any() or (i < j + 128 and j < i + rows):
                    fwd += tile.size
    fwd /= 2 * nb * nb
    # the library bounds a block's factors from its ends, so it keeps a little more than the factors ask for
    assert fwd <= got["forward_fermi"] < fwd + 0.03
    assert 0.5 < got["back_mulliken"] < 1.0
