"""The spectrum of a prepared expansion point (chemical potential, occupations) at the sizes where
its one block changes path: fewer levels than a wave, a few levels past the block's registers
(9 per thread and spin), and spectra whose electron count is flat at N_e (an insulator), where
the chemical potential comes from the plain bisection.

S = Z = Q = I, one orbital per atom, so that the charges are the occupations themselves. Bounds:
mu to 1e-13 relative to the spectrum's width where the count fixes it, occupations to 1e-12 (the
count's rounding over its slope, times beta)."""

import numpy as np
import pytest

from tests.gpu_helpers import t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle.fermi import fermi, solve_mu  # noqa: E402
from paper_2303_03529_amd import krylov  # noqa: E402

KT = 0.25


def charges(e_up, e_dn, n_e, atoms):
    nb = len(e_up)
    eye = torch.eye(nb, dtype=torch.float64, device="cuda")
    off = np.linspace(0, nb, atoms + 1).astype(np.int32)
    h = krylov.Handle()
    try:
        h.prepare(off, eye, eye, eye, eye, t(e_up), t(e_dn), torch.eye(atoms, dtype=torch.float64, device="cuda"),
                  -0.4, KT, n_e)
        return off, h.mu, h.ground_state_charges().cpu().numpy()
    finally:
        h.close()


@pytest.mark.parametrize("nb,n_e", [(1, 0.7), (2, 2.0), (63, 50.0), (65, 0.01), (128, 255.9), (1025, 900.0),
                                    (9217, 8100.0)])
def test_mu_and_occupations(nb, n_e):
    rng = np.random.default_rng(nb)
    e_up, e_dn = (np.sort(rng.uniform(-30.0, 25.0, nb)) for _ in range(2))
    atoms = min(nb, 64)
    off, mu, q = charges(e_up, e_dn, n_e, atoms)
    ref = solve_mu([e_up, e_dn], n_e, KT)
    f = [np.add.reduceat(fermi(e, ref, KT), off[:-1]) for e in (e_up, e_dn)]
    assert abs(mu - ref) <= 1e-13 * 55.0, (mu, ref)
    assert np.allclose(q, np.concatenate([f[0] + f[1], f[0] - f[1]]), rtol=0.0, atol=1e-12 * max(1.0, nb / atoms))


@pytest.mark.parametrize("gap", [30.0, 60.0, 200.0])
def test_insulator(gap):
    """Six levels below a gap of many kT, six electrons: any mu well inside fills them exactly."""
    e = np.array([-3.0, -2.0, -1.0, gap, gap + 1.0, gap + 2.0])
    _, mu, q = charges(e, e, 6.0, 6)
    assert -1.0 + 30 * KT < mu < gap - 30 * KT
    assert np.allclose(q, [2, 2, 2, 0, 0, 0] + [0] * 6, rtol=0.0, atol=1e-12)


@pytest.mark.parametrize("nb", [255, 256, 257, 511, 512, 513, 1024])
def test_block_sizes(nb):
    """Both sides of where the block grows from 256 to 512 and 1024 threads; a metal, with the levels
    in any order, and an insulator."""
    rng = np.random.default_rng(nb)
    e_up, e_dn = (rng.uniform(-30.0, 25.0, nb) for _ in range(2))
    off, mu, q = charges(e_up, e_dn, 1.7 * nb, 50)
    ref = solve_mu([np.sort(e_up), np.sort(e_dn)], 1.7 * nb, KT)
    f = [np.add.reduceat(fermi(e, ref, KT), off[:-1]) for e in (e_up, e_dn)]
    assert abs(mu - ref) <= 1e-13 * 55.0, (mu, ref)
    assert np.allclose(q, np.concatenate([f[0] + f[1], f[0] - f[1]]), rtol=0.0, atol=1e-12 * nb / 50)
    n_full = nb // 3
    e = np.concatenate([rng.uniform(-9.0, -1.0, n_full), rng.uniform(40.0, 50.0, nb - n_full)])
    _, mu, q = charges(e, e, 2.0 * n_full, nb)
    assert -1.0 + 30 * KT < mu < 40.0 - 30 * KT
    assert np.allclose(q, np.where(np.arange(2 * nb) < n_full, 2.0, 0.0), rtol=0.0, atol=1e-12)
