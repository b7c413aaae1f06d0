"""The chemical potential to the bit: kk_prepare leaves out the counts whose outcome is known, and the split
products, whose rounding follows mu's last bit, need it where the plain bisection (every halving counted, then
Newton) ends. tests/golden/mu_bits.json holds what the library returned with the plain bisection,
for levels spread evenly, in two groups with gaps of many kT, and rounded to 0.1 (degenerate)."""

import json
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2303_03529_amd import krylov  # noqa: E402

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "mu_bits.json")
ATOMS = (1, 8, 28, 57, 128, 250)


def chemical_potentials(atoms):
    """{name: hex} over the spectra of a size."""
    nb = 9 * atoms
    eye = torch.eye(nb, dtype=torch.float64, device="cuda")
    gamma = torch.eye(atoms, dtype=torch.float64, device="cuda")
    out = {}
    h = krylov.Handle()
    try:
        for seed in range(4):
            rng = np.random.default_rng(100 * atoms + seed)
            for kT in (0.25, 0.02, 3.0):
                spectra = dict(even=rng.uniform(-30.0, 30.0, (2, nb)),
                               groups=np.where(rng.uniform(size=(2, nb)) < 0.4, rng.uniform(-7.0, -3.0, (2, nb)),
                                               rng.uniform(2.0, 10.0, (2, nb))),
                               rounded=np.round(rng.uniform(-10.0, 10.0, (2, nb)), 1))
                n_e = (8.0 * nb / 9.0, nb * (0.1 + 0.45 * seed), float(int(0.8 * nb)), 0.37 * nb)[seed]
                for name, e in spectra.items():
                    e = [torch.as_tensor(np.sort(x), device="cuda") for x in e]
                    h.prepare(np.arange(0, nb + 1, 9, dtype=np.int32), eye, eye, eye, eye, *e, gamma, -0.4, kT, n_e, 0)
                    out[f"{atoms} {name} {kT} {seed}"] = float(h.mu).hex()
    finally:
        h.close()
    return out


@pytest.mark.parametrize("atoms", ATOMS)
def test_mu_bits(atoms):
    golden = json.load(open(GOLDEN))
    got = chemical_potentials(atoms)
    assert len(got) == 36
    assert got == {k: golden[k] for k in got}
