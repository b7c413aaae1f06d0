"""Window tables (blocks of levels whose divided differences are negligible): the same system with
its levels in ascending order, where the transforms leave out every block between deep filled or
between high empty levels, and with levels and eigenvector columns in a random order, where
no block can be left out. Both orders are the same system, so every result has to agree.

Levels spread over 60 eV at kT = 0.25 eV, S = I, atoms of 9 orbitals. Sizes: each tile class
and form of the forward transform (padded 768: K-split; 1280: one round of 128 x 128 tiles; 1536:
64 x 64 tiles in FP64, stream-K products in the split forms; 2432 and 2688: the two forms of the
large tiles, the 256 x 128 split tiles). Bounds: FP64 1e-11 (the sums' order), split forms
2e-6 (each order within 1e-6 of FP64).
"""

import numpy as np
import pytest

from tests.gpu_helpers import rel, t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2303_03529_amd import krylov  # noqa: E402

TOL = {krylov.KK_FP64: 1e-11, krylov.KK_MIXED_F16: 2e-6, krylov.KK_MIXED_BF16: 2e-6}
PRECISIONS = [krylov.KK_FP64, krylov.KK_MIXED_F16, krylov.KK_MIXED_BF16]
IDS = ["fp64", "f16x3", "bf16"]


def make(atoms, seed, gap=0.0):
    """A system of `atoms` atoms; gap: no level within gap / 2 of 0, N_e at the middle of it."""
    rng = np.random.default_rng(seed)
    nb = 9 * atoms
    q = [torch.linalg.qr(torch.as_tensor(rng.standard_normal((nb, nb))))[0] for _ in range(2)]
    e = [np.sort(rng.uniform(-30.0, 30.0, nb)) for _ in range(2)]
    for x in e:
        x += np.where(x < 0.0, -0.5, 0.5) * gap
    n_e = float(sum((x < 0.0).sum() for x in e)) if gap else 8.0 * atoms
    d = np.abs(np.arange(atoms)[:, None] - np.arange(atoms)[None, :])
    return dict(offsets=np.arange(0, nb + 1, 9, dtype=np.int32), S=torch.eye(nb, dtype=torch.float64, device="cuda"),
                gamma=t(10.0 / (1.0 + d)), Q=q, e=e, n_e=n_e, seed=seed)


def arguments(y, shuffled):
    perm = [np.random.default_rng(y["seed"] + 1 + s).permutation(len(y["e"][0])) if shuffled
            else np.arange(len(y["e"][0])) for s in range(2)]
    Q = [y["Q"][s][:, torch.as_tensor(perm[s])].contiguous().cuda() for s in range(2)]
    return (y["offsets"], y["S"], y["S"], Q[0], Q[1], t(y["e"][0][perm[0]]), t(y["e"][1][perm[1]]), y["gamma"], -0.4,
            0.25, y["n_e"])


def results(y, shuffled, precision, v, delta, m):
    h = krylov.Handle()
    try:
        h.prepare(*arguments(y, shuffled), precision)
        r = h.density_response_batch(t(v)).cpu().numpy()
        k = [h.krylov_kernel_apply(t(delta), m)[0].cpu().numpy() for _ in range(2)]
        assert np.array_equal(k[0], k[1])
        return list(r) + [k[0]]
    finally:
        h.close()


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("atoms", [80, 140, 170, 265, 295])
def test_ascending_and_shuffled_levels_agree(atoms, precision):
    y = make(atoms, 100 + atoms)
    rng = np.random.default_rng(atoms)
    v, delta = rng.standard_normal((3, 2 * atoms)), 0.01 * rng.standard_normal(2 * atoms)
    a, b = (results(y, shuffled, precision, v, delta, 4) for shuffled in (False, True))
    err = [rel(p, q) for p, q in zip(a, b)]
    print(atoms, precision, err, flush=True)
    assert max(err) < TOL[precision], err


@pytest.mark.parametrize("atoms", [140, 170, 265])
def test_gradients_agree(atoms):
    """The reverse pass, whose back-transforms and commutator sums go by the same windows. The
    gradient with respect to H is a matrix in the orbital basis, the same for both orders; its
    commutators cancel, which costs digits (bound 1e-9)."""
    y = make(atoms, 300 + atoms)
    delta = t(0.01 * np.random.default_rng(atoms).standard_normal(2 * atoms))
    got = []
    for shuffled in (False, True):
        h = krylov.Handle()
        try:
            h.prepare(*arguments(y, shuffled), krylov.KK_FP64)
            x, _ = h.krylov_kernel_apply(delta, 3)
            g = h.krylov_kernel_adjoint(delta, 3, 2.0 * x, reuse_forward=True)
            got.append([g[k].cpu().numpy() for k in ("delta", "gamma", "W", "H_up", "H_dn")])
        finally:
            h.close()
    err = [rel(a, b) for a, b in zip(*got)]
    print(atoms, err, flush=True)
    assert max(err) < 1e-9, err


@pytest.mark.parametrize("gap", [8.0, 40.0])
def test_insulator(gap):
    """A gap of 32 and 160 kT at N_e: the smallest kept factor is 1 / (width of the spectrum), far
    below the metal's beta / 4, and the whole filled and empty blocks are left out."""
    y = make(140, 7, gap)
    rng = np.random.default_rng(7)
    v, delta = rng.standard_normal((2, 280)), 0.01 * rng.standard_normal(280)
    a, b = (results(y, shuffled, krylov.KK_FP64, v, delta, 4) for shuffled in (False, True))
    err = [rel(p, q) for p, q in zip(a, b)]
    print(gap, err, flush=True)
    assert max(err) < TOL[krylov.KK_FP64], err


def test_prepare_again_with_another_window():
    """One handle prepared with shuffled, then ascending, then shuffled levels: a block that one
    window leaves out is computed again in the next (same buffers, same graph)."""
    y = make(140, 9)
    delta = t(0.01 * np.random.default_rng(9).standard_normal(280))
    h = krylov.Handle()
    try:
        got = []
        for shuffled in (True, False, True, False):
            h.prepare(*arguments(y, shuffled), krylov.KK_FP64)
            got.append(h.krylov_kernel_apply(delta, 4)[0].cpu().numpy())
    finally:
        h.close()
    assert np.array_equal(got[0], got[2]) and np.array_equal(got[1], got[3])
    assert rel(got[0], got[1]) < TOL[krylov.KK_FP64]


@pytest.mark.parametrize("precision", PRECISIONS[:2], ids=IDS[:2])
@pytest.mark.parametrize("small_np_max", [0, 1 << 30])
def test_batch(precision, small_np_max):
    ys = [make(n, 200 + n) for n in (80, 31, 113)]
    rng = np.random.default_rng(3)
    deltas = [t(0.01 * rng.standard_normal(2 * n)) for n in (80, 31, 113)]
    got = []
    for shuffled in (False, True):
        names = ("offsets", "S", "Z", "Q_up", "Q_dn", "eps_up", "eps_dn", "gamma", "W", "kT", "n_electrons")
        b = krylov.Batch().prepare([dict(zip(names, arguments(y, shuffled))) for y in ys], precision)
        try:
            b.set_tuning(small_np_max, 2)
            got.append([x.cpu().numpy() for x in b.krylov_kernel_apply(deltas, 4)[0]])
        finally:
            b.close()
    err = [rel(p, q) for p, q in zip(*got)]
    assert max(err) < TOL[precision], err


@pytest.mark.parametrize("precision", PRECISIONS[:2], ids=IDS[:2])
@pytest.mark.parametrize("small_np_max", [0, 1 << 30])
@pytest.mark.parametrize("copies", [1, 6])
def test_batch_tiles_at_once_and_from_queues(copies, small_np_max, precision):
    """Launches of either tile class that hold at most one tile for each co-resident workgroup (one
    system of 640 and one of 1024 padded levels) and that take their tiles from the queues (six of
    each), each system against its own handle."""
    ys = [make(n, 400 + n + 7 * i) for i in range(copies) for n in (113, 66)]
    rng = np.random.default_rng(copies)
    deltas = [t(0.01 * rng.standard_normal(2 * (len(y["offsets"]) - 1))) for y in ys]
    names = ("offsets", "S", "Z", "Q_up", "Q_dn", "eps_up", "eps_dn", "gamma", "W", "kT", "n_electrons")
    b = krylov.Batch().prepare([dict(zip(names, arguments(y, False))) for y in ys], precision)
    try:
        b.set_tuning(small_np_max, 2)
        got = [[x.cpu().numpy() for x in b.krylov_kernel_apply(deltas, 4)[0]] for _ in range(2)]
    finally:
        b.close()
    for i, (y, delta) in enumerate(zip(ys, deltas)):
        h = krylov.Handle()
        try:
            h.prepare(*arguments(y, False), precision)
            want = h.krylov_kernel_apply(delta, 4)[0].cpu().numpy()
        finally:
            h.close()
        assert rel(got[0][i], want) < TOL[precision], i
        assert np.array_equal(got[0][i], got[1][i]), i


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("atoms", [171, 250, 320])
def test_last_round_in_pieces(atoms, precision):
    """Sizes whose shuffled levels leave a last round of few tiles, run in quarters (FP64 at 250 and
    320 atoms: 136 and 34 tiles past the last multiple of 256) or halves (FP16 x 3 at 171 atoms: 82;
    FP16 x 3 and BF16 at 320: 40), against the ascending order with its other tile count."""
    y = make(atoms, 600 + atoms)
    rng = np.random.default_rng(atoms)
    v, delta = rng.standard_normal((1, 2 * atoms)), 0.01 * rng.standard_normal(2 * atoms)
    a, b = (results(y, shuffled, precision, v, delta, 3) for shuffled in (False, True))
    err = [rel(p, q) for p, q in zip(a, b)]
    print(atoms, precision, err, flush=True)
    assert max(err) < TOL[precision], err


@pytest.mark.parametrize("atoms", [86, 99, 114, 118, 160])
def test_small_tiles_with_windows(atoms):
    """FP64 on unsplit 64 x 64 tiles by window tables: both ends of the two ranges that are not K-split
    (padded sizes 896 and 1152), a last round in quarters (99 atoms shuffled: 136 tiles past 256; 160
    atoms: 128 past 1024) and one that is not cut (118 atoms ascending)."""
    y = make(atoms, 700 + atoms)
    rng = np.random.default_rng(atoms)
    v, delta = rng.standard_normal((3, 2 * atoms)), 0.01 * rng.standard_normal(2 * atoms)
    a, b = (results(y, shuffled, krylov.KK_FP64, v, delta, 4) for shuffled in (False, True))
    err = [rel(p, q) for p, q in zip(a, b)]
    print(atoms, err, flush=True)
    assert max(err) < TOL[krylov.KK_FP64], err
