"""H.psi on grids whose passes run on two-step transforms (n = A B within one
wave), against the dense oracle: every plane and column length they cover."""
import numpy as np
import pytest

import oracle
from paper_0906_2569_amd import pwgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SQUARE = [24, 25, 27, 30, 45, 50, 54, 60, 64, 72, 75, 81, 90, 100, 108, 120, 125, 135]
PAIRS = [(24, 25), (25, 30), (30, 36), (36, 40), (40, 45), (45, 50), (50, 54), (54, 60), (60, 64), (64, 72), (72, 75),
         (75, 80), (80, 81), (81, 90), (90, 96), (96, 100), (100, 108), (108, 120), (120, 125)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_2569_amd import pwdft
    return pwdft.Context(0)


def _err(ctx, p, nb, **kw):
    from paper_0906_2569_amd import pwdft
    plan = pwdft.Plan(ctx, p, precision=0, nb_max=nb, ndim_max=0, **kw)
    x = torch.from_numpy(p.psi0[:nb].copy()).cuda()
    got = plan.hpsi(x).cpu().numpy()
    plan.close()
    return got


def _box_cell(seed, nr, nb, natoms=2, a=6.5, ng=240):
    """A set of G vectors that fills the box |m_d| <= (n_d - 1) / 4 at random and
    reaches its faces, with a random potential on the whole grid."""
    rng = np.random.default_rng(seed)
    p = pwgen.tiny_cell(seed, a=a, ecut_ry=3.0, natoms=natoms, nb=nb, kfrac=(0.25, -0.125, 0.375))
    h = [(n - 1) // 4 for n in nr]
    m = [tuple(int(rng.integers(-x, x + 1)) for x in h) for _ in range(ng)]
    m += [(0, 0, 0)] + [tuple(s * x if d == e else 0 for e, x in enumerate(h)) for d in range(3) for s in (1, -1)]
    p.miller = np.array(sorted(set(m)), dtype=np.int32)
    p.kpg = p.kpt + 2 * np.pi / a * p.miller
    p.nr = nr
    p.vloc_r = 0.5 * rng.standard_normal((nr[2], nr[1], nr[0]))
    npw = len(p.miller)
    beta = rng.standard_normal((4 * natoms, npw)) + 1j * rng.standard_normal((4 * natoms, npw))
    p.beta = beta / np.linalg.norm(beta, axis=1, keepdims=True)
    p.psi0 = pwgen.random_psi(rng, nb, npw)
    return p


def _check(ctx, nr, nb):
    p = _box_cell(900 + nr[0] + nr[2], nr, nb)
    got = _err(ctx, p, nb)
    ref = oracle.hpsi(oracle.dense_h_of(p), p.psi0)
    err = (np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()
    assert err <= 1e-11, err


# n3 odd and even, one band and several (one and several planes per workgroup)
@pytest.mark.parametrize("nb,n3", [(1, 27), (7, 32)])
@pytest.mark.parametrize("n", SQUARE)
def test_square_planes(ctx, n, nb, n3):
    _check(ctx, (n, n, n3), nb)


@pytest.mark.parametrize("a,b", PAIRS)
def test_unequal_planes(ctx, a, b):
    _check(ctx, (a, b, 30), 3)
    _check(ctx, (b, a, 30), 3)


@pytest.mark.parametrize("n3", [24, 25, 27, 30, 45, 50, 54, 75, 81, 90, 100, 108, 120, 135])
def test_column_lengths(ctx, n3):
    _check(ctx, (30, 32, n3), 5)


@pytest.mark.parametrize("n", [30, 45, 54, 72, 90, 120])
def test_gamma_pairs(ctx, n):
    # two bands share a transform; odd band counts leave the last one alone
    g = pwgen.gamma_cell(6.5, 20.0, 2, 5, 950 + n, nr=(n, n, n))
    got = g.expand(_err(ctx, g, 5, gamma=1))
    ref = oracle.hpsi(oracle.dense_h_of(g.full), g.expand(g.psi0))
    err = (np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()
    assert err <= 1e-11, err


# band sums over groups of transforms: one band, fewer than and more than one per group
@pytest.mark.parametrize("nb", [1, 5, 40])
@pytest.mark.parametrize("nr", [(24, 24, 30), (30, 30, 25), (50, 45, 27), (60, 60, 24), (72, 72, 24), (96, 100, 25),
                                (120, 120, 25), (128, 128, 24)])
def test_density(ctx, nr, nb):
    from paper_0906_2569_amd import pwdft
    p = _box_cell(70 + nr[0] + nb, nr, nb, ng=60)
    w = np.random.default_rng(nb).uniform(0.0, 2.0, nb)
    plan = pwdft.Plan(ctx, p, precision=0, nb_max=nb, ndim_max=0, density=1)
    x = torch.from_numpy(p.psi0).cuda()
    got = plan.density(x, w, 275.0)
    again = plan.density(x, w, 275.0).cpu().numpy()
    twice = plan.density(x, w, 275.0, rho=got.clone(), accumulate=True).cpu().numpy()
    got = got.cpu().numpy()
    plan.close()
    f = np.zeros((nb, nr[2], nr[1], nr[0]), dtype=complex)
    m = p.miller
    f[:, m[:, 2] % nr[2], m[:, 1] % nr[1], m[:, 0] % nr[0]] = p.psi0
    r = np.fft.ifftn(f, axes=(1, 2, 3)) * (nr[0] * nr[1] * nr[2])
    ref = np.einsum("b,bzyx->zyx", w, r.real ** 2 + r.imag ** 2) / 275.0
    # rounding of three transforms (about 2 log2 N ulp of the largest value) and of the band sum
    tol = 1e-13 * np.abs(ref).max()
    np.testing.assert_allclose(got, ref, atol=tol, rtol=0)
    np.testing.assert_array_equal(got, again)
    np.testing.assert_allclose(twice, 2 * ref, atol=2 * tol, rtol=0)


@pytest.mark.parametrize("n", [45, 72])
def test_density_gamma(ctx, n):
    from paper_0906_2569_amd import pwdft
    g = pwgen.gamma_cell(6.5, 20.0, 2, 5, 960 + n, nr=(n, n, n))
    w = np.array([2.0, 1.0, 0.5, 0.0, 1.5])
    plan = pwdft.Plan(ctx, g, precision=0, nb_max=5, ndim_max=0, density=1, gamma=1)
    got = plan.density(torch.from_numpy(g.psi0).cuda(), w, 100.0).cpu().numpy()
    plan.close()
    f = np.zeros((5, n, n, n), dtype=complex)
    m = g.full.miller
    f[:, m[:, 2] % n, m[:, 1] % n, m[:, 0] % n] = g.expand(g.psi0)
    r = np.fft.ifftn(f, axes=(1, 2, 3)) * n ** 3
    ref = np.einsum("b,bzyx->zyx", w, r.real ** 2 + r.imag ** 2) / 100.0
    np.testing.assert_allclose(got, ref, atol=1e-13 * np.abs(ref).max(), rtol=0)
