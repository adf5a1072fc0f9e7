"""The two-step plane kernels with several z planes per workgroup (enough bands
to fill the device, a last group that is short), where plane_mode 3 alone may
take them, and their density at every plane they cover."""
import numpy as np
import pytest

import oracle
from test_gpu_wave_plane import PAIRS, _box_cell

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_2569_amd import pwdft
    return pwdft.Context(0)


def _hpsi_error(ctx, p, nb, plane_mode=0):
    from paper_0906_2569_amd import pwdft
    plan = pwdft.Plan(ctx, p, precision=0, nb_max=nb, ndim_max=0, plane_mode=plane_mode)
    form = plan.info()["plane64"]
    got = plan.hpsi(torch.from_numpy(p.psi0[:nb].copy()).cuda()).cpu().numpy()
    plan.close()
    ref = oracle.hpsi(oracle.dense_h_of(p), p.psi0[:nb])
    return form, (np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()


# up to 6 planes per workgroup: 130 bands make 650 groups and more, over the 512
# from which the kernels take several planes; no group size above 3 (2) divides 27 (32, but 4)
@pytest.mark.parametrize("n1,n2", [(24, 24), (25, 25), (27, 27), (30, 30), (45, 45), (50, 50), (54, 54), (64, 64),
                                   (72, 72), (36, 30), (30, 36), (45, 50), (75, 72)])
@pytest.mark.parametrize("n3", [27, 32])
def test_groups_of_planes(ctx, n1, n2, n3):
    p = _box_cell(700 + n1 + n3, (n1, n2, n3), 130)
    form, err = _hpsi_error(ctx, p, 130)
    assert form == 3
    assert err <= 1e-11


@pytest.mark.parametrize("n", [75, 81, 90, 100, 108, 120, 125, 135])
def test_form_of_large_planes(ctx, n):
    p = _box_cell(800 + n, (n, n, 25), 24, ng=60)
    form, err = _hpsi_error(ctx, p, 24)
    assert form == 3
    assert err <= 1e-11


# measured at plan creation: the register or the two-step kernel
@pytest.mark.parametrize("n", [32, 36, 40, 48])
@pytest.mark.parametrize("nb", [2, 130])
def test_measured_form(ctx, n, nb):
    p = _box_cell(850 + n, (n, n, 27), nb)
    form, err = _hpsi_error(ctx, p, nb, plane_mode=3)
    assert form in (0, 3)
    assert err <= 1e-11


@pytest.mark.parametrize("n1,n2", [(n, n) for n in (25, 27, 32, 36, 40, 45, 48, 50, 54, 64, 75, 80, 81, 90, 96, 100, 108,
                                                    125, 135)] + PAIRS + [(b, a) for a, b in PAIRS])
def test_density(ctx, n1, n2):
    from paper_0906_2569_amd import pwdft
    nr, nb = (n1, n2, 24), 3
    p = _box_cell(60 + n1 + n2, nr, nb, ng=60)
    w = np.array([2.0, 0.5, 1.25])
    plan = pwdft.Plan(ctx, p, precision=0, nb_max=nb, ndim_max=0, density=1)
    got = plan.density(torch.from_numpy(p.psi0).cuda(), w, 275.0).cpu().numpy()
    plan.close()
    f = np.zeros((nb, nr[2], nr[1], nr[0]), dtype=complex)
    m = p.miller
    f[:, m[:, 2] % nr[2], m[:, 1] % nr[1], m[:, 0] % nr[0]] = p.psi0
    r = np.fft.ifftn(f, axes=(1, 2, 3)) * (nr[0] * nr[1] * nr[2])
    ref = np.einsum("b,bzyx->zyx", w, r.real ** 2 + r.imag ** 2) / 275.0
    # as in test_gpu_wave_plane: rounding of three transforms and of the band sum
    np.testing.assert_allclose(got, ref, atol=1e-13 * np.abs(ref).max(), rtol=0)
