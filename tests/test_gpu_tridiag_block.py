"""Davidson solves whose reduced problems take the one-workgroup
tridiagonalization, alone (up to 96 rows) and as the tail of the cooperative
one, against the dense oracle: bases of nb up to ndim nb rows around the edges
of its forms (32, 48, 64 and 96 rows)."""
import numpy as np
import pytest

import oracle
from paper_0906_2569_amd import pwgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_2569_amd import pwdft
    return pwdft.Context(0)


@pytest.fixture(scope="module")
def cell():
    p = pwgen.make_cell(10.0, 15.0, 8, 60, 4242, nr=(30, 30, 30))
    return p, oracle.eigh_lowest(oracle.dense_h_of(p), 60)[0]


@pytest.mark.parametrize("nb,ndim", [(1, 2), (2, 8), (4, 8), (11, 3), (12, 4), (16, 2), (16, 4), (17, 4), (24, 4),
                                     (31, 2), (32, 3), (33, 3), (48, 2), (49, 2), (50, 4), (60, 3)])
def test_eigenvalues(ctx, cell, nb, ndim):
    from paper_0906_2569_amd import pwdft
    p, w = cell
    plan = pwdft.Plan(ctx, p, nb_max=nb, ndim_max=ndim)
    x = torch.from_numpy(p.psi0[:nb].copy()).cuda()
    st, eig, resid, _ = plan.davidson(x, opts=pwdft.default_opts(ndim=ndim, max_iter=400))
    psi = x.cpu().numpy()
    plan.close()
    assert st == 0 and resid.max().item() <= 1e-6
    np.testing.assert_allclose(eig.cpu().numpy(), w[:nb], atol=5e-9, rtol=0)
    np.testing.assert_allclose(psi.conj() @ psi.T, np.eye(nb), atol=1e-10)


@pytest.mark.parametrize("nb", [9, 40])
def test_real_reduced_problem(ctx, nb):
    # Gamma: the reduced matrices are real
    from paper_0906_2569_amd import pwdft
    g = pwgen.gamma_cell(8.0, 12.0, 5, nb, 77)
    w = oracle.eigh_lowest(oracle.dense_h_of(g.full), nb)[0]
    plan = pwdft.Plan(ctx, g, nb_max=nb, ndim_max=3, gamma=1)
    x = torch.from_numpy(g.psi0.copy()).cuda()
    st, eig, _, _ = plan.davidson(x, opts=pwdft.default_opts(ndim=3, max_iter=400))
    plan.close()
    assert st == 0
    np.testing.assert_allclose(eig.cpu().numpy(), w, atol=5e-9, rtol=0)


@pytest.mark.parametrize("nb,k", [(7, (0.0, 0.0, 0.0)), (13, (0.0, 0.0, 0.0)), (20, (0.25, 0.1, 0.0))])
def test_decoupled_blocks(ctx, nb, k):
    # no potential and no projectors: plane waves as trial vectors give reduced
    # problems whose tridiagonal has exact zeros and multiple eigenvalues
    from paper_0906_2569_amd import pwdft
    p = pwgen.make_cell(8.0, 12.0, 2, nb, 5, kfrac=k, with_vloc=False, with_beta=False)
    w = oracle.eigh_lowest(oracle.dense_h_of(p), nb)[0]
    kin = np.real(np.diag(oracle.dense_h_of(p)))
    order = np.argsort(kin, kind="stable")
    x0 = np.zeros((nb, p.npw), dtype=np.complex128)
    x0[np.arange(nb), order[:nb]] = 1.0
    x0[-1] += 1e-3 * p.psi0[0]     # one of them still to converge
    plan = pwdft.Plan(ctx, p, nb_max=nb, ndim_max=4)
    x = torch.from_numpy(x0).cuda()
    st, eig, resid, _ = plan.davidson(x, opts=pwdft.default_opts(ndim=4, max_iter=400))
    plan.close()
    assert st == 0 and resid.max().item() <= 1e-6
    np.testing.assert_allclose(eig.cpu().numpy(), w, atol=5e-9, rtol=0)
