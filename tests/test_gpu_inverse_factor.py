"""The reduced eigenproblem at the edges of the forms of the inverse factor
(64, 128, 256, 512 and 1024 rows), against LAPACK.

Tolerance: 64 n u times the norm of the matrix, divided by the smallest
eigenvalue of S (here at least 0.5), for eigenvalues of a pencil whose factor
and inverse are formed explicitly.
"""
import numpy as np
import pytest
import scipy.linalg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 2, 5, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1024, 1025])
def test_eigenvalues(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_2569_amd import pwdft
    rng = np.random.default_rng(n)
    a = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    h = (a + a.conj().T) / (2.0 * np.sqrt(n))
    b = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    s = np.eye(n) + 0.1 * (b + b.conj().T) / (2.0 * np.sqrt(n))
    nev = min(n, 6)
    ctx = pwdft.Context(0)
    try:
        w, c, _ = pwdft.reduced_eigh(ctx, torch.from_numpy(h.T.copy()).cuda(), torch.from_numpy(s.T.copy()).cuda(), nev)
        w, c = w.cpu().numpy(), c.cpu().numpy().T
    finally:
        ctx.close()
    smin = np.linalg.eigvalsh(s)[0]
    assert smin >= 0.5
    want = scipy.linalg.eigh(h, s, eigvals_only=True)[:nev]
    tol = 64 * n * np.finfo(float).eps * np.linalg.norm(h, 2) / smin
    np.testing.assert_allclose(w, want, atol=tol, rtol=0)
    assert np.abs(h @ c - (s @ c) * w).max() <= 4 * tol
    assert np.abs(c.conj().T @ s @ c - np.eye(nev)).max() <= 4 * tol
