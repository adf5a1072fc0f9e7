"""Bands far apart in memory: a Gamma block whose stride takes a 64-row tile's
offsets past 32 bits gives what the packed block gives."""
import numpy as np
import pytest

from paper_0906_2569_amd import pwgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# 63 strides of 2 ld values: 2^32 - 130 (32-bit offsets still hold), 2^32 + 122, 1.25 times 2^32
@pytest.mark.parametrize("ld", [34087041, 34087043, 42608801])
@pytest.mark.parametrize("mixed", [0, 1])
def test_gamma_block(ld, mixed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0906_2569_amd import pwdft
    nb = 65
    g = pwgen.gamma_cell(6.5, 20.0, 2, nb, 41)
    ctx = pwdft.Context(0)
    plan = pwdft.Plan(ctx, g, precision=mixed, nb_max=nb, ndim_max=0, gamma=1)
    x = torch.from_numpy(g.psi0).cuda()
    want = plan.hpsi(x, prec=mixed).cpu().numpy()
    far = torch.empty(((nb - 1) * ld + plan.npw,), dtype=torch.complex128, device="cuda")
    y = far.as_strided((nb, plan.npw), (ld, 1))
    y.copy_(x)
    got = plan.hpsi(y, out=torch.empty_like(x), prec=mixed).cpu().numpy()
    del far, y
    torch.cuda.empty_cache()
    ctx.close()
    np.testing.assert_array_equal(got, want)
