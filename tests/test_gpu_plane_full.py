"""The plane pass of H.X and of the density with spheres that reach beyond the
middle half of the grid, at every FFT size whose default split has a pruned
form (first factor 8) and that other tests reach only with smaller spheres."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(32, 3), (40, 3), (64, 2), (80, 2), (96, 2)])
def test_plane_pass_beyond_the_middle_half(torch_cuda, n, nb):
    torch = torch_cuda
    from paper_0707_3405_amd import Context, PW_PREC_MIXED
    rng = np.random.default_rng(n)
    r = n // 4 + 1.05
    v = rng.standard_normal((n, n, n))
    ctx = Context(0)
    npw = ctx.init_basis(np.eye(3) * 2 * np.pi, (0.02, -0.03, 0.01), 0.5 * r * r, (n, n, n))
    mil = ctx.get_miller()
    assert (mil[:, 0] > n // 4).any() and (mil[:, 1] < -(n // 4)).any()
    ctx.set_local_potential(v)
    ctx.alloc_workspace(nb, nb, PW_PREC_MIXED)
    x = rng.standard_normal((nb, npw)) + 1j * rng.standard_normal((nb, npw))
    xd = torch.from_numpy(x).cuda()
    i = np.mod(mil, n)
    g = np.zeros((nb, n, n, n), complex)
    g[:, i[:, 0], i[:, 1], i[:, 2]] = x
    psi = np.fft.ifftn(g, axes=(1, 2, 3))
    ref = np.fft.fftn(psi * v, axes=(1, 2, 3))[:, i[:, 0], i[:, 1], i[:, 2]] + ctx.get_kinetic() * x
    hn = (np.abs(v).max() + 0.5 * r * r) * np.linalg.norm(x, axis=1)   # norms of the two terms' operators
    y = torch.empty_like(xd)
    ctx.apply_H(xd, y)
    err = np.linalg.norm(y.cpu().numpy() - ref, axis=1) / hn
    assert err.max() <= 1e-13, err.max()
    x32 = xd.to(torch.complex64)
    y32 = torch.empty_like(x32)
    ctx.apply_H(x32, y32, prec=PW_PREC_MIXED)
    err = np.linalg.norm(y32.cpu().numpy() - ref, axis=1) / hn   # the rounding of x itself included
    assert err.max() <= 1e-6, err.max()
    occ = rng.uniform(0.0, 2.0, nb)
    rho = torch.empty((n, n, n), dtype=torch.float64, device="cuda")
    ctx.density(xd, occ, rho)
    want = (occ[:, None, None, None] * np.abs(psi * n ** 3) ** 2).sum(0) / (2 * np.pi) ** 3
    assert np.abs(rho.cpu().numpy() - want).max() <= 1e-12 * want.max()
    ctx.close()
