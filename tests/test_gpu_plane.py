"""The plane pass of H.X and of the density over its shapes: every FFT size with
a sphere inside the middle half of the grid (the pruned first and last stages)
and with one that fills it, up to the widest kept-column set LDS holds, in both
precisions, against numpy FFTs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = (16, 20, 24, 32, 36, 40, 48, 60, 64, 72, 80, 96, 108, 120, 128)


def _problem(n, r, k):
    """Cube of side 2 pi (so |k + G| = |n + k|), sphere of radius r, random potential."""
    rng = np.random.default_rng(n * 1000 + int(r * 10))
    return np.eye(3) * 2 * np.pi, k, 0.5 * r * r, rng.standard_normal((n, n, n)), rng


def _grid(mil, x, n):
    g = np.zeros((x.shape[0], n, n, n), complex)
    i = np.mod(mil, n)
    g[:, i[:, 0], i[:, 1], i[:, 2]] = x
    return np.fft.ifftn(g, axes=(1, 2, 3)), i


# (n, radius, k, bands): half-grid spheres, full ones where LDS holds every
# column, and the widest of the largest grids
LOOSE = [(n, (n - 1) // 4 + 0.05, (0.02, -0.03, 0.01), 3) for n in SIZES]
TIGHT = [(n, (n - 1) // 2 + 0.05, (0.02, 0.03, -0.01), 2) for n in (16, 20, 24, 36, 48, 60, 72)]
WIDEST = [(108, 45.05, (0.02, 0.0, 0.0), 1), (120, 41.0, (0.5, 0.1, 0.0), 1), (128, 38.05, (0.02, 0.0, 0.0), 1)]


@pytest.mark.parametrize("n,r,k,nb", LOOSE + TIGHT + WIDEST)
def test_plane_pass(torch_cuda, n, r, k, nb):
    torch = torch_cuda
    from paper_0707_3405_amd import Context, PW_PREC_MIXED
    cell, k, ecut, v, rng = _problem(n, r, k)
    ctx = Context(0)
    npw = ctx.init_basis(cell, k, ecut, (n, n, n))
    mil = ctx.get_miller()
    ctx.set_local_potential(v)
    ws = torch.empty((nb * n * 4 * n * n * 16 >> 2) + 64 * npw * 16 + (256 << 20), dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:])
    x = rng.standard_normal((nb, npw)) + 1j * rng.standard_normal((nb, npw))
    xd = torch.from_numpy(x).cuda()
    psi, i = _grid(mil, x, n)
    kin = ctx.get_kinetic()
    ref = np.fft.fftn(psi * v, axes=(1, 2, 3))[:, i[:, 0], i[:, 1], i[:, 2]] + kin * x
    # sum of the norms of the two terms' operators
    hn = (np.abs(v).max() + ecut) * np.linalg.norm(x, axis=1)
    y = torch.empty_like(xd)
    ctx.apply_H(xd, y)
    err = np.linalg.norm(y.cpu().numpy() - ref, axis=1) / hn
    assert err.max() <= 1e-13, err.max()
    x32 = xd.to(torch.complex64)
    y32 = torch.empty_like(x32)
    ctx.apply_H(x32, y32, prec=PW_PREC_MIXED)
    # the rounding of x itself is 2^-24 relative: part of the bar
    err = np.linalg.norm(y32.cpu().numpy() - ref, axis=1) / hn
    assert err.max() <= 1e-6, err.max()
    occ = rng.uniform(0.0, 2.0, nb)
    rho = torch.empty((n, n, n), dtype=torch.float64, device="cuda")
    ctx.density(xd, occ, rho)
    want = (occ[:, None, None, None] * np.abs(psi * n ** 3) ** 2).sum(0) / (2 * np.pi) ** 3
    assert np.abs(rho.cpu().numpy() - want).max() <= 1e-12 * want.max()
    ctx.close()


def test_plane_too_wide(torch_cuda):
    """One column more than LDS holds is refused, as an argument error."""
    torch = torch_cuda
    from paper_0707_3405_amd import Context, PWError, PW_ERR_ARG
    cell, k, ecut, v, _ = _problem(128, 39.0, (0.5, 0.1, 0.0))   # 78 columns
    ctx = Context(0)
    npw = ctx.init_basis(cell, k, ecut, (128,) * 3)
    ctx.set_local_potential(v)
    ws = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:])
    x = torch.zeros((1, npw), dtype=torch.complex128, device="cuda")
    with pytest.raises(PWError) as e:
        ctx.apply_H(x, torch.empty_like(x))
    assert e.value.status == PW_ERR_ARG
    ctx.close()


@pytest.mark.parametrize("n,r", [(36, 8.05), (96, 20.05), (120, 25.05)])
def test_density_groups(torch_cuda, n, r):
    """Bands dealt over several groups (a workspace with room) and one group (the
    smallest workspace), several chunks, against each other and numpy."""
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    cell, k, ecut, v, rng = _problem(n, r, (0.1, 0.2, 0.3))
    nb, block = 21, 8
    ctx = Context(0)
    npw = ctx.init_basis(cell, k, ecut, (n, n, n))
    ctx.set_local_potential(v)
    x = rng.standard_normal((nb, npw)) + 1j * rng.standard_normal((nb, npw))
    xd, occ = torch.from_numpy(x).cuda(), rng.uniform(0.0, 2.0, nb)
    psi, _ = _grid(ctx.get_miller(), x, n)
    want = (occ[:, None, None, None] * np.abs(psi * n ** 3) ** 2).sum(0) / (2 * np.pi) ** 3
    out = []
    full = ctx.workspace_size(nb, block)
    for nbytes in (full, full + 64 * n ** 3 * 8):
        ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        ctx.set_workspace(ws[(-ws.data_ptr()) % 256:][:nbytes])
        rho = torch.empty((n, n, n), dtype=torch.float64, device="cuda")
        ctx.density(xd, occ, rho)
        out.append(rho.cpu().numpy())
        assert np.abs(out[-1] - want).max() <= 1e-12 * want.max()
    ctx.close()
