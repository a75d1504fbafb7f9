"""pw_density gives the same bits whatever the workspace: the least the call
takes, any number of grids more, a large one, and a plan of other block sizes
(other chunks of bands); and the oracle's density to rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,nb", [(20, 4.05, 1), (36, 8.05, 21), (96, 20.05, 37), (120, 25.05, 21)])
def test_density_does_not_depend_on_the_workspace(torch_cuda, n, r, nb):
    torch = torch_cuda
    from paper_0707_3405_amd import Context, PWError, PW_ERR_NOMEM
    cell, k, ecut = np.eye(3) * 2 * np.pi, (0.1, 0.2, 0.3), 0.5 * r * r
    rng = np.random.default_rng(n + nb)
    out = []
    for block in (1, 8, min(nb, 64)):
        ctx = Context(0)
        npw = ctx.init_basis(cell, k, ecut, (n, n, n))
        mil = ctx.get_miller()
        if block > 1:
            ctx.workspace_size(nb, min(nb, block))
        full = ctx.workspace_size(nb, min(nb, block)) if block > 1 else 0
        if not out:
            x = rng.standard_normal((nb, npw)) + 1j * rng.standard_normal((nb, npw))
            occ = rng.uniform(0.0, 2.0, nb)
        xd = torch.from_numpy(x).cuda()
        # the least: stick buffer of a chunk, one grid, the occupations
        nst = len({(a, b) for a, b in mil[:, :2].tolist()})
        up = lambda v: (v + 255) // 256 * 256
        least = up(min(nb, block) * n * ((nst + 15) // 16 * 16) * 16) + up(8 * nb) + up(8 * n ** 3)
        sizes = [full, full + 80 * n ** 3 * 8] if full else [least, least + 3 * n ** 3 * 8, least + 80 * n ** 3 * 8]
        for nbytes in sizes:
            ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
            ctx.set_workspace(ws[(-ws.data_ptr()) % 256:][:nbytes])
            rho = torch.full((n, n, n), float("nan"), dtype=torch.float64, device="cuda")
            ctx.density(xd, occ, rho)
            out.append(rho.cpu().numpy())
        if not full:
            ws = torch.empty(least, dtype=torch.uint8, device="cuda")
            ctx.set_workspace(ws[(-ws.data_ptr()) % 256:][:least - 256])
            with pytest.raises(PWError) as e:
                ctx.density(xd, occ, rho)
            assert e.value.status == PW_ERR_NOMEM
        ctx.close()
    i = np.mod(mil, n)
    want = np.zeros((n, n, n))
    for j in range(nb):
        g = np.zeros((n, n, n), complex)
        g[i[:, 0], i[:, 1], i[:, 2]] = x[j]
        want += occ[j] * np.abs(np.fft.ifftn(g) * n ** 3) ** 2
    want /= (2 * np.pi) ** 3
    for rho in out:
        assert np.abs(rho - want).max() <= 1e-12 * want.max()
        assert np.array_equal(rho, out[0])
