"""The waves of a plane workgroup follow from the kept columns, the precision and
the number of planes (few: up to 12 waves; many: four, or eight or six in FP32),
and change no bit: a column of a block, applied with all others and alone, is
the same, and the block's is numpy's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec_name", ["fp64", "mixed"])
@pytest.mark.parametrize("n,r", [(36, 8.05), (64, 27.05), (72, 22.05), (72, 31.05), (96, 14.05), (96, 30.05), (96, 38.05),
                                 (108, 26.05), (120, 29.05), (128, 31.05)])
def test_waves_change_no_bit(torch_cuda, n, r, prec_name):
    torch = torch_cuda
    from paper_0707_3405_amd import Context, PW_PREC_FP64, PW_PREC_MIXED
    prec = PW_PREC_FP64 if prec_name == "fp64" else PW_PREC_MIXED
    rng = np.random.default_rng(n + int(r))
    v = rng.standard_normal((n, n, n))
    ctx = Context(0)
    npw = ctx.init_basis(np.eye(3) * 2 * np.pi, (0.02, -0.03, 0.01), 0.5 * r * r, (n, n, n))
    mil = ctx.get_miller()
    ctx.set_local_potential(v)
    nb = 9
    ctx.alloc_workspace(nb, nb, prec)
    x = rng.standard_normal((nb, npw)) + 1j * rng.standard_normal((nb, npw))
    xd = torch.from_numpy(x).cuda().to(torch.complex128 if prec == PW_PREC_FP64 else torch.complex64)
    y = torch.empty_like(xd)
    ctx.apply_H(xd, y, prec=prec)
    for j in (0, 4, nb - 1):
        alone = torch.empty_like(xd[:1])
        ctx.apply_H(xd[j:j + 1], alone, prec=prec)
        assert torch.equal(alone[0], y[j]), j
    x0 = xd[4].cpu().numpy().astype(complex)
    i = np.mod(mil, n)
    g = np.zeros((n, n, n), complex)
    g[i[:, 0], i[:, 1], i[:, 2]] = x0
    ref = np.fft.fftn(np.fft.ifftn(g) * v)[i[:, 0], i[:, 1], i[:, 2]] + ctx.get_kinetic() * x0
    hn = (np.abs(v).max() + 0.5 * r * r) * np.linalg.norm(x0)   # norms of the two terms' operators
    err = np.linalg.norm(y[4].cpu().numpy() - ref) / hn
    assert err <= (1e-13 if prec == PW_PREC_FP64 else 1e-6), err
    ctx.close()
