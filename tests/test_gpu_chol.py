"""Cholesky inverse factor at the edges of its 16-row panels, with leading
dimensions above n: R^-1 against numpy, its exact zeros, and the backward error
|R^H R - G| of an elimination, n eps |G| up to a small factor (the diagonal shift
1e-15 n max G_ii is part of the definition)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pad", [(2, 0), (15, 3), (16, 0), (17, 0), (31, 1), (32, 0), (33, 0), (47, 0), (48, 5), (49, 0),
                                   (64, 2)])
def test_chol_panels(torch_cuda, n, pad):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
    cond = 1e4
    G = (Q * np.logspace(0, np.log10(cond), n)) @ Q.conj().T
    G = 0.5 * (G + G.conj().T)
    Gd = torch.full((n, n + pad), float("nan"), dtype=torch.complex128, device="cuda")
    Gd[:, :n] = torch.from_numpy(np.ascontiguousarray(G.T)).cuda()
    Rd = torch.full((n, n + pad), 7.0, dtype=torch.complex128, device="cuda")
    ctx.chol_inv(Gd[:, :n], n, Rd[:, :n])
    out = Rd.cpu().numpy()
    assert np.all(out[:, n:] == 7.0)
    Rinv = out[:, :n].T
    shift = 1e-15 * n * np.diag(G).real.max()
    eps = np.finfo(float).eps
    ref = np.linalg.inv(np.linalg.cholesky(G + shift * np.eye(n)).conj().T)
    assert np.abs(Rinv - ref).max() <= 8 * n * eps * np.sqrt(cond) * np.abs(ref).max()
    assert np.all(np.tril(Rinv, -1) == 0)
    R = np.linalg.inv(Rinv)
    back = np.abs(R.conj().T @ R - G - shift * np.eye(n)).max()
    assert back <= 8 * n * eps * np.sqrt(cond) * np.abs(G).max()   # numpy's inverse of R^-1 included
    ctx.close()
