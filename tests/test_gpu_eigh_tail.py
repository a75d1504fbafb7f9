"""The eigensolver's tail at the edges of its kernels: the 16-step groups and the
lost-scale fallback of the Sturm counts (diagonal and split matrices), the
rows-per-lane variants of inverse iteration and back-transform (n across
multiples of 64 up to 1024), and both forms of the re-orthogonalisation
(eigenvectors near the identity's Gram or clustered; clusters side by side for
larger blocks).  Against LAPACK through numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _matrix(rng, n, kind):
    """(Hermitian matrix, exact eigenvalues ascending or None)"""
    if kind == "identity":
        return np.eye(n, dtype=complex), np.ones(n)
    if kind == "diagonal":      # uncoupled, every value repeated
        lam = np.sort(np.repeat(np.arange(1, n // 2 + 2), 2)[:n].astype(float))
        return np.diag(rng.permutation(lam)).astype(complex), lam
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
    if kind == "clusters":      # runs of three values 1e-9 apart, runs 1 apart
        lam = np.arange(n) // 3 + 1e-9 * (np.arange(n) % 3)
    else:
        lam = np.arange(n) * 1.0
    A = (Q * lam) @ Q.conj().T
    return 0.5 * (A + A.conj().T), lam


@pytest.mark.parametrize("n,k,kind", [
    (16, 16, "spread"), (17, 17, "spread"), (18, 3, "spread"), (33, 33, "diagonal"), (64, 64, "identity"),
    (65, 63, "spread"), (192, 64, "clusters"), (48, 17, "clusters"), (208, 64, "spread"),
    (209, 64, "clusters"), (257, 5, "spread"), (384, 65, "clusters"), (385, 385, "spread"),
    (512, 512, "clusters"), (513, 70, "diagonal"), (768, 3, "spread"), (769, 70, "clusters"), (1024, 1, "spread")])
def test_eigh_tail(torch_cuda, n, k, kind):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:])
    rng = np.random.default_rng(n * 37 + k)
    A, lam = _matrix(rng, n, kind)
    w = torch.zeros(k, dtype=torch.float64, device="cuda")
    V = torch.zeros((k, n), dtype=torch.complex128, device="cuda")
    ctx.small_eigh(torch.from_numpy(np.ascontiguousarray(A.T)).cuda(), n, k, w, V)
    wn, Vn, nrm = w.cpu().numpy(), V.cpu().numpy().T, np.abs(lam).max()
    assert np.abs(wn - lam[:k]).max() <= 1e-13 * nrm * max(1, np.sqrt(n) / 4)
    assert np.abs(A @ Vn - Vn * wn).max() <= 1e-12 * nrm
    # clusters are re-orthogonalised in full; between them (a gap of 1)
    # larger blocks keep the solves' backward error over the gap
    orth = max(1e-12, n * np.finfo(float).eps * nrm)
    assert np.abs(Vn.conj().T @ Vn - np.eye(k)).max() <= orth
    ctx.close()
