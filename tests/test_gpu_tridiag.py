"""The reduction to tridiagonal form with a launch per column (n > 192): tile and
thread-count edges (tiles of 4, 8 and 32 rows by 128 columns, 256, 512 and 1024
rows per launch), matrices that need no reflector in some or all columns, and a
leading dimension above n.  Against LAPACK through numpy; both eigenvalues and
residuals of backward-stable reductions stay within a small multiple of
n eps |A|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _matrix(rng, n, kind):
    z = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    A = z + z.conj().T
    if kind == "tridiagonal":   # complex subdiagonal: a phase, nothing to annihilate
        A = np.triu(np.tril(A, 1), -1)
    elif kind == "blocks":      # uncoupled at an odd row: one column without any reflector
        h = n // 2 + 1
        A[h:, :h] = 0.0
        A[:h, h:] = 0.0
    elif kind == "graded":
        d = np.logspace(0, -8, n)
        A = A * d[:, None] * d[None, :]
    return A


@pytest.mark.parametrize("n,k,kind,pad", [
    (193, 7, "dense", 0), (255, 3, "dense", 5), (256, 4, "blocks", 0), (257, 9, "dense", 0), (300, 2, "tridiagonal", 3),
    (384, 3, "dense", 0), (385, 5, "graded", 0), (511, 3, "dense", 1), (512, 4, "blocks", 0), (513, 6, "dense", 0),
    (641, 3, "tridiagonal", 0), (896, 2, "blocks", 7), (1023, 3, "dense", 0), (1024, 3, "dense", 0)])
def test_reduction(torch_cuda, n, k, kind, pad):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:])
    A = _matrix(np.random.default_rng(n + 7 * k), n, kind)
    ref = np.linalg.eigvalsh(A)
    buf = torch.full((n, n + pad), float("nan"), dtype=torch.complex128, device="cuda")
    buf[:, :n] = torch.from_numpy(np.ascontiguousarray(A.T)).cuda()
    w = torch.zeros(k, dtype=torch.float64, device="cuda")
    V = torch.zeros((k, n), dtype=torch.complex128, device="cuda")
    ctx.small_eigh(buf[:, :n], n, k, w, V)
    wn, Vn = w.cpu().numpy(), V.cpu().numpy().T
    tol = 4 * n * np.finfo(float).eps * np.abs(ref).max()
    assert np.abs(wn - ref[:k]).max() <= tol
    assert np.linalg.norm(A @ Vn - Vn * wn, axis=0).max() <= tol
    ctx.close()


@pytest.mark.parametrize("n,k,kind,pad", [
    (96, 96, "dense", 0), (97, 97, "dense", 3), (98, 5, "blocks", 0), (127, 4, "tridiagonal", 0), (129, 129, "dense", 0),
    (160, 64, "graded", 0), (191, 3, "blocks", 1), (192, 64, "dense", 0), (223, 3, "dense", 0), (225, 3, "tridiagonal", 2)])
def test_last_columns(torch_cuda, n, k, kind, pad):
    """The last 96 columns are reduced by one workgroup: the handover, on either side of it."""
    test_reduction(torch_cuda, n, k, kind, pad)
