"""A Hermitian matrix with a non-finite entry is refused by the eigensolver's
entry points with PW_ERR_NUMERIC, on every route of the reduction (one
workgroup up to 96 rows, a launch per column above) and wherever the entry
lies; the context then solves a finite matrix as if nothing had happened."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NAN, INF = float("nan"), float("inf")


def _context(torch, n):
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:])
    return ctx


@pytest.mark.parametrize("entry", ["small_eigh", "small_eigh_noalloc"])
@pytest.mark.parametrize("n", [1, 2, 33, 96, 97, 192, 256, 257, 300, 513])
def test_nonfinite_matrix_is_refused(torch_cuda, n, entry):
    torch = torch_cuda
    from paper_0707_3405_amd import PWError, PW_ERR_NUMERIC
    ctx = _context(torch, n)
    k = min(n, 40)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    A = 0.5 * (A + A.conj().T)
    solve = getattr(ctx, entry)
    w = torch.empty(k, dtype=torch.float64, device="cuda")
    V = torch.empty((k, n), dtype=torch.complex128, device="cuda")
    bad = [np.full((n, n), complex(NAN, NAN)), np.full((n, n), complex(INF, 0.0)), np.diag(np.full(n, INF)).astype(complex)]
    for i, j in ((0, 0), (n - 1, n - 1), (n - 1, 0), (n // 2, n // 3)):
        for x in (NAN, -INF):
            b = A.copy()
            b[i, j] = x
            bad.append(b)
            b = np.diag(np.arange(n) + 0j)   # the reduction of a diagonal matrix reflects nothing
            b[i, j] = x
            bad.append(b)
    for c, b in enumerate(bad):
        with pytest.raises(PWError) as e:
            solve(torch.from_numpy(b).cuda(), n, k, w, V)
        assert e.value.status == PW_ERR_NUMERIC, c
    solve(torch.from_numpy(np.ascontiguousarray(A.T)).cuda(), n, k, w, V)
    ref = np.linalg.eigvalsh(A)
    assert np.abs(w.cpu().numpy() - ref[:k]).max() <= 1e-12 * max(1.0, np.abs(ref).max())
    ctx.close()
