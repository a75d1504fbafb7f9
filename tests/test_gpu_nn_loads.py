"""Loads of the row-block matrix product Y = A C: whole and last k-blocks, rows and
columns past the operands (leading dimensions padded with NaN, which must not
reach a result), the upper row blocks of long operands, and a coefficient
matrix whose leading dimension leaves the short offsets.  Against a complex128
product; rounding bound of p products and sums in the block's type, twice for the
three-multiplication form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx64", [False, True])
@pytest.mark.parametrize("K,p,q,pad,ldc", [
    (16, 1, 1, 0, 0), (17, 15, 17, 3, 0), (100, 16, 64, 0, 2), (33, 33, 65, 1, 5), (1201, 48, 16, 0, 0),
    (40003, 17, 64, 2, 1), (34208, 31, 40, 0, 0), (70001, 32, 5, 0, 0), (257, 35, 3, 0, 1 << 20)])
def test_nn_loads(torch_cuda, K, p, q, pad, ldc, cplx64):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    dt = torch.complex64 if cplx64 else torch.complex128
    g = torch.Generator(device="cuda").manual_seed(K + p)
    nan = float("nan")
    A = torch.full((p, K + pad), nan, dtype=dt, device="cuda")
    A[:, :K] = torch.randn(p, K, dtype=dt, device="cuda", generator=g)
    C = torch.full((q, p + ldc), nan, dtype=torch.complex128, device="cuda")
    C[:, :p] = torch.randn(q, p, dtype=torch.complex128, device="cuda", generator=g)
    Y = torch.full((q, K + pad), 7.0, dtype=dt, device="cuda")
    ctx.block_update(A[:, :K], C[:, :p], Y[:, :K])
    out = Y.cpu().numpy()
    assert np.all(out[:, K:] == 7.0)
    a, c = A[:, :K].cpu().numpy().astype(complex), C[:, :p].cpu().numpy()
    if cplx64:
        c = c.astype(np.complex64).astype(complex)
    eps = np.finfo(np.float32 if cplx64 else np.float64).eps
    err = np.abs(out[:, :K] - c @ a)
    bound = 2 * (p + 4) * eps * (np.abs(c) @ np.abs(a))
    assert np.all(err <= bound)
    ctx.close()
