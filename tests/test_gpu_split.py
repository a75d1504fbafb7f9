"""The work split of the two block products at its edges, FP64 and complex64:
chunk lengths of the split-K Gram (one k-block, the 3-, 5- and 8-block rules, one
and two tiles, more tiles than slots, tuned caps, a small workspace) and row
ranges of the update (fewer row blocks than workgroups, one round, several,
more column tiles than a round), against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _blocks(K, p, q, dtype):
    rng = np.random.default_rng(K + 3 * p + 7 * q)
    f = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(dtype)
    return f(p, K), f(q, K), rng.standard_normal((q, p)) + 1j * rng.standard_normal((q, p))


# relative to the norms of the rows and columns: the bars of the per-step tests
TOL = {np.complex128: 1e-14, np.complex64: 5e-6}


@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("K,p,q,cap,ws_mb", [
    (1, 1, 1, 0, 64), (15, 65, 3, 0, 64), (16, 64, 64, 0, 64), (17, 2, 129, 0, 64), (1023, 64, 64, 0, 64),
    (1030, 100, 7, 0, 64), (8192, 60, 64, 0, 64), (8209, 65, 64, 0, 64), (20000, 130, 70, 0, 256),
    (2000, 1500, 1500, 0, 64), (5000, 96, 80, 1, 64), (5000, 96, 80, 1024, 256), (5000, 96, 80, 0, 1)])
def test_gram_splits(torch_cuda, dtype, K, p, q, cap, ws_mb):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    ws = torch.empty((ws_mb << 20) + 256, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:][:ws_mb << 20])
    if cap:
        ctx.set_tuning(gemm_split_workgroups=cap)
    A, B, _ = _blocks(K, p, q, dtype)
    C = torch.full((q, p), complex(np.nan, np.nan), dtype=torch.complex128, device="cuda")
    ctx.gram(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), C)
    ref = A.astype(np.complex128).conj() @ B.astype(np.complex128).T
    scale = np.linalg.norm(A, axis=1)[:, None] * np.linalg.norm(B, axis=1)[None, :]
    err = np.abs(C.cpu().numpy().T - ref) / scale
    assert err.max() <= TOL[dtype], err.max()
    ctx.close()


@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("K,p,q", [(1, 1, 1), (16, 5, 64), (33, 64, 65), (8191, 20, 64), (8193, 20, 64),
                                   (40977, 17, 16), (13000, 33, 300), (300, 9, 40000)])
def test_update_ranges(torch_cuda, dtype, K, p, q):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    A, Y, Cm = _blocks(K, p, q, dtype)
    Yd = torch.from_numpy(Y).cuda()
    ctx.block_update(torch.from_numpy(A).cuda(), torch.from_numpy(Cm).cuda(), Yd, alpha=-1.0, beta=1.0)
    ref = Y.astype(np.complex128) - (A.astype(np.complex128).T @ Cm.T).T
    scale = np.linalg.norm(A, axis=0)[None, :] * np.linalg.norm(Cm, axis=1)[:, None] + np.abs(Y)
    err = np.abs(Yd.cpu().numpy() - ref) / scale
    assert err.max() <= TOL[dtype], err.max()
    ctx.close()
