"""gemm_split_workgroups is a cap: a value at or above what the default takes
changes nothing (the Gram's bits show its K chunks), one below it takes fewer
chunks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype_name", ["complex128", "complex64"])
@pytest.mark.parametrize("K,p,q", [(34181, 16, 16), (34181, 64, 64), (34181, 128, 64), (20000, 128, 128), (3000, 200, 64)])
def test_split_cap(torch_cuda, dtype_name, K, p, q):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    ws = torch.empty((128 << 20) + 256, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:])
    rng = np.random.default_rng(K + p)
    f = lambda m: torch.from_numpy(rng.standard_normal((m, K)) + 1j * rng.standard_normal((m, K))).cuda().to(
        getattr(torch, dtype_name))
    A, B = f(p), f(q)

    def gram(cap):
        ctx.set_tuning(gemm_split_workgroups=cap)
        C = torch.empty((q, p), dtype=torch.complex128, device="cuda")
        ctx.gram(A, B, C)
        return C
    default = gram(0)
    for cap in (768, 1024):
        assert torch.equal(gram(cap), default), cap
    assert not torch.equal(gram(8), default)
    ctx.close()
