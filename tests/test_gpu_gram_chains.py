"""Length of the FP32 sums of the complex64 Gram.  Every row adds 1 to every
output but one row, which adds 2^27: an FP32 sum that has met it drops the ones
that follow (even four of them at once are half a unit in its last place), so
the ones missing from the result are the rows that went into one FP32 sum after
it.  At most 128 rows may, whatever the number of K chunks; a further sum of such
partial sums in FP32 rounds by at most half of 2^27's unit of 16 for each
partial sum of less than 128 rows (the chunk's last)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CHAIN = 192


@pytest.mark.parametrize("K,p,q", [(300, 70, 70), (2000, 300, 200), (4200, 748, 64), (11401, 256, 23), (34181, 1, 1),
                                   (34181, 128, 64), (34181, 192, 192), (34181, 432, 64), (34181, 512, 512),
                                   (82561, 748, 64)])
def test_fp32_sums_stay_short(torch_cuda, K, p, q):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    ws = torch.empty((256 << 20) + 256, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:])
    B = torch.ones((q, K), dtype=torch.complex64, device="cuda")
    C = torch.empty((q, p), dtype=torch.complex128, device="cuda")
    for at in (0, 7, K // 3, K // 2 + 1, K - 150):
        A = torch.ones((p, K), dtype=torch.complex64, device="cuda")
        A[:, at] = 2.0 ** 27
        ctx.gram(A, B, C)
        got = C.cpu().numpy()
        assert (got.imag == 0.0).all()
        missing = 2.0 ** 27 + K - 1 - got.real
        assert missing.max() <= CHAIN + 16 and missing.min() >= -16, (at, missing.min(), missing.max())
    ctx.close()
