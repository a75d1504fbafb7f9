"""Every row of the contraction enters the Gram once, whatever the chunks of K and
the FP32 runs within them: small whole numbers, whose sums are exact in FP32 and
FP64, give the exact product.  Sizes on both sides of each line of the split
rule (one- and two-block chunks up to half of the compute units, three blocks,
one to three workgroups per unit, 16 k-blocks and 16 runs in complex64, a
partial last block), tuned caps and a workspace for few partials."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (17, 3, 2), (255, 700, 500), (256, 748, 64), (257, 748, 64), (2047, 5, 5), (2049, 60, 64),
         (4095, 64, 64), (4099, 64, 64), (6200, 64, 3), (1030, 128, 64), (1900, 192, 64), (3000, 130, 130), (3070, 512, 512),
         (3100, 512, 512), (5200, 432, 64), (11401, 128, 64), (11401, 192, 192), (20011, 192, 64), (34181, 70, 1),
         (40000, 432, 64), (82561, 130, 129)]


@pytest.mark.parametrize("dtype_name", ["complex128", "complex64"])
@pytest.mark.parametrize("K,p,q", SIZES)
def test_gram_of_whole_numbers_is_exact(torch_cuda, K, p, q, dtype_name):
    torch = torch_cuda
    from paper_0707_3405_amd import Context
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    ws = torch.empty((256 << 20) + 256, dtype=torch.uint8, device="cuda")
    off = (-ws.data_ptr()) % 256
    ctx.set_workspace(ws[off:][:256 << 20])
    rng = np.random.default_rng(K + 3 * p + 7 * q)
    f = lambda m: torch.from_numpy(rng.integers(-2, 3, (m, K)) + 1j * rng.integers(-2, 3, (m, K))).cuda()
    A, B = f(p), f(q)
    # |sum| <= 8 K and the sums of the three products of the complex form <= 16 K, below 2^24
    ref = torch.conj(A).resolve_conj()
    ref = B @ ref.T.contiguous()
    A, B = A.to(getattr(torch, dtype_name)), B.to(getattr(torch, dtype_name))
    for cap, ws_mb in ((0, 256), (1, 256), (24, 256), (1024, 256), (0, max(1, -(-p * q * 16 * 3 >> 20)))):
        ctx.set_tuning(gemm_split_workgroups=cap)
        ctx.set_workspace(ws[off:][:ws_mb << 20])
        C = torch.full((q, p), float("nan"), dtype=torch.complex128, device="cuda")
        ctx.gram(A, B, C)
        assert torch.equal(C, ref), (cap, ws_mb)
    ctx.close()
