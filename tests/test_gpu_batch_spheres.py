"""pw_apply_H_batch over k-points of which some have their sphere inside the
middle half of the grid and some reach beyond it gives every context's
pw_apply_H bitwise, in every order of the contexts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec_name", [(32, "fp64"), (48, "mixed"), (96, "fp64"), (96, "mixed"), (128, "fp64")])
def test_spheres_on_both_sides_of_the_middle_half(torch_cuda, n, prec_name):
    torch = torch_cuda
    from paper_0707_3405_amd import Context, apply_H_batch, PW_PREC_FP64, PW_PREC_MIXED
    prec = PW_PREC_FP64 if prec_name == "fp64" else PW_PREC_MIXED
    rng = np.random.default_rng(n)
    v = rng.standard_normal((n, n, n))
    r = n // 4 - 0.3   # inside at k = 0, one plane of points beyond at k = -1/2
    nb, ctxs, Xs, sides = 5, [], [], []
    for k in ((0.0, 0.01, 0.02), (-0.5, 0.0, 0.0), (0.03, -0.5, 0.0), (0.0, 0.1, 0.4)):
        ctx = Context(0)
        npw = ctx.init_basis(np.eye(3) * 2 * np.pi, k, 0.5 * r * r, (n, n, n))
        xy = ctx.get_miller()[:, :2]
        sides.append(bool((xy >= -n // 4).all() and (xy < n // 4).all()))
        ctx.set_local_potential(v)
        ctx.alloc_workspace(8, 8, prec)
        x = rng.standard_normal((nb, npw)) + 1j * rng.standard_normal((nb, npw))
        ctxs.append(ctx)
        Xs.append(torch.from_numpy(x).cuda().to(torch.complex128 if prec == PW_PREC_FP64 else torch.complex64))
    assert True in sides and False in sides, sides
    alone = [torch.empty_like(X) for X in Xs]
    for c, X, Y in zip(ctxs, Xs, alone):
        c.apply_H(X, Y, prec=prec)
    for order in ((0, 1, 2, 3), (1, 0, 3, 2), (2, 3), (3, 0), (1, 2)):
        Ys = [torch.empty_like(Xs[i]) for i in order]
        apply_H_batch([ctxs[i] for i in order], [Xs[i] for i in order], Ys, prec=prec)
        torch.cuda.synchronize()
        for i, Y in zip(order, Ys):
            assert torch.equal(Y.view(torch.uint8), alone[i].view(torch.uint8)), (order, i)   # signs of zeros too
    for c in ctxs:
        c.close()
