"""A host-only context sizes the workspace at every FFT size, for small spheres and
for the widest the grid holds, without asking a device."""
import numpy as np
import pytest


@pytest.mark.parametrize("n", [16, 20, 24, 32, 36, 40, 48, 60, 64, 72, 80, 96, 108, 120, 128])
def test_workspace_size_needs_no_device(n):
    from paper_0707_3405_amd import Context, PW_PREC_MIXED
    for r in (n / 4 - 0.6, min((n - 1) / 2, 38.0)):
        ctx = Context(-1)
        npw = ctx.init_basis(np.eye(3) * 2 * np.pi, (0.02, 0.03, -0.01), 0.5 * r * r, (n, n, n))
        last = 0
        for nb in (1, 5, 16, 40):
            if nb + 3 * nb > npw:
                break
            size = ctx.workspace_size(nb, nb)
            assert size >= n ** 3 * 8 and size > last
            assert ctx.workspace_size(nb, nb, PW_PREC_MIXED) >= size
            last = size
        ctx.close()
