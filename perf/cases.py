"""Performance cases of the plane-wave block-LOBPCG library.

Each case is one piece of work a program has the library do, through the ctypes
binding's public calls, from the smallest cells (where launches and latency
count) to the largest served one:

  apply      Y = H X of one k-point (pw_apply_H): an SCF or spectrum program's
             operator, FP64 or complex64 (the mixed form's blocks)
  kpoints    the same for several k-points of one cell at once (pw_apply_H_batch)
  ritz       a Rayleigh-Ritz step as a caller writes it from the building blocks:
             Gram of the basis with H times the basis, lowest eigenpairs, rotation
  rotate     rotation of a complex64 basis and of H times it (pw_block_update_mixed)
  directions new search directions: residuals and preconditioner, then CholQR
             (Gram, factor, right multiply)
  density    electron density of the bands (pw_density)
  solve      the whole eigensolve and the density of its bands, as a
             self-consistent program calls them (pw_lobpcg_solve, pw_density);
             the vectors' phases are free, the density is not

Cells are cubes with Gaussian wells of depth 2 Ha and width 1 bohr and four
Kleinman-Bylander projectors per well, as in the repository's workloads.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_0707_3405_amd import PW_PREC_FP64, PW_PREC_MIXED
from paper_0707_3405_amd._binding import Context, apply_H_batch

DEV = "cuda:0"
LM4 = ((0, 0), (1, -1), (1, 0), (1, 1))
FFT_SIZES = (16, 20, 24, 32, 36, 40, 48, 60, 64, 72, 80, 96, 108, 120, 128)
PREC = {"fp64": PW_PREC_FP64, "mixed": PW_PREC_MIXED}


# ---- the cases ---------------------------------------------------------------
def listed():
    tiny = dict(L=8.0, ecut=4.0, n=20, natom=2, kx=0.1, ky=0.2, kz=0.3)
    mid = dict(L=12.0, ecut=8.0, n=36, natom=6, kx=0.25, ky=0.0, kz=0.5)
    kpts = dict(L=16.0, ecut=15.0, n=72, natom=64)
    paper = dict(L=20.0, ecut=20.0, n=96, natom=108, kx=0.25, ky=0.25, kz=0.25)
    largest = dict(L=24.0, ecut=25.0, n=120, natom=187, kx=0.3, ky=0.1, kz=0.7)
    return [
        # one small block of the smallest cell: launches and latency
        dict(name="apply_tiny", kind="apply", prec="fp64", nb=4, **tiny),
        # the solver's block of 64 on the 108-well cell, in both block types
        dict(name="apply_108", kind="apply", prec="fp64", nb=64, **paper),
        dict(name="apply_108_c64", kind="apply", prec="mixed", nb=64, **paper),
        # the largest served cell (82561 plane waves, 748 projectors)
        dict(name="apply_187", kind="apply", prec="fp64", nb=64, **largest),
        # four k-points of the 64-well cell, a partly converged block of 23
        dict(name="kpoints_64", kind="kpoints", prec="fp64", nb=23, nk=4, **kpts),
        # the Rayleigh-Ritz step of one full iteration at the 108-well cell
        dict(name="ritz_iter", kind="ritz", npw=34181, n=192, k=64),
        # the final Rayleigh-Ritz over every band of that cell
        dict(name="ritz_final", kind="ritz", npw=34181, n=512, k=512),
        # rotation in the mixed form, a ragged active set at one k-point
        dict(name="rotate_c64", kind="rotate", npw=11401, n=83, k=58),
        # residuals, preconditioner and CholQR of a full block
        dict(name="directions_108", kind="directions", nb=64, **paper),
        # the density of an occupied half of the 108-well cell's bands
        dict(name="density_108", kind="density", nb=256, **paper),
        # a whole small solve, and the lowest bands of the 108-well cell
        dict(name="solve_small", kind="solve", nbands=48, block=16, tol=1e-7, **mid),
        dict(name="solve_108", kind="solve", nbands=96, block=64, tol=1e-6, **paper),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _cell(rng, L_hi, ecut_hi):
    """A cell as the serving rule builds it: wells by volume, the grid by the sphere."""
    L = round(_log_uniform(rng, 8.0, L_hi), 3)
    ecut = round(_log_uniform(rng, 4.0, ecut_hi), 3)
    nmax = math.ceil(L * math.sqrt(2.0 * ecut) / (2 * math.pi) + 1.0)
    n = next(s for s in FFT_SIZES if s >= 4 * nmax + 1)
    natom = max(1, round(0.0135 * L ** 3))
    k = [round(rng.uniform(0.02, 0.98), 4) for _ in range(3)]
    return dict(L=L, ecut=ecut, n=n, natom=natom, kx=k[0], ky=k[1], kz=k[2])


def draw(rng):
    kind = rng.choice(("apply", "apply", "apply", "kpoints", "ritz", "ritz", "rotate", "directions",
                       "density", "solve"))
    if kind == "apply":
        return dict(kind=kind, prec=rng.choice(("fp64", "mixed")), nb=round(_log_uniform(rng, 1, 64)),
                    **_cell(rng, 23.5, 24.0))
    if kind == "kpoints":
        c = _cell(rng, 16.0, 15.0)
        for key in ("kx", "ky", "kz"):
            del c[key]
        return dict(kind=kind, prec=rng.choice(("fp64", "mixed")), nb=rng.randint(1, 32), nk=rng.randint(2, 6), **c)
    if kind == "ritz":
        npw = round(_log_uniform(rng, 600, 34000))
        if rng.random() < 0.25:   # a final Rayleigh-Ritz: every pair of the bands
            n = round(_log_uniform(rng, 16, min(500, npw // 4)))
            return dict(kind=kind, npw=npw, n=n, k=n)
        k = round(_log_uniform(rng, 2, 64))
        return dict(kind=kind, npw=npw, n=k + rng.randint(1, 2 * k), k=k)
    if kind == "rotate":
        k = rng.randint(2, 64)
        return dict(kind=kind, npw=round(_log_uniform(rng, 600, 82000)), n=k + rng.randint(1, 2 * k),
                    k=k + rng.randint(0, k))
    if kind == "directions":
        return dict(kind=kind, nb=rng.randint(1, 64), **_cell(rng, 23.5, 24.0))
    if kind == "density":
        return dict(kind=kind, nb=round(_log_uniform(rng, 1, 250)), **_cell(rng, 20.0, 20.0))
    c = _cell(rng, 12.0, 8.0)
    block = rng.choice((16, 32))
    return dict(kind="solve", nbands=rng.randint(block, 48), block=block, tol=1e-7, **c)


# ---- inputs ------------------------------------------------------------------
def _kfrac(case, i=0):
    if "kx" in case:
        return (case["kx"], case["ky"], case["kz"])
    # k-points of a regular mesh, away from points of high symmetry
    return (0.03 + 0.25 * (i % 2), 0.07 + 0.25 * (i // 2 % 2), 0.11 + 0.25 * (i // 4))


def _sphere(case, kfrac):
    """Miller indices [npw, 3] and k + G vectors [npw, 3] in the library's order
    (lexicographic), 1/2 |k+G|^2 <= ecut."""
    b = 2.0 * math.pi / case["L"]
    lim = math.ceil(math.sqrt(2.0 * case["ecut"]) / b) + 2
    ax = np.arange(-lim, lim + 1)
    m = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    q = (m + np.asarray(kfrac)) * b
    keep = 0.5 * (q * q).sum(1) <= case["ecut"]
    return m[keep], q[keep]


def _rng(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _crandn(gen, *shape):
    return torch.randn(*shape, dtype=torch.complex128, device=DEV, generator=gen)


def _wells(case, seed):
    """Well positions (fcc sites with jitter where the count allows, else uniform) and couplings."""
    rng = np.random.default_rng(int(seed))
    L, na = case["L"], case["natom"]
    reps = round((na / 4) ** (1 / 3))
    if na == 4 * reps ** 3:
        cells = np.stack(np.meshgrid(*[np.arange(reps)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
        basis = np.array([[0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]])
        pos = ((cells + basis) * (L / reps)).reshape(-1, 3) + rng.uniform(-0.2, 0.2, (na, 3))
        pos = np.mod(pos, L)
    else:
        pos = rng.uniform(0.0, L, (na, 3))
    return pos, rng.uniform(0.5, 1.5, na * len(LM4))


def _potential(case, pos):
    """Periodic sum of the wells on the grid, [x][y][z]."""
    L, n = case["L"], case["n"]
    x = torch.arange(n, dtype=torch.float64, device=DEV) * (L / n)
    t = torch.arange(-3, 4, dtype=torch.float64, device=DEV) * L
    p = torch.from_numpy(pos).to(DEV)
    g = torch.exp(-0.5 * (x[None, None, :, None] - p[:, :, None, None] - t) ** 2).sum(-1)   # [atom, axis, n]
    yz = (g[:, 1, :, None] * g[:, 2, None, :]).reshape(len(pos), n * n)
    return (-2.0 * (g[:, 0].T.contiguous() @ yz)).reshape(n, n, n).contiguous()


def _projectors(case, q, pos):
    """Projector table [nproj, npw]: Gaussian s and p projectors at every well."""
    q = torch.from_numpy(q).to(DEV)
    q2 = (q * q).sum(1)
    pref = math.sqrt(32.0 * math.pi ** 2.5) / math.sqrt(case["L"] ** 3)
    rad = pref * torch.exp(-0.5 * q2)
    qn = q2.sqrt()
    unit = torch.where(qn[:, None] > 0, q / qn.clamp_min(1e-300)[:, None], torch.zeros_like(q))
    c1 = math.sqrt(3.0 / (4.0 * math.pi))
    y = torch.stack([torch.full_like(qn, 0.5 / math.sqrt(math.pi)), c1 * unit[:, 1], c1 * unit[:, 2],
                     c1 * unit[:, 0]])                      # LM4 order: 00, 1-1 (y), 10 (z), 11 (x)
    ph = torch.from_numpy(pos).to(DEV) @ q.T                # [atom, npw]
    e = torch.polar(torch.ones_like(ph), -ph)
    return (e[:, None, :] * (rad * y)[None]).reshape(-1, q.shape[0])


def _context(case, seed, kfrac, nbands, block, prec, stream=None):
    pos, D = _wells(case, seed)
    ctx = Context(0, stream)
    ctx.init_basis(np.eye(3) * case["L"], kfrac, case["ecut"], (case["n"],) * 3)
    ctx.set_local_potential(_potential(case, pos))
    ctx.set_projectors(pos, LM4, D)
    ctx.alloc_workspace(nbands, block, prec)
    return ctx


def _bands(gen, nb, kin):
    """Random bands damped towards low kinetic energy, unit norm, [nb, npw]."""
    x = _crandn(gen, nb, kin.numel()) / (1.0 + kin)
    return x / torch.linalg.vector_norm(x, dim=1, keepdim=True)


def _kin(q):
    return torch.from_numpy(0.5 * (q * q).sum(1)).to(DEV)


def _apply_inputs(case, seed):
    """Per k-point: (miller, q, X) of the block H is applied to."""
    gen, out = _rng(seed), []
    for i in range(case.get("nk", 1)):
        m, q = _sphere(case, _kfrac(case, i))
        x = _bands(gen, case["nb"], _kin(q))
        out.append((m, q, x if case["prec"] == "fp64" else x.to(torch.complex64)))
    return out


def _ritz_inputs(case, seed):
    """Orthonormal basis Z [n, npw] of columns with different decay, and H Z for a
    diagonal H with a spectrum like the kinetic energies'."""
    gen = _rng(seed)
    npw, n = case["npw"], case["n"]
    t = 20.0 * torch.rand(npw, dtype=torch.float64, device=DEV, generator=gen) ** (2.0 / 3.0)
    s = torch.rand(n, 1, dtype=torch.float64, device=DEV, generator=gen)
    z = _crandn(gen, n, npw) * torch.exp(-t * s)
    for _ in range(2):   # Cholesky QR, twice
        z = z / torch.linalg.vector_norm(z, dim=1, keepdim=True)
        r = torch.linalg.cholesky(z.conj() @ z.T)
        z = torch.linalg.solve_triangular(r.conj(), z, upper=False)
    return z.contiguous(), (z * t).contiguous()


def _rotate_inputs(case, seed):
    gen = _rng(seed)
    z = _crandn(gen, case["n"], case["npw"]).to(torch.complex64)
    hz = _crandn(gen, case["n"], case["npw"]).to(torch.complex64)
    c = _crandn(gen, case["k"], case["n"]) / math.sqrt(case["n"])
    return z, hz, c


def _directions_inputs(case, seed):
    gen = _rng(seed)
    _, q = _sphere(case, _kfrac(case))
    kin = _kin(q)
    x = _bands(gen, case["nb"], kin)
    hx = x * (kin - 5.0) + 0.5 * _bands(gen, case["nb"], kin)   # H X of unconverged bands
    return kin, x, hx


def _density_inputs(case, seed):
    gen = _rng(seed)
    m, q = _sphere(case, _kfrac(case))
    x = _bands(gen, case["nb"], _kin(q))
    occ = np.random.default_rng(int(seed)).uniform(0.0, 2.0, case["nb"])
    return m, x, occ


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, kind=kind)
    if kind in ("apply", "kpoints"):
        prec, nb = PREC[case["prec"]], case["nb"]
        ins = _apply_inputs(case, seed)
        st["ctxs"] = [_context(case, seed, _kfrac(case, i), nb, nb, prec) for i in range(len(ins))]
        st["X"] = [x for _, _, x in ins]
        st["Y"] = [torch.empty_like(x) for x in st["X"]]
        st["prec"] = prec
    elif kind == "ritz":
        n, k = case["n"], case["k"]
        st["Z"], st["HZ"] = _ritz_inputs(case, seed)
        st["ctx"] = _block_context(n)
        st["A"] = torch.empty((n, n), dtype=torch.complex128, device=DEV)
        st["w"] = torch.empty(k, dtype=torch.float64, device=DEV)
        st["V"] = torch.empty((k, n), dtype=torch.complex128, device=DEV)
        st["X"] = torch.empty((k, case["npw"]), dtype=torch.complex128, device=DEV)
    elif kind == "rotate":
        st["Z"], st["HZ"], st["C"] = _rotate_inputs(case, seed)
        st["ctx"] = _block_context(case["n"])
        st["X"] = torch.empty((case["k"], case["npw"]), dtype=torch.complex64, device=DEV)
        st["HX"] = torch.empty_like(st["X"])
    elif kind == "directions":
        nb = case["nb"]
        _, st["X"], st["HX"] = _directions_inputs(case, seed)
        ctx = st["ctx"] = Context(0)
        ctx.init_basis(np.eye(3) * case["L"], _kfrac(case), case["ecut"], (case["n"],) * 3)
        ctx.alloc_workspace(nb, nb)
        st["theta"], st["res"] = (torch.empty(nb, dtype=torch.float64, device=DEV) for _ in range(2))
        st["W"], st["Q"] = torch.empty_like(st["X"]), torch.empty_like(st["X"])
        st["G"], st["R"] = (torch.empty((nb, nb), dtype=torch.complex128, device=DEV) for _ in range(2))
    elif kind == "density":
        _, st["X"], st["occ"] = _density_inputs(case, seed)
        ctx = st["ctx"] = Context(0)
        ctx.init_basis(np.eye(3) * case["L"], _kfrac(case), case["ecut"], (case["n"],) * 3)
        ctx.alloc_workspace(case["nb"], min(64, case["nb"]))
        st["rho"] = torch.empty((case["n"],) * 3, dtype=torch.float64, device=DEV)
    else:
        ctx = st["ctx"] = _context(case, seed, _kfrac(case), case["nbands"], case["block"], PW_PREC_FP64)
        st["X"] = torch.zeros((case["nbands"], ctx.npw), dtype=torch.complex128, device=DEV)
        j = np.arange(case["nbands"])   # smeared occupation, empty towards the top band
        st["occ"] = 2.0 / (1.0 + np.exp((j + 1 - 0.7 * len(j)) / (0.05 * len(j))))
        st["rho"] = torch.empty((case["n"],) * 3, dtype=torch.float64, device=DEV)
    return st


def _block_context(n):
    """A context for the building blocks on bases of up to n columns: any basis,
    and a workspace with room for the split Gram and the eigensolver."""
    ctx = Context(0)
    ctx.init_basis(np.eye(3) * 8.0, (0.1, 0.2, 0.3), 4.0, (20, 20, 20))
    nbytes = max(64 << 20, 256 * n * n * 16)
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEV)
    ctx.set_workspace(ws[(-ws.data_ptr()) % 256:][:nbytes])
    return ctx


# ---- one pass ----------------------------------------------------------------
def run(st):
    kind = st["kind"]
    if kind == "apply":
        st["ctxs"][0].apply_H(st["X"][0], st["Y"][0], prec=st["prec"])
        return st["Y"][0]
    if kind == "kpoints":
        return apply_H_batch(st["ctxs"], st["X"], st["Y"], prec=st["prec"])
    ctx = st["ctx"]
    if kind == "ritz":
        n, k = st["case"]["n"], st["case"]["k"]
        ctx.gram(st["Z"], st["HZ"], st["A"])
        ctx.small_eigh(st["A"], n, k, st["w"], st["V"])
        ctx.block_update(st["Z"], st["V"], st["X"])
        return dict(w=st["w"], V=st["V"], X=st["X"])
    if kind == "rotate":
        ctx.block_update(st["Z"], st["C"], st["X"])
        ctx.block_update(st["HZ"], st["C"], st["HX"])
        return dict(X=st["X"], HX=st["HX"])
    if kind == "directions":
        nb = st["case"]["nb"]
        ctx.residuals(st["X"], st["HX"], nb, st["theta"], st["res"], st["W"])
        ctx.gram(st["W"], st["W"], st["G"])
        ctx.chol_inv(st["G"], nb, st["R"])
        ctx.block_update(st["W"], st["R"], st["Q"])
        return dict(theta=st["theta"], res=st["res"], W=st["W"], R=st["R"], Q=st["Q"])
    if kind == "density":
        return ctx.density(st["X"], st["occ"], st["rho"])
    eig, _ = ctx.lobpcg_solve(st["case"]["nbands"], st["case"]["block"], st["case"]["tol"], 300, st["X"])
    return dict(eig=eig, rho=ctx.density(st["X"], st["occ"], st["rho"]))


# ---- what a pass cannot do without -------------------------------------------
def _fft_flops(case):
    """One transform pruned to the sphere: sticks along z, kept columns along y, rows along x."""
    n = case["n"]
    r = case["L"] * math.sqrt(2.0 * case["ecut"]) / (2 * math.pi)
    return 5.0 * n * math.log2(n) * (math.pi * r * r + (2 * r + 1) * n + n * n)


def _npw(case):
    return (case["L"] * math.sqrt(2.0 * case["ecut"]) / (2 * math.pi)) ** 3 * 4.0 * math.pi / 3.0


def _apply_work(case, nb, e):
    npw, nproj, n3 = _npw(case), 4 * case["natom"], case["n"] ** 3
    return (npw * nb * 2 * e + npw * nproj * e + n3 * e / 2,
            nb * (2 * _fft_flops(case) + 16.0 * npw * nproj))


def work(case):
    kind = case["kind"]
    if kind in ("apply", "kpoints"):
        nk = case.get("nk", 1)
        b, f = _apply_work(case, case["nb"], 16 if case["prec"] == "fp64" else 8)
        v = case["n"] ** 3 * (8 if case["prec"] == "fp64" else 4)
        return dict(bytes=nk * (b - v) + v, flops=nk * f)
    if kind == "ritz":
        K, n, k = case["npw"], case["n"], case["k"]
        return dict(bytes=16.0 * (K * (2 * n + k) + n * k), flops=8.0 * K * n * (n / 2 + k) + 16 / 3 * n ** 3 + 8.0 * n * n * k)
    if kind == "rotate":
        K, n, k = case["npw"], case["n"], case["k"]
        return dict(bytes=2 * 8.0 * K * (n + k) + 16.0 * n * k, flops=2 * 8.0 * K * n * k)
    if kind == "directions":
        nb, npw = case["nb"], _npw(case)
        return dict(bytes=npw * nb * 16.0 * 4 + 16.0 * nb * nb, flops=npw * nb * (30 + 12.0 * nb))
    if kind == "density":
        n3 = case["n"] ** 3
        return dict(bytes=_npw(case) * case["nb"] * 16.0 + n3 * 8.0, flops=case["nb"] * (_fft_flops(case) + 4.0 * n3))
    # a solve: about ten iterations a block, each one apply and one Rayleigh-Ritz
    npw, m = _npw(case), case["block"]
    its = 10.0 * math.ceil(case["nbands"] / (m - m // 5))
    b, f = _apply_work(case, m, 16)
    return dict(bytes=its * (b + npw * 16.0 * 12 * m) + case["n"] ** 3 * 8.0,
                flops=its * (f + 8.0 * npw * m * m * 20) + case["nbands"] * _fft_flops(case))


# ---- the same in 64 bits from torch alone ------------------------------------
def _on_grid(m, n):
    i = torch.from_numpy(np.mod(m, n)).to(DEV)
    return (i[:, 0] * n + i[:, 1]) * n + i[:, 2]


def _apply_exact(case, seed):
    pos, D = _wells(case, seed)
    v = _potential(case, pos)
    n, d, out = case["n"], torch.from_numpy(D).to(DEV), []
    for m, q, x in _apply_inputs(case, seed):
        x = x.to(torch.complex128)
        at, kin = _on_grid(m, n), _kin(q)
        y = torch.empty_like(x)
        for j in range(x.shape[0]):
            g = torch.zeros(n ** 3, dtype=torch.complex128, device=DEV)
            g[at] = x[j]
            r = torch.fft.ifftn(g.view(n, n, n)) * v
            y[j] = torch.fft.fftn(r).reshape(-1)[at] + kin * x[j]
        b = _projectors(case, q, pos)
        c = (b.conj() @ x.T) * d[:, None]
        out.append(y + (b.T.contiguous() @ c).T)
    return out


def _dense_eigenvalues(case, seed):
    """Lowest eigenvalues of the dense Galerkin matrix."""
    pos, D = _wells(case, seed)
    m, q = _sphere(case, _kfrac(case))
    n = case["n"]
    vt = torch.fft.fftn(_potential(case, pos)).cpu().numpy() / n ** 3
    i = np.mod(m[:, None, :] - m[None, :, :], n)
    h = vt[i[..., 0], i[..., 1], i[..., 2]]
    b = _projectors(case, q, pos).cpu().numpy()
    h += (b.T * D) @ b.conj()
    h[np.diag_indices(len(m))] += 0.5 * (q * q).sum(1)
    return np.linalg.eigvalsh(h)[:case["nbands"]]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("apply", "kpoints"):
        out = _apply_exact(case, seed)
        return out[0] if kind == "apply" else out
    if kind == "ritz":
        z, hz = _ritz_inputs(case, seed)
        a = (z.conj() @ hz.T).cpu().numpy()
        # vectors are fixed up to a phase only: no value of their own
        return dict(w=np.linalg.eigvalsh(0.5 * (a + a.conj().T))[:case["k"]], V=None, X=None)
    if kind == "rotate":
        z, hz, c = _rotate_inputs(case, seed)
        return dict(X=c @ z.to(torch.complex128), HX=c @ hz.to(torch.complex128))
    if kind == "directions":
        kin, x, hx = _directions_inputs(case, seed)
        theta = (x.conj() * hx).sum(1).real
        r = hx - theta[:, None] * x
        t = kin / (kin * x.abs() ** 2).sum(1, keepdim=True).clamp_min(1e-3)
        num = 27.0 + 18.0 * t + 12.0 * t ** 2 + 8.0 * t ** 3
        w = r * (num / (num + 16.0 * t ** 4))
        g = w.conj() @ w.T
        nb = case["nb"]
        shift = 1e-15 * nb * g.diagonal().real.max()   # the factor's documented diagonal shift
        low = torch.linalg.cholesky(g + shift * torch.eye(nb, dtype=g.dtype, device=DEV))   # G = L L^H, R = L^H
        rinv = torch.linalg.solve_triangular(low, torch.eye(nb, dtype=g.dtype, device=DEV), upper=False).mH
        rinv = rinv.contiguous()
        return dict(theta=theta, res=torch.linalg.vector_norm(r, dim=1), W=w, R=rinv.T.contiguous(),
                    Q=rinv.T.contiguous() @ w)
    if kind == "density":
        m, x, occ = _density_inputs(case, seed)
        n = case["n"]
        at = _on_grid(m, n)
        rho = torch.zeros((n, n, n), dtype=torch.float64, device=DEV)
        for j in range(x.shape[0]):
            g = torch.zeros(n ** 3, dtype=torch.complex128, device=DEV)
            g[at] = x[j]
            r = torch.fft.ifftn(g.view(n, n, n)) * float(n) ** 3
            rho += float(occ[j]) * (r.real ** 2 + r.imag ** 2)
        return rho / case["L"] ** 3
    if _npw(case) < 2200:
        return dict(eig=_dense_eigenvalues(case, seed), rho=None)   # rho carries the solve's tolerance
    return None
