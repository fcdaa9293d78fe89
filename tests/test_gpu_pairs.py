"""The two-stage pair form (W of every pair of a block through a batch buffer, then the sums)
at the sizes where its blocks and tiles end: one field, a target tile (8 fields) less and more
than full, a group of 64 fields and one more, several rows of blocks with rectangles beside
the triangle, k-points whose bands end inside a tile, more than 16 bands (two FP32 partial
sums per k-point). Every k-point against torch's complex128 FFTs over the oracle's kernel
tables, with u as targets and sources (each pair transformed once) and with separate targets
(one-sided).

The tolerances are the forms' stated ones, per k-point: 1e-6 in FP32, 1e-10 in FP64."""

import os

import numpy as np
import pytest

from paper_1507_05156_amd import synth

pytestmark = pytest.mark.gpu

OMEGA = synth.OMEGA_HSE


def make(n, mesh, nb, prec, cap=None):
    from paper_1507_05156_amd.api import Plan
    cell = synth.cubic_cell()
    kp = synth.gamma_mesh(mesh[0], cell, mesh[1], mesh[2])
    if cap is not None:
        os.environ["FOCKMI_WORKSPACE_CAP"] = str(cap)
    try:
        return Plan(dict(n=n, a=cell, kpts=kp, nb=nb, omega=OMEGA), prec=prec), kp
    finally:
        os.environ.pop("FOCKMI_WORKSPACE_CAP", None)


class Ref:
    """sum over (k', j) of M_jk' IDFT(K DFT(conj(P_jk') X_ik)) / -N_k, one k-point pair at a time."""

    def __init__(self, n, kp):
        import torch
        from oracle.kernel import kernel_table
        B = synth.reciprocal_rows(synth.cubic_cell())
        n = (n,) * 3 if isinstance(n, int) else n
        self.nk, tab = len(kp), {}
        for t in range(self.nk):
            for s in range(self.nk):
                q = tuple(np.round(kp[t] - kp[s], 12))
                if q not in tab:
                    tab[q] = torch.from_numpy(np.ascontiguousarray(kernel_table(kp[t] - kp[s], t == s, n, B, OMEGA))).to("cuda:0")
        self.K = [[tab[tuple(np.round(kp[t] - kp[s], 12))] for s in range(self.nk)] for t in range(self.nk)]

    def sum(self, x, p, m):
        import torch
        out = torch.zeros_like(x)
        for t in range(self.nk):
            for s in range(self.nk):
                for j in range(p.shape[1]):
                    w = torch.fft.fftn(p[s, j].conj() * x[t], dim=(1, 2, 3)) * self.K[t][s]
                    out[t] += m[s, j] * torch.fft.ifftn(w, dim=(1, 2, 3))
        return out / -self.nk

    def apply(self, u, phi=None):
        return self.sum(u if phi is None else phi, u, u)

    def vjp(self, u, phi, g):
        return self.sum(u, phi, g) + self.sum(u, g, phi), self.sum(g, u, u)


def fields(nk, nb, n, seed):
    """Random fields with the spectrum of orbitals (the FP32 error bound assumes a decaying one)."""
    import torch
    n = (n,) * 3 if isinstance(n, int) else n
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    x = torch.randn((nk, nb) + n, dtype=torch.complex128, device="cuda:0", generator=g)
    f = [torch.fft.fftfreq(m, dtype=torch.float64, device="cuda:0") * m for m in n]
    k2 = f[0][:, None, None] ** 2 + f[1][None, :, None] ** 2 + f[2][None, None, :] ** 2
    return torch.fft.ifftn(x * torch.exp(-k2 / 16.0), dim=(2, 3, 4)).contiguous()


def per_k(a, b):
    return max(float((a[k] - b[k]).norm() / b[k].norm()) for k in range(a.shape[0]))


@pytest.mark.parametrize("mesh,nb,cap", [((1, 1, 1), 1, None), ((7, 1, 1), 1, None), ((3, 1, 1), 3, None),
                                         ((2, 2, 1), 16, None), ((5, 1, 1), 13, None), ((5, 1, 1), 13, 1100 << 20),
                                         ((3, 1, 1), 19, 40 << 20)])
def test_fp32_32cube_blocks(device, mesh, nb, cap):
    print(f"[gpu] pair form 32^3 mesh={mesh} nb={nb} cap={cap}", flush=True)
    plan, kp = make(32, mesh, nb, "fp32", cap)
    ref, nk = Ref(32, kp), len(kp)
    u = fields(nk, nb, 32, 11 + nb)
    got = plan.apply(u)
    assert bool((plan.apply(u) == got).all())
    assert per_k(got, ref.apply(u)) < 1e-6
    phi = fields(nk, 3, 32, 12)
    assert per_k(plan.apply(u, phi), ref.apply(u, phi)) < 1e-6
    k0 = nk // 2
    part = plan.apply_krange(u, k0, nk - k0, phi[k0:].contiguous())
    assert bool((part == plan.apply(u, phi)[k0:]).all())   # a target's sum does not depend on the blocks


@pytest.mark.parametrize("n,prec,mesh,nb,cap", [
    (16, "fp64f", (1, 1, 1), 1, None), (16, "fp64f", (3, 1, 1), 3, None), (16, "fp64f", (3, 1, 1), 11, None),
    (16, "fp64f", (5, 1, 1), 13, 270 << 20), (16, "fp64f", (3, 1, 1), 11, 400 << 10), (20, "fp64f", (5, 1, 1), 13, None), (20, "fp64f", (7, 1, 1), 1, 3 << 20),
    (24, "fp64f", (2, 2, 2), 4, None), (24, "fp64f", (5, 1, 1), 13, 910 << 20), (24, "fp64f", (3, 1, 1), 17, None),
    (16, "fp32", (2, 2, 2), 4, None), (20, "fp32", (3, 1, 1), 19, None), (24, "fp32", (1, 1, 1), 7, None),
    (24, "fp32", (19, 1, 1), 16, None)])
def test_small_cube_blocks(device, n, prec, mesh, nb, cap):
    """16^3 to 24^3 with few fields (the pair form in both precisions) and, in FP32, 304 fields
    of 24^3 (the pair symmetry); caps that leave one row of 64 fields beside a second row, and
    blocks of a few sources; a cap without room for any batch (the fused kernel)."""
    print(f"[gpu] pair form {n}^3 {prec} mesh={mesh} nb={nb} cap={cap}", flush=True)
    tol = 1e-6 if prec == "fp32" else 1e-10
    plan, kp = make(n, mesh, nb, prec, cap)
    ref, nk = Ref(n, kp), len(kp)
    u = fields(nk, nb, n, 21 + nb)
    every_call(plan, ref, n, nk, nb, tol)


def every_call(plan, ref, n, nk, nb, tol):
    u = fields(nk, nb, n, 21 + nb)
    got = plan.apply(u)
    assert bool((plan.apply(u) == got).all())
    assert per_k(got, ref.apply(u)) < tol
    phi = fields(nk, 3, n, 22)
    full = plan.apply(u, phi)
    assert per_k(full, ref.apply(u, phi)) < tol
    assert bool((plan.apply_krange(u, nk // 2, nk - nk // 2, phi[nk // 2:].contiguous()) == full[nk // 2:]).all())
    g = fields(nk, 3, n, 23)
    for a, b in zip(plan.vjp(u, phi, g), ref.vjp(u, phi, g)):
        assert per_k(a, b) < tol


@pytest.mark.parametrize("n,prec,nb,nphi", [(24, "fp64f", 1, 33), (24, "fp64f", 2, 31), (24, "fp32", 24, 7), (20, "fp32", 24, 13)])
def test_separate_targets_of_either_form(device, n, prec, nb, nphi):
    """phi apart from u with the targets on either side of a full device in FP64 (264 in the fused
    kernel, whose 24^3 transposes take three rounds; 248 in pairs) and few of them in FP32 (pairs,
    two partial sums per k-point); a k-range's bits are the full application's."""
    print(f"[gpu] separate targets {n}^3 {prec} nb={nb} nphi={nphi}", flush=True)
    plan, kp = make(n, (2, 2, 2), nb, prec)
    u, phi = fields(8, nb, n, 51), fields(8, nphi, n, 52)
    full = plan.apply(u, phi)
    assert per_k(full, Ref(n, kp).apply(u, phi)) < (1e-6 if prec == "fp32" else 1e-10)
    assert bool((plan.apply_krange(u, 3, 2, phi[3:5].contiguous()) == full[3:5]).all())


LENGTHS = (16, 20, 24, 32)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n2", LENGTHS)
@pytest.mark.parametrize("n3", LENGTHS)
def test_plane_passes(device, n2, n3, prec):
    """Every plane shape of the passes that serve grids without a one-CU kernel (n1 cycles through
    the lengths), and 32^3 in FP64; 3 k-points x 9 bands: 27 fields, whose last tile has 3."""
    n = (LENGTHS[(LENGTHS.index(n2) + LENGTHS.index(n3) + 1) % 4], n2, n3)
    if n[0] == n2 == n3:
        n = (16 if n2 != 16 else 32, n2, n3)
    if (n2, n3, prec) == (32, 32, "fp64"):
        n = (32, 32, 32)
    print(f"[gpu] plane passes {n} {prec}", flush=True)
    plan, kp = make(n, (3, 1, 1), 9, prec)
    every_call(plan, Ref(n, kp), n, len(kp), 9, 1e-6 if prec == "fp32" else 1e-10)


@pytest.mark.parametrize("n,mesh,nb,cap", [((32, 32, 32), (1, 1, 1), 1, None), ((32, 32, 32), (5, 1, 1), 13, 2200 << 20),
                                           ((24, 32, 16), (2, 1, 1), 40, 12 << 20), ((16, 16, 16), (2, 1, 1), 20, None),
                                           ((24, 24, 24), (5, 1, 1), 13, 910 << 20)])
def test_fp64_blocks(device, n, mesh, nb, cap):
    """The FP64 precision: one field, rows of 64 fields with a second row, a cap of a few sources
    per block, and cubic grids whose field fits on a CU."""
    print(f"[gpu] fp64 blocks {n} mesh={mesh} nb={nb} cap={cap}", flush=True)
    plan, kp = make(n, mesh, nb, "fp64", cap)
    every_call(plan, Ref(n, kp), n, len(kp), nb, 1e-10)


@pytest.mark.parametrize("n,prec,nb", [(24, "fp64f", 9), (32, "fp32", 5)])
def test_pair_form_in_a_graph(device, n, prec, nb):
    """Captured once (every buffer sized by an eager call before), replayed on changed inputs with
    eager work between the replays: each replay gives the eager call's bits."""
    import torch
    print(f"[gpu] pair form captured, {n}^3 {prec}", flush=True)
    plan, kp = make(n, (4, 1, 1), nb, prec)
    nk = len(kp)
    u = fields(nk, nb, n, 31)
    out = torch.empty_like(u)
    plan.apply(u, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.apply(u, out=out)
    for seed in (32, 33, 34):
        u.copy_(fields(nk, nb, n, seed))
        g.replay()
        torch.cuda.synchronize()
        replay = out.clone()
        assert bool((replay == plan.apply(u)).all())


def test_few_targets_first_under_capture(device):
    """FP32 at 16^3: 512 targets eagerly (the fused kernel), then 56 for the first time inside a
    capture, where their pair form finds no batch. Either form is within 1e-6 of the exact sum."""
    import torch
    print("[gpu] few targets first under capture", flush=True)
    plan, _ = make(16, (2, 2, 2), 40, "fp32")
    u, phi = fields(8, 40, 16, 61), fields(8, 7, 16, 62)
    plan.apply(u, fields(8, 64, 16, 63))
    out = torch.empty_like(phi)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        plan.apply(u, phi, out=out)
    for seed in (64, 65):
        phi.copy_(fields(8, 7, 16, seed))
        g.replay()
        torch.cuda.synchronize()
        a = out.clone()
        assert per_k(a, plan.apply(u, phi)) < 2e-6


def test_first_call_under_capture(device):
    """A plan's first FP64 application at 16^3 inside a capture, where the pair form's buffers
    cannot be allocated, and an orthonormalisation: both replay to the eager result (to rounding:
    the eager calls that follow may use the buffers)."""
    import torch
    print("[gpu] first call under capture", flush=True)
    plan, kp = make(16, (2, 1, 1), 3, "fp64f")
    u = fields(2, 3, 16, 41)
    out = torch.empty_like(u)
    psi = u.clone()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        plan.apply(u, out=out)
        plan.orthonormalize(psi)
    for seed in (42, 43):
        u.copy_(fields(2, 3, 16, seed))
        psi.copy_(u)
        g.replay()
        torch.cuda.synchronize()
        a, b = out.clone(), psi.clone()
        assert per_k(a, plan.apply(u)) < 1e-13
        assert per_k(b, plan.orthonormalize(u.clone())) < 1e-13


@pytest.mark.parametrize("n,nk,nb", [(16, 1, 1), (16, 3, 4), (16, 2, 5), (20, 3, 16), (32, 1, 9), (16, 2, 17)])
def test_orthonormalize_routes(device, n, nk, nb):
    """Gram-Schmidt in band order against the oracle's, through the Gram matrix (up to 16 bands)
    and beyond it; a k-point with two fields 1e-5 apart (left to modified Gram-Schmidt, whose
    error is about their condition number, 1e5 eps) beside well-conditioned ones; a vanishing
    field on one k-point leaves the others as they were."""
    import oracle
    import torch
    print(f"[gpu] orthonormalize {n}^3 nk={nk} nb={nb}", flush=True)
    plan, kp = make(n, (nk, 1, 1), nb, "fp64")
    u = fields(nk, nb, n, 51 + nb)
    u = u / u.abs().max()
    close = nk > 1 and nb > 3
    if close:
        u[1, 3] = u[1, 1] + 1e-5 * u[1, 3]
    ref = torch.from_numpy(oracle.gram_schmidt(u.cpu().numpy(), synth.cubic_cell())).to("cuda:0")
    got = plan.orthonormalize(u.clone())
    for k in range(nk):
        tol = 1e-9 if close and k == 1 else 1e-13
        assert float((got[k] - ref[k]).norm() / ref[k].norm()) < tol, k
        q = got[k].reshape(nb, -1)
        s = (q.conj() @ q.t().contiguous()) * (synth.LATTICE_A ** 3 / q.shape[1])
        assert float((s - torch.eye(nb, dtype=s.dtype, device=s.device)).abs().max()) < tol
    if nk > 1:
        v = u.clone()
        v[nk - 1, 0] = 0
        assert bool((plan.orthonormalize(v)[:nk - 1] == got[:nk - 1]).all())


@pytest.mark.parametrize("n,prec,mesh,nb,nphi,cap", [
    (16, "fp64f", (2, 2, 1), 5, 3, None), (24, "fp64f", (3, 1, 1), 25, 23, 900 << 20), (20, "fp32", (2, 1, 1), 9, 33, None),
    (32, "fp32", (2, 1, 1), 3, 37, 200 << 20), ((16, 20, 24), "fp64", (2, 1, 1), 6, 5, None),
    ((24, 16, 16), "fp32", (3, 1, 1), 2, 7, None), (32, "fp64", (2, 1, 1), 3, 2, None)])
def test_adjoint_shares_the_transforms(device, n, prec, mesh, nb, nphi, cap):
    """Both cotangents in one call run the pairs of g_phi once for both (targets and sources of
    different counts, several rows and blocks); each cotangent alone runs its own sums. Both
    against the reference, and against each other."""
    print(f"[gpu] adjoint {n} {prec} mesh={mesh} nb={nb} nphi={nphi}", flush=True)
    tol = 1e-6 if prec == "fp32" else 1e-10
    plan, kp = make(n, mesh, nb, prec, cap)
    nk, ref = len(kp), Ref(n, kp)
    u, phi, g = fields(nk, nb, n, 61), fields(nk, nphi, n, 62), fields(nk, nphi, n, 63)
    gu, gp = plan.vjp(u, phi, g)
    ru, rp = ref.vjp(u, phi, g)
    assert per_k(gu, ru) < tol and per_k(gp, rp) < tol
    assert per_k(plan.vjp(u, phi, g, need_phi=False)[0], gu) < tol
    assert per_k(plan.vjp(u, phi, g, need_u=False)[1], gp) < tol


def test_adjoint_shares_the_transforms_downsampled(device):
    import oracle
    import torch
    print("[gpu] adjoint, down-sampled", flush=True)
    from paper_1507_05156_amd.api import Plan
    cell = synth.cubic_cell()
    kp = synth.gamma_mesh(4, cell, 2, 1)
    src = [0, 2, 5]
    plan = Plan(dict(n=16, a=cell, kpts=kp, nb=3, omega=OMEGA, src=src), prec="fp64f")
    u, phi, g = fields(8, 3, 16, 71), fields(8, 2, 16, 72), fields(8, 2, 16, 73)
    gu, gp = plan.vjp(u, phi, g)
    ru, rp = oracle.fock_vjp(u.cpu().numpy(), phi.cpu().numpy(), g.cpu().numpy(), kp, cell, OMEGA, src=src)
    ru, rp = torch.from_numpy(ru).to("cuda:0"), torch.from_numpy(rp).to("cuda:0")
    assert float((gu - ru).norm() / ru.norm()) < 1e-10 and per_k(gp, rp) < 1e-10
