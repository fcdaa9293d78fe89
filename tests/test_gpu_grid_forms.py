"""The fused kernels of 16^3 to 24^3 (one workgroup per target) at counts of fields where they are not the
default any more in FP32, or only for separate targets in FP64: in FP32 19 bands (two partial sums per k-point) and
more targets than CUs. FP32 against the FP64 form, with the kernel's variant named by a tuning file; FP64
against the pair form's symmetric sum of the same fields."""

import json

import pytest

from paper_1507_05156_amd import synth

pytestmark = pytest.mark.gpu

OMEGA = synth.OMEGA_HSE


def fields(nk, nb, n, seed):
    """Random fields with a decaying spectrum, as orbitals have."""
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    x = torch.randn((nk, nb, n, n, n), dtype=torch.complex128, device="cuda:0", generator=g)
    f = torch.fft.fftfreq(n, dtype=torch.float64, device="cuda:0") * n
    k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + f[None, None, :] ** 2
    return torch.fft.ifftn(x * torch.exp(-k2 / 16.0), dim=(2, 3, 4)).contiguous()


def per_k(a, b):
    return max(float((a[k] - b[k]).norm() / b[k].norm()) for k in range(a.shape[0]))


def desc(n, mesh, nb):
    cell = synth.cubic_cell()
    return dict(n=n, a=cell, kpts=synth.gamma_mesh(mesh[0], cell, mesh[1], mesh[2]), nb=nb, omega=OMEGA)


@pytest.mark.parametrize("n,mesh,nb,variant", [(16, (6, 3, 3), 19, 0), (16, (6, 3, 3), 19, 1), (20, (7, 2, 2), 19, 0),
                                               (20, (7, 2, 2), 19, 1), (24, (17, 1, 1), 19, 0)])
def test_fp32_grid_forms(device, tmp_path, n, mesh, nb, variant):
    import torch
    from paper_1507_05156_amd.api import Plan
    print(f"[gpu] FP32 grid form, {n}^3 mesh={mesh} nb={nb} variant {variant}", flush=True)
    d = desc(n, mesh, nb)
    nk = len(d["kpts"])
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({f"{arch}/fp32/fused/n{n}x{n}x{n}/nt{nk}/ns{nk}/nb{nb}/nx{nb}":
                                {"variant": variant, "xcd_map": 1}}))
    u = fields(nk, nb, n, 31 + n)
    plan = Plan(d, prec="fp32", tune_cache=str(path))
    got = plan.apply(u)
    assert bool((plan.apply(u) == got).all())
    assert per_k(got, Plan(d, prec="fp64").apply(u)) < 1e-6


@pytest.mark.parametrize("n,mesh,nb", [(16, (3, 3, 3), 19), (20, (7, 2, 1), 18), (24, (2, 2, 2), 32)])
def test_fp64_fused_kernel_and_symmetric_pairs(device, n, mesh, nb):
    from paper_1507_05156_amd.api import Plan
    print(f"[gpu] FP64 fused kernel, {n}^3 mesh={mesh} nb={nb}", flush=True)
    d = desc(n, mesh, nb)
    u = fields(len(d["kpts"]), nb, n, 41 + n)
    plan = Plan(d, prec="fp64f")
    a, b = plan.apply(u, u.clone()), plan.apply(u)
    assert per_k(a, b) < 1e-13
