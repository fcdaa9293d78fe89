"""FOCKMI_SPLIT_SYM=0 at plan creation: an application with u as targets runs every pair, as a k-range of
it does, and gives the k-range's bits; the symmetric application agrees with it to rounding."""

import os

import pytest

from paper_1507_05156_amd import synth

pytestmark = pytest.mark.gpu

OMEGA = synth.OMEGA_HSE


@pytest.mark.parametrize("n,prec,nb,tol", [(24, "fp32", 26, 1e-6), (32, "fp32", 9, 1e-6), (20, "fp64f", 9, 1e-12),
                                           (32, "fp64", 9, 1e-12), ((16, 20, 24), "fp64", 9, 1e-12)])
def test_every_pair_gives_the_k_range_bits(device, n, prec, nb, tol):
    import torch
    from paper_1507_05156_amd.api import Plan
    print(f"[gpu] symmetry switch, {n} {prec}", flush=True)
    cell = synth.cubic_cell()
    kp = synth.gamma_mesh(3, cell, 2, 2)
    shape = (n,) * 3 if isinstance(n, int) else n
    g = torch.Generator(device="cuda:0").manual_seed(17)
    u = torch.randn((12, nb) + shape, dtype=torch.complex128, device="cuda:0", generator=g)
    u = torch.fft.ifftn(u * torch.exp(-4.0 * torch.rand(shape, device="cuda:0", generator=g)), dim=(2, 3, 4)).contiguous()
    desc = dict(n=n, a=cell, kpts=kp, nb=nb, omega=OMEGA)
    os.environ["FOCKMI_SPLIT_SYM"] = "0"
    try:
        every = Plan(desc, prec=prec)
    finally:
        os.environ.pop("FOCKMI_SPLIT_SYM")
    full = every.apply(u)
    assert bool((every.apply_krange(u, 5, 4) == full[5:9]).all())
    sym = Plan(desc, prec=prec).apply(u)
    assert float((sym - full).norm() / full.norm()) < tol
