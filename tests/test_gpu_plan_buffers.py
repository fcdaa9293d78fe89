"""Plan buffers on the device: graphs captured from a plan whose buffers eager calls grow between the
replays (an adjoint of the same orbitals, a larger cell of the plan)."""

import numpy as np
import pytest

from paper_1507_05156_amd import synth

pytestmark = pytest.mark.gpu

OMEGA = synth.OMEGA_HSE


def fields(nk, nb, n, seed):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    return torch.randn((nk, nb, n, n, n), dtype=torch.complex128, device="cuda:0", generator=g)


def desc(n, mesh, nb):
    cell = synth.cubic_cell()
    return dict(n=n, a=cell, kpts=synth.gamma_mesh(mesh[0], cell, mesh[1], mesh[2]), nb=nb, omega=OMEGA)


@pytest.mark.parametrize("n,prec,mesh,nb", [(24, "fp32", (4, 4, 4), 16), (24, "fp64f", (3, 3, 2), 16),
                                            (20, "fp64f", (3, 3, 3), 12), (16, "fp64", (2, 2, 2), 4)])
def test_replays_after_the_buffers_grew(device, n, prec, mesh, nb):
    """Every replay gives the bits of the captured call's own kind run before any growth."""
    import torch
    from paper_1507_05156_amd.api import Plan
    print(f"[gpu] replay after growth, {n}^3 {prec} mesh={mesh} nb={nb}", flush=True)
    plan = Plan([desc(n, mesh, nb), desc(n, mesh, nb + 4)], prec=prec)
    nk = int(np.prod(mesh))
    u = fields(nk, nb, n, 91)
    psi0 = fields(nk, nb, n, 92)
    out, psi = torch.empty_like(u), psi0.clone()
    plan.apply(u, out=out)
    plan.orthonormalize(psi)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.apply(u, out=out)
        plan.orthonormalize(psi)

    def replay():
        out.zero_()
        psi.copy_(psi0)
        g.replay()
        torch.cuda.synchronize()
        return out.clone(), psi.clone()

    first = replay()
    phi, c = fields(nk, nb, n, 93), fields(nk, nb, n, 94)
    v = fields(nk, nb + 4, n, 95)
    for step in (lambda: plan.vjp(u, phi, c), lambda: plan.apply(v, cell=1), lambda: plan.orthonormalize(v, cell=1)):
        step()
        again = replay()
        assert bool((again[0] == first[0]).all()) and bool((again[1] == first[1]).all())
    plan.close()
