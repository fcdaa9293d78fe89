"""Calls on one plan from two threads, each with a stream of its own, for the calls that the C ABI lets
run so: every result has the bits of the same call alone."""

import threading

import pytest

from paper_1507_05156_amd import synth

pytestmark = pytest.mark.gpu

OMEGA = synth.OMEGA_HSE


@pytest.mark.parametrize("n,prec", [(16, "fp64f"), (20, "fp64f"), (16, "fp32"), (32, "fp64")])  # the last two: orthonormalisation
def test_two_threads_two_streams(device, n, prec):
    import torch
    from paper_1507_05156_amd.api import Plan
    print(f"[gpu] two threads, {n}^3 {prec}", flush=True)
    cell = synth.cubic_cell()
    kp = synth.gamma_mesh(2, cell)
    nb = 4
    plan = Plan(dict(n=n, a=cell, kpts=kp, nb=nb, omega=OMEGA), prec=prec)
    g = torch.Generator(device="cuda:0").manual_seed(7 + n)
    u = [torch.randn((8, nb, n, n, n), dtype=torch.complex128, device="cuda:0", generator=g) for _ in range(2)]

    def calls(x, y):
        r = [plan.orthonormalize(x.clone())]
        if prec == "fp64f":
            r += [plan.apply(x), plan.apply_krange(x, 3, 4), *plan.vjp(x, y, x), plan.energy_vjp(x, 1.0)]
        return r

    want = [calls(u[i], u[1 - i]) for i in range(2)]
    torch.cuda.synchronize()
    bad, errors = [0, 0], []

    def work(i):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(30):
                    bad[i] += sum(not bool((a == b).all()) for a, b in zip(calls(u[i], u[1 - i]), want[i]))
        except Exception as e:  # the assertion below shows it
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert errors == [] and bad == [0, 0]
    plan.close()
