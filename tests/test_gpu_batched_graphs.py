"""The batched call's captured graph, every form forced through the tuning cache: replays on changed inputs,
with eager work in between, against each cell's own application (without a tuning cache these small cells
run one after another, and no graph is captured)."""

import ctypes as C
import json

import numpy as np
import pytest

from tests.test_gpu_batched import cells_small, rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("odd16", [False, True])
@pytest.mark.parametrize("form", [0, 1, 2])
def test_replays_track_inputs(device, tmp_path, form, odd16):
    import torch
    from paper_1507_05156_amd import _native as N
    from paper_1507_05156_amd.api import Plan
    print(f"[gpu] batched graph replay, form {form} odd16={odd16}", flush=True)
    path = str(tmp_path / "tune.json")
    cs = cells_small(odd16=odd16)
    descs = [{k: v for k, v in c.items() if k != "u"} for c in cs]
    us = [to_dev(c["u"]) for c in cs]
    Plan(descs, prec="fp32", tune_cache=path).apply_batched(us)
    data = json.load(open(path))
    key = [k for k in data if "/batched/" in k][0]
    data[key].update(form=form, wg_per_cu=1)
    json.dump(data, open(path, "w"))
    plan = Plan(descs, prec="fp32", tune_cache=path)
    single = [Plan(d, prec="fp64") for d in descs]
    outs = [torch.empty_like(u) for u in us]
    nc = len(cs)
    up = (C.c_void_p * nc)(*[u.data_ptr() for u in us])
    op = (C.c_void_p * nc)(*[o.data_ptr() for o in outs])
    npv = (C.c_int * nc)(*[c["nb"] for c in cs])
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    for rep in range(4):
        if rep:
            for u in us:
                u.mul_(np.exp(0.3j * rep) * (1.0 + 0.1 * rep))
        N.check(plan._lib.fock_apply_batched(plan._h, up, up, npv, op, st))
        torch.cuda.synchronize()
        for o, u, p in zip(outs, us, single):
            assert rel(o.cpu().numpy(), p.apply(u).cpu().numpy()) < 1e-6, rep
