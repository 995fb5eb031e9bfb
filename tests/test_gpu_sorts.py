"""The counting sorts of the larger queries (points by index box, records by argmin cell): one
block or several scan the bins, a bin a point at most by default, and places come from atomics
in no set order.  A point's answer does not depend on the order, so every granularity and any
order of the points gives the one-kernel form's bits.
"""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import scenes
from tests.test_gpu_group import OUT, _fitted, _sphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scene,n", [("sphere", 196609), ("room", 196609), ("room", 400000)])
def test_every_granularity_and_order_gives_the_same_answers(scene, n):
    print(f"[gpu-case] sorts {scene} {n}", flush=True)
    wl = _sphere(64) if scene == "sphere" else scenes.small_room_workload(n_queries=4099, cfg_id=47, uneven=True)
    model, _ = _fitted(wl)
    reps = -(-n // len(wl.queries))
    q = torch.from_numpy(np.tile(wl.queries, (reps, 1))[:n]).cuda()
    sg = torch.from_numpy(np.tile(wl.sign, reps)[:n]).cuda()
    step = torch.arange(reps * len(wl.queries), device="cuda")[:n] // len(wl.queries)
    q[:, 0] += step * 2.0 ** -12   # distinct points, sorted within each repeat as the scene's are
    model.set_tuning(query_split=0)
    want = model.query(q, sg, grad_var=True)
    order = torch.randperm(n, generator=torch.Generator().manual_seed(3)).cuda()
    model.set_tuning(query_split=1)
    for sub in (0, 1, 2, 4):
        model.set_tuning(query_sub=sub)
        got = model.query(q, sg, grad_var=True)
        mixed = model.query(q[order], sg[order], grad_var=True)
        for k in OUT:
            assert torch.equal(got[k], want[k]), (k, sub)
            assert torch.equal(mixed[k], want[k][order]), (k, sub)
    model.set_tuning(query_sub=0)
    one = model.query(q[:1].expand(n, 3).contiguous(), sg[:1].expand(n).contiguous(), grad_var=True)
    for k in OUT:
        assert torch.equal(one[k], want[k][:1].expand_as(one[k])), k
