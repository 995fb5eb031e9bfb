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


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("m_max,k_fuse", [(1, 8), (7, 16), (9, 8), (63, 8), (64, 9), (65, 8), (128, 16)])
def test_per_lane_cells_give_the_same_answers(kernel, m_max, k_fuse):
    """Past the eight-lane kernel's limit and below 96 points a cell every lane walks its own
    cells: cells of every remainder of eight samples, points far outside, the last wave partial."""
    print(f"[gpu-case] lanes {kernel} m<={m_max} k={k_fuse}", flush=True)
    wl = _sphere(m_max, n_queries=3001)
    model, cells = _fitted(wl, kernel=kernel, k_fuse=k_fuse)
    assert cells.m.max() == m_max
    n = 196609
    reps = -(-n // 3001)
    q = torch.from_numpy(np.tile(wl.queries, (reps, 1))[:n]).cuda()
    q[::97] *= 40
    sg = torch.from_numpy(np.tile(wl.sign, reps)[:n]).cuda()
    model.set_tuning(query_split=0)
    want = model.query(q, sg, grad_var=True)
    model.set_tuning(query_split=1, query_lanes=1)
    for block in (64, 256):
        model.set_tuning(query_block=block)
        got = model.query(q, sg, grad_var=True)
        for k in OUT:
            assert torch.equal(got[k], want[k]), (k, block)
