"""The two-kernel query at sizes past the eight-lane kernel's: wave-shared cells (many points per
cell) and per-lane cells, for both kernels, K to 16 and cells of every size class, against the
one-kernel form bit for bit; in two calls (bucket, query), with tied candidates, and replayed from
a graph.  And the backward with a var_f cotangent in argmin order (past 16,384 points)."""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import scenes
from tests.test_gpu_dispatch import _form
from tests.test_gpu_group import OUT, _fitted, _sphere

pytestmark = pytest.mark.gpu

N = 196609


def _tiled(wl, n):
    reps = -(-n // len(wl.queries))
    q = torch.from_numpy(np.tile(wl.queries, (reps, 1))[:n]).cuda()
    return q, torch.from_numpy(np.tile(wl.sign, reps)[:n]).cuda()


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("m_max,k_fuse", [(1, 8), (7, 16), (9, 8), (63, 8), (64, 9), (65, 8), (128, 16)])
def test_wave_shared_cells_give_the_same_answers(kernel, m_max, k_fuse):
    """80 cells: 2,457 points a cell, far past every limit of the per-lane form."""
    print(f"[gpu-case] wave-shared {kernel} m<={m_max} k={k_fuse}", flush=True)
    wl = _sphere(m_max, n_queries=3001)
    model, cells = _fitted(wl, kernel=kernel, k_fuse=k_fuse)
    assert cells.m.max() == m_max and N > 400 * cells.n
    q, sg = _tiled(wl, N)
    q[::97] *= 40
    model.set_tuning(query_split=0)
    want = model.query(q, sg, grad_var=True)
    for block in (64, 256):
        model.set_tuning(query_split=1, query_lanes=0, query_block=block)
        form, _ = _form(model, q)
        got = model.query(q, sg, grad_var=True)
        assert form == "two"
        for k in OUT:
            assert torch.equal(got[k], want[k]), (k, block)
    model.close()


@pytest.mark.parametrize("k_fuse", [8, 16])
@pytest.mark.parametrize("tuning", [dict(query_lanes=0, query_block=64), dict(query_lanes=0, query_block=256),
                                    dict(query_lanes=1, query_block=64), dict(query_lanes=1, query_block=256),
                                    dict(query_pairs=1)])
def test_uneven_room_in_two_calls(k_fuse, tuning):
    """430,000 points for 4,434 cells of 8 to 128 samples: over 96 a cell, where waves share them;
    bucket and query in two calls give the bits of one."""
    print(f"[gpu-case] uneven room k={k_fuse} {tuning}", flush=True)
    wl = scenes.small_room_workload(n_queries=43000, cfg_id=47, uneven=True)
    model, cells = _fitted(wl, k_fuse=k_fuse)
    n = 430000
    assert n > 96 * cells.n and cells.m.max() == 128
    q, sg = _tiled(wl, n)
    model.set_tuning(query_split=0)
    want = model.query(q[:43000].contiguous(), sg[:43000].contiguous(), grad_var=True)
    model.set_tuning(query_split=1, **tuning)
    got = model.query(q, sg, grad_var=True)
    ws = model.new_workspace(n)
    model.bucket(q, workspace=ws)
    two = model.query(q, sg, grad_var=True, workspace=ws, bucketed=True)
    for k in OUT:
        assert torch.equal(got[k], two[k]), k
        if "query_pairs" not in tuning:   # pairs may re-evaluate other near-ties in float-float
            assert torch.equal(got[k], torch.cat([want[k]] * 10)), k
    model.close()


@pytest.mark.parametrize("lanes", [0, 1])
def test_tied_candidates_in_any_order(lanes):
    """Points midway between cell centres, whose candidate distances tie: the two-kernel form of
    either kind gives the one-kernel bits in any order of the points."""
    print(f"[gpu-case] ties, lanes={lanes}", flush=True)
    wl = _sphere(20, n_queries=16)
    half = wl.h / 2
    ax = torch.arange(-5, 6, device="cuda", dtype=torch.float32) * half
    z = torch.linspace(-1.3, 1.3, 1700, device="cuda")
    q = torch.cartesian_prod(ax, ax, z).contiguous()
    assert len(q) > 196608
    model, cells = _fitted(wl)
    model.set_tuning(query_split=0)
    want = model.query(q)
    model.set_tuning(query_split=1, query_lanes=lanes)
    order = torch.randperm(len(q), generator=torch.Generator().manual_seed(3)).cuda()
    form, _ = _form(model, q)
    assert form == "two"
    got, mixed = model.query(q), model.query(q[order].contiguous())
    for k in want:
        assert torch.equal(got[k], want[k]) and torch.equal(mixed[k], want[k][order]), k
    model.close()


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("lanes", [0, 1])
def test_replayed_from_a_graph(kernel, lanes):
    print(f"[gpu-case] graph {kernel} lanes={lanes}", flush=True)
    wl = _sphere(40, n_queries=3001)
    model, _ = _fitted(wl, kernel=kernel)
    q, sg = _tiled(wl, N)
    model.set_tuning(query_split=1, query_lanes=lanes)
    out, ws = model._out(N, q.device), model.new_workspace(N)
    model.query(q, sg, out=out, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        model.query(q, sg, out=out, workspace=ws)
    for step in range(3):
        q.mul_(0.97).add_(0.003 * step)
        g.replay()
        torch.cuda.synchronize()
        got = {k: v.clone() for k, v in out.items()}
        want = model.query(q, sg)
        torch.cuda.synchronize()
        for k in want:
            assert torch.equal(got[k], want[k]), (k, step)
    model.close()


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("m_max", [9, 64, 128])
def test_var_f_backward_in_argmin_order(kernel, m_max):
    """Past 16,384 points the eight lanes of a point take it from the argmin-sorted order: its
    gradient has the bits that it has in calls small enough to stay in the caller's order, and the
    hyperparameter gradient is their sum (added in float-float, 2^-44 a step)."""
    print(f"[gpu-case] sorted var_f backward {kernel} m<={m_max}", flush=True)
    wl = _sphere(m_max, n_queries=20003)
    model, _ = _fitted(wl, kernel=kernel, adjoint_var_f=True)
    q, sg = torch.from_numpy(wl.queries).cuda(), torch.from_numpy(wl.sign).cuda()
    n = len(q)
    gen = torch.Generator(device="cuda").manual_seed(1)
    cot = [torch.rand(*s, generator=gen, device="cuda") for s in ((n,), (n, 3), (n,), (n,))]
    am = model.query(q, sg)["argmin"]
    dp, dh = model.backward(q, sg, *cot, argmin=am)
    again, _ = model.backward(q, sg, *cot)     # the argmin found by the call
    assert torch.equal(dp, again)
    parts, sums = [], []
    for a, b in ((0, 10000), (10000, n)):
        s = slice(a, b)
        p, h = model.backward(q[s].contiguous(), sg[s].contiguous(), *(c[s].contiguous() for c in cot), argmin=am[s].contiguous())
        parts.append(p)
        sums.append(h)
    assert torch.equal(dp, torch.cat(parts))
    each = sum(h.abs() for h in sums)
    assert bool(((dh - sums[0] - sums[1]).abs() <= 2.0 ** -30 * each).all())
    model.close()
