"""Eight lanes per query: the query and backward kernels that answer small and medium calls,
at the sizes where their blocks of eight and their dispatch turn.

The FP32 query kernel keeps the order of every operation of the one-kernel form
(query_split=0), so all outputs agree bit for bit; it is used up to 196,608 points and sorts
them above 131,072.  The backward is held to the oracle's VJP, and to the per-thread kernels
that answer larger calls: both take the same terms and sums in the same order and differ in
the fused multiply-adds of a handful of final operations, a few 2^-24 of the parts of a
point's gradient.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes
from tests.test_gpu_backward import _compare, _cotangents, _gpu_vjp, _setup

pytestmark = pytest.mark.gpu

OUT = ("mean", "grad", "var", "var_f", "grad_var", "argmin", "status")


def _sphere(m_max, n_samples=9000, n_queries=1000, dtype=np.float32):
    wl = scenes.sphere_workload(n_samples=n_samples, n_queries=n_queries)
    return dataclasses.replace(wl, points=wl.points.astype(dtype), queries=wl.queries.astype(dtype),
                               m_max=m_max)


def _fitted(wl, **kw):
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, wl.m_max, 1)
    model = ksdf.Model(cells, len(wl.points), wl.origin, wl.h, ell=wl.ell, noise_var=wl.noise_var, **kw)
    model.fit(torch.from_numpy(wl.points).cuda())
    return model, cells


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("m_max", [1, 7, 8, 9, 63, 64, 65, 128])
@pytest.mark.parametrize("k_fuse", [1, 8, 9, 16])
def test_query_equals_the_one_kernel_form(kernel, m_max, k_fuse):
    print(f"[gpu-case] group query {kernel} m<={m_max} k={k_fuse}", flush=True)
    wl = _sphere(m_max)
    model, cells = _fitted(wl, kernel=kernel, k_fuse=k_fuse)
    assert cells.m.max() == m_max
    q = torch.from_numpy(wl.queries).cuda()
    q[::5] *= 40   # outside the candidate index: every cell is scanned
    sg = torch.from_numpy(wl.sign).cuda()
    for n in (1, 7, 8, 9, 65, 1000):
        model.set_tuning(query_split=0)
        want = model.query(q[:n], sg[:n], grad_var=True)
        model.set_tuning(query_split=1)
        got = model.query(q[:n], sg[:n], grad_var=True)
        few = model.query(q[:n], sg[:n], var_f=False, argmin=False, status=False)
        for k in OUT:
            assert torch.equal(got[k], want[k]), (k, n)
        for k in few:
            assert torch.equal(few[k], want[k]), (k, n)


@pytest.mark.parametrize("n", [131072, 131073, 196608, 196609])
def test_query_and_bucketed_query_at_the_dispatch_edges(n):
    print(f"[gpu-case] group query, {n} points", flush=True)
    wl = scenes.small_room_workload(n_queries=n, cfg_id=47, uneven=True)
    model, _ = _fitted(wl)
    q, sg = torch.from_numpy(wl.queries).cuda(), torch.from_numpy(wl.sign).cuda()
    model.set_tuning(query_split=0)
    want = model.query(q, sg, grad_var=True)
    model.set_tuning(query_split=1)
    got = model.query(q, sg, grad_var=True)
    ws = model.new_workspace(n)
    model.bucket(q, workspace=ws)
    two = model.query(q, sg, grad_var=True, workspace=ws, bucketed=True)
    for k in OUT:
        assert torch.equal(got[k], want[k]) and torch.equal(two[k], want[k]), k


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("m_max", [1, 7, 9, 64, 65, 128])
def test_backward_with_var_f_matches_the_oracle(precision, m_max):
    print(f"[gpu-case] group backward {precision} m<={m_max}", flush=True)
    wl = _sphere(m_max, n_queries=203, dtype=np.float32 if precision == "fp32" else np.float64)
    model, cells, dt = _setup(wl, precision, var_f=True)
    cot = _cotangents(len(wl.queries), 5, grad=precision == "fp64")
    dp, dh, am = _gpu_vjp(model, wl.queries, wl.sign, cot, dt)
    _compare(dp, dh, am, wl, cells, wl.queries, wl.sign, cot, precision)


@pytest.mark.parametrize("precision,kernel,limit", [("fp32", "rbf", 196608), ("fp32", "matern32", 196608),
                                                    ("fp64", "rbf", 65536)])
def test_backward_equals_the_per_thread_kernels(precision, kernel, limit):
    print(f"[gpu-case] group backward against one thread per query, {precision} {kernel}", flush=True)
    wl = scenes.small_room_workload(n_queries=4099, cfg_id=36, uneven=True)
    model, _, dt = _setup(wl, precision, kernel=kernel)
    reps = limit // len(wl.queries) + 1
    q = torch.from_numpy(wl.queries).to("cuda", dt)
    sg = torch.from_numpy(wl.sign).cuda()
    g = torch.Generator(device="cuda").manual_seed(1)
    cot = [torch.randn(*s, generator=g, device="cuda", dtype=dt) for s in ((4099,), (4099, 3), (4099,))]
    am = model.query(q, sg)["argmin"]
    a, ah = model.backward(q, sg, *cot, argmin=am)
    rep = lambda t: t.repeat(reps, *([1] * (t.dim() - 1)))   # noqa: E731
    b, bh = model.backward(rep(q), rep(sg), *(rep(c) for c in cot), argmin=rep(am))
    eps = 2.0 ** (-24 if precision == "fp32" else -53)
    b = b[:4099]
    big = a.abs().amax(1, keepdim=True)
    # the parts of a gradient exceed it by what cancels between them: 2^10 covers all but
    # points whose gradient nearly vanishes, which the median's share of the bound covers
    assert bool(((a - b).abs() <= eps * 2 ** 10 * (big + big.median())).all())
    assert torch.allclose(ah * reps, bh, rtol=eps * 2 ** 10, atol=0)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_hyperparameter_sums_where_one_block_ends(precision):
    """d_hyper of up to 4,096 points is summed by one block, beyond by 256: the same as the sum
    over two halves, to the FP64 rounding of the few additions that are ordered otherwise (FP32
    partials are added in float-float, 2^-44 a step)."""
    print(f"[gpu-case] hyperparameter sums {precision}", flush=True)
    wl = scenes.small_room_workload(n_queries=4097, cfg_id=36)
    model, _, dt = _setup(wl, precision)
    q, sg = torch.from_numpy(wl.queries).to("cuda", dt), torch.from_numpy(wl.sign).cuda()
    g = torch.Generator(device="cuda").manual_seed(1)
    cot = [torch.rand(*s, generator=g, device="cuda", dtype=dt) for s in ((4097,), (4097, 3), (4097,))]
    am = model.query(q, sg)["argmin"]

    def sums(a, b):
        s = slice(a, b)
        return model.backward(q[s], sg[s], *(c[s].contiguous() for c in cot), argmin=am[s])[1].clone()

    each = torch.stack([sums(i, i + 1) for i in range(0, 4097, 64)]).abs().sum(0) * 64   # their size
    eps = 2.0 ** (-40 if precision == "fp32" else -46)
    for n in (1, 255, 256, 257, 4096, 4097):
        assert bool(((sums(0, n) - sums(0, n // 2) - sums(n // 2, n)).abs() <= eps * each).all()), n


@pytest.mark.parametrize("m_max", [1, 7, 16])
def test_fp64_var_f_backward_of_small_cells_by_one_thread(m_max):
    """FP64 models of up to 16 samples a cell: past 40,960 points one thread answers a point with
    a var_f cotangent too.  Its sums are the eight lanes' but for the order within the two
    triangular solves and the fused steps, a few 2^-53 of the parts of a point's gradient."""
    print(f"[gpu-case] one thread with var_f m<={m_max}", flush=True)
    wl = _sphere(m_max, n_queries=2003, dtype=np.float64)
    model, _, dt = _setup(wl, "fp64", var_f=True)
    q, sg = torch.from_numpy(wl.queries).to("cuda", dt), torch.from_numpy(wl.sign).cuda()
    g = torch.Generator(device="cuda").manual_seed(1)
    n, reps = len(q), 40960 // len(q) + 1
    cot = [torch.randn(*s, generator=g, device="cuda", dtype=dt) for s in ((n,), (n, 3), (n,), (n,))]
    am = model.query(q, sg)["argmin"]
    a, ah = model.backward(q, sg, *cot, argmin=am)
    rep = lambda t: t.repeat(reps, *([1] * (t.dim() - 1)))   # noqa: E731
    b, bh = model.backward(rep(q), rep(sg), *(rep(c) for c in cot), argmin=rep(am))
    assert torch.equal(b[:n], b[-n:])
    big = a.abs().amax(1, keepdim=True)
    # 2^-53 of the parts, which exceed a gradient by what cancels between them and by the
    # cells' condition (below 2^18: 16 samples of variance 1e-4 and more)
    eps = 2.0 ** -53
    assert bool(((a - b[:n]).abs() <= eps * 2 ** 18 * (big + big.median())).all())
    assert torch.allclose(ah * reps, bh, rtol=eps * 2 ** 18, atol=0)
