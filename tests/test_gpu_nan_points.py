"""Points with a NaN coordinate are near no cell: every launch shape answers them "no valid
cell" and leaves the other points of the call as they are.  Infinite coordinates
have no valid cell either."""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf
from tests.test_gpu_group import OUT, _fitted, _sphere

pytestmark = pytest.mark.gpu

BAD = [[np.nan, 0, 0], [0, np.nan, 0], [0.1, 0.2, np.nan], [np.nan] * 3, [np.inf, 0, 0], [0, -np.inf, 0],
       [np.inf, np.nan, 0], [np.inf, -np.inf, 0]]


def _points(n):
    """The sphere's queries repeated, with a bad point here and there and a run of 300 of them."""
    wl = _sphere(20, n_queries=3001)
    reps = -(-n // 3001)
    q = torch.from_numpy(np.tile(wl.queries, (reps, 1))[:n]).cuda()
    bad = torch.zeros(n, dtype=torch.bool, device="cuda")
    bad[::67] = True
    bad[n // 2:n // 2 + 300] = True
    rows = torch.tensor(BAD, dtype=torch.float32, device="cuda")
    good = q.clone()
    q[bad] = rows[torch.arange(int(bad.sum()), device="cuda") % len(BAD)]
    return wl, good, q, bad


def _check(got, want, bad):
    for k in OUT:
        assert torch.equal(got[k][~bad], want[k][~bad]), k
    assert bool((got["argmin"][bad] == -1).all())
    assert bool((got["status"][bad] & ksdf.Q_NO_VALID_CELL).all())
    assert bool(torch.isposinf(got["mean"][bad]).all()) and bool(torch.isposinf(got["var"][bad]).all())
    assert bool((got["grad"][bad] == 0).all()) and bool((got["var_f"][bad] == 1).all())


SHAPES = [dict(query_split=0, query_block=64), dict(query_split=0, query_block=256), dict(query_split=1),
          dict(query_split=1, query_lanes=1), dict(query_split=1, query_block=64),
          dict(query_split=1, query_pairs=1), dict(query_split=1, query_mfma=1)]


CASES = [(kernel, k, s) for kernel in ("rbf", "matern32") for k in (8, 16) for s in SHAPES
         if kernel == "rbf" or "query_mfma" not in s]


@pytest.mark.parametrize("n", [700, 200001])
@pytest.mark.parametrize("kernel,k_fuse,shape", CASES)
def test_every_fp32_launch_shape(n, kernel, k_fuse, shape):
    print(f"[gpu-case] NaN points {n} {kernel} k={k_fuse} {shape}", flush=True)
    wl, good, q, bad = _points(n)
    model, _ = _fitted(wl, kernel=kernel, k_fuse=k_fuse, dense_inverse=True)
    model.set_tuning(**shape)
    want = model.query(good, grad_var=True)
    got = model.query(q, grad_var=True)
    _check(got, want, bad)
    model.close()


@pytest.mark.parametrize("k_fuse", [8, 16])
def test_fp64_and_the_fused_launch(k_fuse):
    print(f"[gpu-case] NaN points, FP64 and fused k={k_fuse}", flush=True)
    wl, good, q, bad = _points(20001)
    model, _ = _fitted(wl, precision="fp64", k_fuse=k_fuse)
    _check(model.query(q.double(), grad_var=True), model.query(good.double(), grad_var=True), bad)
    model.close()
    model, _ = _fitted(wl, k_fuse=k_fuse)
    pts = torch.from_numpy(wl.points).cuda()
    for fused in (0, 1):
        model.set_tuning(fused=fused)
        _check(model.fit_query(pts, q, grad_var=True), model.fit_query(pts, good, grad_var=True), bad)
    model.close()


@pytest.mark.parametrize("n", [700, 200001])
def test_backward(n):
    """Such a point has no gradient, whether its argmin is given or found."""
    print(f"[gpu-case] NaN points, backward of {n}", flush=True)
    wl, good, q, bad = _points(n)
    model, _ = _fitted(wl, adjoint=True)
    one = torch.ones(n, device="cuda")
    am = model.query(q)["argmin"]
    for argmin in (am, None):
        got, _ = model.backward(q, None, one, argmin=argmin)
        want, _ = model.backward(good, None, one, argmin=argmin)
        assert torch.equal(got[~bad], want[~bad]) and bool((got[bad] == 0).all())
    model.close()
