"""Samples of infinite variance (a sample that a caller masks out): the FP64 factorisation
gives them the weight 0 that division by an infinite pivot gives, in FP64 models and in the
FP64 refit of FP32 cells, so that every other output is the one of a variance too large to
matter."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("precision,m_max", [("fp64", 1), ("fp64", 13), ("fp64", 64), ("fp64", 101),
                                             ("fp32", 13), ("fp32", 64), ("fp32", 101)])
def test_an_infinite_variance_is_a_sample_left_out(precision, m_max, kernel):
    print(f"[gpu-case] infinite variance {precision} m<={m_max} {kernel}", flush=True)
    wl = scenes.sphere_workload(n_samples=9000, n_queries=2001)
    dt = torch.float64 if precision == "fp64" else torch.float32
    wl = dataclasses.replace(wl, m_max=m_max)
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, m_max, 1)
    n = len(wl.points)
    pts = torch.from_numpy(wl.points).to("cuda", dt)
    q = torch.from_numpy(wl.queries).to("cuda", dt)
    model = ksdf.Model(cells, n, wl.origin, wl.h, ell=wl.ell, noise_var=wl.noise_var, precision=precision,
                       kernel=kernel)
    # a third of the samples, the nearest of some cells, the farthest of others, among them
    out = {}
    gone = torch.from_numpy(np.random.default_rng(7).random(n) < 0.33).cuda()
    # 1e30 against kernel sums of up to m: a weight of 1e-30, below any rounding of the others
    for name, big in (("inf", float("inf")), ("large", 1e30)):
        var = torch.where(gone, big, wl.noise_var).to(dt)
        status = torch.full((cells.n,), 255, dtype=torch.uint8, device="cuda")
        model.fit(pts, var, cell_status=status)
        out[name] = dict(model.query(q), cells=status)
    a, b = out["inf"], out["large"]
    assert not bool((a["cells"] & ksdf.C_FAILED).any())
    assert torch.equal(a["argmin"], b["argmin"]) and torch.equal(a["status"], b["status"])
    has = a["argmin"] >= 0
    assert int(has.sum()) > 1000
    # the same operations but for the terms below rounding: a few roundings of the results
    tol = 1e-12 if precision == "fp64" else 1e-6
    for k in ("mean", "grad", "var_f"):
        x, y = a[k][has], b[k][has]
        assert bool(torch.isfinite(x).all()) and torch.allclose(x, y, rtol=tol, atol=tol), k
    if precision == "fp64":
        # a cell's softmin variance is infinite where such a sample has a share in it
        masked = torch.from_numpy(np.logical_or.reduceat(gone.cpu().numpy()[cells.samples], cells.offsets[:-1])).cuda()
        there = masked[a["argmin"].clamp_min(0).long()] & has
        assert bool(torch.isinf(a["var"][there & (b["var"] > 1e12)]).all())
        assert torch.equal(a["var"][has & ~there], b["var"][has & ~there])


def _one_cell(m, precision):
    """One cell of m samples, the nearest its centre of infinite variance."""
    dt = torch.float64 if precision == "fp64" else torch.float32
    rng = np.random.default_rng(m)
    p = np.array([0.5, 0.5, 0.5]) + rng.uniform(0.05, 0.3, (m, 3)) * rng.choice([-1, 1], (m, 3))
    p[0] = [0.51, 0.5, 0.5]
    cells = ksdf.CellSet(np.array([0, m], np.int32), np.arange(m, dtype=np.int32), np.zeros((1, 3), np.int32))
    var = torch.full((m,), 1e-4, dtype=dt, device="cuda")
    var[0] = float("inf")
    model = ksdf.Model(cells, m, (0.0, 0.0, 0.0), 1.0, ell=0.2, k_fuse=1, precision=precision, adjoint_var_f=True)
    model.fit(torch.from_numpy(p).to("cuda", dt), var)
    return model, torch.from_numpy(rng.uniform(0.1, 0.9, (64, 3))).to("cuda", dt)


@pytest.mark.parametrize("var_f", [False, True])
@pytest.mark.parametrize("m", [2, 7, 8, 9, 60, 127])
def test_hyperparameter_gradient_of_an_infinite_softmin_variance(var_f, m):
    """Through an infinite softmin variance the FP64 gradient is infinite, not NaN: the eight lanes
    of a point pad its samples to a multiple of eight with terms that are 0."""
    print(f"[gpu-case] gradient of an infinite variance {var_f} m={m}", flush=True)
    model, q = _one_cell(m, "fp64")
    one, zero = torch.ones(1, dtype=q.dtype, device="cuda"), torch.zeros(1, dtype=q.dtype, device="cuda")
    am = torch.zeros(1, dtype=torch.int32, device="cuda")
    for i in range(3):
        _, dh = model.backward(q[i:i + 1].contiguous(), None, zero, None, one, one if var_f else None, argmin=am)
        assert bool(torch.isinf(dh[0])) and float(dh[1]) == 0.0, dh
    model.close()


@pytest.mark.parametrize("precision,most", [("fp64", 40960), ("fp32", 196608)])
@pytest.mark.parametrize("m", [1, 7, 9, 60, 127])
def test_point_gradients_of_an_infinite_softmin_variance(precision, most, m):
    """The eight lanes of a point give an infinity or NaN where the one thread of a larger call
    gives it, which sums the cell's own samples only."""
    print(f"[gpu-case] point gradients of an infinite variance {precision} m={m}", flush=True)
    model, q = _one_cell(m, precision)
    n, reps = len(q), most // len(q) + 1
    one, am = torch.ones(n, dtype=q.dtype, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    a, _ = model.backward(q, None, one, None, one, argmin=am)
    b, _ = model.backward(q.repeat(reps, 1), None, one.repeat(reps), None, one.repeat(reps), argmin=am.repeat(reps))
    b = b[:n]
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
    assert not bool(torch.isfinite(a).all())
    model.close()
