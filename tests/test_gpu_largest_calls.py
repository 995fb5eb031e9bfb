"""Calls whose kernels take more threads than one launch holds (2^32): FP64 queries and
backwards of 2^29 points and more, with eight lanes a point, and the dA/dl of 2^24 cells, with a
workgroup a cell."""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes

pytestmark = pytest.mark.gpu

N = 4099
REPS = (1 << 29) // N + 2


def _model(precision, kernel):
    wl = scenes.sphere_workload(n_samples=300, n_queries=N)
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, 4, 1)
    dt = torch.float64 if precision == "fp64" else torch.float32
    model = ksdf.Model(cells, len(wl.points), wl.origin, wl.h, ell=wl.ell, noise_var=wl.noise_var, k_fuse=1,
                       precision=precision, kernel=kernel, adjoint_var_f=True)
    model.fit(torch.from_numpy(wl.points).to("cuda", dt))
    return model, torch.from_numpy(wl.queries).to("cuda", dt)


def test_fp64_query():
    print("[gpu-case] FP64 query of 2^29 points", flush=True)
    model, q = _model("fp64", "rbf")
    want = model.query(q, var_f=False, status=False)
    got = model.query(q.repeat(REPS, 1), var_f=False, status=False)
    assert len(got["mean"]) > 1 << 29
    for k in ("mean", "grad", "var", "argmin"):
        assert bool((got[k].view(REPS, *want[k].shape) == want[k]).all()), k
    model.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("precision,kernel", [("fp64", "rbf"), ("fp32", "rbf"), ("fp32", "matern32")])
def test_backward_with_var_f(precision, kernel):
    print(f"[gpu-case] backward of 2^29 points {precision} {kernel}", flush=True)
    model, q = _model(precision, kernel)
    one = torch.ones(N, dtype=q.dtype, device="cuda")
    am = model.query(q)["argmin"]
    want, _ = model.backward(q, None, one, None, None, one, argmin=am)
    got, _ = model.backward(q.repeat(REPS, 1), None, one.repeat(REPS), None, None, one.repeat(REPS),
                            argmin=am.repeat(REPS))
    assert bool((got.view(REPS, N, 3) == want).all())
    model.close()
    torch.cuda.empty_cache()


def test_fit_with_the_matrix_derivatives():
    print("[gpu-case] fit of 2^24 cells with dA/dl", flush=True)
    side = 256
    keys = np.stack(np.meshgrid(*[np.arange(side, dtype=np.int32)] * 3, indexing="ij"), -1).reshape(-1, 3)
    n = len(keys)
    cells = ksdf.CellSet(np.arange(n + 1, dtype=np.int32), np.zeros(n, np.int32), keys)
    model = ksdf.Model(cells, 1, (0.0, 0.0, 0.0), 1.0, k_fuse=1, adjoint_var_f=True)
    status = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    model.fit(torch.full((1, 3), 0.5, device="cuda"), cell_status=status)
    assert int(status.max()) == 0
    model.close()
    torch.cuda.empty_cache()
