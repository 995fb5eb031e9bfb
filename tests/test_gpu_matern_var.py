"""The Matern backward's variance term: d var / d z_i is a difference of terms that mostly cancel,
added per sample in both forms of the FP32 kernel."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m_max", [1, 7, 16, 64, 128])
def test_a_variance_cotangent_alone(m_max):
    """Eight lanes per point (4,001 points) are as near the FP64 model as one thread per point
    (200,050), and with one sample a cell, whose variance does not depend on the point, give 0."""
    print(f"[gpu-case] Matern variance cotangent m<={m_max}", flush=True)
    wl = scenes.small_room_workload(n_queries=4001, cfg_id=47, uneven=True)
    p = wl.points.astype(np.float32)
    cells = ksdf.build_cells(p, wl.origin, wl.h, wl.margin, m_max, 1)
    out, argmin = {}, None
    for precision, dt, reps in (("fp64", torch.float64, 1), ("fp32", torch.float32, 1), ("fp32", torch.float32, 50)):
        model = ksdf.Model(cells, len(p), wl.origin, wl.h, ell=wl.ell, noise_var=wl.noise_var, precision=precision,
                           kernel="matern32", adjoint=True)
        model.fit(torch.from_numpy(p).to("cuda", dt))
        q = torch.from_numpy(wl.queries.astype(np.float32)).to("cuda", dt)
        if argmin is None:
            argmin = model.query(q)["argmin"].clone()
        one = torch.ones(len(q) * reps, dtype=dt, device="cuda")
        dx, _ = model.backward(q.repeat(reps, 1), None, torch.zeros_like(one), None, one, argmin=argmin.repeat(reps))
        out[precision, reps] = dx[:len(q)].double()
        model.close()
    if m_max == 1:
        assert not bool(out["fp32", 1].any()) and not bool(out["fp32", 50].any())
        return
    err = {k: float((v - out["fp64", 1]).norm() / out["fp64", 1].norm()) for k, v in out.items()}
    print(f"off FP64: eight lanes {err['fp32', 1]:.2e}, one thread {err['fp32', 50]:.2e}", flush=True)
    assert err["fp32", 1] <= 1.02 * err["fp32", 50]
