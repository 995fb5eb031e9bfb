"""A cell's outputs come from its own samples: what lies behind its last one in memory, another
cell's samples or past the last cell whatever the memory held before, takes no part."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes

pytestmark = pytest.mark.gpu


def _fill_free_memory(value):
    """Blocks that the next allocations are cut from, full of value."""
    torch.cuda.empty_cache()
    blocks = [torch.full((1 << 16,), value, device="cuda") for _ in range(64)]
    blocks.append(torch.full((1 << 24,), value, device="cuda"))
    torch.cuda.synchronize()
    del blocks


@pytest.mark.parametrize("m", [1, 3, 7, 9, 61, 127])
def test_gradients_do_not_read_past_the_last_cell(m):
    """One cell, whose points take eight lanes each in a call of 64 and one thread in a call of
    more than 196,608: the same bits, and finite, wherever the model's memory has been."""
    print(f"[gpu-case] memory past the last cell, m={m}", flush=True)
    rng = np.random.default_rng(m)
    p = np.array([0.5, 0.5, 0.5]) + rng.uniform(0.05, 0.3, (m, 3)) * rng.choice([-1, 1], (m, 3))
    cells = ksdf.CellSet(np.array([0, m], np.int32), np.arange(m, dtype=np.int32), np.zeros((1, 3), np.int32))
    q = torch.from_numpy(rng.uniform(0.1, 0.9, (64, 3))).to("cuda", torch.float32)
    pts = torch.from_numpy(p).to("cuda", torch.float32)
    n, reps = len(q), 196608 // len(q) + 1
    one, am = torch.ones(n, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    many = (q.repeat(reps, 1), None, one.repeat(reps), None, one.repeat(reps))
    for value in (float("nan"), float("inf"), 1e30):
        _fill_free_memory(value)
        model = ksdf.Model(cells, m, (0.0, 0.0, 0.0), 1.0, ell=0.2, k_fuse=1, noise_var=1e-4, adjoint=True)
        model.fit(pts)
        few, _ = model.backward(q, None, one, None, one, argmin=am)
        dx, dh = model.backward(*many, argmin=am.repeat(reps))
        assert bool(torch.isfinite(dx).all()) and bool(torch.isfinite(dh).all()), value
        assert torch.equal(dx.view(reps, n, 3)[0], few) and torch.equal(dx.view(reps, n, 3)[-1], few)
        model.close()


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("m_max", [7, 13, 61, 127])
@pytest.mark.parametrize("form", [None, dict(query_split=0), dict(query_split=1, query_lanes=0),
                                  dict(query_split=1, query_lanes=1)])
def test_an_infinite_variance_stays_in_its_cell(form, m_max, kernel):
    """A sample of infinite variance has no part in another cell's softmin variance, in each form
    of the query (None: eight lanes a point)."""
    print(f"[gpu-case] infinite variance {form} m<={m_max} {kernel}", flush=True)
    wl = dataclasses.replace(scenes.sphere_workload(n_samples=9000, n_queries=4001), m_max=m_max)
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, m_max, 1)
    n = len(wl.points)
    # the first sample of every third cell, the last one of every fifth
    at = np.full(n, False)
    for c in range(cells.n):
        s = cells.samples[cells.offsets[c]:cells.offsets[c + 1]]
        at[s[0]] |= c % 3 == 0
        at[s[-1]] |= c % 5 == 0
    holds = np.logical_or.reduceat(at[cells.samples], cells.offsets[:-1])
    assert 0 < holds.sum() < cells.n
    gone = torch.from_numpy(at).cuda()
    pts, q = (torch.from_numpy(x).to("cuda", torch.float32) for x in (wl.points, wl.queries))
    if form and form["query_split"]:
        q = q.repeat(49, 1)   # 196,049 points
    model = ksdf.Model(cells, n, wl.origin, wl.h, ell=wl.ell, noise_var=wl.noise_var, kernel=kernel)
    out = []
    for big in (float("inf"), 1e30):
        model.fit(pts, torch.where(gone, big, wl.noise_var).to(torch.float32))
        if form:
            model.set_tuning(**form)
        out.append({k: v.clone() for k, v in model.query(q, grad_var=True).items()})
    a, b = out
    has = a["argmin"] >= 0
    assert torch.equal(a["argmin"], b["argmin"]) and int(has.sum()) > 1000
    there = torch.from_numpy(holds).cuda()[a["argmin"].clamp_min(0).long()] & has
    assert int(there.sum()) > 100 and int((has & ~there).sum()) > 100
    for k in ("var", "grad_var"):
        assert torch.equal(a[k][has & ~there], b[k][has & ~there]), k
    model.close()
