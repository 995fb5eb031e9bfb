"""FP32 fits by size of cell: a cell is factored inside the smallest matrix of 16, 32, 64 or 128
rows that holds it, or a larger one (fit_min_bucket), and the rows past its samples add zeros
only, so its fit has the same bits in each; lists known to the host (fit) or to the device
(refit) give the same fits.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes
from tests.test_gpu_group import OUT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("noise_var", [1e-4, 2e-5])
def test_a_fit_has_the_same_bits_in_every_bucket(kernel, noise_var):
    """noise_var 1e-4: most cells' condition is bounded by their row sums; 2e-5: estimated, and
    many cells go on to FP64."""
    print(f"[gpu-case] fit buckets {kernel} {noise_var}", flush=True)
    wl = scenes.small_room_workload(n_queries=3001, cfg_id=47, uneven=True)
    p = wl.points
    keep = (p[:, 0] > np.median(p[:, 0])) | (np.arange(len(p)) % 24 == 0)   # few samples in half of the cells
    wl = dataclasses.replace(wl, points=np.ascontiguousarray(p[keep]), m_max=128)
    pts = torch.from_numpy(wl.points).cuda()
    q, sg = torch.from_numpy(wl.queries).cuda(), torch.from_numpy(wl.sign).cuda()
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, wl.m_max, 1)
    assert cells.m.min() < 16 and cells.m.max() == 128 and len(set(cells.m.tolist())) > 40
    cot = [torch.rand(*s, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
           for s in ((len(q),), (len(q), 3), (len(q),), (len(q),))]

    def answers(model):
        out = model.query(q, sg, grad_var=True)
        dp, dh = model.backward(q, sg, *cot, argmin=out["argmin"])
        return [out[k] for k in OUT] + [dp, dh]

    model = ksdf.Model(cells, len(pts), wl.origin, wl.h, ell=wl.ell, noise_var=noise_var, kernel=kernel,
                       adjoint_var_f=True)
    model.fit(pts)
    want = answers(model)
    for bucket in (32, 64):
        model.set_tuning(fit_min_bucket=bucket)
        model.fit(pts)
        assert all(torch.equal(a, b) for a, b in zip(answers(model), want)), bucket
    model.set_tuning(fit_min_bucket=16)
    n = len(cells.m)
    model.fit(pts * 0.5)
    ids, count = model.refit(pts, torch.ones(n, device="cuda"), torch.ones(n, device="cuda"), 0.5, n)
    assert int(count) == n
    assert all(torch.equal(a, b) for a, b in zip(answers(model), want))


@pytest.mark.parametrize("kernel", ["rbf", "matern32"])
@pytest.mark.parametrize("m_max,shares", [(1, None), (4, None), (5, None), (8, None), (12, (0.3, 0.3)),
                                          (16, (0.3, 0.05)), (16, (0.05, 0.4))])
def test_cells_of_few_samples(kernel, m_max, shares):
    """Cells of up to 4 and up to 8 samples are factored in matrices of 4 and 8 rows where they are
    many (over 1,024) or no others are fewer than 17: the bits are those of the larger matrices,
    adjoint vectors and dA/dl among them."""
    print(f"[gpu-case] small cells {kernel} m<={m_max} {shares}", flush=True)
    wl = scenes.small_room_workload(n_queries=3001, cfg_id=47, uneven=False)
    cap, lo = None, (0, 0, 0)
    if shares:
        lo, dims = (-4, -4, -4), (64, 64, 32)
        u = np.random.default_rng(3).random(dims)
        cap = np.where(u < shares[0], 1 + (u * 1000).astype(int) % 4,
                       np.where(u < sum(shares), 5 + (u * 1000).astype(int) % 4, m_max)).astype(np.uint8)
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, m_max, 1, cap, lo)
    assert cells.m.max() == m_max
    pts = torch.from_numpy(wl.points).cuda()
    q, sg = torch.from_numpy(wl.queries).cuda(), torch.from_numpy(wl.sign).cuda()
    cot = [torch.rand(*s, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
           for s in ((len(q),), (len(q), 3), (len(q),), (len(q),))]
    model = ksdf.Model(cells, len(pts), wl.origin, wl.h, ell=wl.ell, noise_var=wl.noise_var, kernel=kernel,
                       adjoint_var_f=True)

    def answers(bucket):
        model.set_tuning(fit_min_bucket=bucket)
        model.fit(pts)
        out = model.query(q, sg, grad_var=True)
        return [out[k] for k in OUT] + list(model.backward(q, sg, *cot, argmin=out["argmin"]))

    small, large = answers(16), answers(32)
    assert all(torch.equal(a, b) for a, b in zip(small, large))
    model.close()
