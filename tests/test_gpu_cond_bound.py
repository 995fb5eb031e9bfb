"""The bound that replaces the condition estimate holds where the FP32 solves are reliable only:
with a threshold far above 1e6 the estimate is formed, and cells whose FP32 factor is no longer
of use go on to FP64 although the bound of their condition lies below the threshold."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes

pytestmark = pytest.mark.gpu


def test_a_high_threshold_is_held_against_the_estimate():
    print("[gpu-case] condition estimate above 1e6", flush=True)
    wl = scenes.small_room_workload(n_queries=16, cfg_id=47, uneven=True)
    wl = dataclasses.replace(wl, m_max=128)
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, wl.m_max, 1)
    pts = torch.from_numpy(wl.points).cuda()
    noise = 1e-7   # row sums of up to 128: a bound of 1.3e9

    def refitted(threshold):
        model = ksdf.Model(cells, len(pts), wl.origin, wl.h, ell=wl.ell, noise_var=noise,
                           cond_threshold=threshold)
        st = torch.zeros(cells.n, dtype=torch.uint8, device="cuda")
        model.fit(pts, cell_status=st)
        model.close()
        return (st & ksdf.C_FP64).cpu().numpy().astype(bool)

    failed = refitted(1e30)                       # the cells whose FP32 pivots fail
    at = refitted(10 * 128 / noise)               # beyond every bound (1.25 * 128 / noise)
    below = refitted(2e6)
    assert np.all(at >= failed) and np.all(below >= at)
    print(f"refits: pivots {failed.sum()}, estimate {at.sum()}, threshold 2e6 {below.sum()}", flush=True)
    assert at.sum() > failed.sum()


@pytest.mark.parametrize("uneven,m_max", [(False, 4), (False, 8), (False, 13), (False, 64), (True, 128)])
def test_a_variance_beyond_the_estimate_goes_to_fp64(uneven, m_max):
    """The estimate's squared norms overflow FP32 where a sample's variance is 1e30, and the cell
    goes to FP64, also where its bound is small since every variance is that large."""
    print(f"[gpu-case] variances of 1e30, m<={m_max}", flush=True)
    wl = scenes.small_room_workload(n_queries=16, cfg_id=47, uneven=uneven)
    wl = dataclasses.replace(wl, m_max=m_max)
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, wl.m_max, 1)
    pts = torch.from_numpy(wl.points).cuda()
    rng = np.random.default_rng(3)
    large = np.zeros(len(pts), bool)
    for c in range(0, cells.n, 2):   # whole cells, and single samples of others
        s = cells.samples[cells.offsets[c]:cells.offsets[c + 1]]
        large[s if c % 4 == 0 else rng.choice(s, 1)] = True
    holds = np.logical_or.reduceat(large[cells.samples], cells.offsets[:-1])
    var = torch.from_numpy(np.where(large, 1e30, 1e-2)).to("cuda", pts.dtype)
    model = ksdf.Model(cells, len(pts), wl.origin, wl.h, ell=wl.ell)
    st = torch.zeros(cells.n, dtype=torch.uint8, device="cuda")
    model.fit(pts, var, cell_status=st)
    model.close()
    assert np.array_equal((st & ksdf.C_FP64).cpu().numpy().astype(bool), holds)
