"""The box of a point is the floor of the FP64 quotient (x - origin) / box for every edge that a
layout may have, the smallest and largest doubles among them."""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("box", [5e-324, 1e-308, 2.5e-308, 7e-308, 1e-300, 1e-280, 0.16, 1e300, 1.1e307])
@pytest.mark.parametrize("copies", [1, 20000])   # the sorted form and, past 2^21 points, the gathered one
def test_box_of_a_point_by_the_quotients_floor(box, copies):
    print(f"[gpu-case] bhm box {box} x {copies}", flush=True)
    dims, nh = (9, 1, 1), 2
    x = []
    for k in range(-2, 13):
        v = float(k) * box
        x += [v] + [np.nextafter(v, s * np.inf) for s in (-1, 1)]
    x = np.array(x)
    pts = np.zeros((len(x), 3))
    pts[:, 0] = x
    maps = np.where(np.arange(9) % 2 == 0, np.arange(9) // 2, -1).astype(np.int32)   # every other box
    weights = torch.ones(5 * (nh ** 3 + 1), dtype=torch.float64, device="cuda")
    q = torch.from_numpy(pts).cuda().repeat(copies, 1)
    sign, lo = ksdf.bhm_sign(q, (0.0, 0.0, 0.0), box, dims, nh, 1e-3, torch.from_numpy(maps).cuda(), weights,
                             logodds=True)
    with np.errstate(over="ignore"):
        key = np.floor(x / box)
    inside = (key >= 0) & (key < 9)
    have = np.where(inside, maps[np.clip(key, 0, 8).astype(int)] >= 0, False)
    lo = lo.cpu().numpy().reshape(copies, -1)
    assert np.array_equal(~np.isneginf(lo), np.broadcast_to(have, lo.shape))
    assert bool((sign.cpu().numpy().reshape(copies, -1)[:, ~have] == 1).all())
