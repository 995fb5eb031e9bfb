"""The box of a point is the floor of the FP64 quotient (x - origin) / box for every edge that a
layout may have, the smallest and largest doubles among them."""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf, scenes

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


@pytest.mark.parametrize("hinges,dtype,most", [(3, torch.float32, 1 << 21), (3, torch.float64, 1 << 21),
                                               (7, torch.float32, 1 << 21), (4, torch.float32, 1 << 23),
                                               (5, torch.float64, 1 << 23), (6, torch.float32, 1 << 23),
                                               (7, torch.float64, 1 << 23), (8, torch.float32, 1 << 23)])
def test_the_forms_agree_where_one_ends(hinges, dtype, most):
    """A point's log-odds have the same bits in a small call and in calls of the most points that
    the sorted form takes and of one more, for each kind of call that has its own limit."""
    print(f"[gpu-case] bhm forms {hinges} {dtype} {most}", flush=True)
    wl = scenes.small_room_workload(n_queries=4099)
    b = scenes.bhm_weights(wl, hinges=hinges)
    args = (b["origin"], b["box"], b["dims"], b["hinges"], b["gamma"], torch.from_numpy(b["box_bhm"]).cuda(),
            torch.from_numpy(b["weights"]).cuda())
    q = torch.cat([torch.from_numpy(wl.points[:4099]), torch.from_numpy(wl.queries)]).to("cuda", dtype)
    sign, lo = ksdf.bhm_sign(q, *args, logodds=True)
    assert not bool(torch.isneginf(lo[:4099]).any()) and bool(torch.isneginf(lo).any())
    reps = most // len(q) + 1
    many = q.repeat(reps, 1)
    for n in (most, most + 1):
        s, l = ksdf.bhm_sign(many[:n].contiguous(), *args, logodds=True)
        assert torch.equal(s, sign.repeat(reps)[:n])
        assert torch.equal(l.view(torch.int64), lo.repeat(reps)[:n].view(torch.int64))
