"""GPU sign from local BHM weights (eq. sign_prediction) and the threshold update
(eq. online_surf_logodds) against the oracle, on synthetic weights for the small room.
Double points: log-odds within 1e-12 (FP64, a different summation order: the GPU
separates the RBF by axis).  Float points (FP32 arithmetic with a compensated outer
sum): log-odds within 100 float roundings of sum |w_h k(x, h)| (the FP32 exp and the
products and inner sums carry a few roundings each).  Signs identical wherever |l - tau|
exceeds the tolerance, and the sign feeding a query."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_29227_amd import ksdf, scenes
from tests.bhm_bound import abs_terms

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-case] {msg}", flush=True)


def _setup(hinges=7):
    wl = scenes.small_room_workload(n_queries=20000)
    b = scenes.bhm_weights(wl, hinges=hinges)
    rng = np.random.default_rng(3)
    near = wl.points[rng.choice(len(wl.points), 20000)] + rng.normal(0, 0.02, (20000, 3))
    q = np.concatenate([near, wl.queries.astype(np.float64)])
    return wl, b, q


def _args(b):
    return (b["origin"], b["box"], b["dims"], b["hinges"], b["gamma"],
            torch.from_numpy(b["box_bhm"]).cuda(), torch.from_numpy(b["weights"]).cuda())


@pytest.mark.parametrize("dtype,hinges", [(torch.float64, 7), (torch.float32, 7), (torch.float32, 5)])
def test_bhm_sign_matches_oracle(dtype, hinges):
    """7 hinges per axis runs the FP32 form unrolled for that count; 5 the general one."""
    _say(f"bhm sign {dtype}, {hinges} hinges per axis")
    wl, b, q = _setup(hinges)
    qt = torch.from_numpy(q).to("cuda", dtype)
    qd = qt.double().cpu().numpy()
    for tau in (0.0, 0.3):
        sign, lo = ksdf.bhm_sign(qt, *_args(b), tau=tau, logodds=True)
        torch.cuda.synchronize()
        olo, have, osign = oracle.bhm(qd, b["origin"], b["box"], b["dims"], b["hinges"],
                                      b["gamma"], b["box_bhm"], b["weights"], tau=tau)
        g = lo.cpu().numpy()
        h = have == 1
        assert np.all(np.isneginf(g[~h]))
        tol = 1e-12 if dtype == torch.float64 else 100 * 2.0 ** -24 * abs_terms(qd, b)
        err = np.abs(g[h] - olo[h])
        print(f"bhm {dtype} tau {tau}: max |dl| {err.max():.3g}, max |dl| / tol "
              f"{(err / np.broadcast_to(tol, g.shape)[h]).max():.3g}", flush=True)
        assert np.all(err <= np.broadcast_to(tol, g.shape)[h])
        s = sign.cpu().numpy().astype(np.int32)
        clear = ~h | (np.abs(olo - tau) > tol)
        print(f"ambiguous signs: {int((~clear).sum())} of {len(s)}", flush=True)
        assert np.array_equal(s[clear], osign[clear])
        assert h.mean() > 0.3 and (osign == -1).any() and (osign == 1).any()


def test_bhm_tau_update_and_query_sign():
    _say("bhm tau update, sign into a query")
    wl, b, q = _setup()
    hits = torch.from_numpy(np.asarray(wl.points[:5000], np.float32)).cuda()
    tau = torch.tensor([0.4], dtype=torch.float64, device="cuda")
    ksdf.bhm_update_tau(hits, *_args(b), 0.25, tau)
    torch.cuda.synchronize()
    olo, _, _ = oracle.bhm(hits.double().cpu().numpy(), b["origin"], b["box"], b["dims"],
                           b["hinges"], b["gamma"], b["box_bhm"], b["weights"])
    # float hits: FP32 log-odds (tolerance as above), summed in float-float
    tol = 100 * 2.0 ** -24 * abs_terms(hits.double().cpu().numpy(), b).mean() * 0.25 + 1e-12
    assert float(tau.item()) == pytest.approx(oracle.bhm_update_tau(0.4, olo, 0.25), abs=tol)
    tau64 = torch.tensor([0.4], dtype=torch.float64, device="cuda")
    ksdf.bhm_update_tau(hits.double(), *_args(b), 0.25, tau64)
    torch.cuda.synchronize()
    assert float(tau64.item()) == pytest.approx(oracle.bhm_update_tau(0.4, olo, 0.25), abs=1e-12)
    # the sign goes straight into the query: d = s u
    cells = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, wl.m_max, wl.m_min)
    model = ksdf.Model(cells, len(wl.points), wl.origin, wl.h, ell=wl.ell, noise_var=wl.noise_var)
    model.fit(torch.from_numpy(wl.points).cuda())
    qt = torch.from_numpy(wl.queries).cuda()
    sign = ksdf.bhm_sign(qt, *_args(b), tau=float(tau.item()))
    out = model.query(qt, sign)
    plain = model.query(qt)
    torch.cuda.synchronize()
    assert torch.equal(out["mean"], plain["mean"] * sign.float())
    model.close()


@pytest.mark.parametrize("dtype,hinges", [(torch.float64, 7), (torch.float32, 7), (torch.float32, 5)])
def test_bhm_sign_does_not_depend_on_the_call(dtype, hinges):
    """A point's log-odds have the same bits whether its workgroup meets a few maps (staged in
    LDS), more than it has room for, or only this point, and in the sorted form (up to 2^21
    points) or the gathered one; points on the boxes' faces, far away, infinite or NaN are +1 or in
    the box that the FP64 quotient's floor names."""
    _say(f"bhm sign in several calls {dtype} {hinges}")
    wl, b, q = _setup(hinges)
    q = q[:9001]
    key = np.floor((q - np.asarray(b["origin"])) / b["box"])
    q[:500] = np.asarray(b["origin"]) + key[:500] * b["box"]                 # corners of boxes
    q[500:506] = [[np.inf, 0, 0], [-np.inf, 1, 1], [np.nan, 0, 0], [1e30, 1, 1], [-3e9, 1, 1], [1, 1, 1e12]]
    key = np.where(np.isfinite(q), np.floor((q - np.asarray(b["origin"])) / b["box"]), 0)
    order = np.lexsort(key.T)
    qt = torch.from_numpy(q[order]).to("cuda", dtype)
    args = _args(b)
    sign, lo = ksdf.bhm_sign(qt, *args, logodds=True)                        # neighbours share maps
    assert bool((sign[torch.isneginf(lo)] == 1).all())
    x = qt.double().cpu().numpy()
    k = np.floor((x - np.asarray(b["origin"])) / b["box"])
    inside = np.all(np.isfinite(x) & (k >= 0) & (k < np.asarray(b["dims"])), axis=1)
    flat = np.ravel_multi_index(k[inside].astype(np.int64).T, b["dims"])
    have = np.zeros(len(x), bool)
    have[inside] = b["box_bhm"][flat] >= 0
    fin = np.isfinite(x).all(1)
    assert np.array_equal(~np.isneginf(lo.cpu().numpy())[fin], have[fin])
    mix = torch.from_numpy(np.random.default_rng(1).permutation(len(q))).cuda()
    s2, l2 = ksdf.bhm_sign(qt[mix].contiguous(), *args, logodds=True)        # and mostly do not
    many = qt.repeat((1 << 21) // len(q) + 1, 1)
    s3, l3 = ksdf.bhm_sign(many, *args, logodds=True)
    one = [ksdf.bhm_sign(qt[i:i + 1].contiguous(), *args, logodds=True) for i in range(0, len(q), 600)]
    bits = lambda t: t.contiguous().view(torch.int64)   # noqa: E731
    assert torch.equal(s2, sign[mix]) and torch.equal(bits(l2), bits(lo[mix]))
    n = len(many) // len(q)
    s4, l4 = ksdf.bhm_sign(many[torch.randperm(len(many), device="cuda", generator=torch.Generator("cuda").manual_seed(2))],
                           *args, logodds=True)
    assert torch.equal(bits(l4).sort()[0], bits(l3).sort()[0]) and int(s4.sum()) == int(s3.sum())
    assert torch.equal(s3, sign.repeat(n)) and torch.equal(bits(l3), bits(lo.repeat(n)))
    for i, (s, l) in zip(range(0, len(q), 600), one):
        assert int(s[0]) == int(sign[i]) and torch.equal(bits(l), bits(lo[i:i + 1]))
