"""A cell's outputs come from its own samples: what lies behind its last one in memory, another
cell's samples or past the last cell whatever the memory held before, takes no part."""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import ksdf

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
