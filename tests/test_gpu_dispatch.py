"""Which form answers an FP32 query, by the kernel, K, the cells' samples and the points per cell:
seen from the parts of the caller's workspace that the call has written (nothing: eight lanes a
point in the caller's order; the sort: eight lanes a point, sorted; the regrouped records too:
two kernels)."""
import numpy as np
import pytest
import torch

from paper_2603_29227_amd import scenes
from tests.test_gpu_group import OUT, _fitted, _sphere

pytestmark = pytest.mark.gpu


def _form(model, q):
    n = len(q)
    size = model._lib.ksdf_query_workspace_bytes(model._h, n)
    ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
    out = model.query(q, workspace=ws, grad_var=True)
    up = lambda v: -(-v // 256) * 256   # noqa: E731
    nc = model.n_cells + 1
    tail = 2 * up(4 * nc) + up(4 * (-(-nc // 4096)))
    records = ws[size - tail - up(16 * n):size - tail]   # the regrouped records
    if bool((records != 0xA5).any()):
        return "two", out
    return "sorted" if bool((ws != 0xA5).any()) else "unsorted", out


# the sphere has 80 cells (dense), the room 4,434
CASES = [("sphere", 32, 8, "rbf", [(131072, "unsorted"), (196608, "sorted"), (196609, "two")]),
         ("sphere", 64, 8, "rbf", [(131072, "unsorted"), (147456, "sorted"), (147457, "two")]),
         ("sphere", 64, 16, "rbf", [(131072, "unsorted"), (147457, "two")]),
         ("room", 64, 16, "rbf", [(147457, "sorted"), (196608, "sorted"), (196609, "two")]),
         ("sphere", 128, 8, "rbf", [(65536, "unsorted"), (65537, "sorted"), (98304, "sorted"), (98305, "two")]),
         ("room", 128, 8, "rbf", [(98305, "sorted"), (147456, "sorted"), (147457, "two")]),
         ("sphere", 32, 8, "matern32", [(131072, "unsorted"), (131073, "two")]),
         ("sphere", 64, 8, "matern32", [(65536, "unsorted"), (65537, "two")]),
         ("room", 128, 8, "matern32", [(57344, "unsorted"), (57345, "two")])]


@pytest.mark.parametrize("scene,m_max,k_fuse,kernel,at", CASES)
def test_form_by_size(scene, m_max, k_fuse, kernel, at):
    print(f"[gpu-case] dispatch {scene} m<={m_max} k={k_fuse} {kernel}", flush=True)
    if scene == "sphere":
        wl = _sphere(m_max, n_samples=20000, n_queries=4099)
    else:
        wl = scenes.small_room_workload(n_queries=4099, cfg_id=47, uneven=m_max > 64)
    model, cells = _fitted(wl, k_fuse=k_fuse, kernel=kernel)
    assert (cells.m.max() > 64) == (m_max > 64) and (scene == "room" or cells.m.max() == m_max)
    most = max(n for n, _ in at)
    q = torch.from_numpy(np.tile(wl.queries, (-(-most // 4099), 1))[:most]).cuda()
    model.set_tuning(query_split=0)
    want = model.query(q, grad_var=True)
    model.set_tuning(query_split=1)
    for n, form in at:
        got, out = _form(model, q[:n].contiguous())
        assert got == form, (n, got)
        for k in OUT:
            assert torch.equal(out[k], want[k][:n]), (n, k)
    model.close()
