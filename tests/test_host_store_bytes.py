"""A model's store holds the arrays of its own precision only (host query, no GPU)."""
from paper_2603_29227_amd import ksdf, scenes
from tests.test_abi import _bytes


def test_an_fp32_store_holds_no_fp64_arrays():
    wl = scenes.small_room_workload(n_queries=8)
    c = ksdf.build_cells(wl.points, wl.origin, wl.h, wl.margin, wl.m_max, wl.m_min)
    nnz, factor = int(c.offsets[-1]), int((c.m.astype(int) * (c.m + 1) // 2).sum())
    f32, f64 = _bytes(c, wl), _bytes(c, wl, precision=ksdf.FP64)
    # per factor entry 4 against 8 bytes; per sample (p, a), their low parts and sigma^2, 36,
    # against (p, a) and sigma^2, 40; the rest is equal but for a list of the cells and padding
    assert abs((f64 - f32) - (4 * factor + 4 * nnz)) < 8 * c.n + 8192
