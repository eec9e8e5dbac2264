"""Host-only checks of the planner: fp32 tile numbers that run on a ring tile
are planned in that tile's K-stages (workspace queries, no launch)."""
import ctypes

import pytest

from paper_2602_00125_amd import binding as b


def _t(shape, ptr):
    t = b.MtTensor()
    t.data, t.dtype, t.ndim = ptr, 0, len(shape)
    stride = 1
    for i in reversed(range(len(shape))):
        t.shape[i], t.stride[i] = shape[i], stride
        stride *= shape[i]
    return t


def _dw_workspace(cfg, M, N, K):
    n, g = ctypes.c_size_t(0), 1 << 32
    x, w, dy, dw = _t([M, K], g), _t([N, K], 2 * g), _t([M, N], 3 * g), _t([N, K], 4 * g)
    b.debug_set("cfg", cfg)
    b.debug_set("splits", 64)
    try:
        r = ctypes.byref
        assert b.lib.mt_linear_bwd_workspace(r(x), r(w), r(dy), None, r(dw), None, r(n)) == 0
    finally:
        b.debug_set("cfg", -1)
        b.debug_set("splits", 0)
    return n.value


@pytest.mark.parametrize("cfg,ring", [(0, 6), (1, 8), (2, 9), (3, 10), (5, 6)])
@pytest.mark.parametrize("M", [64, 96, 1000])
def test_fp32_tiles_are_planned_as_the_ring_tiles_they_run_on(cfg, ring, M):
    assert _dw_workspace(cfg, M, 512, 256) == _dw_workspace(ring, M, 512, 256) > 0
