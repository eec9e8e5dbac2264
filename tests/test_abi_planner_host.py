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


def _workspace(fn, *args):
    n = ctypes.c_size_t(0)
    assert fn(*args, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("n,parts", [(1, 0), (5120, 0), (12288, 0), (12289, 4), (1 << 20, 256)])
def test_a_small_mean_squared_error_is_one_launch(n, parts):
    """(no parts: no second launch adds them)"""
    g = 1 << 32
    p, t = _t([n], g), _t([n], 2 * g)
    assert _workspace(b.lib.mt_mse_loss_workspace, ctypes.byref(p), ctypes.byref(t)) == 4 * parts


@pytest.mark.parametrize("M,N,parts", [(512, 1024, 16), (4096, 1024, 128), (4000, 1001, 32), (300, 8191, 4),
                                       (8192, 8192, 8), (16384, 1024, 64), (20, 64, 0)])
def test_row_slices_of_the_activation_pullback(M, N, parts):
    """About 512 blocks, counted in the columns a block takes (64 where rows
    are odd); 256 where long rows fill every CU by themselves."""
    g = 1 << 36
    z, dy, dz, db = _t([M, N], g), _t([M, N], 2 * g), _t([M, N], 3 * g), _t([N], 4 * g)
    r = ctypes.byref
    assert _workspace(b.lib.mt_act_bwd_workspace, 4, r(z), r(dy), r(dz), r(db)) == 4 * parts * N
