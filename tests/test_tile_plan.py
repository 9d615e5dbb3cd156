"""Host-only tests of the decomposition of the matrix products
(regenvc_linear_plan_query, regenvc_vae_conv3d_plan_query): the queries make
no HIP call, so a device of 256 compute units is assumed."""
import ctypes

import pytest

from paper_2607_28144_amd import _lib

N_CU = 256
ALL = 2 ** 63 - 1  # as much workspace as the call can use


def linear_plan(M, N, K, epi, ws=ALL, n_cu=N_CU):
    p = _lib.TilePlan()
    _lib.check(_lib.load().regenvc_linear_plan_query(M, N, K, epi, n_cu, ws, ctypes.byref(p)), "plan query")
    return p.rows, p.cols, p.waves, p.k_ranges


def conv_plan(T, H, W, Cin, Cout, ws=ALL, n_cu=N_CU):
    p = _lib.TilePlan()
    _lib.check(_lib.load().regenvc_vae_conv3d_plan_query(T, H, W, 1, Cin, Cout, n_cu, ws, ctypes.byref(p)), "plan query")
    return p.rows, p.cols, p.waves, p.k_ranges


def linear_bytes(M, N, K, epi):
    b = ctypes.c_int64()
    _lib.check(_lib.load().regenvc_linear_workspace(M, N, K, epi, N_CU, ctypes.byref(b)), "workspace query")
    return b.value


def conv_bytes(T, H, W, Cin, Cout):
    b = ctypes.c_int64()
    _lib.check(_lib.load().regenvc_vae_conv3d_workspace(T, H, W, 1, Cin, Cout, N_CU, ctypes.byref(b)), "workspace query")
    return b.value


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(1, 16, 64), (300, 1536, 8960), (1365, 1536, 8960), (700, 1552, 8896), (10920, 4608, 1536),
                                   (65520, 5120, 5120), (300, 16, 1 << 22), (300, 16, 0)])
def test_linear_ranges_and_workspace_agree(M, N, K, epi):
    """One f32 plane of the output per range, at least 8 K steps in each, at
    most 8 ranges, fewer where the workspace holds fewer planes."""
    ranges = linear_plan(M, N, K, epi)[3]
    assert 1 <= ranges <= 8 and (ranges == 1 or K // 64 >= 8 * ranges)
    assert linear_bytes(M, N, K, epi) == (ranges * M * N * 4 if ranges > 1 else 0)
    for planes in range(9):
        assert linear_plan(M, N, K, epi, planes * M * N * 4 + 255)[3] <= max(1, planes)


@pytest.mark.parametrize("T,H,W,Cin,Cout", [(1, 17, 19, 64, 64), (7, 34, 34, 384, 384), (7, 60, 104, 384, 384),
                                            (1, 2, 3, 155392, 64)])
def test_conv_ranges_and_workspace_agree(T, H, W, Cin, Cout):
    rows, cols, _, ranges = conv_plan(T, H, W, Cin, Cout)
    assert 1 <= ranges <= 8 and (ranges == 1 or 27 * Cin // 64 >= 8 * ranges)
    assert conv_bytes(T, H, W, Cin, Cout) == (ranges * T * H * W * Cout * 4 if ranges > 1 else 0)
    for planes in range(9):
        assert conv_plan(T, H, W, Cin, Cout, planes * T * H * W * Cout * 4 + 255)[3] <= max(1, planes)
    if 27 * Cin >= 1 << 22:
        assert (rows, cols) == (128, 128)


def test_bad_queries_are_refused():
    lib, p = _lib.load(), _lib.TilePlan()
    linear = lambda *a: lib.regenvc_linear_plan_query(*a, ctypes.byref(p))  # noqa: E731
    conv = lambda *a: lib.regenvc_vae_conv3d_plan_query(*a, ctypes.byref(p))  # noqa: E731
    for a in [(-1, 16, 64, 0, 256, 0), (1, 16, 64, 3, 256, 0), (1, 16, 64, 0, 0, 0), (1, 16, 64, 0, 256, -1)]:
        assert linear(*a) == _lib.ERR_INVALID_ARG
    assert linear(1, 17, 64, 0, 256, 0) == linear(1, 16, 65, 0, 256, 0) == _lib.ERR_UNSUPPORTED
    assert lib.regenvc_linear_plan_query(1, 16, 64, 0, 256, 0, None) == _lib.ERR_INVALID_ARG
    for a in [(0, 1, 1, 1, 64, 64, 256, 0), (1, 1, 1, 17, 64, 64, 256, 0), (1, 1, 1, 1, 64, 64, 0, 0), (1, 1, 1, 1, 64, 64, 256, -1)]:
        assert conv(*a) == _lib.ERR_INVALID_ARG
    assert conv(1, 1, 1, 1, 65, 64, 256, 0) == _lib.ERR_UNSUPPORTED
    assert lib.regenvc_vae_conv3d_plan_query(1, 1, 1, 1, 64, 64, 256, 0, None) == _lib.ERR_INVALID_ARG


@pytest.mark.parametrize("M,N,K,epi,slow", [
    (32760, 1536, 1536, 2, [(288, 256, 8)]),                  # 218 us; 187 on 256 x 256 by four waves
    (2730, 8960, 1536, 2, [(288, 256, 8)]),                   # 111; 98
    (16384, 4608, 1536, 2, [(288, 256, 8)]),                  # 340; 270 to 325 on the others
    (65520, 2048, 128, 0, [(64, 128, 4), (128, 128, 4)]),     # 88; 76 on 256 x 256 by eight waves
])
def test_tiles_measured_slow_are_not_chosen(M, N, K, epi, slow):
    """Launches for which tiles are known that take 7 to 15 % less time than these."""
    rows, cols, waves, ranges = linear_plan(M, N, K, epi)
    assert (rows, cols, waves) not in slow and ranges == 1


def test_eight_waves_on_256_rows_where_k_is_short():
    assert linear_plan(65520, 2048, 128, 0) == linear_plan(32760, 512, 512, 2) == (256, 256, 8, 1)


TILES = [(64, 128, 4), (128, 128, 4), (128, 192, 4), (160, 256, 4), (192, 192, 4), (256, 256, 4), (256, 256, 8), (288, 256, 8)]
CONV_TILES = [(128, 128, 4), (128, 192, 4), (192, 192, 4), (256, 192, 4), (256, 256, 4)]


def test_the_gpu_tests_run_every_linear_kernel():
    """The shapes of test_linear_on_every_tile are planned as they say, and
    between them reach every kernel: each tile with each epilogue (eight
    waves on 256 rows are never chosen for the GELU), each four-wave tile
    split over K, and the second kernel of a split with each epilogue."""
    from test_gpu_dit import LINEAR_PLANS
    assert [linear_plan(*c[:4]) for c in LINEAR_PLANS] == [c[4] for c in LINEAR_PLANS]
    whole = {(p[:3], epi) for _, _, _, epi, p in LINEAR_PLANS if p[3] == 1}
    assert whole == {(t, e) for t in TILES for e in range(3)} - {((256, 256, 8), 1)}
    assert {p[:3] for *_, p in LINEAR_PLANS if p[3] > 1} == {t for t in TILES if t[2] == 4}
    assert {epi for _, _, _, epi, p in LINEAR_PLANS if p[3] > 1} == {0, 1, 2}


def test_the_gpu_tests_run_every_convolution_kernel():
    """The same for test_conv_tiles, which runs each shape with and without
    the activation."""
    from test_gpu_vae import CONV_PLANS
    assert [conv_plan(*c[:5]) for c in CONV_PLANS] == [c[5] for c in CONV_PLANS]
    for split in (False, True):
        assert {p[:3] for *_, p in CONV_PLANS if (p[3] > 1) == split} == set(CONV_TILES)
    assert any(27 * c[3] >= 1 << 22 for c in CONV_PLANS)
