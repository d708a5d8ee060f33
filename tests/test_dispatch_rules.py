"""Rules that pick between two kernels for one call, against the faster of the two as measured (host computations of the library,
no device work)."""
import os

import pytest


@pytest.fixture(scope="module")
def libqii():
    from paper_2601_22813_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build(force=True)
    return binding


# whole MS-EDEN calls along the columns of a bf16 matrix, us: abs-max by column blocks, by 128 x 128 tiles, with one cleared word and atomics in
# both, as qii_absmax measures (a quantizer call whose blocks leave words goes by WORDS_US); shapes where the two differ by more than their
# repeated runs do
ABSMAX_US = {
    (128, 8192): (12.7, 10.8), (1024, 2048): (13.0, 12.5), (4096, 512): (13.0, 12.5), (128, 16384): (15.5, 11.8),
    (3328, 1024): (12.8, 14.3), (2048, 2048): (14.6, 15.7), (896, 8192): (15.8, 17.9), (4096, 2048): (17.0, 18.8),
    (8320, 2048): (32.9, 35.6), (8704, 2048): (34.7, 36.0), (2176, 8192): (25.9, 30.2), (1152, 16384): (27.8, 32.4),
    (3712, 5120): (26.9, 32.5), (4096, 5120): (27.5, 32.6), (20480, 1024): (27.3, 31.5), (3712, 6144): (31.3, 35.0),
    (28672, 1024): (34.2, 35.3), (2176, 16384): (42.8, 44.6), (5376, 4096): (39.8, 36.8), (10240, 2048): (38.0, 36.0),
    (22528, 1024): (43.0, 37.6), (6144, 5120): (51.8, 43.4), (4096, 8192): (41.1, 37.5), (8448, 4096): (52.8, 49.1),
    (5120, 8192): (47.5, 45.2), (10240, 4096): (61.0, 52.9), (8192, 8192): (66.0, 62.6),
}


@pytest.mark.parametrize("rows,cols", ABSMAX_US)
def test_the_faster_abs_max_pass_along_columns(libqii, rows, cols):
    columns, tiles = ABSMAX_US[rows, cols]
    assert bool(libqii.lib().qii_absmax_takes_tiles(rows, cols)) == (tiles < columns)


# whole quantizer calls that measure their tensor, us: one maximum, cleared by a launch and kept by atomics; a word per block.  f32 or
# not, rows, cols, along the columns or not, rotation
F32, BF16 = 0, 1
WORDS_US = {   # (MS-EDEN or SR with the rotation, RTN, 4/6 or SR without)
    # along the rows: the row quads that a wave takes one after the other decide, not the elements
    (BF16, 32382, 128, 0, 128): (29.93, 57.03), (BF16, 20480, 128, 0, 128): (22.43, 37.70), (F32, 16384, 256, 0, 128): (19.96, 31.25),
    (BF16, 10239, 256, 0, 128): (21.46, 26.57), (F32, 7038, 384, 0, 128): (15.33, 17.85), (BF16, 4685, 768, 0, 128): (17.26, 18.22),
    (BF16, 510, 5376, 0, 128): (12.56, 12.89), (BF16, 512, 7040, 0, 128): (12.72, 12.41), (BF16, 184, 13056, 0, 128): (12.04, 11.91),
    (F32, 381, 9600, 0, 128): (13.98, 13.37), (BF16, 640, 1664, 0, 128): (9.48, 8.70), (F32, 126, 640, 0, 128): (8.78, 7.28),
    (BF16, 31439, 16, 0, 0): (16.98, 20.81), (BF16, 25389, 48, 0, 0): (17.17, 18.69), (F32, 28064, 96, 0, 0): (21.36, 29.30),
    (F32, 13967, 80, 0, 0): (19.54, 21.97), (BF16, 12445, 256, 0, 0): (16.82, 16.22), (BF16, 7902, 144, 0, 0): (14.48, 11.65),
    (F32, 245, 14464, 0, 128): (11.17, 13.03), (F32, 10357, 32, 0, 0): (16.51, 14.73), (BF16, 16510, 144, 0, 0): (19.29, 18.23), (F32, 12663, 32, 0, 0): (14.99, 13.87),
    (F32, 7549, 16, 0, 0): (12.93, 10.43), (F32, 5598, 192, 0, 0): (12.58, 10.20),
    # along the columns of bf16 matrices that the 128 x 128 tiles take
    (BF16, 5760, 512, 1, 128): (11.56, 13.17), (BF16, 4352, 896, 1, 128): (12.58, 13.89), (BF16, 1664, 1408, 1, 128): (13.13, 14.32),
    (BF16, 18560, 128, 1, 128): (11.60, 13.00), (BF16, 9984, 384, 1, 128): (13.72, 14.70), (BF16, 256, 16000, 1, 128): (14.98, 14.72),
    (BF16, 384, 5760, 1, 128): (14.32, 14.03), (BF16, 2048, 2048, 1, 128): (14.31, 13.32), (BF16, 1408, 2816, 1, 128): (19.11, 17.77),
    (BF16, 13184, 256, 1, 128): (15.31, 14.51), (BF16, 1536, 2304, 1, 128): (15.61, 14.58), (BF16, 14848, 256, 1, 128): (14.26, 13.42),
    (BF16, 7936, 128, 1, 128): (13.30, 11.51), (BF16, 640, 2944, 1, 128): (12.38, 11.30),
}


@pytest.mark.parametrize("call", WORDS_US)
def test_blocks_leave_words_where_that_is_faster(libqii, call):
    clearing, words = WORDS_US[call]
    n = libqii.lib().qii_absmax_words(*call)
    assert 0 <= n <= 64
    assert (n > 0) == (words < clearing)


# whole post hoc calls along the rows of a bf16 matrix, us: a wave per row, a wave per four rows
ROWS_US = {
    (1023, 1024): (8.15, 10.19), (2559, 1024): (9.86, 10.42), (3071, 1024): (10.01, 10.52), (3583, 1024): (10.83, 10.63),
    (4799, 1024): (12.55, 12.15), (1535, 2048): (9.94, 10.52), (1999, 2048): (10.89, 10.59), (339, 2304): (8.73, 10.14), (679, 2304): (9.86, 10.35),
    (1191, 2304): (12.57, 11.91), (1331, 2304): (12.59, 11.93), (679, 2560): (9.89, 10.36), (851, 2560): (10.59, 10.41), (1023, 2560): (10.81, 10.55),
    (1331, 2560): (12.57, 12.06), (679, 3072): (9.89, 10.30), (1023, 3072): (10.67, 10.50), (1331, 3072): (12.79, 12.05), (767, 4096): (9.94, 10.57),
    (895, 4096): (10.80, 10.57), (611, 5120): (10.04, 10.57), (715, 5120): (10.69, 10.58), (511, 6144): (10.03, 10.53), (663, 6144): (10.88, 10.64),
    (435, 7168): (9.89, 10.53), (567, 7168): (10.82, 10.66), (383, 8192): (9.93, 10.55), (447, 8192): (10.79, 10.59),
}


@pytest.mark.parametrize("rows,cols", ROWS_US)
def test_the_faster_wave_of_the_post_hoc_quantizer(libqii, rows, cols):
    one, four = ROWS_US[rows, cols]
    assert libqii.lib().qii_rows_per_wave(rows, cols, libqii.MS_EDEN_PH) == (1 if one < four else 4)


MAIN, NO_WORKSPACE, T64, T128, T128_WIDE = range(5)


def scales_bytes(M, N, K):
    return ((M + 255) // 256 * 256 + (N + 255) // 256 * 256) * (K // 16)


@pytest.mark.parametrize("M,N,K", [(512, 128, 26624), (300, 520, 30720), (256, 256, 32768), (2816, 2048, 16384), (8448, 2048, 8192)])
def test_a_route_is_priced_for_the_workspace_it_has(libqii, M, N, K):
    """These products share the tiles of their last round between blocks, partial tiles in the workspace.  Where that holds the
    scales only, the main kernel would run one block per tile (512 x 128 x 26624: 433 us; 64 x 64 tiles 78, shared 70)."""
    L = libqii.lib()
    full = libqii.qii_gemm_workspace_bytes(M, N, K)
    assert full > scales_bytes(M, N, K)
    assert L.qii_gemm_route(M, N, K, full, 0) == MAIN
    for too_small in (scales_bytes(M, N, K), full - 256):
        assert L.qii_gemm_route(M, N, K, too_small, 0) == L.qii_gemm_route(M, N, K, 0, 0) != MAIN


# products of one or two 256 x 256 tiles, us: 64 x 64 tiles, the shared main kernel (its re-tiling launch included)
SHARED_US = {
    (128, 128, 19968): (60.6, 55.6), (128, 128, 24320): (71.2, 59.5), (256, 128, 22528): (66.3, 60.2), (256, 256, 19456): (58.4, 56.9),
    (256, 256, 24320): (72.1, 61.2), (256, 512, 19712): (61.2, 58.9), (256, 512, 22784): (70.1, 62.9), (384, 256, 22272): (66.6, 62.3),
}


@pytest.mark.parametrize("M,N,K", SHARED_US)
def test_one_or_two_shared_tiles_are_priced_without_spans(libqii, M, N, K):
    """No block's range of such a plan spans two tiles, whatever its length, so that no block stores two partial tiles."""
    import ctypes
    L = libqii.lib()
    small, main = SHARED_US[M, N, K]
    route = L.qii_gemm_route(M, N, K, libqii.qii_gemm_workspace_bytes(M, N, K), 0)
    assert main < small and route == MAIN
    plan = (ctypes.c_int32 * 3)()
    L.qii_gemm_sharing_plan(ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int64(K), plan)
    segments = (ctypes.c_int32 * 64)()
    assert plan[0] == 0 and plan[1] in (1, 2)
    assert all(L.qii_gemm_sharing_segments(plan[1], K // 256, plan[2], b, segments) == 1 for b in range(plan[2]))


# whole backward passes T x d_in -> d_out in bf16, us: dX and dW in a launch each, both in one launch of 64 x 64 tiles, of 128 x 128 tiles in
# two and in four K groups
PASS_US = {
    (896, 256, 384): (31.86, 26.69, 32.56, 32.93), (128, 304, 128): (28.56, 23.73, 26.65, 27.79), (512, 512, 256): (28.07, 24.35, 27.42, 28.46),
    (128, 2432, 1408): (31.06, 24.23, 31.57, 30.13), (128, 2048, 3968): (56.59, 48.40, 68.50, 59.84), (1280, 512, 4864): (64.29, 52.29, 72.92, 61.94),
    (896, 1280, 4480): (79.51, 64.96, 78.14, 71.06), (1280, 7552, 2304): (149.26, 155.40, 136.43, 148.79), (896, 3072, 2176): (75.61, 69.47, 64.02, 73.67),
    (1920, 6144, 1408): (128.89, 121.71, 105.75, 118.24), (512, 6528, 512): (46.41, 43.42, 40.05, 47.27), (640, 4992, 896): (50.75, 43.28, 39.39, 45.66),
    (6912, 640, 3840): (129.08, 124.61, 123.78, 112.09), (2688, 5792, 640): (81.03, 91.66, 89.86, 88.78), (6656, 6912, 256): (115.57, 134.98, 144.82, 144.61),
    (5120, 3968, 512): (82.69, 90.89, 111.24, 97.96), (4992, 5616, 128): (83.01, 96.38, 103.96, 110.89), (6912, 3840, 256): (79.18, 91.88, 103.58, 102.64),
    (1536, 1872, 768): (36.7, 33.6, 37.5, 39.6), (768, 2304, 1280): (35.1, 32.3, 33.2, 35.7),
    # the four-group form, whose blocks of both products share the rounds
    (2560, 512, 6656): (84.8, 74.8, 91.0, 69.1), (6144, 1536, 4608): (197.1, 226.3, 198.6, 182.4), (8192, 256, 7168): (140.7, 135.5, 138.8, 116.2),
    (9728, 256, 4352): (128.0, 113.5, 132.0, 102.3), (3072, 624, 2816): (54.6, 50.4, 50.1, 44.0),
    # which product is long and which comes first decides as much as the sum: a long one behind many short blocks keeps few units busy at the end
    (17920, 1280, 256): (102.1, 124.3, 181.7, 140.3), (14848, 1648, 512): (117.5, 138.2, 182.9, 149.2), (10240, 3328, 256): (113.0, 131.5, 155.3, 148.3),
    (128, 1792, 14208): (97.2, 79.7, 149.0, 106.9), (384, 1296, 9856): (95.8, 80.8, 126.2, 99.7), (128, 2448, 12160): (101.3, 85.9, 137.1, 101.6),
    (256, 7344, 7936): (151.5, 150.9, 129.1, 168.0), (128, 14592, 1152): (67.9, 69.3, 59.3, 72.3), (1920, 2816, 8064): (257.2, 258.1, 222.1, 235.7),
    (7040, 256, 6528): (131.5, 130.0, 125.3, 109.6), (11136, 384, 7808): (285.9, 275.6, 267.8, 247.5), (3712, 512, 3968): (78.9, 73.7, 70.7, 63.9),
}


@pytest.mark.parametrize("T,d_in,d_out", PASS_US)
def test_dx_and_dw_share_a_launch_where_that_is_faster(libqii, T, d_in, d_out):
    size = max(libqii.qii_gemm_workspace_bytes(T, d_in, d_out), libqii.qii_gemm_workspace_bytes(d_out, d_in, T))
    ways = dict(zip((-1, T64, T128, T128_WIDE), PASS_US[T, d_in, d_out]))
    assert libqii.lib().qii_linear_bwd_gemm_route(T, d_in, d_out, size, 1) == min(ways, key=ways.get)


def test_products_of_different_routes_share_a_launch(libqii):
    """dX alone is faster in 128 x 128 tiles, dW in 64 x 64 ones; with a launch each the pass took 86.2 us, with one 80.6."""
    L = libqii.lib()
    T, d_in, d_out = 3840, 1280, 1024
    dx, dw = libqii.qii_gemm_workspace_bytes(T, d_in, d_out), libqii.qii_gemm_workspace_bytes(d_out, d_in, T)
    assert (L.qii_gemm_route(T, d_in, d_out, dx, 0), L.qii_gemm_route(d_out, d_in, T, dw, 0)) == (T128, T64)
    assert L.qii_linear_bwd_gemm_route(T, d_in, d_out, max(dx, dw), 0) == T64
    for bad in ((0, 16, 128), (128, 0, 128), (128, 16, 0), (64, 16, 128), (128, 16, 64), (128, 8, 128)):
        assert L.qii_linear_bwd_gemm_route(*bad, 1 << 30, 0) == -1


# products with an incomplete last round of 256 x 256 tiles, us: one block per tile, the last round's tiles shared, the fastest other kernel
# (re-tiling included)
LAST_ROUND_US = {
    (3072, 2816, 10240): (183.8, 156.6, 186.9), (8448, 1024, 10240): (188.8, 157.2, 187.6), (8448, 2048, 3072): (128.2, 106.4, 114.8),
    (11264, 2048, 6144): (249.8, 224.5, 254.0), (18432, 2048, 3072): (199.6, 188.5, 206.8), (8448, 3072, 12288): (474.8, 444.1, 520.3),
    (7168, 5376, 3840): (250.6, 243.9, 277.8), (4096, 2816, 2048): (50.0, 73.8, 53.0), (5632, 1664, 17664): (317.6, 267.3, 307.5),
    (8960, 1280, 32256): (654.0, 560.9, 602.4), (6912, 4992, 4864): (310.4, 273.5, 330.5), (2304, 5248, 3328): (73.8, 98.0, 80.9),
    (11520, 1024, 2560): (59.8, 83.8, 61.1),
}


@pytest.mark.parametrize("M,N,K", LAST_ROUND_US)
def test_the_last_round_is_shared_where_that_is_faster(libqii, M, N, K):
    """And the product then takes the main kernel, where its time so shared is the least: the plan's figure is the route's."""
    import ctypes
    plain, shared, other = LAST_ROUND_US[M, N, K]
    plan = (ctypes.c_int32 * 3)()
    libqii.lib().qii_gemm_sharing_plan(ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int64(K), plan)
    assert (plan[1] > 0) == (shared < plain)
    assert min(plain, shared) < other
    assert libqii.lib().qii_gemm_route(M, N, K, libqii.qii_gemm_workspace_bytes(M, N, K), 0) == MAIN


MAIN_TILES = 5


def call_route(libqii, M, N, K, c_dt, ldc, c=1 << 20, a_scales=1 << 21, ws=1 << 22, tiled=0):
    """qii_gemm_call_route for operands at made-up addresses."""
    import ctypes
    A, B = (libqii._NVFP4(1 << 23, s, 1 << 24, r, K) for r, s in ((M, a_scales), (N, 1 << 21)))
    size = libqii.qii_gemm_workspace_bytes(M, N, K) if ws else 0
    return libqii.lib().qii_gemm_call_route(ctypes.byref(A), ctypes.byref(B), c, c_dt, ldc, ws, size, tiled)


def test_the_route_of_a_call_heeds_its_result_and_its_scale_bytes(libqii):
    """Blocks take several tiles from three rounds of tiles on, where C's rows lie on 128-byte lines and are whole 16-byte pieces."""
    M, N, K = 16384, 8192, 2048
    assert libqii.lib().qii_gemm_route(M, N, K, libqii.qii_gemm_workspace_bytes(M, N, K), 0) == MAIN
    for dt in (BF16, F32):
        line = 64 if dt == BF16 else 32
        assert call_route(libqii, M, N, K, dt, N) == MAIN_TILES
        assert call_route(libqii, M, N - line // 8, K, dt, N) == MAIN_TILES
        assert call_route(libqii, M, N - line // 8, K, dt, N - line // 8) == MAIN       # rows off the lines
        assert call_route(libqii, M, N - 1, K, dt, N) == MAIN                           # a piece cut
        assert call_route(libqii, M, N, K, dt, N, c=(1 << 20) + 16) == MAIN             # C off the lines
        assert call_route(libqii, 2048, N, K, dt, N) == MAIN                            # one round
    # without a workspace, or with scale bytes that the re-tiling kernel cannot load, the main kernel is out of the question
    assert call_route(libqii, M, N, K, BF16, N, ws=None) == call_route(libqii, M, N, K, BF16, N, a_scales=(1 << 21) + 8) == T128
    assert call_route(libqii, M, N, K, BF16, N, a_scales=(1 << 21) + 8, tiled=1) == MAIN_TILES
    for bad in ((0, N, K), (M, 0, K), (M, N, 24)):
        assert call_route(libqii, *bad, BF16, N, ws=None) == -1
    assert call_route(libqii, M, N, K, 7, N) == call_route(libqii, M, N, K, BF16, N - 1) == call_route(libqii, M, N, 128, BF16, N, tiled=1) == -1
    # the routes differ by the type of the result alone
    assert call_route(libqii, 5376, 5376, 512, BF16, 5376) == MAIN and call_route(libqii, 5376, 5376, 512, F32, 5376) == T128


# products, us: the main kernel (re-tiling included, the last round shared where the plan says so), tiles of 64 x 64, of 128 x 128 in two K
# groups, in four
ROUTE_US = {
    # short K: 64 x 64 tiles, though the four-group form takes less per K tile than it did
    (1856, 1664, 768, F32): (22.3, 9.5, 11.5, 11.3), (226, 11243, 768, BF16): (26.3, 10.5, 12.6, 12.3),
    (4352, 512, 1024, F32): (24.1, 10.7, 13.1, 12.0), (256, 9216, 1024, F32): (24.3, 10.8, 13.3, 12.3), (1280, 2304, 768, BF16): (19.2, 9.3, 10.8, 10.5),
    (768, 4096, 768, BF16): (19.3, 9.3, 10.8, 10.5), (576, 3648, 1024, F32): (27.0, 10.2, 13.2, 12.3),
    # few tiles of long K: a shared round is not as much cheaper as a whole one
    (6016, 256, 11520, F32): (62.7, 59.3, 98.8, 59.0), (450, 2419, 9216, F32): (51.4, 44.7, 76.4, 47.3),
    # f32 results at short K: memory, whose time the main kernel's price has per round
    (11584, 3776, 512, F32): (67.3, 76.9, 63.6, 99.5), (14848, 3008, 512, F32): (68.1, 76.5, 64.8, 104.5), (9216, 2368, 1536, F32): (78.2, 80.1, 72.9, 84.0),
    (2376, 22776, 768, F32): (118.8, 123.6, 105.4, 150.6), (7320, 4872, 1280, F32): (114.6, 122.6, 100.8, 126.4),
    # but not where its blocks take several tiles
    (25344, 15616, 512, F32): (423.4, 736.3, 523.7, 808.6), (32768, 2560, 512, F32): (105.6, 149.4, 113.7, 181.7),
}


@pytest.mark.parametrize("M,N,K,c_dt", ROUTE_US)
def test_the_fastest_kernel_of_a_product(libqii, M, N, K, c_dt):
    """Within 3 %."""
    us = dict(zip((MAIN, T64, T128, T128_WIDE), ROUTE_US[M, N, K, c_dt]))
    us[MAIN_TILES] = us[MAIN]
    assert us[call_route(libqii, M, N, K, c_dt, N)] <= 1.03 * min(us.values())


def test_routes_of_refused_and_smallest_sizes(libqii):
    L = libqii.lib()
    for bad in ((0, 8, 16, 0, 0), (8, 0, 16, 0, 0), (8, 8, 0, 0, 0), (8, 8, 24, 0, 0), (8, 8, 128, 0, 1)):
        assert L.qii_gemm_route(*bad) == -1
    assert L.qii_gemm_route(1, 1, 16, 0, 0) == T64
    # beyond 2^23 columns the main kernel's 32-bit offsets do not reach
    assert L.qii_gemm_route(512, 512, (1 << 23) + 256, 1 << 40, 0) != MAIN
    # nor those of the 64 x 64 and two-group 128 x 128 kernels beyond 2^25
    for M, N in ((1, 1), (64, 64), (512, 512), (2048, 2048)):
        assert L.qii_gemm_route(M, N, 1 << 25, 0, 0) in (T64, T128, T128_WIDE, NO_WORKSPACE)
        for K in ((1 << 25) + 16, (1 << 25) + 128, (1 << 25) + 256, 1 << 28):
            for ws in (0, 1 << 40):
                assert L.qii_gemm_route(M, N, K, ws, 0) in (T128_WIDE, NO_WORKSPACE)
    assert L.qii_gemm_route(64, 64, 1 << 25, 0, 0) == T64
