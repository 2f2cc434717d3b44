"""Which kernel the library's cost models send a call to: the GPU tests of the tiled kernel reach every instance of it (CPU, no launch)."""
import ctypes

import paper_2506_23025_amd as tl
import test_gpu_tile as shapes

_instance = tl.raw().tl_internal_tile_instance           # not in tl.h: for the tests alone
_instance.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 4
_instance.restype = ctypes.c_int

TWO_BIT, ONE_POINT_SIX, SCALES, TWO_BIT_FORCED = range(4)
_runs = tl.raw().tl_internal_runs
_runs.argtypes = _instance.argtypes
_runs.restype = ctypes.c_int
PLAIN, STREAMS, TILED = range(3)
_grouped = tl.raw().tl_internal_grouped_tiled
_grouped.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
_grouped.restype = None
RAGGED = 100                                               # first instance of the forms for odd K


def instance(form, M, N, K, group=0):
    """Place of the tiled kernel's instance in the table of its form, or -1 where another kernel takes the call."""
    return _instance(form, M, N, K, group)


def runs(form, M, N, K, group=0):
    """The kernel that a call of its own runs in: PLAIN, STREAMS or TILED."""
    return _runs(form, M, N, K, group)


def _of_jobs(form, jobs):
    flat = (ctypes.c_int64 * (4 * len(jobs)))(*[v for j in jobs for v in (tuple(j) + (0,))[:4]])
    out = (ctypes.c_int * len(jobs))()
    _grouped(form, flat, len(jobs), out)
    return list(out)


def grouped(form, jobs):
    """Per job (M, N, K[, group]) of a grouped call, whether the tiled kernel takes it from the launches that others share."""
    return [v == 1 for v in _of_jobs(form, jobs)]


def shares(form, jobs):
    """Per job of a grouped call, whether it shares the streaming kernel's launches."""
    return [v == 0 for v in _of_jobs(form, jobs)]


def test_tile_shapes_reach_every_instance():
    assert {instance(TWO_BIT_FORCED, *s) for s in shapes.TILE_SHAPES} == set(range(6))
    assert {instance(ONE_POINT_SIX, *s) for s in shapes.TILE3_SHAPES} - {-1} == set(range(5))
    assert {instance(SCALES, *s) for s in shapes.TILE_GS_SHAPES} - {-1} == set(range(7))


def test_odd_k_shapes_reach_every_instance():
    assert {instance(TWO_BIT, *s) for s in shapes.RAGGED_SHAPES} - {-1} == {RAGGED + i for i in range(4)}
    assert {instance(ONE_POINT_SIX, *s) for s in shapes.RAGGED_SHAPES} - {-1} == {RAGGED + i for i in range(3)}
    assert all(instance(ONE_POINT_SIX, 2000, 2050, K) >= RAGGED for K in (9, 15, 33))
    assert {instance(SCALES, *s, group) for s in shapes.RAGGED_SHAPES for group in (16, 144, 8192)} - {-1} == {RAGGED + i for i in range(3)}


def test_shapes_beyond_the_form_are_left_to_others():
    assert instance(TWO_BIT, 16, 4096, 4096) == -1         # few rows
    assert instance(ONE_POINT_SIX, 16, 4096, 4096) == -1
    assert instance(SCALES, 16, 4096, 4096, 128) == -1
    for form in (TWO_BIT, ONE_POINT_SIX, SCALES):
        assert instance(form, 1024, 4096, 7, 16) == -1     # K of less than a piece
        assert instance(form, 1 << 25, 16, 100, 16) == -1  # rows past 2^24


def test_a_call_is_told_from_those_of_other_kernels():
    assert runs(SCALES, 16, 4096, 4096, 128) == STREAMS and runs(SCALES, 16, 4096, 4096, 16) == TILED and runs(SCALES, 1, 1, 5344, 128) == PLAIN
    assert shares(SCALES, [(16, 4096, 4096, 128), (16, 4096, 4096, 16), (16, 4099, 4096, 128), (2, 300, 777, 32)]) == [True, False, False, False]
    assert runs(TWO_BIT, 16, 4099, 4090) == STREAMS and runs(TWO_BIT, 2000, 2050, 33) == TILED and runs(TWO_BIT, 1, 16, 7) == PLAIN
    assert shares(TWO_BIT, [(16, 4099, 4090), (9, 4099, 4090), (16, 4099, 63)]) == [True, True, False]
    assert runs(ONE_POINT_SIX, 16, 4096, 4096) == STREAMS and runs(ONE_POINT_SIX, 512, 14336, 4096) == TILED and runs(ONE_POINT_SIX, 1, 16, 7) == PLAIN
    assert shares(ONE_POINT_SIX, [(16, 4096, 4800), (16, 4096, 4801), (16, 4096, 63), (17, 4096, 63)]) == [True, False, True, False]


def test_two_bit_words_at_many_rows():
    # measured (us), small-M / tiled: 14701 x 2304 at M = 1295 141 / 93, 15104 x 2688 at 1421 152 / 104, 5447 x 1920 at 884 30.9 / 30.4, 16384 x 512
    # at 192 11.7 / 9.2, 384 18.9 / 14.0, 512 29.7 / 15.0; 16384 x 1024 at 384 23.0 / 19.1; 2048 x 2048 at 192 8.8 / 6.9.  And where the
    # small-M kernel is ahead: 2048 x 2048 at 48 5.3 / 6.7, at 96 6.1 / 6.7; 4096 x 4096 at 96 9.0 / 10.3.
    for M, N, K in ((1295, 14701, 2304), (1421, 15104, 2688), (884, 5447, 1920), (192, 16384, 512), (384, 16384, 512), (512, 16384, 512), (384, 16384, 1024),
                    (192, 2048, 2048)):
        assert tl.tl_ternary_gemm_which(M, N, K) == tl.TL_PATH_MFMA, (M, N, K)
    for M, N, K in ((48, 2048, 2048), (96, 2048, 2048), (96, 4096, 4096), (16, 16384, 512)):
        assert tl.tl_ternary_gemm_which(M, N, K) == tl.TL_PATH_GEMV, (M, N, K)


def test_two_bit_words_of_short_k_at_more_than_16_rows():
    # measured (us), streaming / tiled: 3.40 / 2.69, 3.55 / 2.91, 4.19 / 3.49, 3.53 / 2.98, 3.64 / 3.31, 4.59 / 3.89; the other way round
    # 3.62 / 4.25, 3.58 / 4.20
    for M, N, K in ((24, 128, 128), (75, 576, 128), (46, 1696, 192), (81, 576, 64), (128, 768, 256), (113, 1072, 320)):
        assert tl.tl_ternary_gemm_which(M, N, K) == tl.TL_PATH_MFMA, (M, N, K)
    for M, N, K in ((26, 1344, 448), (66, 1024, 448)):
        assert tl.tl_ternary_gemm_which(M, N, K) == tl.TL_PATH_GEMV, (M, N, K)


def test_one_point_six_bit_codes_at_many_rows():
    # measured (us), streaming / best tile: narrow layers 4224 x 832 at M = 1311 25.2 / 27.5, 1024 x 64 at 2048 6.4 / 7.3; 17 to 36 rows of long
    # ones 8704 x 4260 at 18 17.9 / 22.7, 13184 x 5554 at 19 25.1 / 31.5, 6776 x 4928 at 21 15.5 / 18.4; and the other way round 4096 x 14336
    # at 512 112 / 58, 11008 x 4096 at 64 42 / 27, 704 x 15020 at 805 73 / 47
    for M, N, K in ((1311, 832, 4224), (2048, 64, 1024), (18, 4260, 8704), (19, 5554, 13184), (21, 4928, 6776)):
        assert instance(ONE_POINT_SIX, M, N, K) == -1, (M, N, K)
    for M, N, K in ((512, 14336, 4096), (64, 4096, 11008), (805, 15020, 704)):
        assert instance(ONE_POINT_SIX, M, N, K) >= 0, (M, N, K)


def test_one_point_six_bit_codes_in_one_pass():
    # measured (us), streaming / best tile, K in one pass of 15 half slices: 4672 -> 4647 at M = 20 7.5 / 14.4, 4736 -> 572 at 228 7.3 / 14.6, 4560 -> 2624
    # at 31 6.5 / 14.5; K past it and wide layers at many rows the other way round: 11008 -> 4096 at 60, 4096 -> 14336 at 512 56
    for M, N, K in ((20, 4647, 4672), (228, 572, 4736), (31, 2624, 4560), (31, 2624, 4800)):
        assert instance(ONE_POINT_SIX, M, N, K) == -1, (M, N, K)
    for M, N, K in ((60, 4096, 11008), (512, 14336, 4096), (2048, 4096, 1024)):
        assert instance(ONE_POINT_SIX, M, N, K) >= 0, (M, N, K)


def test_one_point_six_bit_codes_in_several_passes():
    # measured (us), streaming / best tile: a block of 16 rows costs a pass more than one of few.  9536 -> 10688 at M = 47 34.0 / 29.8, 9536 -> 768 at 258
    # 26.9 / 25.2, 8320 -> 14080 at 24 25.2 / 22.7; 13248 -> 1920 at 25 10.3 / 31.9, 14208 -> 6592 at 28 24.2 / 34.1
    for M, N, K in ((47, 10688, 9536), (258, 768, 9536), (24, 14080, 8320)):
        assert instance(ONE_POINT_SIX, M, N, K) >= 0, (M, N, K)
    for M, N, K in ((18, 4260, 8704), (25, 1920, 13248), (28, 6592, 14208)):
        assert instance(ONE_POINT_SIX, M, N, K) == -1, (M, N, K)


def test_short_k_of_one_point_six_bit_codes():
    # measured (us), streaming / best tile: 500 x 4100 x 1600 16.3 / 18.0, 700 x 1100 x 952 6.8 / 8.0; one step of K 33 x 20754 x 64 6.1 / 5.4,
    # 1279 x 512 x 128 5.7 / 5.2, 846 x 832 x 152 5.8 / 5.3
    for M, N, K in ((500, 4100, 1600), (700, 1100, 952)):
        assert instance(ONE_POINT_SIX, M, N, K) == -1, (M, N, K)
    for M, N, K in ((33, 20754, 64), (1279, 512, 128), (846, 832, 152)):
        assert instance(ONE_POINT_SIX, M, N, K) >= 0, (M, N, K)


def test_scales_that_do_not_stream():
    # measured (us), plain / tiled: groups or N that the streaming kernel does not take, short K and many rows above all, whose chunks of 1024 weights cost the plain
    # kernel as much as whole ones; and the other way round one or two rows of few columns
    for M, N, K, group in ((3, 12363, 1088, 32), (1566, 433, 85, 16), (5042, 209, 64, 256), (52, 4032, 128, 80), (730, 261, 192, 256), (229, 320, 384, 16),   # 19.8 / 6.9, 57 / 5.1, 80 / 5.4, 19 / 3.4, 20 / 3.9, 12 / 4.3
                           (490, 9, 384, 16), (5, 695, 1344, 384), (3, 1721, 2304, 64), (3, 8003, 2496, 128), (6, 6, 1088, 32), (2, 64, 16, 80)):            # 9.4 / 4.2, 10.4 / 6.8, 12.0 / 8.2, 15.6 / 9.7, 9.6 / 6.0, 5.3 / 3.2
        assert instance(SCALES, M, N, K, group) >= 0, (M, N, K, group)
    for M, N, K, group in ((1, 1, 5344, 128), (2, 2, 13292, 16), (2, 4, 3041, 48), (1, 22, 1888, 256)):                                                      # 11.5 / 17.7, 27 / 39, 9.4 / 12.1, 6.7 / 8.2
        assert instance(SCALES, M, N, K, group) == -1, (M, N, K, group)


def test_two_bit_words_that_do_not_stream():
    # measured (us), plain / tiled: K below 64 or more than 4096 rows: 42 / 5.2, 18 / 4.9, 16 / 4.5, 183 / 11.4, 388 / 25
    for M, N, K in ((19384, 25, 84), (8760, 3, 235), (8496, 1, 308), (1844, 1406, 51), (13509, 179, 1427), (1, 16, 8), (4, 20, 63)):
        assert instance(TWO_BIT, M, N, K) >= RAGGED, (M, N, K)
    assert instance(TWO_BIT, 4, 20, 7) == -1               # K of less than a piece


def test_scales_of_more_rows_than_one_launch_streams():
    # measured (us), streaming, 4096 rows to a launch / tiled
    for M, N, K, group in ((21027, 36, 192, 128), (14334, 8, 128, 256), (27651, 16, 448, 128), (18991, 64, 832, 256)):    # 27 / 6.2, 15 / 3.9, 28 / 7.6, 33 / 9.5
        assert instance(SCALES, M, N, K, group) >= 0, (M, N, K, group)
    assert instance(SCALES, 1311, 832, 512, 256) == -1


def test_scales_of_short_k_at_more_than_16_rows():
    # measured (us), streaming / tiled: 4.7 / 3.7, 4.7 / 3.7, 4.6 / 3.7, 4.3 / 3.6, 4.3 / 3.6, 4.2 / 3.5, 4.5 / 4.0; the other way round 4.0 / 4.6, 3.8 / 4.9, 3.8 / 5.0
    for M, N, K, group in ((96, 2912, 64, 256), (305, 896, 64, 256), (30, 5948, 64, 256), (1572, 96, 128, 128), (493, 352, 128, 128), (641, 36, 128, 128), (29, 320, 256, 32)):
        assert runs(SCALES, M, N, K, group) == TILED, (M, N, K, group)
    for M, N, K, group in ((98, 112, 320, 128), (19, 1408, 448, 256), (64, 272, 448, 256)):
        assert runs(SCALES, M, N, K, group) == STREAMS, (M, N, K, group)


def test_one_point_six_bit_codes_of_more_rows_than_one_launch_streams():
    # measured (us), streaming, 4096 rows to a launch / tiled
    for M, N, K in ((29569, 20, 171), (14561, 37, 703), (10488, 62, 743), (24042, 62, 1251), (5936, 144, 107), (4872, 8, 354)):    # 36 / 16, 24 / 12, 21 / 12, 50 / 29, 12 / 7, 8 / 6
        assert instance(ONE_POINT_SIX, M, N, K) >= RAGGED, (M, N, K)


def test_workgroups_of_the_streaming_kernel_fit_on_a_compute_unit():
    # 160 KB of LDS in units of 1280 bytes, at most 16 waves; a wave's area (16 rows of 656 bytes) and the table of 2 KB
    fn = tl.raw().tl_internal_stream3_per_cu
    fn.argtypes = [ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    for waves in range(1, 16):
        lds = ctypes.c_int()
        count = fn(waves, ctypes.byref(lds))
        assert lds.value % 1280 == 0 and lds.value >= waves * 16 * 656 + 2048, waves
        assert count >= 1 and count * lds.value <= 160 * 1024 and count * waves <= 16, waves


def test_small_launches_find_their_jobs_in_a_table_unless_captured():
    # measured (us), records / table: 2 x 2048 x 2048 in a loop 5.4 / 4.3, replayed 3.1 / 3.3; 18 x 4672 x 4096 (two blocks of rows, 9.1 MB) 5.6 / 5.9
    fn = tl.raw().tl_internal_jobs_by_table
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_int64, ctypes.c_int]
    mb = 1 << 20
    for captured in (0, 1):
        assert fn(2, 1, 1, 0, 2 * mb, captured) == 1 - captured
        assert fn(16, 1, 1, 0, 8 * mb - 1, captured) == 1 - captured
        assert not fn(2, 1, 1, 0, 9 * mb, captured) and not fn(2, 1, 1, 1, 9 * mb, captured)
        assert fn(2, 1, 1, 1, 2 * mb, captured)            # several workgroups to a CU: equal on the device, cheaper on the host
        assert fn(2, 1, 0, 0, 90 * mb, captured)           # nothing else takes it
        assert not fn(1, 1, 1, 0, mb, captured) and not fn(17, 1, 1, 0, mb, captured) and not fn(2, 0, 0, 0, mb, captured)
        assert fn(32, 1, 0, 1, mb, captured) and not fn(33, 1, 0, 1, mb, captured)


def test_grouped_jobs_share_launches_where_that_is_faster():
    # measured (us), all streaming / each as if alone: 16 layers at M = 256, 2-bit words 512 x 1024 68.7 / 83.2, 768 x 2048 87.2 / 108.3, 1.6-bit codes
    # 512 x 1024 102.5 / 119.6
    for form, M, N, K in ((TWO_BIT, 256, 512, 1024), (TWO_BIT, 256, 768, 2048), (ONE_POINT_SIX, 256, 512, 1024)):
        assert not any(grouped(form, [(M, N, K)] * 16)), (form, M, N, K)

    def block(M, group=0):
        return [(M, 12288, 4096, group), (M, 4096, 4096, group), (M, 22016, 4096, group), (M, 4096, 11008, group)]

    assert not any(grouped(SCALES, block(32, 128)))
    assert all(grouped(SCALES, block(256, 128)))           # 662 / 132
    assert all(grouped(ONE_POINT_SIX, [(256, n, k) for _, n, k, _ in block(256)][:3]))
    # a job alone is taken as its single call takes it, and what a group tiles a single call tiles too
    for form, group in ((TWO_BIT, 0), (ONE_POINT_SIX, 0), (SCALES, 128), (SCALES, 256)):
        for M in (16, 17, 40, 100, 250, 600, 2000):
            for N, K in ((512, 512), (1024, 2048), (4096, 4096), (14336, 4096), (768, 4096), (16384, 512)):
                alone = instance(form, M, N, K, group) >= 0
                assert grouped(form, [(M, N, K, group)]) == [alone], (form, M, N, K)
                assert alone or not any(grouped(form, [(M, N, K, group)] * 5)), (form, M, N, K)


def test_jobs_of_many_rows_leave_the_shared_launches():
    # measured (us), 2 to 8 alike jobs that share launches / as calls of their own: 2-bit words 43.4 / 16.5, 16.0 / 13.9; scales 64.4 / 36.0, 27.6 / 21.6; 1.6-bit
    # codes 75.4 / 65.7 and 30.6 / 25.4 (two of several); and the other way round 5.1 / 13.4, 8.2 / 9.5, 8.0 / 16.4, and of different ones 22.4 / 27.9
    assert not any(shares(TWO_BIT, [(834, 2624, 128), (834, 6054, 488)]))
    assert not shares(TWO_BIT, [(57, 96, 208), (302, 3520, 64)])[1]                    # K = 64 in the form for any K: 15.7 / 8.1
    for form, n, job in ((TWO_BIT, 4, (1479, 80, 512)), (TWO_BIT, 2, (506, 272, 453)), (SCALES, 2, (787, 4128, 273, 64)),
                         (SCALES, 4, (482, 328, 621, 64)), (ONE_POINT_SIX, 4, (835, 2432, 80)), (ONE_POINT_SIX, 2, (1197, 272, 1071))):
        assert not any(shares(form, [job] * n)), (form, job)
    assert all(shares(SCALES, [(33, 8032, 640, 256), (33, 10312, 8064, 256)])) and all(shares(ONE_POINT_SIX, [(2, 3200, 136), (445, 208, 384)]))
    for form, n, job in ((TWO_BIT, 4, (99, 272, 318)), (SCALES, 2, (70, 2176, 576, 32)), (ONE_POINT_SIX, 4, (129, 350, 400))):
        assert all(shares(form, [job] * n)), (form, job)
