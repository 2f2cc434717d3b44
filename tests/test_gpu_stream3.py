"""The weight-streaming kernel of the 1.6-bit forms at the edges of its geometry: half slices of 320 weights (64 packed bytes, four 16-byte
chunks), up to 15 waves, items of up to three tiles, several passes beyond, one and two workgroups per CU in a grouped launch."""
import numpy as np
import pytest

import oracle
import paper_2506_23025_amd as tl
import synth_inputs as si
from parity import assert_close, launches, to_dev
from test_tile_choice import ONE_POINT_SIX, STREAMS, runs, shares

pytestmark = pytest.mark.gpu

FORMS = [(tl.TL_FMT_1P6BIT, tl.tl_pack_1p6bit, tl.tl_ternary_gemm_1p6), (tl.TL_FMT_1P6BIT_FX, tl.tl_pack_1p6bit_fx, tl.tl_ternary_gemm_1p6_fx)]


def check(y, x, W, g, what):
    N = W.shape[0]
    cols = np.unique(np.r_[0:min(N, 16), max(0, N - 16):N, np.random.default_rng(N).choice(N, min(N, 100), replace=False)])
    assert_close(y[:, cols], oracle.gemm(x, np.ascontiguousarray(W[cols]), g), x, g, what)


# one chunk; a half slice less, full and one group over; 14 and 15 waves full, one weight group over into a second pass; passes of unequal waves;
# columns: one, a tile less one, full and over, rows of y at odd places, runs of one to four tiles and more
@pytest.mark.parametrize("fmt,pack,call", FORMS)
@pytest.mark.parametrize("M,N,K", [(1, 1, 8), (3, 15, 80), (16, 16, 312), (2, 17, 320), (5, 33, 328), (1, 4100, 4480), (16, 1022, 4800),
                                   (7, 4097, 4808), (16, 48, 9600), (1, 5000, 9608), (9, 8211, 6400), (4, 12304, 4872), (12, 16400, 640)])
def test_shapes_at_the_edges(M, N, K, fmt, pack, call):
    assert runs(ONE_POINT_SIX, M, N, K) == STREAMS
    x, W, g = si.layer(41000 + M + N + K, M, N, K)
    xd, wd = to_dev(x.view(np.int16)), to_dev(pack(W))
    yd = to_dev(np.full((M, N), -21555, dtype=np.int16))
    call(xd, wd, si.gamma_bits(g), yd, M, N, K)
    check(yd.cpu().numpy().view(np.float16), x, W, g, f"{M}x{N}x{K}")


# one to seven half slices, tiles for all workgroups of the chip and for twice as many
@pytest.mark.parametrize("M,N,K", [(1, 32784, 320), (5, 65552, 264), (16, 16400, 640), (2, 32768, 584), (16, 16399, 960), (3, 33000, 904), (9, 12304, 1280),
                                   (16, 8208, 1600), (1, 16384, 1320), (7, 24577, 1528), (33, 9000, 1600), (40, 20000, 960), (4, 16400, 2240)])
def test_several_workgroups_per_cu(M, N, K):
    assert runs(ONE_POINT_SIX, M, N, K) == STREAMS
    x, W, g = si.layer(43000 + M + N + K, M, N, K)
    xd, wd = to_dev(x.view(np.int16)), to_dev(tl.tl_pack_1p6bit(W))
    yd = to_dev(np.full((M, N), -21555, dtype=np.int16))
    tl.tl_ternary_gemm_1p6(xd, wd, si.gamma_bits(g), yd, M, N, K)
    check(yd.cpu().numpy().view(np.float16), x, W, g, f"{M}x{N}x{K}")


# K that leaves two workgroups to a CU (up to 2240) and one over, with tiles for both; a wave without a part of a shorter K
@pytest.mark.parametrize("specs", [[(16, 14336, 1024), (16, 18448, 640)], [(1, 16384, 2240), (9, 16400, 2240)],
                                   [(2, 16384, 2248), (5, 16384, 2240)], [(3, 32768, 320), (1, 30, 2240)]])
def test_grouped_launches_of_one_and_two_workgroups_per_cu(specs):
    assert all(shares(ONE_POINT_SIX, specs))
    jobs, want = [], []
    for i, (M, N, K) in enumerate(specs):
        x, W, g = si.layer(42000 + i + M + N + K, M, N, K)
        yd = to_dev(np.full((M, N), -21555, dtype=np.int16))
        jobs.append((to_dev(x.view(np.int16)), to_dev(tl.tl_pack_1p6bit(W)), si.gamma_bits(g), yd, M, N, K))
        want.append((yd, x, W, g))
    tl.tl_ternary_gemm_1p6_grouped(jobs, tl.TL_FMT_1P6BIT)
    for yd, x, W, g in want:
        check(yd.cpu().numpy().view(np.float16), x, W, g, f"{yd.shape}")


# A NaN and an infinity in two rows of x: every other row is exactly what it is without them.  One pass, several workgroups per CU, several passes;
# rows that are no power of two and a second block of rows.
@pytest.mark.parametrize("M,N,K", [(5, 272, 4096), (13, 4100, 960), (7, 1000, 6400), (16, 33, 320), (21, 2000, 11008)])
@pytest.mark.parametrize("fmt,pack,call", FORMS)
def test_non_finite_activations_stay_in_their_row(M, N, K, fmt, pack, call):
    assert runs(ONE_POINT_SIX, M, N, K) == STREAMS
    x, W, g = si.layer(44000 + M + N + K, M, N, K)
    wd = to_dev(pack(W))

    def run(x):
        yd = to_dev(np.full((M, N), -21555, dtype=np.int16))
        call(to_dev(x.view(np.int16)), wd, si.gamma_bits(g), yd, M, N, K)
        return yd.cpu().numpy().view(np.float16)

    clean, bad = run(x), x.copy()
    bad[1, K - 3] = np.float16(np.nan)
    bad[3, 7] = np.float16(np.inf)
    y = run(bad)
    for m in set(range(M)) - {1, 3}:
        assert np.array_equal(y[m].view(np.uint16), clean[m].view(np.uint16)), m
    assert not np.isfinite(y[1].astype(np.float32)).any()
    assert not np.isfinite(y[3].astype(np.float32)).any()


# K that is no multiple of 8, whose rows of x start at any even address: the pieces of one to ten rounds of a wave (1, 4, 8 and 16 rows), the last piece
# of a row cut at every place, a half slice less one, one over and one piece over, passes with one, two and more rows ahead of their tiles
@pytest.mark.parametrize("fmt,pack,call", FORMS)
@pytest.mark.parametrize("M,N,K", [(1, 1, 9), (16, 40, 15), (2, 33, 319), (5, 50, 321), (8, 17, 322), (9, 100, 323), (4, 4099, 2045), (16, 1030, 4799),
                                   (3, 4099, 644), (1, 300, 4801), (6, 4100, 5002), (16, 4098, 9603), (4, 8211, 9607), (7, 12304, 4873), (2, 16400, 4805),
                                   (16, 12300, 9611), (40, 700, 1001), (33, 130, 8190), (20, 9000, 1013)])
def test_any_k(M, N, K, fmt, pack, call):
    assert runs(ONE_POINT_SIX, M, N, K) == STREAMS
    x, W, g = si.layer(45000 + M + N + K, M, N, K)
    xd, wd = to_dev(x.view(np.int16)), to_dev(pack(W))
    yd = to_dev(np.full((M, N), -21555, dtype=np.int16))
    call(xd, wd, si.gamma_bits(g), yd, M, N, K)
    check(yd.cpu().numpy().view(np.float16), x, W, g, f"{M}x{N}x{K}")


# such jobs share a launch with others, bit for bit what they give alone; a NaN in the row that follows a row's last piece stays there
def test_any_k_in_a_grouped_launch():
    specs = [(16, 2050, 1001), (3, 1024, 1024), (9, 515, 641), (16, 300, 4799), (1, 40, 9)]
    assert all(shares(ONE_POINT_SIX, specs))
    jobs, alone = [], []
    for i, (M, N, K) in enumerate(specs):
        x, W, g = si.layer(46000 + i, M, N, K)
        if M > 1:
            x[1, 0], x[M - 1, K - 1] = np.nan, np.inf
        xd, wd = to_dev(x.view(np.int16)), to_dev(tl.tl_pack_1p6bit(W))
        yd, ya = (to_dev(np.full((M, N), -21555, dtype=np.int16)) for _ in range(2))
        jobs.append((xd, wd, si.gamma_bits(g), yd, M, N, K))
        tl.tl_ternary_gemm_1p6(xd, wd, si.gamma_bits(g), ya, M, N, K)
        alone.append((ya, yd, x, W, g))
    tl.tl_ternary_gemm_1p6_grouped(jobs, tl.TL_FMT_1P6BIT)
    for ya, yd, x, W, g in alone:
        assert np.array_equal(ya.cpu().numpy(), yd.cpu().numpy())
        clean = np.isfinite(x).all(axis=1)
        y = yd.cpu().numpy().view(np.float16)
        check(y[clean], np.ascontiguousarray(x[clean]), W, g, f"{x.shape}")
        assert not np.isfinite(y[~clean].astype(np.float32)).any()


# a grouped call of one job is one launch however many rows, and gives the bits of the call of its own; so is the one of several that the others leave alone
@pytest.mark.parametrize("M,N,K,others", [(1080, 62, 274, []), (905, 16, 108, []), (1311, 832, 512, []), (600, 48, 1280, []), (600, 48, 1280, [(512, 14336, 4096)]), (512, 62, 273, []), (3, 100, 40, [])])
def test_one_job(M, N, K, others):
    tl.tl_init()
    jobs = []
    for m, n, k in [(M, N, K), *others]:
        x, W, g = si.layer(47000 + m, m, n, k)
        jobs.append((to_dev(x.view(np.int16)), to_dev(tl.tl_pack_1p6bit(W)), si.gamma_bits(g), to_dev(np.full((m, n), -21555, dtype=np.int16)), m, n, k))
    ya = to_dev(np.full((M, N), -21555, dtype=np.int16))
    tl.tl_ternary_gemm_1p6(*jobs[0][:3], ya, M, N, K)
    tl.tl_ternary_gemm_1p6_grouped(jobs, tl.TL_FMT_1P6BIT)
    assert np.array_equal(ya.cpu().numpy(), jobs[0][3].cpu().numpy())
    assert launches(lambda stream: tl.tl_ternary_gemm_1p6_grouped(jobs, tl.TL_FMT_1P6BIT, stream)) == len(jobs)
