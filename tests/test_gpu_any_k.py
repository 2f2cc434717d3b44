"""2-bit words with a K that is no multiple of 64 in the weight-streaming kernel: rows of packed words start at multiples of 4 bytes, rows of x and y
at any even address, and a row's last 64 weights overlap the ones before."""
import numpy as np
import pytest

import oracle
import paper_2506_23025_amd as tl
import synth_inputs as si
from parity import assert_close, dev_u32, launches, to_dev
from test_tile_choice import STREAMS, TWO_BIT, runs, shares

pytestmark = pytest.mark.gpu


def product(M, N, K, seed, x=None):
    """y of a call, its guard behind it untouched, and its inputs."""
    x0, W, g = si.layer(seed, M, N, K)
    x = x0 if x is None else x
    yd = to_dev(np.full(M * N + 64, -21555, dtype=np.int16))
    tl.tl_ternary_gemm(to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), si.gamma_bits(g), yd, M, N, K)
    y = yd.cpu().numpy()
    assert (y[M * N:] == -21555).all()
    return y[:M * N].view(np.float16).reshape(M, N), x, W, g


def check(y, x, W, g, what):
    N = W.shape[0]
    cols = np.unique(np.r_[0:min(N, 20), max(0, N - 20):N, np.random.default_rng(N).choice(N, min(N, 100), replace=False)])
    assert_close(y[:, cols], oracle.gemm(x, np.ascontiguousarray(W[cols]), g), x, g, what)


# the last chunk of a row of every kind (a word, a weight or all but one of them), one slice of 512 and its edges, rows of every class of the
# staging (1, 4, 8, 16), runs of one tile to several items, two blocks of rows; up to 8 slices, from 9 on one or two tiles to a workgroup, beyond
# that and beyond 32 slices several passes
@pytest.mark.parametrize("M,N,K", [(1, 1, 65), (4, 17, 79), (2, 40, 80), (3, 33, 81), (4, 100, 111), (1, 64, 112), (1, 300, 127), (2, 7, 511), (3, 1030, 513),
                                   (4, 4099, 1000), (1, 16390, 520), (2, 9000, 2047), (8, 2050, 4090), (16, 4099, 4094), (5, 20000, 4081), (37, 4099, 4090), (9, 8200, 3583),
                                   (1, 100, 4097), (4, 4099, 4104), (16, 4099, 8211), (7, 8190, 11009), (20, 2000, 9001), (1, 8200, 4161), (3, 20000, 6001), (13, 20000, 4999),
                                   (2, 600, 16385), (16, 1030, 32767), (13, 30, 16383), (64, 515, 4111)])
def test_any_k(M, N, K):
    y, x, W, g = product(M, N, K, 47000 + M + N + K)
    assert runs(TWO_BIT, M, N, K) == STREAMS
    check(y, x, W, g, f"{M}x{N}x{K}")


# what stands behind a row's last weight, the next row's first, is not multiplied in; a NaN or an infinity stays in its row
@pytest.mark.parametrize("M,N,K", [(4, 200, 1003), (16, 200, 4087), (7, 100, 5001), (16, 4099, 8211), (12, 20000, 4999)])
def test_rows_stay_apart(M, N, K):
    x, W, g = si.layer(48000 + K, M, N, K)
    x[1, 0], x[2, K - 1], x[M - 1, 5] = np.inf, np.nan, -np.inf
    y, x, W, g = product(M, N, K, 48000 + K, x)
    assert runs(TWO_BIT, M, N, K) == STREAMS
    clean = np.setdiff1d(np.arange(M), [1, 2, M - 1])
    check(y[clean], np.ascontiguousarray(x[clean]), W, g, "rows beside a NaN")
    assert np.isnan(y[2]).all() and not np.isfinite(y[[1, M - 1]].astype(np.float32)).any()


# such jobs among others: short and long K side by side (waves without a slice, several passes), many rows, runs too long for what one launch keeps
@pytest.mark.parametrize("specs", [[(16, 4099, 4090), (16, 4096, 1024), (3, 640, 4099), (1, 40, 65)],
                                   [(37, 5952, 1984), (37, 1984, 1984), (37, 8416, 1984), (37, 1984, 4208)],
                                   [(2, 12288, 4096), (2, 4096, 4096), (2, 22016, 4096), (2, 4096, 11000)],
                                   [(200, 512, 999), (8, 512, 999), (300, 4096, 4096)], [(4, 300, 77)],
                                   [(1, 60000, 4100), (1, 60000, 4100), (1, 60000, 4100)], [(3, 100, 30), (3, 100, 100)]])
def test_grouped(specs):
    assert shares(TWO_BIT, specs) == [K >= 64 for M, N, K in specs]
    jobs, want = [], []
    for i, (M, N, K) in enumerate(specs):
        x, W, g = si.layer(49000 + i + M + N + K, M, N, K)
        yd = to_dev(np.full(M * N + 64, -21555, dtype=np.int16))
        jobs.append((to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), si.gamma_bits(g), yd, M, N, K))
        want.append((yd, x, W, g))
    tl.tl_ternary_gemm_grouped(jobs)
    for (yd, x, W, g), (M, N, K) in zip(want, specs):
        y = yd.cpu().numpy()
        assert (y[M * N:] == -21555).all()
        check(y[:M * N].view(np.float16).reshape(M, N), x, W, g, f"{M}x{N}x{K}")


def test_the_forced_path_still_refuses_it():
    x, W, g = si.layer(50000, 2, 64, 100)
    yd = to_dev(np.zeros((2, 64), dtype=np.int16))
    xd, wd = to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W))
    for path in (tl.TL_PATH_GEMV, tl.TL_PATH_MFMA):
        with pytest.raises(RuntimeError):
            tl.tl_ternary_gemm_path(xd, wd, si.gamma_bits(g), yd, 2, 64, 100, path=path)
    assert tl.tl_ternary_gemm_which(2, 64, 100) == tl.TL_PATH_GENERIC


# K a multiple of 64 up to 2048 and more than 16 rows: one launch with the blocks of rows in the grid's second dimension.  One wave to four per
# workgroup, a last block of one row, several tiles per workgroup, the most blocks that a launch has
@pytest.mark.parametrize("M,N,K", [(17, 16, 64), (33, 48, 512), (64, 2048, 1024), (37, 4096, 2048), (100, 1040, 1600), (20, 14336, 2048), (300, 528, 512), (47, 2064, 1472), (4096, 16, 64)])
def test_blocks_of_rows_in_one_launch(M, N, K):
    x, W, g = si.layer(49000 + M + N + K, M, N, K)
    yd = to_dev(np.full(M * N + 64, -21555, dtype=np.int16))
    tl.tl_ternary_gemm_path(to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), si.gamma_bits(g), yd, M, N, K, path=tl.TL_PATH_GEMV)
    y = yd.cpu().numpy()
    assert (y[M * N:] == -21555).all()
    check(y[:M * N].view(np.float16).reshape(M, N), x, W, g, f"{M}x{N}x{K}")


# what one launch keeps of the sums of several passes is 32 tiles a workgroup, 8192 in all: jobs beyond that are two launches, not one for each block of 16 rows
@pytest.mark.parametrize("specs,most", [([(2, 14336, 4608 + 8)] * 12, 2), ([(17, 14336, 4608), (17, 100, 999)] * 6, 3), ([(1, 60000, 4100)] * 3, 2), ([(3, 640, 4099), (16, 4096, 1024)], 1)])
def test_launches_of_long_runs(specs, most):
    tl.tl_init()
    jobs, want, layers = [], [], {}
    for M, N, K in specs:
        if (M, N, K) not in layers:
            x, W, g = si.layer(51000 + M + N + K, M, N, K)
            layers[M, N, K] = (x, W, g, to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)))
        x, W, g, xd, wd = layers[M, N, K]
        yd = to_dev(np.full(M * N, -21555, dtype=np.int16))
        jobs.append((xd, wd, si.gamma_bits(g), yd, M, N, K))
        want.append((yd, x, W, g))
    assert all(shares(TWO_BIT, specs))
    assert launches(lambda stream: tl.tl_ternary_gemm_grouped(jobs, stream)) <= most
    tl.tl_ternary_gemm_grouped(jobs)
    for (yd, x, W, g), (M, N, K) in zip(want, specs):
        check(yd.cpu().numpy().view(np.float16).reshape(M, N), x, W, g, f"{M}x{N}x{K}")


# Aligned jobs of short K that fill launches of their own leave those to them, since the form for any K has fewer workgroups there; others share its launches
@pytest.mark.parametrize("specs,count", [([(64, 32, 512)] * 9 + [(64, 15, 1296 + 1)], 3), ([(64, 32, 512)] * 7 + [(64, 15, 1296 + 1)], 1), ([(16, 48, 4096)] * 40 + [(16, 15, 1001)], 2)])
def test_launches_beside_aligned_jobs(specs, count):
    tl.tl_init()
    jobs, want = [], []
    for i, (M, N, K) in enumerate(specs):
        x, W, g = si.layer(52000 + i, M, N, K)
        yd = to_dev(np.full(M * N, -21555, dtype=np.int16))
        jobs.append((to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), si.gamma_bits(g), yd, M, N, K))
        want.append((yd, x, W, g))
    assert all(shares(TWO_BIT, specs))
    assert launches(lambda stream: tl.tl_ternary_gemm_grouped(jobs, stream)) == count
    tl.tl_ternary_gemm_grouped(jobs)
    for (yd, x, W, g), (M, N, K) in zip(want, specs):
        check(yd.cpu().numpy().view(np.float16).reshape(M, N), x, W, g, f"{M}x{N}x{K}")
