"""The tiled matrix-core kernel at the edges of its tiles, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2506_23025_amd as tl
import synth_inputs as si
from parity import REL_TOL, assert_close, dev_u32, floors, to_dev

pytestmark = pytest.mark.gpu


def _sampled(N, seed, most=300):
    """Columns to compare: all of a small matrix, else a sample with both ends and a tile edge."""
    if N <= 1100:
        return np.arange(N)
    cols = np.sort(np.random.default_rng(seed).choice(N, most, replace=False))
    cols[:2], cols[-2:] = (0, 255), (N - 2, N - 1)
    return np.unique(cols)


# The shapes take, by the library's cost model, tiles of 256 x 256 (rows and columns past the edge; 2, 3 and 1 steps
# of K, fewer than the ring is deep), 128 x 256, 128 x 128, 128 x 64, 64 x 64 and 32 x 64, with an N that is a multiple
# of 8 or not (16-byte or single stores) and a K whose last step is half empty (K % 128 = 64) where steps are 128.
TILE_SHAPES = [
    (1030, 8200, 128), (1030, 8201, 192), (2500, 2700, 64), (2048, 3000, 192), (300, 9000, 704), (515, 4099, 256),
    (117, 14340, 4096), (700, 1500, 320), (640, 2500, 1152), (129, 1030, 1088), (65, 1030, 192), (17, 70, 64),
    (512, 14340, 256), (400, 2050, 320),
]


@pytest.mark.parametrize("M,N,K", TILE_SHAPES)
def test_tile_2bit(M, N, K):
    x, W, g = si.layer(31000 + M + N + K, M, N, K)
    xd, wd = to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W))
    yd = to_dev(np.full((M, N), -1, dtype=np.int16))
    tl.tl_ternary_gemm_path(xd, wd, si.gamma_bits(g), yd, M, N, K, path=tl.TL_PATH_MFMA)
    y = yd.cpu().numpy().view(np.float16)
    cols = _sampled(N, M)
    assert np.isfinite(y).all()
    assert_close(y[:, cols], oracle.gemm(x, np.ascontiguousarray(W[cols]), g), x, g, f"tile {M}x{N}x{K}")


# 1.6-bit codes: 128 x 256, 128 x 128, 64 x 128, 64 x 64 and 32 x 64; K inside one step, one byte into the next, ending
# in a byte with 3 weights, in the first half of a 32-k block, and long; N with and without 16-byte stores.
TILE3_SHAPES = [
    (512, 14340, 4096), (2050, 2056, 1288), (500, 4100, 1600), (1030, 2050, 168), (500, 1030, 648), (700, 1100, 952),
    (60, 4096, 11008), (500, 600, 328), (190, 10000, 488),
    # as those of K = 1600, 168, 648 and 952 above, which the weight-streaming kernel takes since it is the faster one there (500 x 4100 x 1600
    # 18.0 / 16.3 us, 700 x 1100 x 952 8.0 / 6.8)
    (2050, 4100, 1600), (1700, 1884, 168), (2500, 1030, 648), (2100, 1430, 952), (82, 7958, 8008), (60, 9004, 5608),
]


@pytest.mark.parametrize("fx", [False, True])
@pytest.mark.parametrize("M,N,K", TILE3_SHAPES)
def test_tile_1p6(M, N, K, fx):
    x, W, g = si.layer(32000 + M + N + K, M, N, K)
    Wp = tl.tl_pack_1p6bit_fx(W) if fx else tl.tl_pack_1p6bit(W)
    yd = to_dev(np.full((M, N), -1, dtype=np.int16))
    (tl.tl_ternary_gemm_1p6_fx if fx else tl.tl_ternary_gemm_1p6)(to_dev(x.view(np.int16)), to_dev(Wp), si.gamma_bits(g), yd, M, N, K)
    y = yd.cpu().numpy().view(np.float16)
    cols = _sampled(N, M)
    assert np.isfinite(y).all()
    assert_close(y[:, cols], oracle.gemm(x, np.ascontiguousarray(W[cols]), g), x, g, f"tile 1.6 {M}x{N}x{K}")


# Group scales: every tile shape (and three calls so small that they go elsewhere); groups of 64 and more (one scale per 64 k), of 32, 48, 16 (one per 16 k), longer than K,
# ending inside a step and inside a group; N with and without 16-byte stores.
TILE_GS_SHAPES = [
    (1030, 8200, 192, 64), (2048, 3000, 192, 128), (300, 9000, 704, 256), (300, 9001, 704, 48), (117, 14340, 4096, 32),
    (640, 2500, 1152, 96), (129, 1030, 1088, 16), (40, 300, 1024, 128), (17, 70, 64, 4096), (16, 333, 4096, 64), (5, 40, 320, 64),
    (300, 9004, 704, 128), (300, 2050, 1024, 64), (300, 4100, 320, 32), (512, 14340, 256, 64),
]


@pytest.mark.parametrize("M,N,K,group", TILE_GS_SHAPES)
def test_tile_group_scales(M, N, K, group):
    rng = np.random.default_rng(33000 + M + N + K)
    x, W, _ = si.layer(33000 + M + N + K, M, N, K)
    s = si.group_scales(rng, -(-K // group), N)
    yd = to_dev(np.full((M, N), -1, dtype=np.int16))
    tl.tl_ternary_gemm_gs(to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), to_dev(s.view(np.int16)), group, yd, M, N, K)
    y = yd.cpu().numpy().view(np.float16)
    cols = _sampled(N, M)
    assert np.isfinite(y).all()
    ref = oracle.gemm_group_scales(x, np.ascontiguousarray(W[cols]), np.ascontiguousarray(s[:, cols]), group)
    assert_close(y[:, cols], ref, x, 0.05, f"tile scales {M}x{N}x{K} group {group}")   # no scale is above 0.05


# K that fits no 16-byte piece: X rows at any even byte, W rows at any word; K of one piece (the smallest the form takes),
# one short of and past a block, a piece, a step and the fetch depth; every tile shape of the three forms (the smallest K and
# the smallest matrices go to the plain kernels; the 1.6-bit form's smallest K below); N = 1 and N odd.
RAGGED_SHAPES = [
    (1, 1, 9), (3, 40, 33), (16, 333, 1001), (16, 4099, 255), (37, 4099, 4090), (70, 257, 127), (40, 1030, 129), (200, 2050, 257),
    (150, 8200, 641), (900, 2500, 1100), (1030, 4100, 383), (5, 64, 2044), (33, 130, 8190),
    (1024, 4096, 1001), (700, 2050, 127),
    (79, 4928, 74), (292, 730, 86),                        # 1.6-bit: the smaller tiles, ahead of the streaming kernel for short rows alone
]


@pytest.mark.parametrize("M,N,K", RAGGED_SHAPES)
def test_tile_odd_k(M, N, K):
    x, W, g = si.layer(34000 + M + N + K, M, N, K)
    cols = _sampled(N, M)
    ref = oracle.gemm(x, np.ascontiguousarray(W[cols]), g)
    xd, gb = to_dev(x.view(np.int16)), si.gamma_bits(g)
    yd = to_dev(np.full((M, N), -1, dtype=np.int16))

    def check(what, ref, gamma):
        y = yd.cpu().numpy().view(np.float16)
        assert np.isfinite(y).all()
        assert_close(y[:, cols], ref, x, gamma, f"odd K {what} {M}x{N}x{K}")
        yd.fill_(-1)

    tl.tl_ternary_gemm(xd, dev_u32(tl.tl_pack_2bit(W)), gb, yd, M, N, K)
    check("2-bit", ref, g)
    for fx in (False, True):
        Wp = to_dev(tl.tl_pack_1p6bit_fx(W) if fx else tl.tl_pack_1p6bit(W))
        (tl.tl_ternary_gemm_1p6_fx if fx else tl.tl_ternary_gemm_1p6)(xd, Wp, gb, yd, M, N, K)
        check(f"1.6-bit fx={fx}", ref, g)
    for group in (16, 144, 8192):
        s = si.group_scales(np.random.default_rng(K + group), -(-K // group), N)
        tl.tl_ternary_gemm_gs(xd, dev_u32(tl.tl_pack_2bit(W)), to_dev(s.view(np.int16)), group, yd, M, N, K)
        sref = oracle.gemm_group_scales(x, np.ascontiguousarray(W[cols]), np.ascontiguousarray(s[:, cols]), group)
        check(f"scales {group}", sref, 0.05)


# K of one piece: rows shorter than a step of X, a fetch of W and a 16-byte store, in the tiled kernel with 1.6-bit codes.  Outputs this small reach
# fp16's subnormal range, where rounding alone is 2^-25 whatever the value.
@pytest.mark.parametrize("K", [9, 15, 33])
def test_tile_smallest_odd_k(K):
    M, N = 2000, 2050
    x, W, g = si.layer(34800 + K, M, N, K)
    xd, gb = to_dev(x.view(np.int16)), si.gamma_bits(g)
    ref = oracle.gemm(x, W, g)
    for fx in (False, True):
        yd = to_dev(np.full((M, N), -1, dtype=np.int16))
        Wp = to_dev(tl.tl_pack_1p6bit_fx(W) if fx else tl.tl_pack_1p6bit(W))
        (tl.tl_ternary_gemm_1p6_fx if fx else tl.tl_ternary_gemm_1p6)(xd, Wp, gb, yd, M, N, K)
        y = yd.cpu().numpy().view(np.float16).astype(np.float64)
        assert (np.abs(y - ref) <= REL_TOL * np.maximum(np.abs(ref), floors(x, g, K)) + 2.0 ** -25).all()


def test_tile_odd_k_keeps_rows_apart():
    # a row of x with an infinity or a NaN next to rows without: the pieces that reach past K must not bring it in
    M, N, K = 40, 200, 1003
    x, W, g = si.layer(34900, M, N, K)
    x[3, 0], x[7, K - 1], x[39, 5] = np.inf, np.nan, -np.inf
    yd = to_dev(np.zeros((M, N), dtype=np.int16))
    tl.tl_ternary_gemm(to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), si.gamma_bits(g), yd, M, N, K)
    y = yd.cpu().numpy().view(np.float16)
    clean = np.setdiff1d(np.arange(M), [3, 7, 39])
    assert np.isfinite(y[clean]).all()
    assert_close(y[clean], oracle.gemm(x[clean], W, g), x[clean], g, "rows beside a NaN")
    assert np.isnan(y[7]).all()


def _with_spare_digits(Wp, K, fx, digit):
    """The packed rows with the digits past K of each row's last byte (the packers write 1) set to `digit`."""
    nb, rem = -(-K // 5), K - 5 * (-(-K // 5) - 1)
    P = Wp.copy()
    last = P[:, nb - 1].astype(int)
    if fx:                                                 # first weight: most significant digit
        v = (last * 243 >> 8) // 3 ** (5 - rem) * 3 ** (5 - rem) + digit * ((3 ** (5 - rem) - 1) // 2)
        last = (v * 256 + 242) // 243
    else:                                                  # first weight: least significant digit
        last = last % 3 ** rem + digit * ((3 ** 5 - 3 ** rem) // 2)
    P[:, nb - 1] = last.astype(np.uint8)
    return P


# K of one to four weights in a row's last byte, that byte first, in the middle and last of what a step and a thread fetch; few rows,
# which the streaming kernel takes, and many
@pytest.mark.parametrize("fx", [False, True])
@pytest.mark.parametrize("M,N,K", [(4, 600, 328), (500, 600, 328), (512, 4100, 4096), (60, 1030, 11008), (1030, 2050, 168), (700, 1100, 952),
                                   (500, 1030, 104), (40, 70, 8)])
def test_spare_digits_of_the_last_byte_do_not_count(M, N, K, fx):
    x, W, g = si.layer(39000 + M + N + K, M, N, K)
    Wp = tl.tl_pack_1p6bit_fx(W) if fx else tl.tl_pack_1p6bit(W)
    xd, gb = to_dev(x.view(np.int16)), si.gamma_bits(g)

    def product(packed):
        yd = to_dev(np.full((M, N), -1, dtype=np.int16))
        (tl.tl_ternary_gemm_1p6_fx if fx else tl.tl_ternary_gemm_1p6)(xd, to_dev(packed), gb, yd, M, N, K)
        return yd.cpu().numpy()

    want = product(Wp)
    for digit in (0, 2):
        other = _with_spare_digits(Wp, K, fx, digit)
        assert not np.array_equal(other, Wp)
        assert np.array_equal(tl.tl_unpack(tl.TL_FMT_1P6BIT_FX if fx else tl.TL_FMT_1P6BIT, other, N, K), W)
        assert np.array_equal(product(other), want), f"spare digits {digit}"


# An infinite scale makes the outputs of its column infinite, with the sign of scale times the group's sum, whatever the number of rows; a NaN
# makes them NaN; the other columns do not notice.  Tiles that store 16 bytes, 8 bytes and single values, with sets of waves side
# by side and not; K that ends inside a step.
@pytest.mark.parametrize("M,N,K,group", [(4, 300, 1024, 128), (40, 300, 1024, 128), (1030, 8200, 192, 128), (1030, 8204, 192, 128), (2048, 3000, 192, 256),
                                         (700, 9000, 704, 256), (300, 9004, 704, 128), (640, 2500, 1152, 384), (512, 4096, 1024, 128), (256, 4096, 512, 4096),
                                         (129, 1030, 1088, 16)])
def test_infinite_group_scales_with_many_rows(M, N, K, group):
    rng = np.random.default_rng(39500 + M + N + K)
    x, W, _ = si.layer(39500 + M + N + K, M, N, K)
    x[:, :] = np.where(x == 0, np.float16(0.5), x)
    s = si.group_scales(rng, -(-K // group), N)
    last = s.shape[0] - 1
    bad = {1: (0, np.inf), 64: (last, np.inf), 66: (last // 2, -np.inf), N - 1: (last, -np.inf), N - 30: (0, np.nan)}
    for n, (gi, v) in bad.items():
        s[gi, n] = v
    yd = to_dev(np.full((M, N), -1, dtype=np.int16))
    tl.tl_ternary_gemm_gs(to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), to_dev(s.view(np.int16)), group, yd, M, N, K)
    y = yd.cpu().numpy().view(np.float16)
    for n, (gi, v) in bad.items():
        k = slice(gi * group, min(K, (gi + 1) * group))
        part = x[:, k].astype(np.float64) @ W[n, k].astype(np.float64)
        if np.isnan(v):
            assert np.isnan(y[:, n]).all()
        else:
            assert (part != 0).all()                       # none here: NaN
            same = y[:, n].astype(np.float64) == np.sign(part) * v
            assert same.all(), f"column {n}: rows {np.flatnonzero(~same)[:8]}"
    cols = np.setdiff1d(_sampled(N, M), list(bad))
    ref = oracle.gemm_group_scales(x, np.ascontiguousarray(W[cols]), np.ascontiguousarray(s[:, cols]), group)
    assert_close(y[:, cols], ref, x, 0.05, f"beside infinite scales {M}x{N}x{K} group {group}")
