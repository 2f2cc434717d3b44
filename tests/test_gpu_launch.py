"""Decode launches: single calls with one job's arguments, at the edges of their split into runs of tiles, and groups with long K and with group scales."""
import numpy as np
import pytest

import oracle
import paper_2506_23025_amd as tl
import synth_inputs as si
from parity import assert_close, dev_u32, to_dev

pytestmark = pytest.mark.gpu


# one tile; fewer, as many and one more than the workgroups of a K (256 / waves per group); runs of 1 to 3 and more with and
# without longer ones; then long K: one and two tiles per workgroup, an odd number of tiles
@pytest.mark.parametrize("M,N,K", [(1, 16, 4096), (1, 4080, 4096), (3, 4096, 4096), (16, 4112, 4096), (2, 8208, 4096), (1, 20496, 4096),
                                   (1, 4096, 512), (5, 16400, 1024), (1, 16, 4160), (4, 4096, 4608), (1, 4112, 8192), (16, 8176, 4672)])
def test_single_decode_call(M, N, K):
    import torch
    x, W, g = si.layer(35000 + M + N + K, M, N, K)
    xd, wd, gb = to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), si.gamma_bits(g)
    yd = to_dev(np.full((M, N), -1, dtype=np.int16))
    tl.tl_ternary_gemm(xd, wd, gb, yd, M, N, K)
    y = yd.cpu().numpy().view(np.float16)
    cols = np.unique(np.r_[0:16, N - 16:N, np.random.default_rng(N).choice(N, min(N, 200), replace=False)])
    assert np.isfinite(y).all()
    assert_close(y[:, cols], oracle.gemm(x, np.ascontiguousarray(W[cols]), g), x, g, f"single call {M}x{N}x{K}")
    # the call goes to the stream that is current, also on a stream that is not the first one used
    side = torch.cuda.Stream()
    yd.fill_(-1)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(2000000)
        tl.tl_ternary_gemm(xd, wd, gb, yd, M, N, K)
        on_side = yd.clone()                               # right behind it on the same stream
    side.synchronize()
    assert np.array_equal(on_side.cpu().numpy(), y.view(np.int16))


# grouped calls with K beyond one pass of the waves: one, two, three tiles in the last item of a run; a second or third pass with one
# wave, some and all waves at work; K ending inside a slice
@pytest.mark.parametrize("M", [1, 5, 16])
@pytest.mark.parametrize("sizes", [[(4096, 4096)] * 3 + [(4096, 11008)], [(1024, 4096), (1040, 4160)], [(6160, 8192), (16400, 4672)],
                                   [(4096, 4096), (8208, 12352)], [(16, 8256), (24576, 4096)]])
def test_grouped_calls_with_long_k(M, sizes):
    jobs, want = [], []
    for i, (N, K) in enumerate(sizes):
        x, W, g = si.layer(36000 + M + i + N + K, M, N, K)
        yd = to_dev(np.full((M, N), -1, dtype=np.int16))
        jobs.append((to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), si.gamma_bits(g), yd, M, N, K))
        cols = np.unique(np.r_[0:16, N - 16:N, np.random.default_rng(N).choice(N, min(N, 200), replace=False)])
        want.append((yd, cols, oracle.gemm(x, np.ascontiguousarray(W[cols]), g), x, g))
    tl.tl_ternary_gemm_grouped(jobs)
    for (yd, cols, ref, x, g), (N, K) in zip(want, sizes):
        y = yd.cpu().numpy().view(np.float16)
        assert np.isfinite(y).all()
        assert_close(y[:, cols], ref, x, g, f"long K in a group {M}x{N}x{K}")


# scales per group of a multiple of 256 weights, N a multiple of 16: groups of half a slice, of one and one and a half slices, of all of K,
# with and without several passes, alone and in a group; one to three tiles in the last item
@pytest.mark.parametrize("M,sizes,group", [(4, [(4096, 4096)] * 2 + [(4096, 11008)], 256), (1, [(1040, 4096), (8208, 4672)], 768), (16, [(16400, 8192)], 512),
                                           (5, [(16, 4096)], 4096), (3, [(4112, 1024), (12304, 1024)], 256), (2, [(2064, 4160)], 256),
                                           # and large enough for the lean kernel as a group, with one pass and with two
                                           (3, [(4112, 1024), (49168, 1024)], 256), (5, [(1040, 4096), (16400, 4672)], 768), (2, [(11584, 5760)], 256)])
def test_decode_with_group_scales(M, sizes, group):
    jobs, want = [], []
    for i, (N, K) in enumerate(sizes):
        x, W, _ = si.layer(37000 + M + i + N + K, M, N, K)
        sc = si.group_scales(np.random.default_rng(N + K), (K + group - 1) // group, N)
        yd = to_dev(np.full((M, N), -1, dtype=np.int16))
        jobs.append((to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), to_dev(sc.view(np.int16)), group, yd, M, N, K))
        cols = np.unique(np.r_[0:16, N - 16:N, np.random.default_rng(N).choice(N, min(N, 200), replace=False)])
        want.append((yd, cols, oracle.gemm_packed2_group_scales(x, tl.tl_pack_2bit(np.ascontiguousarray(W[cols])),
                                                                np.ascontiguousarray(sc[:, cols]), group, K), x, float(sc.max())))
    tl.tl_ternary_gemm_gs_grouped(jobs)
    for (yd, cols, ref, x, g), (N, K) in zip(want, sizes):
        y = yd.cpu().numpy().view(np.float16)
        assert np.isfinite(y).all()
        assert_close(y[:, cols], ref, x, g, f"group scales {M}x{N}x{K} / {group}")


def test_an_infinite_group_scale_stays_in_its_output():
    # K of nine slices: waves without a slice in the second pass must not turn their zeros into NaN
    M, N, K, group = 1, 2048, 4608, 4608
    x, W, _ = si.layer(38001, M, N, K)
    x, W[100] = np.abs(x), 1                               # every partial sum of the column is positive
    sc = si.group_scales(np.random.default_rng(5), 1, N)
    sc[0, 100] = np.inf
    yd = to_dev(np.zeros((M, N), dtype=np.int16))
    tl.tl_ternary_gemm_gs(to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), to_dev(sc.view(np.int16)), group, yd, M, N, K)
    y = yd.cpu().numpy().view(np.float16)[0]
    assert np.isinf(y[100]) and np.isfinite(np.delete(y, 100)).all()


# a group longer than K is the one group there is, however long: few rows (units of 256 and of 128 weights), many rows, odd K
@pytest.mark.parametrize("M,N,K", [(1, 4096, 4096), (16, 48, 11008), (40, 1024, 512), (600, 1030, 1024), (3, 50, 100)])
def test_groups_longer_than_k(M, N, K):
    x, W, _ = si.layer(38100 + M + N + K, M, N, K)
    xd, wd = to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W))
    sd = to_dev(si.group_scales(np.random.default_rng(K), 1, N).view(np.int16))

    def product(group):
        yd = to_dev(np.full((M, N), -1, dtype=np.int16))
        tl.tl_ternary_gemm_gs(xd, wd, sd, group, yd, M, N, K)
        return yd.cpu().numpy()

    for step in (256, 128, 16):                            # multiples of 256, odd multiples of 128, of 16
        first = (K // 256 + 1) * 256 + (step if step < 256 else 0)
        want = product(first)
        assert np.isfinite(want.view(np.float16)).all()
        for base in (1 << 31, 1 << 40, (1 << 63) - 512):
            assert np.array_equal(product(base + (step if step < 256 else 0)), want), f"group {base} + {step}"
