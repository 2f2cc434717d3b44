"""Decode launches: single calls with one job's arguments, at the edges of their split into runs of tiles, and groups with long K."""
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
