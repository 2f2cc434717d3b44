"""Group scales in the weight-streaming kernel: groups that are multiples of 32, 64, 128 and 256 weights, of which each kind has a form of its own."""
import numpy as np
import pytest

import oracle
import paper_2506_23025_amd as tl
import synth_inputs as si
from parity import assert_close, dev_u32, launches, to_dev
from test_tile_choice import SCALES, STREAMS, TILED, TWO_BIT, runs, shares

pytestmark = pytest.mark.gpu


def inputs(M, N, K, group, seed):
    x, W, _ = si.layer(seed, M, N, K)
    return x, W, si.group_scales(np.random.default_rng(seed), -(-K // group), N)


def on_device(x, W, sc, M, N):
    return to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), to_dev(sc.view(np.int16)), to_dev(np.full(M * N + 64, -21555, dtype=np.int16))


def result(yd, M, N):
    y = yd.cpu().numpy()
    assert (y[M * N:] == -21555).all(), "guard behind y"
    return y[:M * N].view(np.float16).reshape(M, N)


def product(M, N, K, group, seed, x=None, sc=None):
    x0, W, sc0 = inputs(M, N, K, group, seed)
    x, sc = x0 if x is None else x, sc0 if sc is None else sc
    xd, wd, sd, yd = on_device(x, W, sc, M, N)
    tl.tl_ternary_gemm_gs(xd, wd, sd, group, yd, M, N, K)
    return result(yd, M, N), x, W, sc


def check(y, x, W, sc, group, what):
    N = W.shape[0]
    cols = np.unique(np.r_[0:min(N, 20), max(0, N - 20):N, np.random.default_rng(N).choice(N, min(N, 100), replace=False)])
    ref = oracle.gemm_group_scales(x, np.ascontiguousarray(W[cols]), np.ascontiguousarray(sc[:, cols]), group)
    assert_close(y[:, cols], ref, x, float(sc.max()), what)


# one slice of 512 weights and its edges, a chunk of 64 and one more, N of a quad, of part of a tile and of many; one tile to several items per
# workgroup; one pass, several, and waves without a slice in the last one; blocks of rows
SHAPES = [(1, 4, 64), (3, 20, 128), (2, 16, 192), (4, 64, 512), (16, 1000, 576), (5, 272, 1088), (16, 4096, 4096), (4, 14336, 4096), (9, 30000, 1024), (1, 100, 4160),
          (16, 2048, 8192), (7, 4096, 11008), (2, 20000, 4608), (3, 528, 32768), (33, 512, 1024), (70, 1040, 4224)]


@pytest.mark.parametrize("group", [32, 64, 96, 128, 192, 256, 384, 1 << 20])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_groups(M, N, K, group):
    assert runs(SCALES, M, N, K, group) == STREAMS
    y, x, W, sc = product(M, N, K, group, 61000 + M + N + K)
    check(y, x, W, sc, group, f"{M}x{N}x{K} group {group}")


# K no multiple of 64: the last chunk of a row starts anywhere in units of 16 weights
@pytest.mark.parametrize("group", [64, 128, 192, 256])
@pytest.mark.parametrize("M,N,K", [(1, 4, 65), (4, 20, 127), (3, 64, 513), (16, 1000, 1003), (4, 4096, 4090), (16, 2048, 4104), (8, 20000, 2049), (5, 9000, 6001), (37, 516, 3000), (1, 100, 32760)])
def test_groups_of_any_k(M, N, K, group):
    assert runs(SCALES, M, N, K, group) == STREAMS
    y, x, W, sc = product(M, N, K, group, 62000 + M + N + K)
    check(y, x, W, sc, group, f"{M}x{N}x{K} group {group}")


# jobs of one call: kinds of groups side by side, short and long K, many rows, runs too long for what one launch keeps of their sums
@pytest.mark.parametrize("specs", [[(4, 12288, 4096, 64), (4, 4096, 4096, 64), (4, 22016, 4096, 64), (4, 4096, 11008, 64)],
                                   [(16, 1536, 512, 32), (3, 512, 512, 128), (7, 2816, 512, 256), (7, 512, 1408, 64), (5, 1000, 1003, 64), (2, 300, 777, 64), (2, 300, 777, 32)],
                                   [(40, 2048, 2048, 128), (40, 516, 2048, 128), (1, 64, 16384, 128)], [(2, 60000, 4608, 64), (2, 60000, 4608, 64), (2, 90000, 4608, 64)]])
def test_groups_in_one_call(specs):
    host = [inputs(M, N, K, group, 63000 + i + M + N + K) for i, (M, N, K, group) in enumerate(specs)]
    dev = [on_device(x, W, sc, M, N) for (x, W, sc), (M, N, K, group) in zip(host, specs)]
    tl.tl_ternary_gemm_gs_grouped([(xd, wd, sd, group, yd, M, N, K) for (xd, wd, sd, yd), (M, N, K, group) in zip(dev, specs)])
    for (x, W, sc), (_, _, _, yd), (M, N, K, group) in zip(host, dev, specs):
        check(result(yd, M, N), x, W, sc, group, f"{M}x{N}x{K} group {group}")
    # all but groups of 32 with a K that is no multiple of 64, which the streaming kernel does not take
    assert shares(SCALES, specs) == [group != 32 or K % 64 == 0 for M, N, K, group in specs]


# a few small jobs, which find their place in a table of jobs: of 2 to 16 jobs, of equal and of different numbers of slices, N of quads, more
# workgroups than 256, one gamma or scales; one job more than the table holds
@pytest.mark.parametrize("group", [0, 64, 256])
@pytest.mark.parametrize("specs", [[(1, 512, 512)] * 2, [(3, 528, 1024)] * 8, [(2, 64, 2048), (16, 4096, 2048), (1, 16, 2048)] * 3, [(i + 1, 512, 1024) for i in range(16)], [(1, 256, 512)] * 17,
                                   [(4, 1024, 512), (4, 20, 1024), (4, 1000, 4096)], [(1, 12288, 1024), (2, 12288, 1024)], [(1, 16, 64), (1, 16, 4096)]])
def test_small_jobs_in_one_call(specs, group):
    assert all(shares(SCALES if group else TWO_BIT, [(*s, group) for s in specs]))
    host = [inputs(M, N, K, group or 1 << 20, 66000 + i + M + N + K) for i, (M, N, K) in enumerate(specs)]
    dev = [on_device(x, W, sc, M, N) for (x, W, sc), (M, N, K) in zip(host, specs)]
    if group:
        tl.tl_ternary_gemm_gs_grouped([(xd, wd, sd, group, yd, M, N, K) for (xd, wd, sd, yd), (M, N, K) in zip(dev, specs)])
    else:
        tl.tl_ternary_gemm_grouped([(xd, wd, si.gamma_bits(np.float16(0.02)), yd, M, N, K) for (xd, wd, sd, yd), (M, N, K) in zip(dev, specs)])
    for (x, W, sc), (_, _, _, yd), (M, N, K) in zip(host, dev, specs):
        sc = sc if group else np.full((1, N), 0.02, dtype=np.float16)
        check(result(yd, M, N), x, W, sc, group or 1 << 20, f"{M}x{N}x{K} group {group}")


# The same calls in a graph, whose launches carry records where the table's look-ups cost more: every replay gives what the call gives
@pytest.mark.parametrize("group", [0, 64, 256])
@pytest.mark.parametrize("specs", [[(1, 2048, 2048)] * 2, [(3, 4096, 4096), (16, 528, 4096)], [(2, 64, 2048), (5, 8192, 2048)], [(18, 512, 512), (1, 512, 512)]])
def test_small_jobs_in_a_graph(specs, group):
    import torch
    assert all(shares(SCALES if group else TWO_BIT, [(*s, group) for s in specs]))
    host = [inputs(M, N, K, group or 1 << 20, 67000 + i + M + N + K) for i, (M, N, K) in enumerate(specs)]
    dev = [on_device(x, W, sc, M, N) for (x, W, sc), (M, N, K) in zip(host, specs)]
    if group:
        jobs = tl.make_gs_jobs([(xd, wd, sd, group, yd, M, N, K) for (xd, wd, sd, yd), (M, N, K) in zip(dev, specs)])
        call = lambda: tl.tl_ternary_gemm_gs_grouped(jobs)
    else:
        jobs = tl.make_jobs([(xd, wd, si.gamma_bits(np.float16(0.02)), yd, M, N, K) for (xd, wd, _, yd), (M, N, K) in zip(dev, specs)])
        call = lambda: tl.tl_ternary_gemm_grouped(jobs)
    tl.tl_init()
    call()
    want = [yd.clone() for _, _, _, yd in dev]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(4):
        for _, _, _, yd in dev:
            yd.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        for w, (_, _, _, yd), (M, N, K) in zip(want, dev, specs):
            assert torch.equal(w[:M * N], yd[:M * N])
        call()


# An infinite scale makes the outputs of its column infinite, with the sign of scale times the group's sum, and leaves the others alone; K that
# ends within a unit, a slice and a pass.  A NaN or an infinity in x stays in its row.
@pytest.mark.parametrize("M,N,K,group", [(4, 64, 448, 64), (4, 64, 4032, 32), (16, 96, 4096, 128), (3, 48, 5056, 64), (5, 64, 8256, 128), (4, 64, 1003, 64), (2, 64, 4800, 32)])
def test_infinite_scales_and_activations(M, N, K, group):
    x, W, sc = inputs(M, N, K, group, 64000 + K)
    last = sc.shape[0] - 1
    bad = {1: (0, np.inf), 17: (last, np.inf), 30: (last // 2, -np.inf), N - 1: (last, -np.inf), N - 2: (0, np.nan)}
    for n, (g, v) in bad.items():
        sc[g, n] = v
    y, _, _, _ = product(M, N, K, group, 64000 + K, x, sc)
    good = np.setdiff1d(np.arange(N), list(bad))
    check(y[:, good], x, W[good], np.ascontiguousarray(sc[:, good]), group, "beside infinite scales")
    for n, (g, v) in bad.items():
        if np.isnan(v):
            assert np.isnan(y[:, n]).all()
            continue
        sums = x[:, g * group:(g + 1) * group].astype(np.float64) @ W[n, g * group:(g + 1) * group].astype(np.float64)
        for m in range(M):
            if sums[m]:
                assert y[m, n] == np.float16(v * sums[m]), (m, n, y[m, n])
    x2, _, sc2 = inputs(M, N, K, group, 64000 + K)
    x2 = x2.copy()
    x2[1, K - 1], x2[0, 3] = np.nan, np.inf
    y2, _, _, _ = product(M, N, K, group, 64000 + K, x2, sc2)
    assert np.isnan(y2[1]).all() and not np.isfinite(y2[0].astype(np.float32)).any()
    if M > 2:
        check(y2[2:], x2[2:], W, sc2, group, "rows beside a NaN")


@pytest.mark.parametrize("M,N,K,group,kernel", [(4096 + 17, 16, 512, 64, TILED), (4096 + 17, 4, 12288, 256, STREAMS)])
def test_rows_of_several_launches(M, N, K, group, kernel):
    assert runs(SCALES, M, N, K, group) == kernel
    x, W, sc = inputs(M, N, K, group, 65000)
    y, _, _, _ = product(M, N, K, group, 65000, x, sc)
    rows = np.r_[0:20, 4080:M]
    check(y[rows], x[rows], W, sc, group, "many rows")


# Shared launches: as many jobs as a launch holds find their place in a table where 256 records do not do (more workgroups, jobs with fewer slices than waves);
# runs too long for what one launch keeps of their sums are two launches
@pytest.mark.parametrize("specs,count", [([(16, 1024, 512, 256)] * 32, 1), ([(5, 528, 1024, 64), (16, 300, 512, 64), (1, 20, 2048, 64)] * 10, 1), ([(9, 516, 1000, 128)] * 24, 1),
                                         ([(70, 1024, 1024, 32)] * 6, 1), ([(70, 1024, 1024, 32)] * 7, 2), ([(2, 14336, 4608, 64)] * 12, 2), ([(2, 14336, 4600, 64)] * 12, 2)])
def test_launches_of_many_jobs(specs, count):
    tl.tl_init()
    assert all(shares(SCALES, specs))
    made, jobs, want = {}, [], []
    for i, (M, N, K, group) in enumerate(specs):
        if (M, N, K, group) not in made:
            x, W, sc = inputs(M, N, K, group, 68000 + M + N + K)
            made[M, N, K, group] = (x, W, sc, to_dev(x.view(np.int16)), dev_u32(tl.tl_pack_2bit(W)), to_dev(sc.view(np.int16)))
        x, W, sc, xd, wd, sd = made[M, N, K, group]
        yd = to_dev(np.full(M * N + 64, -21555, dtype=np.int16))
        jobs.append((xd, wd, sd, group, yd, M, N, K))
        want.append((x, W, sc, yd))
    assert launches(lambda stream: tl.tl_ternary_gemm_gs_grouped(jobs, stream)) == count
    tl.tl_ternary_gemm_gs_grouped(jobs)
    for (x, W, sc, yd), (M, N, K, group) in zip(want, specs):
        check(result(yd, M, N), x, W, sc, group, f"{M}x{N}x{K} group {group}")
