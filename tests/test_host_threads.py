"""The packers' rows dealt out to threads: sizes on both sides of a second thread and beyond the most there are, against the oracle."""
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
import paper_2506_23025_amd as tl
import synth_inputs as si

PACKERS = ((tl.tl_pack_2bit, oracle.pack2), (tl.tl_pack_1p6bit, oracle.pack3le), (tl.tl_pack_1p6bit_fx, oracle.pack3fx))
SIZES = [(1, 2_100_000), (2, 1_000_001), (3, 700_003), (7, 300_001), (33, 61_000), (1999, 1003), (4097, 2050), (300_001, 7)]


@pytest.mark.parametrize("N,K", SIZES)
def test_packers_match_the_oracle(N, K):
    W = si.ternary_weights(np.random.default_rng(N), N, K)
    for pack, ref in PACKERS:
        assert np.array_equal(pack(W), ref(W)), pack.__name__


def test_a_value_that_is_no_weight_is_found_in_every_piece():
    N, K = 2003, 2051
    W = si.ternary_weights(np.random.default_rng(5), N, K)
    for n in list(range(0, N, 61)) + [N - 1]:
        W[n, n % K] = 2
        for pack, _ in PACKERS:
            with pytest.raises(tl.TlError) as e:
                pack(W)
            assert e.value.status == tl.TL_ERR_VALUE
        W[n, n % K] = 0


def test_calls_from_several_threads_and_on_one_cpu():
    W = si.ternary_weights(np.random.default_rng(6), 1201, 3000)
    want = [ref(W) for _, ref in PACKERS]
    with ThreadPoolExecutor(4) as pool:
        got = list(pool.map(lambda i: PACKERS[i % 3][0](W), range(12)))
    assert all(np.array_equal(g, want[i % 3]) for i, g in enumerate(got))
    allowed = os.sched_getaffinity(0)
    try:
        os.sched_setaffinity(0, {min(allowed)})
        assert np.array_equal(tl.tl_pack_2bit(W), want[0])
    finally:
        os.sched_setaffinity(0, allowed)
