"""The packers' eight-at-a-time path: row lengths around its words and bytes, and every value that is no weight."""
import numpy as np
import pytest

import oracle
import paper_2506_23025_amd as tl
import synth_inputs as si

PACKERS = ((tl.tl_pack_2bit, oracle.pack2), (tl.tl_pack_1p6bit, oracle.pack3le), (tl.tl_pack_1p6bit_fx, oracle.pack3fx))


@pytest.mark.parametrize("K", [1, 5, 7, 8, 9, 12, 13, 15, 16, 17, 31, 32, 33, 40, 63, 64, 65, 80, 127, 128, 129, 1003])
def test_packers_match_the_oracle_at_every_row_end(K):
    W = si.ternary_weights(np.random.default_rng(K), 7, K)
    for pack, ref in PACKERS:
        assert np.array_equal(pack(W), ref(W)), pack.__name__


@pytest.mark.parametrize("value", [v for v in range(-128, 128) if v not in (-1, 0, 1)])
def test_packers_refuse_every_other_value(value):
    K = 83
    for k in (0, 7, 8, 15, 16, 40, 74, 75, 77, 79, 80, K - 1):
        W = np.zeros((2, K), dtype=np.int8)
        W[1, k] = value
        for pack, _ in PACKERS:
            with pytest.raises(tl.TlError) as e:
                pack(W)
            assert e.value.status == tl.TL_ERR_VALUE
