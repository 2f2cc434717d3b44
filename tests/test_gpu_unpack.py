"""Device unpacking: rows, blocks and output addresses that its 16-byte pieces do not fit."""
import numpy as np
import pytest

import paper_2506_23025_amd as tl
import synth_inputs as si
from parity import to_dev

pytestmark = pytest.mark.gpu


# K below, at and past a piece, many rows to a piece, a piece across rows in every position, more than one block of
# 16384 weights, K far from and just off multiples of 16 and 5; the output starting at every kind of address.
@pytest.mark.parametrize("N,K", [(1, 1), (1000, 3), (17, 15), (64, 16), (9, 33), (40, 1000), (5, 16384), (3, 16399), (129, 4095), (16, 4096),
                                 # four pieces per thread from 2^22 weights on: whole blocks, a last one of a few pieces, rows across pieces
                                 (1024, 4096), (1100, 4095), (13107, 321)])
@pytest.mark.parametrize("offset", [0, 1, 7, 15])
def test_unpack_any_row_and_address(N, K, offset):
    import torch
    W = si.ternary_weights(np.random.default_rng(7 * N + K), N, K)
    for fmt, P in ((tl.TL_FMT_2BIT, tl.tl_pack_2bit(W).view(np.int32)), (tl.TL_FMT_1P6BIT, tl.tl_pack_1p6bit(W)),
                   (tl.TL_FMT_1P6BIT_FX, tl.tl_pack_1p6bit_fx(W))):
        buf = torch.full((N * K + 64,), 77, dtype=torch.int8, device="cuda")
        out = buf[16 + offset:16 + offset + N * K]
        tl.tl_unpack_dev(fmt, to_dev(P), N, K, out)
        got = buf.cpu().numpy()
        assert np.array_equal(got[16 + offset:16 + offset + N * K].reshape(N, K), W)
        assert (got[:16 + offset] == 77).all() and (got[16 + offset + N * K:] == 77).all()      # nothing beside it


def test_unpack_invalid_codes():
    # code 3 is +2; a byte above 242 has the digits of the byte - 243 (plain) or of floor(243 b / 256) (fixed point)
    import torch
    words = np.array([0xFFFFFFFF, 0xE4E4E4E4], dtype=np.uint32).view(np.int32)
    out = torch.empty(32, dtype=torch.int8, device="cuda")
    tl.tl_unpack_dev(tl.TL_FMT_2BIT, to_dev(words), 1, 32, out)
    assert out.cpu().tolist() == [2] * 16 + [-1, 0, 1, 2] * 4
    b = np.arange(256, dtype=np.uint8)
    out = torch.empty(1280, dtype=torch.int8, device="cuda")
    for fmt, v, order in ((tl.TL_FMT_1P6BIT, b.astype(int) % 243, range(5)), (tl.TL_FMT_1P6BIT_FX, (b.astype(int) * 243) >> 8, range(4, -1, -1))):
        tl.tl_unpack_dev(fmt, to_dev(b), 1, 1280, out)
        ref = np.stack([v // 3 ** i % 3 - 1 for i in order], axis=1).reshape(-1)
        assert np.array_equal(out.cpu().numpy(), ref)
