"""Argument validation of ditango_compose and ditango_attn_block_states, on the
host (nothing is launched)."""
import ctypes

import pytest

FAKE = 0x10000


@pytest.fixture(scope="module")
def compose():
    from paper_2607_15650_amd import _lib
    return _lib.lib().ditango_compose


def call(f, states=FAKE, lse=FAKE, sdt=1, P=4, slots=None, n=0, D=64, q_len=8, out=2 * FAKE, odt=1, lse_out=3 * FAKE,
         w=FAKE, ws=FAKE):
    sl = None if slots is None else (ctypes.c_int32 * max(len(slots), 1))(*slots)
    return f(states, lse, sdt, P, sl, n, 1, 2, D, q_len, out, odt, lse_out, w, ws, None)


def test_compose_argument_validation(compose):
    assert call(compose, states=None) == 1 and call(compose, lse=None) == 1 and call(compose, out=None) == 1
    assert call(compose, w=None) == 1 and call(compose, ws=None) == 1
    assert call(compose, ws=FAKE + 64) == 1                     # not 256-byte aligned
    assert call(compose, sdt=3) == 1 and call(compose, odt=-1) == 1
    assert call(compose, P=0) == 1 and call(compose, P=65) == 2 and call(compose, D=32) == 2
    assert call(compose, q_len=0) == 1
    assert call(compose, slots=[4], n=1) == 1 and call(compose, slots=[0], n=0) == 1


def test_compose_is_not_in_place(compose):
    slot = 8 * 2 * 64 * 2                                       # bytes of one bf16 OUT slot
    rows = 8 * 2 * 4                                            # bytes of one LSE slot
    assert call(compose, out=FAKE + 2 * slot) == 1
    assert call(compose, lse_out=FAKE + 3 * rows) == 1
    assert call(compose, slots=[1, 2], n=2, out=FAKE + 2 * slot) == 1


def test_attn_block_validation():
    from paper_2607_15650_amd import _lib
    f = _lib.lib().ditango_attn_block_states
    o = (ctypes.c_int64 * 3)(0, 5, 10)

    def block(rows, begin, q_len=10, q=FAKE, sel=(0, 0), D=64, ws=None):
        s = (ctypes.c_uint8 * 2)(*sel)
        return f(q, rows, begin, FAKE, FAKE, 1, 1, 2, D, q_len, o, 2, s, 0.1, FAKE, 1, FAKE, ws, 0, None)

    assert block(10, 0) == 0 and block(30, 20) == 0             # nothing selected: nothing launched
    assert block(9, 0) == 1 and block(30, 21) == 1 and block(30, -1) == 1
    assert block(30, 1 << 62) == 1 and block(30, 0, q=None) == 1 and block(30, 0, D=96) == 2
    assert block(30, 0, ws=FAKE + 64) == 1
