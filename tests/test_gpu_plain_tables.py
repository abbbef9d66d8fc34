"""Width tables of plain streams, summed by every workgroup: sizes around the pieces, batches and limits of that, against the
reference codec; bytes that are no width, wherever they are; bytes behind the table's last."""
import numpy as np
import pytest

import gpuutil as u
from paper_2502_18554_amd.binding import ZC_ERR_FORMAT, ZC_OK

pytestmark = pytest.mark.gpu

PIECE = 1024                                       # blocks of a load by a wave


@pytest.fixture(autouse=True)
def plain(zcref):
    u.set_variant(zcref, False)


def _stream(zcref, nb, seed, ragged=5):
    """Blocks of all widths from 0 to 31, most of them narrow."""
    rng = np.random.default_rng(seed)
    w = np.where(rng.random(nb) < 0.05, rng.integers(0, 29, nb), rng.integers(0, 4, nb))
    top = (np.int64(1) << w) - 1
    q = rng.integers(0, 2, (nb, 32)) * top[:, None]
    q[:, 0] = 0
    q[:, 1] = top
    return zcref.encode_codes(q.reshape(-1)[: nb * 32 - ragged].astype(np.int32), 0.5)[1]


# one wave's piece, the pieces asked for ahead (two a wave), the first batch behind them, of one stream (four waves share it), of two (two waves
# each) and of more (a wave each), and the limits up to which every workgroup sums the tables (480 and 512 tiles of 256 blocks)
@pytest.mark.parametrize("nb", [1, 15, 16, 17, PIECE, PIECE + 1, 2 * PIECE + 1, 6 * PIECE, 6 * PIECE + 1, 8 * PIECE + 1, 40 * PIECE, 40 * PIECE + 17,
                                512 * 256, 512 * 256 + 1])
def test_tables(zcref, nb):
    s = [_stream(zcref, nb, 7 * nb + i) for i in range(3)]
    n = nb * 32 - 5
    st, y, _ = u.gpu_decompress(s[0], n)
    assert st == ZC_OK and y.tobytes() == zcref.decompress(s[0])[1].tobytes()
    local = np.zeros(n, np.float32)
    st_ref, ref = zcref.reduce_step(s[0], local)[:2]
    st, r, _ = u.gpu_reduce_step(s[0], local)
    assert st == st_ref and r.tobytes() == ref.tobytes(), u.first_diff(r, ref)
    for k in (2, 3):
        st, ys, _ = u.gpu_decompress_many(s[:k], [n] * k)
        assert st == ZC_OK and all(a[:n].tobytes() == zcref.decompress(b)[1].tobytes() for a, b in zip(ys, s))
        for op in (None, 1):
            st_ref, ref = zcref.reduce(s[:k], op=op or 0)[:2]
            st, r, _ = u.gpu_reduce(s[:k], n, op=op)
            assert st == st_ref and (st != ZC_OK or r.tobytes() == ref.tobytes()), (k, op)


# The limits where tiles are handed out by tickets: 320 tiles of a ring round, 480 of up to four streams, 320, 256 and 192 of more.
@pytest.mark.parametrize("k,tiles", [(1, 320), (1, 321), (2, 240), (2, 241), (8, 40), (8, 41), (16, 16), (16, 17), (24, 8), (24, 9)])
def test_tables_by_tickets(zcref, k, tiles):
    nb = tiles * 256
    n = nb * 32 - 5
    s = [_stream(zcref, nb, 9 * nb + i) for i in range(k)]
    u.set_tickets(True)
    try:
        if k == 1:
            local = np.zeros(n, np.float32)
            st_ref, ref = zcref.reduce_step(s[0], local)[:2]
            st, r, _ = u.gpu_reduce_step(s[0], local)
            assert st == st_ref and r.tobytes() == ref.tobytes(), u.first_diff(r, ref)
        for op in (None, 1):
            st_ref, ref = zcref.reduce(s, op=op or 0)[:2]
            st, r, _ = u.gpu_reduce(s, n, op=op)
            assert st == st_ref == ZC_OK and r.tobytes() == ref.tobytes(), u.first_diff(r, ref)
    finally:
        u.set_tickets(False)


@pytest.mark.parametrize("byte", [32, 33, 0x7F, 0x80, 0x81, 0xE0, 0xFF])
def test_bytes_that_are_no_width(zcref, byte):
    nb = 10 * PIECE + 37
    good = _stream(zcref, nb, 3)
    for at in (0, 3, 2 * PIECE - 1, 9 * PIECE + 2, nb - 1):
        s = good.copy()
        s[32 + at] = byte
        assert zcref.decompress(s)[0] == ZC_ERR_FORMAT
        assert u.gpu_decompress(s, nb * 32)[0] == ZC_ERR_FORMAT, at
        assert u.gpu_reduce([good, s, good], nb * 32)[0] == ZC_ERR_FORMAT, at


def test_padding_of_the_table_does_not_count(zcref):
    nb = 8 * PIECE + 37
    s = _stream(zcref, nb, 4)
    ref = zcref.decompress(s)[1]
    s[32 + nb:32 + u.pad16(nb)] = 0xFF
    st, y, _ = u.gpu_decompress(s, nb * 32)
    assert st == ZC_OK and y.tobytes() == ref.tobytes()
