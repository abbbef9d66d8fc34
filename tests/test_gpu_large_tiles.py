"""Reduces by tiles of eight segments, which only indexed streams have: the limits of the rule that picks them, and last tiles of one segment, of four and of
five, with wide blocks and without, with both ways to read the chains, against the reference codec; what is wrong in the upper half of a tile; and calls of
which the host takes there to be more tiles than there are."""
import numpy as np
import pytest
import torch

import gpuutil as u
from paper_2502_18554_amd import synth
from paper_2502_18554_amd.binding import ZC_ERR_CAPACITY, ZC_ERR_FORMAT, ZC_ERR_RANGE, ZC_OK

SEG = 2048


@pytest.fixture(autouse=True)
def indexed_streams(zcref):
    u.set_variant(zcref, True)
    yield
    u.set_variant(zcref, False)


@pytest.fixture(params=["loads", "coherent_loads"])
def chains(request):
    u.set_coherent(request.param == "coherent_loads")
    yield request.param
    u.set_coherent(False)


pytestmark = [pytest.mark.gpu]


def _operands(zcref, k, n, seed, wide, first=900.0):
    base = synth.sinusoids(n, seed=seed).numpy()
    eb = synth.abs_bound(torch.from_numpy(base), 1e-3)
    refs = []
    for i in range(k):
        x = np.roll(base, 977 * i) if i else base.copy()
        if wide:
            x[np.random.default_rng(i).integers(0, n, 40)] = 900.0 if i else first      # blocks wider than 15 bits, which most tiles take beside the others ...
            if i == 0:
                x[5 * SEG:6 * SEG:2] = 900.0       # ... and a segment of nothing else, which its tile does not
        refs.append(zcref.compress(x, eb)[1])
    return refs


def _compare(zcref, refs, n, op, ws=None):
    st_ref, ref = zcref.reduce(refs, op=op)[:2]
    st, r, _ = u.gpu_reduce(refs, n, op=op or None, ws=ws)
    assert st == st_ref == ZC_OK and r.tobytes() == ref.tobytes(), u.first_diff(r, ref)


# segments (a tile of the rule's count is four): both sides of 900, 784 and 640 tiles, of 1024, of 1400 and 1536, 1700, 1780, 1850 and 2048
@pytest.mark.parametrize("k,segments", [(2, 900 * 4), (2, 900 * 4 + 1), (3, 784 * 4), (3, 784 * 4 + 5), (5, 640 * 4), (5, 640 * 4 + 1), (2, 1024 * 4 + 3), (5, 1024 * 4 + 1),
                                        (5, 1400 * 4 + 1), (2, 1536 * 4 + 1), (2, 1700 * 4 + 1), (3, 1780 * 4 + 4), (4, 1850 * 4 + 5), (6, 2048 * 4), (6, 2048 * 4 + 1)])
@pytest.mark.parametrize("wide", [False, True])
def test_sum_by_large_tiles(zcref, chains, k, segments, wide):
    n = segments * SEG - 33
    _compare(zcref, _operands(zcref, k, n, 11, wide), n, 0)


# Max and Min: both sides of 784 tiles, of 1024, of 1200 and 1300, 1400 and 1850, and beyond 2400 with two operands
@pytest.mark.parametrize("k,op,segments", [(2, 1, 784 * 4), (2, 2, 784 * 4 + 1), (3, 1, 1024 * 4), (3, 2, 1024 * 4 + 5), (2, 1, 1200 * 4 + 4), (4, 2, 1300 * 4 + 1), (5, 1, 1400 * 4 + 1),
                                           (4, 1, 1850 * 4 + 1), (2, 2, 2400 * 4 + 5)])
@pytest.mark.parametrize("wide", [False, True])
def test_extremes_by_large_tiles(zcref, chains, k, op, segments, wide):
    n = segments * SEG - 33
    _compare(zcref, _operands(zcref, k, n, 12, wide, -900.0), n, op)


# A width that its index does not agree with, in each half of a large tile, and an output that ends inside one.
@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("wide", [False, True])
def test_errors_in_large_tiles(zcref, op, wide):
    segments = 910 * 4
    n = segments * SEG - 33
    refs = _operands(zcref, 2, n, 13, wide)
    nb = (n + 31) // 32
    for seg in (8 * 100 + 2, 8 * 100 + 6, segments - 1):
        broken = refs[1].copy()
        at = u.widths_begin(nb) + 64 * seg + 3
        broken[at] = (int(broken[at]) + 1) % 31
        assert zcref.reduce([refs[0], broken], op=op)[0] == ZC_ERR_FORMAT == u.gpu_reduce([refs[0], broken], n, op=op or None)[0]
    total = zcref.reduce(refs, op=op)[2]
    for cap in (total - 4, (u.tables_end(nb) + total) // 2 // 4 * 4, u.tables_end(nb) + 4, u.tables_end(nb) - 16):
        st, _, need = u.gpu_reduce(refs, n, op=op or None, out_cap=cap)
        assert st == ZC_ERR_CAPACITY and need == total
    _compare(zcref, refs, n, op)


# A sum that leaves the range of codes, in each half of a large tile: the segment before holds just what fits.
@pytest.mark.parametrize("seg", [8 * 50 + 1, 8 * 50 + 5, 8 * 50 + 7])
def test_range_in_large_tiles(zcref, seg):
    n = 910 * 4 * SEG - 33
    q = np.zeros(n, np.int32)
    q[(seg - 1) * SEG + 40:seg * SEG] = 2 ** 29 - 1
    fits = zcref.encode_codes(q, 1e-3)[1]
    _compare(zcref, [fits, fits], n, 0)
    q[seg * SEG + 40:(seg + 1) * SEG] = 2 ** 29 + 5
    beyond = zcref.encode_codes(q, 1e-3)[1]
    assert u.gpu_reduce([beyond, beyond], n)[0] == ZC_ERR_RANGE == zcref.reduce([beyond, beyond])[0]


# A workspace and an output made for many more values: tiles of eight then reduce streams of any size, down to one of a few values.
@pytest.mark.parametrize("n", [33, 2049, 5 * 8192 + 1, 130 * 8192 - 1, 525 * 8192 - 777])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("made_for", [900 * 8192, 3000 * 8192])
def test_few_tiles_in_a_large_workspace(zcref, n, wide, made_for):
    refs = _operands(zcref, 3, n, 14, wide and n > 6 * SEG)
    room = 32 + 10 * (made_for // 32)              # streams whose sizes speak for as many tiles, as far as the host knows
    padded = [np.concatenate([r, np.zeros(max(0, room - r.size), np.uint8)]) for r in refs]
    ws = u.workspace(made_for, 3)
    for op in (0, 1, 2):
        st_ref, ref = zcref.reduce(refs, op=op)[:2]
        st, r, _ = u.gpu_reduce(padded, made_for, op=op or None, ws=ws)
        assert st == st_ref == ZC_OK and r.tobytes() == ref.tobytes(), (op, u.first_diff(r, ref))
