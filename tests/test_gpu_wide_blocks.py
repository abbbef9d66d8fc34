"""Blocks wider than 15 bits in the compressor, which stages them beside the others of their wave: how many of them, where, and up to how
many words of the wave, against the reference codec; both of the kernel's tiles."""
import numpy as np
import pytest

import gpuutil as u
from paper_2502_18554_amd.binding import ZC_ERR_BOUND, ZC_OK

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("stream_variant")]

EB = np.float32(1e-3)
BLOCKS = {"one": [0], "last": [63], "two": [5, 40], "three": [5, 40, 41], "neighbours": [30, 31, 32, 33], "many": list(range(0, 64, 2)), "all": list(range(64))}


def _compare(zcref, x):
    st_ref, ref = zcref.compress(x, EB)[:2]
    st, s, total = u.gpu_compress(x, EB)
    assert st == st_ref and st in (ZC_OK, ZC_ERR_BOUND) and total == ref.size and s.tobytes() == ref.tobytes(), u.first_diff(s, ref)


# 9 tiles of four waves, and 150 tiles of eight; the last wave is ragged, and its last block one value, or 31
@pytest.mark.parametrize("n", [9 * 8192 - 2048 - 31, 300 * 8192 - 2048 - 1])
@pytest.mark.parametrize("which", BLOCKS)
def test_wide_blocks(zcref, n, which):
    rng = np.random.default_rng(n + len(which))
    x = (np.sin(np.arange(n) / 300.0) + rng.normal(0, 1e-3, n)).astype(np.float32)
    for wave in (0, 3, 7, n // 2048):
        for b in BLOCKS[which]:
            at = wave * 2048 + 32 * b + int(rng.integers(0, 32))
            if at < n:
                x[at] = rng.choice((-1, 1)) * rng.uniform(100, 900)
    x[-1] = 700.0                                  # in the last block, which may be all of it
    _compare(zcref, x)


# both sides of the limits from which a wave with wide blocks goes over all its values again: two of them in small tiles, six in large ones
@pytest.mark.parametrize("n", [9 * 8192 - 31, 300 * 8192 - 2048 - 1])
@pytest.mark.parametrize("count", [1, 2, 3, 6, 7, 8])
def test_number_of_wide_blocks(zcref, n, count):
    rng = np.random.default_rng(n + count)
    x = (np.sin(np.arange(n) / 300.0) + rng.normal(0, 1e-3, n)).astype(np.float32)
    for wave in range(0, (n + 2047) // 2048, 2):   # every other wave, the ragged last one among them
        for b in rng.choice(62, count, replace=False):
            at = wave * 2048 + 32 * int(b) + int(rng.integers(0, 32))
            if at < n:
                x[at] = rng.choice((-1, 1)) * rng.uniform(100, 900)
    _compare(zcref, x)


# a wave of constant blocks but for `wide` of 30 planes, 31 words each: 1023 words, 1054, and the whole wave
@pytest.mark.parametrize("wide", [1, 32, 33, 34, 64])
def test_words_of_a_wave(zcref, wide):
    n = 4 * 8192
    x = np.zeros(n, np.float32)
    x[2048:4096:32][:wide] = np.float32(0.0)
    x[2048 + 7:4096:32][:wide] = np.float32(EB * 63 / 32 * 5.0e8)      # code 5e8: 29 bits and the way back
    x[10000] = 0.5
    _compare(zcref, x)
