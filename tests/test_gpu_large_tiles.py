"""Reduces by tiles of eight segments: the limits of the rule that picks them, and last tiles of one segment, of four and of
five, with wide blocks and without, against the reference codec."""
import numpy as np
import pytest
import torch

import gpuutil as u
from paper_2502_18554_amd import synth
from paper_2502_18554_amd.binding import ZC_OK

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("stream_variant")]

SEG = 2048


# segments (a tile of the rule's count is four): both sides of 768 and 640 tiles, of 1024, of 1400, of 1536, 1700 and 1900
@pytest.mark.parametrize("k,segments", [(2, 768 * 4), (2, 768 * 4 + 1), (3, 768 * 4 + 4), (3, 768 * 4 + 5), (5, 640 * 4 + 1), (2, 1024 * 4 + 3), (5, 1024 * 4 + 1),
                                        (5, 1400 * 4 + 1), (2, 1536 * 4 + 1), (2, 1700 * 4 + 1), (4, 1900 * 4 + 5)])
@pytest.mark.parametrize("wide", [False, True])
def test_sum_by_large_tiles(zcref, k, segments, wide):
    n = segments * SEG - 33
    base = synth.sinusoids(n, seed=11).numpy()
    eb = synth.abs_bound(torch.from_numpy(base), 1e-3)
    refs = []
    for i in range(k):
        x = np.roll(base, 977 * i) if i else base.copy()
        if wide:
            at = np.random.default_rng(i).integers(0, n, 40)
            x[at] = 900.0                          # blocks wider than 15 bits, which most tiles sum beside the others ...
            if i == 0:
                x[5 * SEG:6 * SEG:2] = 900.0       # ... and a segment of nothing else, which its tile does not
        refs.append(zcref.compress(x, eb)[1])
    st_ref, ref = zcref.reduce(refs)[:2]
    st, r, _ = u.gpu_reduce(refs, n)
    assert st == st_ref == ZC_OK and r.tobytes() == ref.tobytes(), u.first_diff(r, ref)


# Max and Min: both sides of 768 tiles, of 1024 and of 1400, and beyond 4096 with two operands
@pytest.mark.parametrize("k,op,segments", [(2, 1, 768 * 4), (2, 2, 768 * 4 + 1), (3, 1, 1024 * 4), (3, 2, 1024 * 4 + 5), (2, 1, 1024 * 4 + 4), (4, 1, 1400 * 4 + 1),
                                           (2, 2, 4096 * 4 + 5)])
@pytest.mark.parametrize("wide", [False, True])
def test_extremes_by_large_tiles(zcref, k, op, segments, wide):
    n = segments * SEG - 33
    base = synth.sinusoids(n, seed=12).numpy()
    eb = synth.abs_bound(torch.from_numpy(base), 1e-3)
    refs = []
    for i in range(k):
        x = np.roll(base, 977 * i) if i else base.copy()
        if wide:
            x[np.random.default_rng(i).integers(0, n, 40)] = 900.0 if i else -900.0
            if i == 0:
                x[5 * SEG:6 * SEG:2] = 900.0
        refs.append(zcref.compress(x, eb)[1])
    st_ref, ref = zcref.reduce(refs, op=op)[:2]
    st, r, _ = u.gpu_reduce(refs, n, op=op)
    assert st == st_ref == ZC_OK and r.tobytes() == ref.tobytes(), u.first_diff(r, ref)
