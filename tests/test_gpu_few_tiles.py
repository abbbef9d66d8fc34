"""Streams of few tiles take ways of their own through the kernels that write streams (all tiles run at once then, and
round trips are what counts): sizes around the limits of those ways, against the reference codec."""
import numpy as np
import pytest
import torch

import gpuutil
from paper_2502_18554_amd import synth
from paper_2502_18554_amd.binding import ZC_ERR_ARG, ZC_ERR_CAPACITY, ZC_ERR_FORMAT, ZC_ERR_MISMATCH, ZC_OK, ZC_STREAM_PLAIN

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("stream_variant")]

TILE = 8192                                        # of the ring round and the reduces; the compressor's is twice that


def _values(n, seed):
    """Smooth values with a block wider than 15 bits near the start, so that the mark of such blocks has to travel."""
    x = synth.sinusoids(n, seed=seed).numpy().copy()
    x[37] = 900.0
    return x


# one lane, wave and round of lanes of the direct look-back more than the tile before needs (64, 256 and 512 tiles),
# and both sides of its limits (512 and 1024 tiles)
@pytest.mark.parametrize("tiles", [2, 8, 9, 64, 65, 256, 257, 512, 513, 1024, 1025])
def test_streams_of_few_tiles(zcref, tiles):
    u = gpuutil
    n = tiles * TILE - 4097
    xs = [_values(n, 40 + i) for i in range(4)]
    eb = synth.abs_bound(torch.from_numpy(synth.sinusoids(n, seed=1).numpy()), 1e-3)
    st_ref, ref = zcref.compress(xs[0], eb)[:2]
    st, s, total = u.gpu_compress(xs[0], eb)
    assert st == st_ref and total == ref.size and s.tobytes() == ref.tobytes(), u.first_diff(s, ref)
    refs = [ref] + [zcref.compress(x, eb)[1] for x in xs[1:]]
    for k, op in ((2, None), (4, None), (2, 1)):
        st_ref, red_ref = zcref.reduce(refs[:k], op=op or 0)[:2]
        st, red, _ = u.gpu_reduce(refs[:k], n, op=op)
        assert st == st_ref == ZC_OK and red.tobytes() == red_ref.tobytes(), (k, op, u.first_diff(red, red_ref))
    st_ref, step_ref = zcref.reduce_step(refs[0], xs[1])[:2]
    st, step, _ = u.gpu_reduce_step(refs[0], xs[1])
    assert st == st_ref and step.tobytes() == step_ref.tobytes(), u.first_diff(step, step_ref)
    n2 = 2 * tiles * TILE - 4097                   # the compressor's own tiles: as many
    x = _values(n2, 50)
    st_ref, ref = zcref.compress(x, eb)[:2]
    st, s, total = u.gpu_compress(x, eb)
    assert st == st_ref and total == ref.size and s.tobytes() == ref.tobytes(), u.first_diff(s, ref)


# the same with tiles handed out by tickets, on both sides of both limits
@pytest.mark.parametrize("tiles", [9, 512, 513, 1024, 1025])
def test_streams_of_few_tiles_by_ticket(zcref, tiles):
    gpuutil.set_tickets(True)
    try:
        test_streams_of_few_tiles(zcref, tiles)
    finally:
        gpuutil.set_tickets(False)


# both sides of the size from which ring rounds of indexed streams run with more workgroups per compute unit, and plain ones
# that are indexed ahead
@pytest.mark.parametrize("tickets", [False, True])
@pytest.mark.parametrize("tiles", [2047, 2048])
def test_ring_rounds_of_many_tiles(zcref, tiles, tickets):
    u = gpuutil
    n = tiles * TILE - 4097
    xs = [_values(n, 80 + i) for i in range(2)]
    ref = zcref.compress(xs[0], 1e-3)[1]
    u.set_tickets(tickets)
    try:
        for op in (0, 1, 2):
            st_ref, step_ref = zcref.reduce_step(ref, xs[1], op=op)[:2]
            st, step, _ = u.gpu_reduce_step(ref, xs[1], op=op)
            assert st == st_ref and step.tobytes() == step_ref.tobytes(), u.first_diff(step, step_ref)
    finally:
        u.set_tickets(False)


# the tables of plain streams are summed by every workgroup of the main kernel up to 320 tiles of all streams together (512 from
# 16 streams on), by a kernel ahead of it from there on; parts of four waves (one stream), two and one, and a table of more than one round
@pytest.mark.parametrize("tiles,k", [(4, 1), (5, 1), (17, 1), (512, 1), (513, 1), (3, 2), (256, 2), (257, 2), (5, 3), (170, 3), (171, 3),
                                     (33, 5), (103, 5), (2, 64), (9, 64),
                                     (320, 1), (321, 1), (160, 2), (161, 2), (106, 3), (107, 3), (64, 5), (65, 5), (32, 16), (33, 16), (8, 64)])
def test_decompress_of_few_tiles(zcref, stream_variant, tiles, k):
    u = gpuutil
    n = tiles * TILE - 2049
    eb = 6e-3
    base = _values(n, 60)
    xs = [np.roll(base, 4096 * i) for i in range(k)]
    refs = [zcref.compress(x, eb)[1] for x in xs]
    want = [zcref.decompress(r)[1] for r in refs]
    st, got, ns = u.gpu_decompress_many(refs, [n] * k)
    assert st == ZC_OK and ns == [n] * k
    for w, g in zip(want, got):
        assert np.array_equal(w.view(np.uint32), g[:n].view(np.uint32))
    st, y, got_n = u.gpu_decompress(refs[-1], n)
    assert st == ZC_OK and got_n == n and np.array_equal(y.view(np.uint32), want[-1].view(np.uint32))
    if stream_variant == "indexed":
        return
    # a table that does not add up, or holds a width above 31, far from every tile but its own: nothing is written
    nb = (n + 31) // 32
    for bad in (32, 7 + int(refs[-1][u.widths_begin(nb) + nb - 1])):
        broken = refs[-1].copy()
        broken[u.widths_begin(nb) + nb - 1] = bad
        assert zcref.decompress(broken)[0] == ZC_ERR_FORMAT
        d_out = torch.full((n,), 7.0, device=u.DEV)
        st, _ = u.zc.zc_decompress(u.to_dev(broken), broken.size, d_out, u.workspace(n))
        assert st == ZC_ERR_FORMAT and bool((d_out == 7.0).all())
        st, outs, _ = u.gpu_decompress_many(refs[:-1] + [broken], [n] * k)
        assert st == ZC_ERR_FORMAT and all(np.isnan(o).all() for o in outs)


# both sides of the number of tiles up to which a reduce of plain streams sums their tables itself
@pytest.mark.parametrize("k,tiles", [(1, 320), (1, 321), (2, 160), (2, 161), (12, 26), (12, 27), (16, 16), (16, 17), (24, 8), (24, 9), (25, 1)])
def test_reduces_of_few_tiles(zcref, stream_variant, k, tiles):
    if stream_variant == "indexed":
        return
    u = gpuutil
    n = tiles * TILE - 2049
    base = _values(n, 62)
    refs = [zcref.compress(np.roll(base, 4096 * i), 6e-3)[1] for i in range(k)]
    for op in (None, 1):
        st_ref, want = zcref.reduce(refs, op=op or 0)[:2]
        st, got, _ = u.gpu_reduce(refs, n, op=op)
        assert st == st_ref == ZC_OK and got.tobytes() == want.tobytes(), (op, u.first_diff(got, want))


# the lists of spans (128 tiles each) of plain streams that a kernel ahead has indexed, which are added up in rows of lanes: by
# every wave for itself up to four streams, four streams a wave and round above; one span and several
@pytest.mark.parametrize("k,tiles", [(1, 600), (2, 300), (3, 257), (4, 129), (5, 128), (15, 40), (16, 33), (17, 129), (33, 16), (64, 9)])
def test_plain_streams_indexed_ahead(zcref, stream_variant, k, tiles):
    if stream_variant == "indexed":
        return
    u = gpuutil
    n = tiles * TILE - 2049
    base = _values(n, 61)
    refs = [zcref.compress(np.roll(base, 4096 * i), 6e-3)[1] for i in range(k)]
    for tickets in (False, True):
        u.set_tickets(tickets)
        try:
            for op in (None, 1, 2):
                st_ref, want = zcref.reduce(refs, op=op or 0)[:2]
                st, got, _ = u.gpu_reduce(refs, n, op=op)
                assert st == st_ref == ZC_OK and got.tobytes() == want.tobytes(), (op, u.first_diff(got, want))
        finally:
            u.set_tickets(False)
    want = [zcref.decompress(r)[1] for r in refs]
    st, got, ns = u.gpu_decompress_many(refs, [n] * k)
    assert st == ZC_OK and ns == [n] * k
    for w, g in zip(want, got):
        assert np.array_equal(w.view(np.uint32), g[:n].view(np.uint32))
    # one stream whose table does not add up, or holds a width above 31, in its last block or its first: every tile must know
    nb = (n + 31) // 32
    for s in sorted({0, k // 2, k - 1}):
        for at, bad in ((nb - 1, 32), (0, 1 + int(refs[s][u.widths_begin(nb)]) % 15)):
            broken = refs[s].copy()
            broken[u.widths_begin(nb) + at] = bad
            assert zcref.decompress(broken)[0] == ZC_ERR_FORMAT
            streams = refs[:s] + [broken] + refs[s + 1:]
            assert u.gpu_reduce(streams, n)[0] == ZC_ERR_FORMAT and u.gpu_reduce(streams, n, op=1)[0] == ZC_ERR_FORMAT
            st, outs, _ = u.gpu_decompress_many(streams, [n] * k)
            assert st == ZC_ERR_FORMAT and all(np.isnan(o).all() for o in outs)


@pytest.mark.parametrize("k", [2, 17])
def test_plain_streams_of_more_spans_than_a_row_reads_at_once(stream_variant, k):
    """65 spans: against the indexed streams of the same values, whose positions come from their index."""
    if stream_variant == "indexed":
        return
    u, lib = gpuutil, gpuutil._zc
    n = 64 * 128 * TILE + 5000
    xs = [synth.sinusoids(n, seed=5 + i, device=u.DEV) for i in range(2)]
    ws = u.workspace(n, k)
    results, made = [], []
    for flags in (ZC_STREAM_PLAIN, 0):
        room = torch.empty(lib.zc_compress_bound(n, flags), dtype=torch.uint8, device=u.DEV)
        streams = []
        for x in xs:
            st, size = lib.zc_compress(x, n, 1e-2, room, ws, flags=flags)
            assert st == ZC_OK
            streams.append(room[:size].clone())
        made.append(streams)
        operands = (streams * k)[:k]
        for op in (0, 1):
            st, size = lib.zc_reduce_compressed_op(operands, [s.numel() for s in operands], op, room, ws, flags=flags)
            assert st == ZC_OK
            begin = 32 + (0 if flags else (4 * ((n + 2047) // 2048 + 1) + 15) // 16 * 16)
            results.append(room[begin:size].clone())         # width table, first codes and payload
    assert torch.equal(results[0], results[2]) and torch.equal(results[1], results[3])
    del xs, results
    operands = (made[0] * k)[:k]
    outs = [torch.empty(n, device=u.DEV) for _ in range(k)]
    st, ns = lib.zc_decompress_many(operands, [s.numel() for s in operands], outs, ws, flags=ZC_STREAM_PLAIN)
    assert st == ZC_OK and ns == [n] * k
    for i in range(2):
        y = torch.empty(n, device=u.DEV)
        assert lib.zc_decompress(made[1][i], made[1][i].numel(), y, ws)[0] == ZC_OK
        assert all(torch.equal(y.view(torch.int32), o.view(torch.int32)) for o in outs[i::2])


@pytest.mark.parametrize("tiles", [12, 40])
def test_parts_that_look_back_in_different_ways(zcref, stream_variant, tiles):
    """A part may be given with ZC_CHAINS_COHERENT and the next without, or the other way round: the tiles of a part read
    what those of the parts before it have published, however they looked back themselves."""
    if stream_variant == "plain":
        return
    u, zc = gpuutil, gpuutil.zc
    n = 2 * tiles * TILE - 4097
    xs = [_values(n, 70 + i) for i in range(2)]
    eb = synth.abs_bound(torch.from_numpy(xs[0]), 1e-3)
    refs = [zcref.compress(x, eb)[1] for x in xs]
    d_xs, d_refs, sizes = [u.to_dev(x) for x in xs], [u.to_dev(r) for r in refs], [r.size for r in refs]
    wanted = [refs[0], zcref.reduce(refs)[1], zcref.reduce_step(refs[0], xs[1])[1]]
    cut = tiles // 2 * 2 * TILE
    d_out, ws = torch.empty(zc.zc_compress_bound(n), dtype=torch.uint8, device=u.DEV), u.workspace(n, 2)
    calls = [lambda *part: zc.zc_compress_part(d_xs[0], n, eb, *part, d_out, ws),
             lambda *part: zc.zc_reduce_compressed_part(d_refs, sizes, n, *part, d_out, ws),
             lambda *part: zc.zc_reduce_step_part(d_refs[0], sizes[0], d_xs[1], n, 0, *part, d_out, ws)]
    try:
        for want, call in zip(wanted, calls):
            for first_coherent in (True, False):
                u.set_coherent(first_coherent)
                assert call(0, cut)[0] == ZC_OK
                u.set_coherent(not first_coherent)
                st, total = call(cut, n - cut)
                got = d_out[:total].cpu().numpy()
                assert st == ZC_OK and got.tobytes() == want.tobytes(), u.first_diff(got, want)
    finally:
        u.set_coherent(False)


@pytest.mark.parametrize("tiles", [3, 600])          # plain streams: one launch, and two
def test_a_refused_call_reports_a_size_of_nothing(zcref, stream_variant, tiles):
    """Whatever the workspace held before."""
    u, zc = gpuutil, gpuutil.zc
    n = tiles * TILE - 2049
    x = _values(n, 90)
    ref = zcref.compress(x, 1e-3)[1]
    d_ref, d_x = u.to_dev(ref), u.to_dev(x)
    d_out = torch.empty(zc.zc_compress_bound(n), dtype=torch.uint8, device=u.DEV)
    d_y = torch.empty(n, device=u.DEV)
    offsets = torch.empty(8, dtype=torch.int32, device=u.DEV)
    ws = u.workspace(n)
    for call, want in ((lambda: zc.zc_reduce_step(d_ref, ref.size, d_x, n - 1, d_out, ws), ZC_ERR_MISMATCH),
                       (lambda: zc.zc_decompress_range(d_ref, ref.size, tiles * TILE, 5, d_y, ws), ZC_ERR_ARG),
                       (lambda: (zc.zc_debug_block_offsets(d_ref, ref.size, offsets, ws), u.zc.zc_finish(ws)[1]), ZC_ERR_CAPACITY)):
        ws.fill_(0x5A)
        assert call() == (want, 0)
    if stream_variant == "indexed":                  # (parts are of indexed streams)
        ws.fill_(0x5A)
        assert zc.zc_reduce_compressed_part([d_ref], [ref.size], n - 1, 0, TILE, d_out, ws) == (ZC_ERR_MISMATCH, 0)



@pytest.mark.parametrize("tickets", [False, True])
@pytest.mark.parametrize("k", [1, 2, 5, 12])
def test_a_reduce_in_too_small_a_workspace_is_refused(zcref, k, tickets):
    """n is only known on the GPU, from the streams: every tile of the result needs a place in the workspace."""
    u = gpuutil
    n = 40 * TILE - 2049
    ref = zcref.compress(_values(n, 91), 1e-3)[1]
    d_refs, sizes = [u.to_dev(ref)] * k, [ref.size] * k
    other = zcref.compress(_values(n - 4096, 92), 1e-3)[1]
    d_other = u.to_dev(other)
    d_out = torch.empty(u.zc.zc_compress_bound(n), dtype=torch.uint8, device=u.DEV)
    u.set_tickets(tickets)
    try:
        for small in (1, 16 * TILE, 23 * TILE):
            ws = u.workspace(small, k)
            for op in (0, 1, 2):
                ws.fill_(0x5A)
                assert u.zc.zc_reduce_compressed_op(d_refs, sizes, op, d_out, ws) == (ZC_ERR_ARG, 0), (small, op)
                if k > 1:                                # ahead of anything else that is wrong
                    for d_last, last in ((d_other, other), (u.to_dev(ref[:-1]), ref[:-1])):
                        assert u.zc.zc_reduce_compressed_op(d_refs[:-1] + [d_last], sizes[:-1] + [last.size], op, d_out, ws) == (ZC_ERR_ARG, 0)
        for op in (0, 1, 2):
            want = zcref.reduce([ref] * k, op=op)[1]
            st, total = u.zc.zc_reduce_compressed_op(d_refs, sizes, op, d_out, u.workspace(n, k))
            assert st == ZC_OK and d_out[:total].cpu().numpy().tobytes() == want.tobytes(), op
    finally:
        u.set_tickets(False)


# Sums of few tiles: four segments of a tile by a wave each, two by two and one by four that share its operands; a wave's last batch of
# operands of every size, several batches, one side of every limit and the other; blocks of all classes of widths, and (wide) so many
# wide blocks that they do not fit a wave's place for them; a segment count that is no multiple of a tile's.  Max and Min the same way.
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("k,tiles", [(2, 1), (3, 2), (4, 9), (5, 3), (6, 129), (7, 17), (8, 256), (8, 257), (9, 1), (11, 5), (12, 128), (12, 129),
                                     (13, 2), (16, 16), (17, 3), (64, 2), (4, 512), (4, 513), (2, 1024), (2, 1025), (5, 513),
                                     (4, 64), (4, 65), (7, 128), (8, 129), (12, 512), (12, 513)])
def test_reduces_by_waves_that_share_operands(zcref, stream_variant, k, tiles, wide):
    u = gpuutil
    n = tiles * TILE - 2049 - 31
    g = np.random.default_rng(7 * k + tiles)
    base = _values(n, 63)
    rough = np.repeat(10.0 ** g.uniform(-3, 1 if not wide else 3, (n + 2047) // 2048), 2048)[:n].astype(np.float32)    # a segment's widths
    base += rough * g.standard_normal(n).astype(np.float32)
    refs = [zcref.compress(np.roll(base, 4096 * i), 6e-3)[1] for i in range(min(k, 4))]
    refs = (refs * 16)[:k]
    for op in (None, 1, 2) if tiles <= 513 else (None,):
        st_ref, want = zcref.reduce(refs, op=op or 0)[:2]
        st, got, _ = u.gpu_reduce(refs, n, op=op)
        assert st == st_ref == ZC_OK and got.tobytes() == want.tobytes(), (op, u.first_diff(got, want))
    # one operand whose index says something else than its widths, or whose widths say something else than its size
    nb, at = (n + 31) // 32, int(g.integers(0, (n + 31) // 32))
    broken = refs[-1].copy()
    if stream_variant == "indexed":
        entry = 32 + 4 * (1 + at // 64)
        broken[entry:entry + 4] = np.frombuffer(np.uint32(int.from_bytes(broken[entry:entry + 4].tobytes(), "little") + int(g.integers(1, 1 << 31))).tobytes(), np.uint8)
    else:
        broken[u.widths_begin(nb) + at] = (int(broken[u.widths_begin(nb) + at]) + 1) % 31
    assert zcref.reduce(refs[:-1] + [broken])[0] == ZC_ERR_FORMAT
    for op in (None, 1):
        assert u.gpu_reduce(refs[:-1] + [broken], n, op=op)[0] == ZC_ERR_FORMAT


# The same operands where the kernels for few tiles are not taken: a workspace for many more values (the tiles are told by the streams' sizes
# then, which allow more than there are), and by ticket.  Blocks of all classes of widths, and an operand that is not in order.
@pytest.mark.parametrize("way", ["large_workspace", "tickets"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("k,tiles", [(1, 1), (2, 1), (2, 70), (4, 9), (5, 65), (8, 129), (12, 17), (16, 60), (64, 3)])
def test_reduces_of_few_tiles_by_the_other_kernels(zcref, stream_variant, k, tiles, wide, way):
    u = gpuutil
    n = tiles * TILE - 2049 - 31
    g = np.random.default_rng(9 * k + tiles)
    rough = np.repeat(10.0 ** g.uniform(-3, 1 if not wide else 3, (n + 2047) // 2048), 2048)[:n].astype(np.float32)
    base = _values(n, 64) + rough * g.standard_normal(n).astype(np.float32)
    refs = ([zcref.compress(np.roll(base, 4096 * i), 6e-3)[1] for i in range(min(k, 4))] * 16)[:k]
    nb, at = (n + 31) // 32, int(g.integers(0, (n + 31) // 32))
    broken = refs[-1].copy()
    if stream_variant == "indexed":
        entry = 32 + 4 * (1 + at // 64)
        broken[entry:entry + 4] = np.frombuffer(np.uint32(int.from_bytes(broken[entry:entry + 4].tobytes(), "little") + int(g.integers(1, 1 << 31))).tobytes(), np.uint8)
    else:
        broken[u.widths_begin(nb) + at] = (int(broken[u.widths_begin(nb) + at]) + 1) % 31
    assert zcref.reduce(refs[:-1] + [broken])[0] == ZC_ERR_FORMAT
    ws = u.workspace(1 << 27 if way == "large_workspace" else n, k)
    u.set_tickets(way == "tickets")
    try:
        for op in (None, 1, 2):
            st_ref, want = zcref.reduce(refs, op=op or 0)[:2]
            st, got, _ = u.gpu_reduce(refs, n, op=op, ws=ws)
            assert st == st_ref == ZC_OK and got.tobytes() == want.tobytes(), (op, u.first_diff(got, want))
            assert u.gpu_reduce(refs[:-1] + [broken], n, op=op, ws=ws)[0] == ZC_ERR_FORMAT
    finally:
        u.set_tickets(False)


# calls of one workgroup that somebody waits for: the main kernel itself gives the answer, also to a call that fails (the reduces here are of one workgroup
# for the smallest streams only, see the test below)
@pytest.mark.parametrize("n", [1, 31, 2049, 8192])
def test_calls_of_one_workgroup_answer_themselves(zcref, n):
    u = gpuutil
    x = synth.sinusoids(n, seed=3).numpy()
    st_ref, ref = zcref.compress(x, 1e-3)[:2]
    for _ in range(3):                               # (the slots of the answers before hold their words)
        st, s, total = u.gpu_compress(x, 1e-3)
        assert st == st_ref == ZC_OK and total == ref.size and s.tobytes() == ref.tobytes()
        assert u.gpu_compress(x, 1e-3, out_cap=ref.size - 4)[0] == ZC_ERR_CAPACITY
        want = zcref.decompress(ref)[1]
        st, y, got = u.gpu_decompress(ref, n)
        assert st == ZC_OK and got == n and np.array_equal(y.view(np.uint32), want.view(np.uint32))
        st, ys, ns = u.gpu_decompress_many([ref], [n])
        assert st == ZC_OK and ns == [n] and np.array_equal(ys[0][:n].view(np.uint32), want.view(np.uint32))
        assert u.gpu_decompress(ref, n, in_bytes=ref.size - 1)[0] == ZC_ERR_FORMAT
        want = zcref.reduce_step(ref, x)[1]
        st, s, total = u.gpu_reduce_step(ref, x)
        assert st == ZC_OK and total == want.size and s.tobytes() == want.tobytes()
        bad = x.copy()
        bad[n // 2] = np.nan
        assert u.gpu_reduce_step(ref, bad)[0] == zcref.reduce_step(ref, bad)[0] == u.gpu_compress(bad, 1e-3)[0]
        for op in (None, 1):
            want = zcref.reduce([ref], op=op or 0)[1]
            st, s, total = u.gpu_reduce([ref], n, op=op)
            assert st == ZC_OK and total == want.size and s.tobytes() == want.tobytes()


# reduces of one workgroup, which takes streams whose sizes allow no second tile, and ring rounds and compressions by ticket: they answer
# themselves too, whatever the answer
@pytest.mark.parametrize("tickets", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_reduces_of_one_workgroup_answer_themselves(zcref, stream_variant, k, tickets):
    u = gpuutil
    u.set_tickets(tickets)
    try:
        for n in (1, 31, 700):
            xs = [synth.sinusoids(n, seed=i).numpy() for i in range(k)]
            refs = [zcref.compress(x, 1e-1)[1] for x in xs]
            assert all(r.size <= 32 + 5 * 256 for r in refs)
            for _ in range(2):
                for op in (None, 1, 2):
                    want = zcref.reduce(refs, op=op or 0)[1]
                    st, s, total = u.gpu_reduce(refs, n, op=op)
                    assert st == ZC_OK and total == want.size and s.tobytes() == want.tobytes(), (n, op)
                    assert u.gpu_reduce(refs, n, op=op, out_cap=want.size - 4)[0] == ZC_ERR_CAPACITY
                    cut = refs[:-1] + [refs[-1][:refs[-1].size - 1]]
                    assert u.gpu_reduce(cut, n, op=op)[0] == ZC_ERR_FORMAT
                want = zcref.reduce_step(refs[0], xs[-1])[1]
                st, s, total = u.gpu_reduce_step(refs[0], xs[-1])
                assert st == ZC_OK and total == want.size and s.tobytes() == want.tobytes(), n
                st, s, total = u.gpu_compress(xs[0], 1e-1)
                assert st == ZC_OK and total == refs[0].size and s.tobytes() == refs[0].tobytes(), n
                st, y, got = u.gpu_decompress(refs[0], n, average=True)
                assert st == ZC_OK and got == n and np.array_equal(y.view(np.uint32), zcref.decompress(refs[0])[1].view(np.uint32))
    finally:
        u.set_tickets(False)


# What a call has written is there when it returns: read at once on another stream, which nothing orders behind the call's (the call's own is
# not waited for before the end).  Calls of one workgroup, which answer themselves, and of more.
@pytest.mark.parametrize("n", [31, 5120, 8192, 100003, 1 << 20])
def test_outputs_are_there_when_a_waited_call_returns(zcref, n):
    u, zc = gpuutil, gpuutil.zc
    xs = [synth.sinusoids(n, seed=i).numpy() for i in range(2)]
    refs = [zcref.compress(x, 1e-1)[1] for x in xs]
    d_xs, d_refs, sizes = [u.to_dev(x) for x in xs], [u.to_dev(r) for r in refs], [r.size for r in refs]
    ws, d_out = u.workspace(n, 2), torch.empty(zc.zc_compress_bound(n), dtype=torch.uint8, device=u.DEV)
    copy, d_y, copy_y = torch.empty_like(d_out), torch.empty(n, device=u.DEV), torch.empty(n, device=u.DEV)
    wants = [refs[0], zcref.reduce(refs)[1], zcref.reduce(refs, op=1)[1], zcref.reduce_step(refs[0], xs[1])[1]]
    want_y = zcref.decompress(refs[0])[1].view(np.uint32)
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    calls = [lambda: zc.zc_compress(d_xs[0], n, 1e-1, d_out, ws, stream=mine),
             lambda: zc.zc_reduce_compressed(d_refs, sizes, d_out, ws, stream=mine),
             lambda: zc.zc_reduce_compressed_op(d_refs, sizes, 1, d_out, ws, stream=mine),
             lambda: zc.zc_reduce_step(d_refs[0], sizes[0], d_xs[1], n, d_out, ws, stream=mine)]
    for _ in range(5):
        for call, want in zip(calls, wants):
            d_out.fill_(0xA5)
            torch.cuda.synchronize()
            st, total = call()
            with torch.cuda.stream(other):
                copy.copy_(d_out)
            other.synchronize()
            assert st == ZC_OK and total == want.size and copy[:total].cpu().numpy().tobytes() == want.tobytes()
        for call in (lambda: zc.zc_decompress(d_refs[0], sizes[0], d_y, ws, stream=mine),
                     lambda: zc.zc_decompress_many([d_refs[0]], [sizes[0]], [d_y], ws, stream=mine)):
            d_y.fill_(float("nan"))
            torch.cuda.synchronize()
            st, got = call()
            with torch.cuda.stream(other):
                copy_y.copy_(d_y)
            other.synchronize()
            assert st == ZC_OK and got in (n, [n]) and np.array_equal(copy_y.cpu().numpy().view(np.uint32), want_y)
    torch.cuda.synchronize()


# both sides of the sizes between which the compressor's tiles are of four waves, with narrow and with wider blocks
@pytest.mark.parametrize("tiles", [1, 2, 255, 256, 257, 512, 513, 768, 769])
def test_compression_by_small_tiles(zcref, tiles):
    u = gpuutil
    for n in (tiles * TILE, tiles * TILE - 4097):
        for eb in (2e-2, 1e-5):                      # blocks of at most 7 bits (but for one), and of more
            x = _values(n, 30)
            st_ref, ref = zcref.compress(x, eb)[:2]
            st, s, total = u.gpu_compress(x, eb)
            assert st == st_ref and total == ref.size and s.tobytes() == ref.tobytes(), u.first_diff(s, ref)
