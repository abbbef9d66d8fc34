"""The entry points without flags (zc_compress, zc_decompress, zc_reduce_compressed, zc_reduce_compressed_ex, zc_reduce_step) called as C functions, waited for and not:
the same streams and values as their forms with flags, and the reference codec's.  (The binding reaches them only where its native calls decline.)"""
import ctypes as C

import numpy as np
import pytest
import torch

import gpuutil as u
from paper_2502_18554_amd import binding as b
from paper_2502_18554_amd import synth
from paper_2502_18554_amd.binding import ZC_OK

pytestmark = pytest.mark.gpu

EB = 1e-3


# one workgroup, which answers itself; some; more than a compute unit each
@pytest.mark.parametrize("n", [5120, 262177, 2_500_003])
@pytest.mark.parametrize("sync", [True, False])
def test_entries_without_flags(zcref, n, sync):
    L = b.lib()
    k = 3
    u.set_variant(zcref, True)
    try:
        xs = [synth.power_law_field((10, 512, 512), seed=70 + i).numpy().ravel()[:n] for i in range(k)]
        refs = [zcref.compress(x, EB)[1] for x in xs]
        want_sum, want_step, want_values = zcref.reduce(refs)[1], zcref.reduce_step(refs[0], xs[1])[1], zcref.decompress(refs[0])[1]
    finally:
        u.set_variant(zcref, False)
    ws = u.workspace(n, k)
    streams = [u.to_dev(r) for r in refs]
    d_x = [u.to_dev(x) for x in xs]
    stream = b._stream()
    chunks = (C.c_void_p * k)(*[s.data_ptr() for s in streams])
    sizes = (C.c_size_t * k)(*[s.numel() for s in streams])

    def call(f, out, before, after=(), capacity=None):
        size = C.c_size_t(0)
        out.fill_(0x77)
        st = f(*before, out.data_ptr(), out.numel() if capacity is None else capacity, C.byref(size) if sync else None, ws.data_ptr(), ws.numel(), stream, *after)
        assert st == ZC_OK
        if not sync:
            st, total = b.zc_finish(ws)
            assert st == ZC_OK
            return total
        return size.value

    def room():
        return torch.empty(b.zc_compress_bound(n), dtype=torch.uint8, device=u.DEV)

    def same(plain, with_flags, want):
        out_plain, out_flags = room(), room()
        total = call(plain[0], out_plain, plain[1])
        assert total == want.size == call(with_flags[0], out_flags, with_flags[1], with_flags[2])
        got = out_plain[:total].cpu().numpy()
        assert got.tobytes() == want.tobytes(), u.first_diff(got, want)
        assert torch.equal(out_plain[:total], out_flags[:total])

    x = (d_x[0].data_ptr(), n, C.c_float(EB))
    same((L.zc_compress, x), (L.zc_compress_ex, x, (0,)), refs[0])
    same((L.zc_reduce_compressed, (chunks, sizes, k)), (L.zc_reduce_compressed_op, (chunks, sizes, k, b.ZC_OP_SUM), (0,)), want_sum)
    same((L.zc_reduce_compressed, (chunks, sizes, k)), (L.zc_reduce_compressed_ex, (chunks, sizes, k), (0,)), want_sum)
    step = (streams[0].data_ptr(), streams[0].numel(), d_x[1].data_ptr(), n)
    same((L.zc_reduce_step, step), (L.zc_reduce_step_op, step + (b.ZC_OP_SUM,), (0,)), want_step)

    y = torch.empty(n, dtype=torch.float32, device=u.DEV)
    s = (streams[0].data_ptr(), streams[0].numel())
    assert call(L.zc_decompress, y, s, capacity=n) == n
    assert np.array_equal(y.cpu().numpy().view(np.uint32), want_values.view(np.uint32))
    z = torch.empty_like(y)
    assert call(L.zc_decompress_ex, z, s, (0,), capacity=n) == n and torch.equal(y, z)
