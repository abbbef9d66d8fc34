"""The work that a user of this library has it do, as measurable cases: one pass of each through the public calls.

A case names an operation (`op`), its size (`n` values per buffer, `k` buffers), the data and the value-range-relative
error bound (`rel`), the stream variant (`plain`) and whether the call is the synchronous form that hands back the
stream's size (`wait`) or the asynchronous one that only enqueues (as a step of a pipeline, or bench.py, uses it).

  round_trip   zc_compress, then zc_decompress of what it wrote
  compress     zc_compress
  decompress   zc_decompress
  reduce       zc_reduce_compressed / zc_reduce_compressed_op: k streams -> the stream of their Sum, Max or Min
  step         zc_reduce_step / zc_reduce_step_op: one ring round, a received stream and a local buffer -> a stream
  allgather    zc_decompress_many: k streams -> k buffers

Sizes and data are those of bench.py and tests/: 2^20 sinusoids, 512^3 and 256 x 512 x 512 power-law fields, the hard
mixture of 2^28 values, the paper's 5120-value chunk, and ragged ones between them.
"""
import math

import torch

import paper_2502_18554_amd as zc
from paper_2502_18554_amd import synth
from paper_2502_18554_amd.binding import ZC_OP_MAX, ZC_OP_MIN, ZC_OP_SUM, ZC_STREAM_PLAIN

DEV = "cuda:0"
OPS = {"sum": ZC_OP_SUM, "max": ZC_OP_MAX, "min": ZC_OP_MIN}


def _case(op, n, rel, data="field", k=1, agg="sum", plain=False, wait=False, **more):
    return dict(more, op=op, n=n, k=k, rel=rel, data=data, agg=agg, plain=plain, wait=wait)


def listed():
    return [
        # one chunk of the paper's pipelined codec (5120 values), size handed back so that it can be sent: pure latency
        _case("round_trip", 5120, 1e-4, "sinusoids", wait=True, name="chunk_5120_wait"),
        # the 1D array of the first benchmark configuration, compressed and decompressed
        _case("round_trip", 1 << 20, 1e-4, "sinusoids", name="round_trip_1m"),
        # the 512^3 field of the headline benchmark, each direction, at two of its bounds
        _case("compress", 1 << 27, 1e-4, name="compress_512cube_1e-4"),
        _case("decompress", 1 << 27, 1e-3, name="decompress_512cube_1e-3"),
        # the paper's plain stream (no segment index) on a buffer of no round size, at the loosest bound
        _case("round_trip", 20000003, 1e-2, plain=True, name="round_trip_plain_20m"),
        # the local step of a compressed Allreduce: the headline's 8 x 2^26 values
        _case("reduce", 1 << 26, 1e-4, k=8, name="reduce_8x64m"),
        # ... of a few ranks on hard data (wide and constant blocks) and a ragged size
        _case("reduce", 4194301, 1e-5, "hard", k=4, name="reduce_hard_4x4m"),
        # the Max of 8 ranks
        _case("reduce", 1 << 24, 1e-4, k=8, agg="max", name="reduce_max_8x16m"),
        # rounds of the ring: the headline's buffer, and a small ragged chunk whose size the sender waits for
        _case("step", 1 << 26, 1e-4, name="step_64m"),
        _case("step", 262177, 1e-3, agg="min", wait=True, name="step_min_262177_wait"),
        # the tail of a compressed Allgather: 8 streams of 2^26 values
        _case("allgather", 1 << 26, 1e-3, k=8, name="allgather_8x64m"),
        # the hard-data stress configuration: spikes, steps and constant blocks at a tight bound
        _case("round_trip", 1 << 28, 1e-5, "hard", name="round_trip_hard_256m"),
    ]


def draw(rng):
    op = rng.choice(("round_trip", "compress", "decompress", "reduce", "reduce", "step", "step", "allgather"))
    data = rng.choice(("field", "field", "sinusoids", "hard"))
    k = rng.choice((2, 3, 4, 5, 8, 16)) if op in ("reduce", "allgather") else 1
    most = (1 << 26) // (1 if k == 1 else k // 2)
    n = int(math.exp(rng.uniform(math.log(1000), math.log(most))))
    if rng.random() < 0.4:                      # buffers of a round size are common
        n = max(1024, n // 1024 * 1024)
    rel = 1e-5 if data == "hard" else rng.choice((1e-2, 1e-3, 1e-4))
    agg = rng.choice(("sum", "sum", "max", "min")) if op in ("reduce", "step") else "sum"
    return _case(op, n, rel, data, k=k, agg=agg, plain=rng.random() < 0.2, wait=rng.random() < 0.3)


def _values(data, n, seed):
    if data == "sinusoids":
        return synth.sinusoids(n, seed=seed, device=DEV)
    if data == "hard":
        return synth.hard_mix(n, seed=seed, device=DEV)
    for shape in ((16, 128, 128), (64, 256, 256), (256, 512, 512), (512, 512, 512)):
        if n <= shape[0] * shape[1] * shape[2]:
            return synth.power_law_field(shape, seed=seed, device=DEV)[:n].clone()
    raise ValueError("no field that large")


def _stream_room(n, plain):
    # zeroed, so that what a call leaves unwritten behind its stream is the same every time
    return torch.zeros(zc.zc_compress_bound(n, ZC_STREAM_PLAIN if plain else 0), dtype=torch.uint8, device=DEV)


def _checked(result, what):
    if result[0] != 0:
        raise zc.ZcError(result[0], what)
    return result[1]


def prepare(case, seed):
    n, k, op = case["n"], case["k"], case["op"]
    flags = ZC_STREAM_PLAIN if case["plain"] else 0
    s = dict(case, flags=flags, agg=OPS[case["agg"]], wait=case["wait"],
             ws=torch.empty(zc.zc_workspace_bytes(n, k), dtype=torch.uint8, device=DEV))
    seeds = [(seed * 64 + i) & 0x7fffffff for i in range(k + 1)]
    first = _values(case["data"], n, seeds[0])
    s["eb"] = synth.abs_bound(first, case["rel"])           # one bound for all ranks: that of the first one's range
    if op in ("round_trip", "compress"):
        s["x"] = first
        s["stream"] = _stream_room(n, case["plain"])
    if op in ("decompress", "reduce", "step", "allgather"):  # what has been received
        room = _stream_room(n, case["plain"])
        s["chunks"], s["sizes"] = [], []
        for i in range(k):
            x = first if i == 0 else _values(case["data"], n, seeds[i])
            size = _checked(zc.zc_compress(x, n, s["eb"], room, s["ws"], flags=flags), "compress")
            s["chunks"].append(room[:size].clone())
            s["sizes"].append(size)
        del x
        if op in ("reduce", "step"):
            s["stream"] = room.zero_()
    if op == "step":
        s["local"] = _values(case["data"], n, seeds[k])
    if op in ("round_trip", "decompress", "allgather"):
        s["y"] = [torch.empty(n, dtype=torch.float32, device=DEV) for _ in range(k)]
    return s


def run(s):
    n, ws, flags, wait, op = s["n"], s["ws"], s["flags"], s["wait"], s["op"]
    if op == "round_trip":
        size = _checked(zc.zc_compress(s["x"], n, s["eb"], s["stream"], ws, sync=wait, flags=flags), op)
        _checked(zc.zc_decompress(s["stream"], size if wait else s["stream"].numel(), s["y"][0], ws, sync=wait, flags=flags), op)
        return s["stream"], s["y"][0]
    if op == "compress":
        _checked(zc.zc_compress(s["x"], n, s["eb"], s["stream"], ws, sync=wait, flags=flags), op)
        return s["stream"]
    if op == "decompress":
        _checked(zc.zc_decompress(s["chunks"][0], s["sizes"][0], s["y"][0], ws, sync=wait, flags=flags), op)
        return s["y"]
    if op == "allgather":
        _checked(zc.zc_decompress_many(s["chunks"], s["sizes"], s["y"], ws, sync=wait, flags=flags), op)
        return s["y"]
    if op == "reduce":
        if s["agg"] == ZC_OP_SUM:
            _checked(zc.zc_reduce_compressed(s["chunks"], s["sizes"], s["stream"], ws, sync=wait, flags=flags), op)
        else:
            _checked(zc.zc_reduce_compressed_op(s["chunks"], s["sizes"], s["agg"], s["stream"], ws, sync=wait, flags=flags), op)
        return s["stream"]
    if s["agg"] == ZC_OP_SUM:
        _checked(zc.zc_reduce_step(s["chunks"][0], s["sizes"][0], s["local"], n, s["stream"], ws, sync=wait, flags=flags), op)
    else:
        _checked(zc.zc_reduce_step_op(s["chunks"][0], s["sizes"][0], s["local"], n, s["agg"], s["stream"], ws, sync=wait, flags=flags), op)
    return s["stream"]


# Stream bytes per value, measured on these generators from 2^18 values up (within 3 % of each other; below that the
# fixed parts of a stream add a few per cent).
_BYTES = {("sinusoids", 1e-2): 0.36, ("sinusoids", 1e-3): 0.41, ("sinusoids", 1e-4): 0.67,
          ("field", 1e-2): 0.665, ("field", 1e-3): 1.06, ("field", 1e-4): 1.48, ("hard", 1e-5): 0.77}


def work(case):
    n, k = case["n"], case["k"]
    stream = n * _BYTES[case["data"], case["rel"]]
    summed = stream + n * 0.5 * math.log2(k) / 8            # a sum of k independent fields is sqrt(k) times as rough
    values = 4 * n
    total = {"round_trip": 2 * (values + stream),
             "compress": values + stream,
             "decompress": stream + values,
             "allgather": k * (stream + values),
             "reduce": k * stream + (summed if case["agg"] == "sum" else stream),
             "step": stream + values + stream}[case["op"]]
    return {"bytes": total, "flops": 0}                     # nothing here is a contraction: memory is what it cannot do without


def tolerance(case):
    # streams are defined byte for byte, and a reconstruction is one binary64 product rounded once
    return "exact"
