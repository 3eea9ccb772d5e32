"""The work that users of this library have it do, as cases that can be timed and compared.

The P ranks of a collective are P buffers in one GPU's memory. A case names a collective with its
rank count, sizes, element type and configuration; `prepare` makes what a program holds before the
call (a communicator, the send and receive buffers, for an AllToAllv its counts), `run` makes the
call through the package's public methods (bound once where the method has a bound form, as loops
over the same buffers do) and returns the receive buffers.

Receive buffers are the rows of one zeroed tensor, each row padded to 256 bytes, so that one
tensor holds everything a call wrote, and the bytes that it must not write.
"""
import math

import numpy as np
import torch

import paper_2608_00358_amd as hccl

DEVICE = "cuda:0"
TYPES = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32, "int32": torch.int32}
SIZE = {"bf16": 2, "fp16": 2, "fp32": 4, "int32": 4}
Ki, Mi = 1024, 1024 * 1024
ROOM = 3  # rows that a receive buffer of an AllToAllv holds, over the mean number that it receives

# Fields that a case leaves out.
DEFAULTS = {"op": "sum", "algo": "auto", "order": "ascending", "group": 0, "chunk": 0, "requantize": False,
            "noalloc": False, "offset": 0, "ids": False, "indexed": False}


def listed():
    return [
        # Tensor-parallel inference: the activations of a few tokens, where launch latency is all.
        {"name": "allreduce_p8_fp32_64KiB", "coll": "allreduce", "P": 8, "n": 16 * Ki, "dtype": "fp32", "algo": "direct"},
        # The same in a serving loop that may not allocate: 16 tokens x 8192 bf16 per rank.
        {"name": "allreduce_p8_bf16_noalloc", "coll": "allreduce", "P": 8, "n": 128 * Ki, "dtype": "bf16", "noalloc": True},
        # A gradient bucket of data-parallel training, ring in 64 KiB chunks.
        {"name": "allreduce_p4_fp32_4MiB", "coll": "allreduce", "P": 4, "n": 1 * Mi, "dtype": "fp32", "algo": "ring",
         "chunk": 64 * Ki},
        # A gradient bucket over 64 ranks in 8 groups of 8 (two-level).
        {"name": "allreduce_p64_two_level", "coll": "allreduce", "P": 64, "n": 4 * Mi, "dtype": "bf16", "group": 8},
        # Sharded-optimizer training: the whole gradient scattered, the largest call.
        {"name": "reduce_scatter_p8_bf16_256MiB", "coll": "reduce_scatter", "P": 8, "n": 16 * Mi, "dtype": "bf16"},
        # The same for a parameter group whose shard is no multiple of 16 bytes.
        {"name": "reduce_scatter_p8_fp32_ragged", "coll": "reduce_scatter", "P": 8, "n": 1000003, "dtype": "fp32"},
        # Recursive halving, the order of butterfly networks, at a layer's gradient size.
        {"name": "reduce_scatter_p16_halving", "coll": "reduce_scatter", "P": 16, "n": 256 * Ki, "dtype": "fp16",
         "order": "halving"},
        # Sharded parameters gathered before a layer runs, in bf16 ...
        {"name": "allgather_p8_bf16_4MiB", "coll": "allgather", "P": 8, "n": 2 * Mi, "dtype": "bf16"},
        # ... and a ragged fp32 shard.
        {"name": "allgather_p8_fp32_ragged", "coll": "allgather", "P": 8, "n": 300001, "dtype": "fp32"},
        # Embedding exchange: 2^18 rows of 128 bf16 per rank with their int32 ids, skewed, one group.
        {"name": "alltoallv_p8_rows_ids", "coll": "alltoallv", "P": 8, "n": 256 * Ki, "row": 128, "dtype": "bf16", "ids": True},
        # Expert dispatch with counts that a router wrote on the device: 256 tokens x 4096 per rank ...
        {"name": "dynamic_p8_moe", "coll": "dynamic", "P": 8, "n": 256, "row": 4096, "dtype": "bf16"},
        # ... and over 64 experts' ranks.
        {"name": "dynamic_p64_moe", "coll": "dynamic", "P": 64, "n": 256, "row": 2048, "dtype": "bf16"},
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm; half of them odd, half round."""
    v = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    return max(lo, v | 1) if rng.random() < 0.5 else max(lo, v // 64 * 64)


def draw(rng):
    coll = rng.choice(["allreduce", "allreduce", "reduce_scatter", "allgather", "alltoallv", "dynamic"])
    dtype = rng.choice(["bf16", "bf16", "fp16", "fp32", "int32"])
    c = {"coll": coll, "dtype": dtype}
    size = SIZE[dtype]
    if coll == "alltoallv":
        # rows from a handful to thousands per pair, of an id's size up to an embedding's
        c["P"] = rng.choice([2, 4, 8, 13, 16, 32, 64])
        c["row"] = rng.choice([1, 16, 64, 100, 128, 256])
        c["n"] = _spread(rng, 16 * c["P"], max(64 * c["P"], 512 * Mi // (c["P"] * c["row"] * size) // 2))
        c["ids"] = c["P"] <= 32 and rng.random() < 0.3  # (a group names at most 128 buffers)
        return c
    if coll == "dynamic":
        c["P"] = rng.choice([2, 4, 8, 8, 16, 32, 64])
        c["row"] = rng.choice([128, 1024, 2048, 4096, 7168])
        c["n"] = _spread(rng, 16, max(64, min(16384, 256 * Mi // (c["P"] * c["row"] * size))))
        c["indexed"] = rng.random() < 0.25
        return c
    P = c["P"] = rng.choice([2, 3, 4, 8, 8, 16, 32, 64])
    if coll == "allgather":
        c["n"] = _spread(rng, 256, 512 * Mi // (P * P * size))
        c["offset"] = rng.choice([0, 0, 0, 1])
        return c
    c["op"] = rng.choice(["sum", "sum", "sum", "sum", "max", "min"])
    per_rank = 512 * Mi // P // size
    c["n"] = _spread(rng, 1 * Ki, per_rank) if coll == "allreduce" else _spread(rng, 256, per_rank // P)
    c["order"] = rng.choice(["ascending", "ascending", "ring", "halving" if P & (P - 1) == 0 else "ascending"])
    c["requantize"] = c["op"] == "sum" and size == 2 and rng.random() < 0.25
    c["offset"] = rng.choice([0, 0, 0, 1])  # a view into a flat bucket
    if coll == "allreduce":
        if c["order"] == "ascending" and P >= 16 and rng.random() < 0.5:
            c["group"] = 8
        elif c["order"] == "ascending" and rng.random() < 0.3:
            c["algo"] = "direct"
        c["noalloc"] = c["n"] <= 1 * Mi and rng.random() < 0.3
    return c


def _full(case):
    return {**DEFAULTS, **case}


def _values(g, n, dtype):
    """n values as the path meets them: gradients and activations around zero; ids over their range."""
    if dtype == "int32":
        return torch.randint(-(1 << 31), (1 << 31) - 1, (n,), generator=g, device=DEVICE, dtype=torch.int64).to(torch.int32)
    x = torch.randn(n, generator=g, device=DEVICE, dtype=torch.float32)
    return x.mul_(0.02).to(TYPES[dtype])


def _sends(seed, P, n, dtype, offset=0):
    """P send buffers of n values, `offset` elements into their allocation."""
    out = []
    for r in range(P):
        g = torch.Generator(device=DEVICE)
        g.manual_seed(seed * 1000003 + r)
        out.append(_values(g, n + offset, dtype)[offset:])
    return out


def _whole(P, n, dtype, offset=0):
    """A zeroed tensor with a row of n + offset elements, padded to 256 bytes, for every rank."""
    unit = 256 // SIZE[dtype]
    return torch.zeros((P, (n + offset + unit - 1) // unit * unit), device=DEVICE, dtype=TYPES[dtype])


def _rows(whole, n, offset=0):
    return [whole[r, offset:offset + n] for r in range(whole.shape[0])]


def _counts(case, seed):
    """Rows that each source sends to each destination: every source sends n, skewed (Zipf, 1.1) over
    the destinations in an order of its own, and no destination receives more than it has room for."""
    P, rng = case["P"], np.random.default_rng(seed)
    p = np.arange(1, P + 1, dtype=np.float64) ** -1.1
    p /= p.sum()
    while True:
        counts = np.zeros((P, P), dtype=np.int64)
        for s in range(P):
            counts[s, rng.permutation(P)] = rng.multinomial(case["n"], p)
        if counts.sum(axis=0).max() <= ROOM * case["n"]:
            return counts


def _packed(counts):
    """Offsets [source, destination] of ranges that follow each other by destination."""
    return np.cumsum(counts, axis=1) - counts


def prepare(case, seed):
    c = _full(case)
    P, n, dtype = c["P"], c["n"], c["dtype"]
    if c["coll"] in ("alltoallv", "dynamic"):
        counts = _counts(c, seed)
        return (_prepare_alltoallv if c["coll"] == "alltoallv" else _prepare_dynamic)(c, counts, seed)
    comm = hccl.Comm(P, 0, algo=c["algo"], order=c["order"], group_size=c["group"], chunk_bytes=c["chunk"],
                     requantize=c["requantize"])
    nsend = n * P if c["coll"] == "reduce_scatter" else n
    nrecv = n * P if c["coll"] == "allgather" else n
    send = _sends(seed, P, nsend, dtype, c["offset"])
    whole = _whole(P, nrecv, dtype, c["offset"])
    recv = _rows(whole, nrecv, c["offset"])
    if c["coll"] == "allgather":
        call = comm.bind_allgather(send, recv)
    elif c["coll"] == "reduce_scatter":
        call = comm.bind_reduce_scatter(send, recv, c["op"])
    elif c["noalloc"]:
        def call():
            comm.allreduce_noalloc(send, recv, c["op"])
    else:
        call = comm.bind_allreduce(send, recv, c["op"])
    return {"comm": comm, "calls": [call], "send": send, "out": [whole], "keep": recv}


def _prepare_alltoallv(c, counts, seed):
    P = c["P"]
    comm = hccl.Comm(P, 0)
    calls, send, out = [], [], []
    for row, dtype in ((c["row"], c["dtype"]),) + (((1, "int32"),) if c["ids"] else ()):
        back = np.ascontiguousarray(counts.T)
        most = ROOM * c["n"] * row
        sb, whole = _sends(seed + len(out), P, c["n"] * row, dtype), _whole(P, most, dtype)
        calls.append(comm.bind_alltoallv(sb, counts * row, _packed(counts) * row, _rows(whole, most), back * row,
                                         _packed(back) * row))
        send.append(sb)
        out.append(whole)
    return {"comm": comm, "calls": calls, "send": send, "out": out}


def _prepare_dynamic(c, counts, seed):
    P, row = c["P"], c["row"]
    comm = hccl.Comm(P, 0)
    cap = ROOM * c["n"]
    send = _sends(seed, P, c["n"] * row, c["dtype"])
    whole = torch.zeros((P, cap * row), device=DEVICE, dtype=TYPES[c["dtype"]])
    d_counts = torch.from_numpy(counts).to(DEVICE)
    got = torch.zeros((P, P), device=DEVICE, dtype=torch.int64)
    more = {}
    if c["indexed"]:  # the program lays its ranges out itself
        back = np.ascontiguousarray(counts.T)
        more = {"sdispls": torch.from_numpy(_packed(counts)).to(DEVICE), "rdispls": torch.from_numpy(_packed(back)).to(DEVICE)}
    call = comm.bind_alltoallv_dynamic(send, d_counts, _rows(whole, cap * row), row, recvcounts=got, **more)
    return {"comm": comm, "calls": [call], "send": send, "out": [whole, got], "keep": (d_counts, more)}


def run(state):
    calls = state["calls"]
    if len(calls) == 1:
        calls[0]()
    else:
        with state["comm"].group():
            for call in calls:
                call()
    return state["out"]


def work(case):
    c = _full(case)
    P, n, size = c["P"], c["n"], SIZE[c["dtype"]]
    if c["coll"] == "allreduce":
        return {"bytes": 2 * P * n * size, "flops": (P - 1) * n}
    if c["coll"] == "reduce_scatter":
        return {"bytes": (P * P + P) * n * size, "flops": (P - 1) * P * n}
    if c["coll"] == "allgather":
        return {"bytes": (P + P * P) * n * size, "flops": 0}
    moved = P * n * (c["row"] * size + (4 if c["ids"] else 0))
    return {"bytes": 2 * moved, "flops": 0}


def tolerance(case):
    """The interface fixes the order in which the contributors of an element are folded, FP32
    partials and where they are rounded, so every result is determined to the bit."""
    return "exact"


def exact(case, seed):
    c = _full(case)
    state = prepare(case, seed)
    P, n = c["P"], c["n"]
    send, out = state["send"], [torch.zeros(w.shape, device=DEVICE, dtype=torch.float64 if w.is_floating_point() else w.dtype)
                                for w in state["out"]]
    if c["coll"] in ("alltoallv", "dynamic"):
        counts = _counts(c, seed)
        so, ro = _packed(counts), _packed(np.ascontiguousarray(counts.T))
        for sb, whole, row in zip(send if c["coll"] == "alltoallv" else [send], out, (c["row"], 1)):
            for s in range(P):
                for d in range(P):
                    k = int(counts[s, d]) * row
                    a, b = int(so[s, d]) * row, int(ro[d, s]) * row
                    whole[d, b:b + k] = sb[s][a:a + k]
        if c["coll"] == "dynamic":
            out[1].copy_(torch.from_numpy(np.ascontiguousarray(counts.T)))
        return out
    at = c["offset"]
    if c["coll"] == "allgather":
        out[0][:, at:at + P * n] = torch.cat(send)
        return out
    wide = torch.float64 if send[0].is_floating_point() else torch.int64
    total = send[0].to(wide)
    for x in send[1:]:
        total = total + x if c["op"] == "sum" else torch.maximum(total, x.to(wide)) if c["op"] == "max" else torch.minimum(total, x.to(wide))
    # (an int32 sum wraps: the conversion keeps its low 32 bits)
    out[0][:, at:at + n] = total if c["coll"] == "allreduce" else total.view(P, n)
    return out
