"""GPU parity of the calls that travel in their launch packets (uniform phases and a lone
AllToAllvDynamic), at the edges of their tiles, against the oracle: bit for bit, guard bands included.
With the default tile size a fused call takes these kernels; a configured one takes the executor's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_00358_amd as H
from gpu_helpers import Guarded, MaskedStream, first_mismatch, same_bits, to_device
from test_gpu_dynamic import random_counts, run_dynamic
from test_gpu_orders import lib_shard, run_ar, run_rs
from test_gpu_parity import inputs, run_allgather, run_allreduce, run_reduce_scatter

pytestmark = pytest.mark.gpu

# one element, less than a vector, around a wavefront's vectors, around two, several tiles
SIZES = [1, 5, 511, 513, 1029, 9001]


@pytest.mark.parametrize("dt", ["bf16", "fp16", "fp32", "int32"])
@pytest.mark.parametrize("P", [2, 3, 8, 9, 17, 64])
def test_sum_in_list_order(dt, P):
    for n in SIZES:
        assert run_allreduce(P, n, dt)["inline_launch"] == 1
    run_reduce_scatter(P, 517, dt)


@pytest.mark.parametrize("dt", ["bf16", "fp16", "fp32", "int32"])
@pytest.mark.parametrize("op", ["max", "min"])
@pytest.mark.parametrize("P", [2, 9, 16])
def test_max_min(dt, op, P):
    for n in SIZES:
        assert run_allreduce(P, n, dt, op=op)["inline_launch"] == 1
    run_reduce_scatter(P, 517, dt, op=op, order="ring")


@pytest.mark.parametrize("dt", ["bf16", "fp16", "fp32", "int32"])
@pytest.mark.parametrize("requant", [False, True])
@pytest.mark.parametrize("order,P", [("ring", 3), ("ring", 16), ("halving", 2), ("halving", 4), ("halving", 8),
                                     ("halving", 16), ("halving", 32), ("halving", 64), ("ascending", 8)])
def test_orders_and_requantised_partials(dt, requant, order, P):
    for n in SIZES:
        assert run_ar(P, n, dt, order, requant)["inline_launch"] == 1
    run_rs(P, 517, dt, order, requant)


@pytest.mark.parametrize("dt", ["bf16", "fp32"])
@pytest.mark.parametrize("P,group", [(16, 8), (64, 8), (6, 3)])
@pytest.mark.parametrize("phases", ["auto", "levels"])
def test_two_level_in_one_and_two_phases(dt, P, group, phases):
    for n in (9001, 64 * P * 3):  # unequal sub-shards (the executor's kernels), then equal ones
        info = run_allreduce(P, n, dt, algo="two_level", group_size=group, phases=phases)
        assert info["num_phases"] == (2 if phases == "levels" and P >= 16 else 1)
    assert info["inline_launch"] == 1


@pytest.mark.parametrize("dt", ["bf16", "int32"])
@pytest.mark.parametrize("P", [1, 2, 5, 8, 33, 64])
def test_allgather(dt, P):
    for m in (1, 7, 2047, 2049, 5001):
        run_allgather(P, m, dt)


@pytest.mark.parametrize("P,n,offset,packed", [(32, 262144, 0, 0), (32, 262144, 1, 1), (32, 262147, 0, 1), (32, 200000, 0, 1),
                                               (16, 131072, 0, 1), (16, 131072, 1, 1), (9, 262144, 0, 1), (7, 524288, 0, 1)])
def test_large_allgather(P, n, offset, packed):
    """16 MiB and more to 32 destinations: the executor's long runs for aligned blocks alone. Blocks of
    a power of two bytes, in 1024 tiles and more: a wavefront writes all destinations where they
    are aligned and there are 8 or more."""
    print(f"allgather P={P} n={n} offset {offset}", flush=True)
    rng = np.random.default_rng(n)
    send = [to_device(np.concatenate([np.zeros(offset, np.uint16), rng.integers(0, 1 << 15, n).astype(np.uint16)]), "bf16")[offset:]
            for _ in range(P)]
    whole = torch.zeros((P, P * n + 2 * 64), dtype=torch.bfloat16, device="cuda:0")
    with H.Comm(P, device=0) as c:
        H.hccl_allgather(c.handle, send, [w[64 + offset:64 + offset + P * n] for w in whole], n, "bf16")
        torch.cuda.synchronize()
        assert c.last_program()["inline_launch"] == packed
    want = torch.zeros_like(whole[0]).view(torch.int16)
    want[64 + offset:64 + offset + P * n] = torch.cat(send).view(torch.int16)
    for w in whole:
        assert torch.equal(w.view(torch.int16), want)


@pytest.mark.parametrize("dt,order", [("bf16", "halving"), ("fp16", "ring"), ("fp32", "halving")])
@pytest.mark.parametrize("op", ["sum", "max"])
def test_every_offset_from_a_boundary(dt, order, op):
    """Views that start 1, 2, ... elements into their allocation; sources and results agree or not."""
    P, n = 8, 2100
    rng = np.random.default_rng(3)
    x = rng.standard_normal((P, n)).astype(np.float32)
    bits = np.stack([to_device_bits(v, dt) for v in x])
    want = oracle.allreduce_ordered(bits, dt, order=order, shard=-(-(-(-n // P)) // 64) * 64) if op == "sum" else \
        oracle.allreduce(bits, dt, op=op)
    with H.Comm(P, device=0, order=order) as c:
        for a, b in ((1, 1), (3, 3), (0, 1), (5, 2), (7, 0)):
            print(f"offsets {a} {b} {dt} {op}", flush=True)
            send = [to_device(np.concatenate([np.zeros(a, bits.dtype), bits[r]]), dt)[a:] for r in range(P)]
            outs = [Guarded(n + b, dt) for _ in range(P)]
            H.hccl_allreduce(c.handle, send, [o.view[b:] for o in outs], n, dt, op)
            torch.cuda.synchronize()
            for r in range(P):
                got = outs[r].result()[b:]
                assert same_bits(got, want[r], dt), f"rank {r}: {first_mismatch(got, want[r])}"
                assert outs[r].guards_intact()


# fold, ranks, element type, operator, configuration
IN_PLACE = [
    ("list", 2, "bf16", "sum", {}), ("list", 3, "fp32", "sum", {}), ("list", 8, "fp16", "sum", {}),
    ("list", 9, "bf16", "sum", {}), ("list", 17, "int32", "sum", {}), ("list", 64, "fp32", "sum", {}),
    ("ring", 8, "bf16", "sum", {}), ("ring", 16, "fp32", "sum", {}),
    ("tree", 4, "fp16", "sum", {}), ("tree", 16, "bf16", "sum", {}), ("tree", 32, "fp32", "sum", {}),
    ("tree", 8, "bf16", "sum", {"requantize": 1}), ("list", 12, "fp16", "sum", {"requantize": 1}),
    ("group", 6, "bf16", "sum", {"algo": "two_level", "group_size": 3}),
    ("group", 16, "fp32", "sum", {"algo": "two_level", "group_size": 8}),
    ("group", 16, "bf16", "sum", {"algo": "two_level", "group_size": 8, "phases": "levels"}),
    ("list", 8, "bf16", "max", {}), ("list", 9, "fp32", "min", {}), ("ring", 4, "int32", "max", {}),
]


@pytest.mark.parametrize("fold,P,dt,op,cfg", IN_PLACE)
def test_in_place(fold, P, dt, op, cfg):
    """Results over their own inputs: in the last step of a tile a lane reads again what its neighbour
    is about to overwrite. Views that begin on a boundary, and 1 or 3 elements after one."""
    order = {"ring": "ring", "tree": "halving"}.get(fold, "ascending")
    # (sub-shards of one length: the two-level schedule's phases are then uniform)
    sizes = [64 * P, 64 * P * 3, 64 * P * 17] if fold == "group" else SIZES
    with H.Comm(P, device=0, order=order, **cfg) as c:
        for n in sizes:
            x = inputs(P, n, dt, seed=P * 13 + n)
            if op != "sum":
                want = oracle.allreduce(x, dt, op=op)
            elif fold == "group":
                want = oracle.allreduce(x, dt, group=cfg["group_size"])
            else:
                want = oracle.allreduce_ordered(x, dt, order=order, shard=lib_shard(n, P), requant=bool(cfg.get("requantize")))
            for at in (0, 1, 3):
                print(f"in place {fold} P={P} {dt} {op} n={n} offset {at} {cfg}", flush=True)
                bufs = [Guarded(n + at, dt, fill=np.concatenate([np.zeros(at, x.dtype), x[r]])) for r in range(P)]
                views = [b.view[at:] for b in bufs]
                H.hccl_allreduce(c.handle, views, views, n, dt, op)
                torch.cuda.synchronize()
                assert c.async_error() == 0
                assert c.last_program()["inline_launch"] == 1
                for r in range(P):
                    got = bufs[r].result()
                    assert not got[:at].any()
                    assert same_bits(got[at:], want[r], dt), f"rank {r}: {first_mismatch(got[at:], want[r])}"
                    assert bufs[r].guards_intact()


def to_host_floats(bits, dt):
    t = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16))
    return t.view({"bf16": torch.bfloat16, "fp16": torch.float16}[dt]).to(torch.float32).numpy()


def to_device_bits(v, dt):
    t = torch.from_numpy(v)
    if dt == "fp32":
        return v
    return t.to({"bf16": torch.bfloat16, "fp16": torch.float16}[dt]).view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("op,order,requant", [("sum", "ascending", False), ("sum", "halving", True), ("max", "ring", False)])
@pytest.mark.parametrize("dt", ["bf16", "fp16"])
def test_every_kind_of_value(op, order, requant, dt):
    """Random bit patterns: infinities, NaNs, subnormal and largest numbers."""
    P, n = 4, 20000
    x = np.random.default_rng(5).integers(0, 1 << 16, (P, n)).astype(np.uint16)
    with H.Comm(P, device=0, order=order, requantize=int(requant)) as c:
        send = [to_device(x[r], dt) for r in range(P)]
        outs = [Guarded(n, dt) for _ in range(P)]
        H.hccl_allreduce(c.handle, send, [o.view for o in outs], n, dt, op)
        torch.cuda.synchronize()
    want = oracle.allreduce(x, dt, op=op) if op == "max" else \
        oracle.allreduce_ordered(x, dt, order=order, shard=-(-(-(-n // P)) // 64) * 64, requant=requant)
    for r in range(P):
        assert same_bits(outs[r].result(), want[r], dt), first_mismatch(outs[r].result(), want[r])


def test_large_reductions_on_few_cus():
    """From 1 GiB moved on the tiles depend on the CUs of the stream, the results do not."""
    for P, n in ((8, (1 << 23) + 5), (12, 4 << 20)):
        g = torch.Generator(device="cuda:0").manual_seed(P)
        send = [torch.randn(P * n, generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(P)]
        want = send[0].float()
        for s in send[1:]:
            want += s
        want = want.to(torch.bfloat16).view(P, n)
        torch.cuda.synchronize()
        workers = []
        with MaskedStream(2) as few, H.Comm(P, device=0) as c:
            for stream in (None, few):
                print(f"reduce-scatter P={P} n={n} on {'16 CUs' if stream else 'all CUs'}", flush=True)
                out = [Guarded(n, "bf16") for _ in range(P)]
                torch.cuda.synchronize()
                H.hccl_reduce_scatter(c.handle, send, [o.view for o in out], n, "bf16", stream=stream)
                torch.cuda.synchronize()
                workers.append(c.last_program()["workers"])
                assert c.last_program()["inline_launch"] == 1
                for r in range(P):
                    assert torch.equal(out[r].view, want[r]) and out[r].guards_intact()
        assert workers[1] < workers[0]


def test_bf16_rounding_of_every_sum():
    """Every FP32 value that a sum of bf16 numbers can take (multiples of the smallest subnormal bf16,
    2^-133), each as a sum of three: the result is rounded to nearest, ties to even."""
    P, n = 3, 1 << 26
    recv = [torch.empty(n, dtype=torch.bfloat16, device="cuda:0") for _ in range(P)]
    with H.Comm(P, device=0) as c:
        for k in range(1 << 6):
            if k % 16 == 0:
                print(f"bf16 rounding, patterns from {k << 26:#x}", flush=True)
            u = torch.arange(k * n, (k + 1) * n, device="cuda:0") - (1 << 31)      # all patterns, as int64
            x = u.to(torch.int32).view(torch.float32)
            small = x.abs() < 2.0 ** -110                                          # below, drop the bits under 2^-133
            x = torch.where(small, (x * 2.0 ** 120 * 2.0 ** 13).trunc() * 2.0 ** -120 * 2.0 ** -13, x)
            x = torch.where(torch.isfinite(x), x, torch.zeros_like(x))
            parts, rest = [], x
            for _ in range(P):
                top = (rest.view(torch.int32) & -65536).view(torch.float32)
                parts.append((top.view(torch.int32) >> 16).to(torch.int16).view(torch.bfloat16))
                rest = rest - top
            assert not rest.any()
            c.allreduce(parts, recv)
            assert c.last_program()["inline_launch"] == 1
            b = x.view(torch.int32).to(torch.int64) & 0xFFFFFFFF
            want = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16).to(torch.int16)
            # (a sum that is zero is +0: the first part of -0 carries the sign and the others are +0)
            want = torch.where(x == 0, torch.zeros_like(want), want)
            for r in recv:
                assert torch.equal(r.view(torch.int16), want)


@pytest.mark.parametrize("dt", ["bf16", "fp16"])
def test_vectors_and_single_elements_round_alike(dt):
    """Infinities, NaNs of both kinds and signs, ties, overflow and subnormals, in pairs: the bits of a
    call of whole vectors are those of calls of fewer elements than a vector, payload and sign of a
    NaN included (which of two NaNs a sum keeps is not defined)."""
    special = {"bf16": [0, 0x8000, 1, 0x8001, 0x7F, 0x80, 0x3F80, 0x3F81, 0xBF80, 0x3380, 0x3B80, 0x4380, 0x7F7F, 0xFF7F, 0x7E80, 0x7F80, 0xFF80,
                        0x7F81, 0x7FC0, 0xFFC5, 0xFF81, 0x7FFF],
               "fp16": [0, 0x8000, 1, 0x8001, 0x3FF, 0x400, 0x3C00, 0x3C01, 0xBC00, 0x1000, 0x0C00, 0x6400, 0x7BFF, 0xFBFF, 0x7000, 0x7C00, 0xFC00,
                        0x7C01, 0x7E00, 0xFE05, 0xFC01, 0x7FFF]}[dt]
    x = np.array([(a, b) for a in special for b in special], np.uint16).T.copy()
    x = np.concatenate([x, np.zeros((2, -x.shape[1] % 56), np.uint16)], axis=1)   # whole vectors, and sevens
    P, n = x.shape
    with H.Comm(P, device=0) as c:
        def run(lo, hi):
            outs = [Guarded(hi - lo, dt) for _ in range(P)]
            H.hccl_allreduce(c.handle, [to_device(x[r, lo:hi], dt) for r in range(P)], [o.view for o in outs], hi - lo, dt)
            torch.cuda.synchronize()
            assert c.last_program()["inline_launch"] == 1
            return np.stack([o.result() for o in outs])

        print(f"special values {dt}", flush=True)
        whole = run(0, n)
        single = np.concatenate([run(lo, lo + 7) for lo in range(0, n, 7)], axis=1)
    nan = np.isnan(to_host_floats(x, dt))
    one = ~(nan[0] & nan[1])
    assert nan.any() and np.array_equal(whole[:, one], single[:, one]), first_mismatch(whole[0, one], single[0, one])
    assert all(same_bits(a, b, dt) for a, b in zip(whole, single))
    want = oracle.allreduce(x, dt)
    for r in range(P):
        assert same_bits(whole[r], want[r], dt), first_mismatch(whole[r], want[r])


# ------------------------------------------------------------------ AllToAllvDynamic
@pytest.mark.parametrize("P", [7, 8, 9, 16, 17, 33, 64])
@pytest.mark.parametrize("R,dt", [(1, "bf16"), (5, "int32"), (2048, "bf16"), (3001, "fp32")])
def test_dynamic_layouts(P, R, dt):
    rows = 9 if R < 100 else 3
    counts = random_counts(P, rows, seed=P + R, zero_frac=0.4)
    ok, info = run_dynamic(P, R, dt, counts, int(counts.sum(axis=1).max()) + 1, int(counts.sum(axis=0).max()), seed=P)
    assert ok and info["inline_launch"] == 1
    # explicit offsets, the received ranges in another order with gaps
    rng = np.random.default_rng(P)
    sd, rd, cap = np.cumsum(counts, axis=1) - counts, np.zeros((P, P), np.int64), 0
    for d in range(P):
        at = 0
        for s in rng.permutation(P):
            rd[d, s] = at
            at += counts[s, d] + int(rng.integers(0, 2))
        cap = max(cap, at)
    assert run_dynamic(P, R, dt, counts, int(counts.sum(axis=1).max()), cap, sd=sd, rd=rd, seed=P)[0]


@pytest.mark.parametrize("P", [8, 20, 64])
@pytest.mark.parametrize("case", ["send_over", "recv_over", "negative", "huge", "overlap", "offset_out", "recv_offset_out"])
def test_dynamic_rejects_as_a_workgroup(P, case):
    R = 6
    counts = random_counts(P, 5, seed=P, zero_frac=0.0) + 1
    send_cap, recv_cap = int(counts.sum(axis=1).max()), int(counts.sum(axis=0).max())
    sd = rd = None
    s, d = P - 1, P // 2
    if case == "send_over":
        send_cap -= 1
    elif case == "recv_over":
        recv_cap -= 1
    elif case == "negative":
        counts[s, d] = -1
    elif case == "huge":
        counts[s, d] = (1 << 32) + 1
    elif case in ("overlap", "recv_offset_out"):
        back = counts.T
        rd = np.cumsum(back, axis=1) - back
        rd[d, s] = rd[d, s] - 1 if case == "overlap" else recv_cap - counts[s, d] + 1
    elif case == "offset_out":
        sd = np.cumsum(counts, axis=1) - counts
        sd[s, d] = send_cap - counts[s, d] + 1
    assert not run_dynamic(P, R, "bf16", counts, send_cap, recv_cap, sd=sd, rd=rd, seed=1)[0]
