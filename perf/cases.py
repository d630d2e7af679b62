"""Timed cases of the codec's public entry points.

The codec sits inside GPU communication: a sender compresses a tensor (whole,
or cut into chunks that leave as they finish), a receiver decompresses what
arrived, and a rank of an all-reduce decodes its peers' shares, sums and
recompresses them.  Messages range from 256 KiB to 1 GiB.  Each case is one
such call with the buffers a communication loop keeps (stream buffer,
workspace, size, flags) made beforehand.

Every output is bytes or whole numbers and the stream format defines exactly
one stream per input, so all comparisons are exact.
"""
from __future__ import annotations

import math

import torch

import paper_2604_17172_amd as uz

KIB, MIB = 1 << 10, 1 << 20
ELEM = {"bf16": 2, "fp16": 2, "fp32": 4, "e4m3fn": 2, "e5m2": 2}
FP8 = {"e4m3fn": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}


def listed():
    return [
        # the smallest message of a point-to-point transfer (256 KiB, U[-1, 1]): launches and one block's chain
        {"name": "p2p_send_256KiB", "op": "compress", "dtype": "bf16", "data": "uniform", "n": 131072, "block": 64 * KIB},
        # a received tensor of odd length, about 2 MB
        {"name": "p2p_recv_odd", "op": "decompress", "dtype": "bf16", "data": "normal", "n": 1000003, "block": 64 * KIB},
        # a single activation or weight tensor of 4 MiB
        {"name": "tensor_send_4MiB", "op": "compress", "dtype": "bf16", "data": "normal", "n": 2097152, "block": 64 * KIB},
        # a small gradient bucket of a two-input reduce with the rank's own share added raw, ragged
        {"name": "reduce_small_fp32_local", "op": "reduce", "dtype": "fp32", "data": "grad", "n": 300001, "block": 64 * KIB, "inputs": 2, "local": True},
        # one rank's share of an 8-way all-reduce of activations [8192, 8192]
        {"name": "reduce_8x16MiB", "op": "reduce", "dtype": "bf16", "data": "tokens", "n": 8388608, "block": 64 * KIB, "inputs": 8, "local": False},
        # FP8 activations (value pairs) sent in 4 MiB chunks with a table sampled per chunk
        {"name": "fp8_chunks_sampled_64MiB", "op": "send_chunks", "dtype": "e4m3fn", "data": "fp8", "n": 33554432, "block": 64 * KIB, "chunk": 4 * MIB, "table": "sampled"},
        # a received fp32 gradient of 214 MB
        {"name": "grad_recv_fp32_214MB", "op": "decompress", "dtype": "fp32", "data": "grad", "n": 53500000, "block": 256 * KIB},
        # an fp16 gradient of 512 MiB in large blocks
        {"name": "grad_send_fp16_512MiB", "op": "compress", "dtype": "fp16", "data": "grad", "n": 268435456, "block": 256 * KIB},
        # eight layers' KV cache leaving prefill in 1 MiB chunks, and arriving
        {"name": "kv_send_chunks_512MiB", "op": "send_chunks", "dtype": "bf16", "data": "kv", "n": 268435456, "block": 64 * KIB, "chunk": MIB, "table": "per_block"},
        {"name": "kv_recv_chunks_512MiB", "op": "recv_chunks", "dtype": "bf16", "data": "kv", "n": 268435456, "block": 64 * KIB, "chunk": MIB, "table": "per_block"},
        # weight synchronisation of a 0.5B-parameter model (1 GiB buffer): sender and receiver
        {"name": "weights_send_1GiB", "op": "compress", "dtype": "bf16", "data": "weights", "n": 536870912, "block": 64 * KIB},
        {"name": "weights_recv_1GiB", "op": "decompress", "dtype": "bf16", "data": "weights", "n": 536870912, "block": 64 * KIB},
    ]


def draw(rng):
    """Another call of the same ranges: 256 KiB to 256 MiB of input per call
    (over the logarithm of the size, so any remainder occurs), every type,
    16 KiB to 256 KiB blocks, chunks of 1 to 4 MiB."""
    op = rng.choice(["compress", "compress", "decompress", "decompress", "send_chunks", "recv_chunks", "reduce", "reduce"])
    size = math.exp(rng.uniform(math.log(256 * KIB), math.log(256 * MIB)))
    if op == "reduce":
        dtype = rng.choice(["bf16", "bf16", "fp16", "fp32"])
    else:
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp16", "fp32", "e4m3fn", "e5m2"])
    data = {"bf16": rng.choice(["normal", "uniform", "weights", "kv", "tokens"]), "fp16": "grad", "fp32": "grad",
            "e4m3fn": "fp8", "e5m2": "fp8"}[dtype]
    block = rng.choice([64 * KIB, 64 * KIB, 64 * KIB, 16 * KIB, 32 * KIB, 128 * KIB])
    if data == "grad":
        block = rng.choice([64 * KIB, 256 * KIB])
    case = {"op": op, "dtype": dtype, "data": data, "block": block}
    if op == "reduce":
        case["inputs"] = rng.choice([2, 3, 4, 7, 8])
        case["local"] = rng.random() < 0.5
        size = max(size / case["inputs"], 64 * KIB)
    if op in ("send_chunks", "recv_chunks"):
        case["chunk"] = rng.choice([1, 2, 4]) * MIB
        case["table"] = rng.choice(["per_block", "per_block", "sampled"])
    case["n"] = max(int(size) // ELEM[dtype], 1024)
    return case


# ------------------------------------------------------------------ inputs
def _values(case, g, share=0):
    """The tensor's bit patterns on the GPU (int16, or int32 for fp32)."""
    n, data, dtype = case["n"], case["data"], case["dtype"]
    dev = g.device
    if data == "fp8":
        z = torch.randn(2 * n, generator=g, device=dev)
        return z.to(FP8[dtype]).view(torch.int16)
    if data == "grad":
        # Laplace(0, 1e-4), one entry in a hundred 100 times larger
        x = torch.empty(n, device=dev).exponential_(1.0, generator=g)
        x -= torch.empty(n, device=dev).exponential_(1.0, generator=g)
        x *= 1e-4
        x = torch.where(torch.rand(n, generator=g, device=dev) < 0.01, 100.0 * x, x)
        return x.view(torch.int32) if dtype == "fp32" else x.to(torch.float16).view(torch.int16)
    if data == "uniform":
        x = torch.rand(n, generator=g, device=dev) * 2 - 1
    else:
        x = torch.randn(n, generator=g, device=dev)
        if data == "normal":
            x *= 0.02
        elif data == "weights":
            # embedding N(0, 1), then layers N(0, 0.02) with norm vectors N(1, 0.05)
            embed = min(n // 4, 151936 * 896)
            x[embed:] *= 0.02
            for at in range(embed + 14712320, n, 14714112):
                m = min(1792, n - at)
                x[at:at + m] = 1.0 + 2.5 * x[at:at + m]
        elif data == "kv":
            # [.., 8 heads, 128 channels]: log-normal channel scales, 4 outlier channels a head at 20x
            s = torch.exp(0.5 * torch.randn(8, 128, generator=g, device=dev))
            s.scatter_(1, torch.rand(8, 128, generator=g, device=dev).argsort(1)[:, :4],
                       20.0 * s.gather(1, torch.arange(4, device=dev).expand(8, 4)))
            head = n // 1024 * 1024
            x[:head].view(-1, 1024).mul_(s.view(1, 1024))
        elif data == "tokens":
            # per-token scales, the same for every rank's share
            t = torch.Generator(device=dev).manual_seed(g.initial_seed() - share)
            s = torch.rand((n + 8191) // 8192, generator=t, device=dev) * 1.5 + 0.5
            x *= s.repeat_interleave(8192)[:n]
    return x.to(torch.bfloat16).view(torch.int16)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _bytes(n):
    return torch.zeros(max(n, 16), dtype=torch.uint8, device="cuda")


def _compress_state(case, x):
    dt, n = uz.dtype_code(case["dtype"]), case["n"]
    return {"case": case, "x": x, "out": _bytes(uz.uzip_max_compressed_size(dt, n, case["block"])),
            "ws": _bytes(uz.uzip_workspace_size(uz.OP_COMPRESS, dt, n, case["block"])),
            "size": torch.zeros(1, dtype=torch.int64, device="cuda")}


def _chunks_state(case, x):
    dt, n, e = uz.dtype_code(case["dtype"]), case["n"], ELEM[case["dtype"]]
    ce = case["chunk"] // e
    chunks = (n + ce - 1) // ce
    sampled = case["table"] == "sampled"
    slot = uz.uzip_max_compressed_size(dt, min(n, ce), case["block"]) + (uz.TABLE_BYTES if sampled else 0)
    slot = (slot + 255) // 256 * 256
    op = uz.OP_CHUNKED_TABLE if sampled else uz.OP_CHUNKED
    return {"case": case, "x": x, "out": _bytes(slot * chunks),
            "ws": _bytes(uz.uzip_workspace_size(op, dt, n, case["block"], case["chunk"])),
            "flags": torch.zeros(2 * chunks, dtype=torch.int32, device="cuda")}


def _send(s):
    """A sender's call on state s: the compressed stream or chunk streams."""
    case = s["case"]
    if "chunk" not in case:
        return uz.compress(s["x"], case["block"], dtype=case["dtype"], out=s["out"], ws=s["ws"], size=s["size"])
    if case["table"] == "sampled":
        return uz.compress_chunked_table(s["x"], case["block"], case["chunk"], "sampled", dtype=case["dtype"],
                                         flags=s["flags"], out=s["out"], ws=s["ws"])
    return uz.compress_chunked(s["x"], case["block"], case["chunk"], dtype=case["dtype"], flags=s["flags"],
                               out=s["out"], ws=s["ws"])


def prepare(case, seed):
    op, n = case["op"], case["n"]
    bits = torch.int32 if case["dtype"] == "fp32" else torch.int16
    if op == "reduce":
        streams = []
        for r in range(case["inputs"]):
            st = _compress_state(case, _values(case, _generator(100 * seed + r), r))
            out, size = _send(st)
            streams.append(out[: int(size.item())].clone())
        local = _values(case, _generator(100 * seed + 99), 99) if case["local"] else None
        dt = uz.dtype_code(case["dtype"])
        return {"case": case, "streams": streams, "local": local,
                "out": _bytes(uz.uzip_max_compressed_size(dt, n, case["block"])),
                "ws": _bytes(uz.uzip_workspace_size(uz.OP_REDUCE, dt, n, case["block"], case["inputs"]))}
    x = _values(case, _generator(seed))
    st = _chunks_state(case, x) if "chunk" in case else _compress_state(case, x)
    if op in ("compress", "send_chunks"):
        return st
    sent = _send(st)
    state = {"case": case, "y": torch.zeros(n, dtype=bits, device="cuda"),
             "status": torch.zeros(1, dtype=torch.int32, device="cuda")}
    if op == "decompress":
        state["stream"] = sent[0][: int(sent[1].item())].clone()
    else:
        state["buf"], state["slot"] = sent[0], sent[1]
        torch.cuda.synchronize()
    return state


def run(s):
    case = s["case"]
    op, dtype, n = case["op"], case["dtype"], case["n"]
    if op == "compress":
        return _send(s)
    if op == "send_chunks":
        out, _, sizes, flags = _send(s)
        return out, sizes, flags
    if op == "decompress":
        return uz.decompress(s["stream"], dtype, n, out=s["y"], status=s["status"])
    if op == "recv_chunks":
        return uz.decompress_chunked(s["buf"], s["slot"], dtype, n, case["block"], case["chunk"], out=s["y"],
                                     shared=case["table"] == "sampled")
    return uz.reduce_fused(s["streams"], dtype, n, case["block"], local=s["local"], out=s["out"], ws=s["ws"])


# ------------------------------------------------------------------ what a pass cannot do without
# stream bytes per tensor byte of each distribution (measured; the raw plane
# alone is 1/2, for fp32 3/4)
RATIO = {"uniform": 0.63, "normal": 0.663, "weights": 0.663, "kv": 0.69, "tokens": 0.67, "bf16": 0.67,
         "fp16": 0.806, "fp32": 0.842, "e4m3fn": 0.822, "e5m2": 0.71}


def work(case):
    tensor = case["n"] * ELEM[case["dtype"]]
    stream = tensor * RATIO.get(case["data"], RATIO[case["dtype"]])
    if case["op"] == "reduce":
        # streams in, the local share in, the reduced tensor and its stream out; one addition per value and input
        return {"bytes": case["inputs"] * stream + (tensor if case["local"] else 0) + tensor + stream,
                "flops": (case["inputs"] - 1 + case["local"]) * case["n"]}
    return {"bytes": tensor + stream, "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """What the receiver must get back: the tensor that was sent."""
    if case["op"] in ("decompress", "recv_chunks"):
        return _values(case, _generator(seed)), torch.zeros(1, dtype=torch.int32, device="cuda")
    return None
