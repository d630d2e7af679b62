"""GPU: damaged streams through every decoder.

Which decoder takes a call goes by its blocks (256 compute units): two waves
per block, or the same kernel with one wave per block (a stream of many small
blocks); one wave per block with the ring of table entries or the ring of plain
words; and for a large stream two launches, of which its header picks one.
Each must report damage to a header or a directory entry, must report or show
damage to a section, and must not read outside the stream.  The undamaged
stream is decoded first and last."""
import struct
import sys

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

EB = {"bf16": 2, "fp16": 2, "fp32": 4, "e4m3fn": 2}
HEADER = (0, 4, 5, 6, 7, 8, 12, 16, 24)   # magic, version, type, bits, mode, block size, blocks, elements, bytes


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def uz():
    import paper_2604_17172_amd as m
    return m


def tensor(dtype, n, seed):
    m = min(n, 1 << 20)
    x = (W.normal_bf16(m, seed=seed) if dtype == "bf16" else W.grad_fp16(m, seed=seed) if dtype == "fp16" else
         W.grad_fp32(m, seed=seed) if dtype == "fp32" else W.normal_fp8_pairs(m, dtype, seed=seed))
    t = torch.from_numpy(x.view(np.int16 if EB[dtype] == 2 else np.int32)).cuda()
    return t.repeat(-(-n // m))[:n].contiguous()


def put(s, at, value):
    s[at:at + len(value)] = torch.tensor(list(value), dtype=torch.uint8, device="cuda")


def check_damage(decode, s, at, n_blocks, raw_bytes, x, label, uz, shared):
    """`decode(s)` -> (output, status); a stream of n_blocks blocks at byte
    `at` of the buffer s is damaged a byte at a time and restored."""
    def run():
        y, status = decode(s)
        torch.cuda.synchronize()
        return y.view(x.dtype), int(status.item())

    y, status = run()
    assert status == 0 and torch.equal(y, x), label
    pad = lambda v: (v + 15) // 16 * 16
    dir_at = at + 32
    ends = [e & 0x7FFFFFFF for e in struct.unpack(f"<{n_blocks}I", s[dir_at:dir_at + 4 * n_blocks].cpu().numpy().tobytes())]
    coded = at + 32 + pad(4 * n_blocks) + (512 if shared else 0) + pad(raw_bytes)
    mid = n_blocks // 2
    start, end = coded + 16 * ends[mid - 1], coded + 16 * ends[mid]
    always = [(f"header byte {o}", at + o, 0x5A) for o in HEADER]
    # an entry that ends before it starts, one past the stream, and the last
    always += [("first directory entry", dir_at + 3, 0x40), ("a directory entry", dir_at + 4 * mid + 3, 0x40),
               ("the last directory entry", dir_at + 4 * (n_blocks - 1), 0x01)]
    if shared:
        always.append(("the stream's table", at + 32 + pad(4 * n_blocks) + 2, 0x01))
    else:
        always += [("a section's presence bits", start + 256 + 20, 0x10), ("a section's table", start + 288, 0x01)]
    always.append(("a section's first state", start + 3, 0x80))
    rng = np.random.Generator(np.random.PCG64(n_blocks))
    shown = [(f"section byte {o}", start + o, 1 << int(rng.integers(0, 8)))
             for o in sorted(rng.integers(256 if shared else 800, end - start - 16, 12))]
    for what, byte, flip in always + shown:
        old = int(s[byte].item())
        say(f"[damage] {label}: {what}")
        put(s, byte, [old ^ flip])
        y, status = run()
        put(s, byte, [old])
        if (what, byte, flip) in always:
            assert status == uz.ECORRUPT, (label, what)
        else:
            assert status != 0 or not torch.equal(y, x), (label, what)
    y, status = run()
    assert status == 0 and torch.equal(y, x), label


# bf16: ring of entries to 3072 blocks and past 4096, plain words between (and
# past it for FP8 and under a stream's table); fp32 plain words from 1409 on
@pytest.mark.parametrize("dtype,mode,blocks", [("bf16", "per_block", 700), ("bf16", "per_block", 800),
                                               ("bf16", "per_block", 3500), ("bf16", "per_block", 4200),
                                               ("e4m3fn", "per_block", 4200), ("fp16", "sampled", 700),
                                               ("fp16", "sampled", 800), ("fp16", "sampled", 4200),
                                               ("fp32", "per_block", 1000), ("fp32", "per_block", 1500)])
def test_chunk_streams(uz, dtype, mode, blocks):
    bb, per_chunk = 8192, 100
    e = EB[dtype]
    be = bb // e
    n = blocks * be
    x = tensor(dtype, n, seed=blocks)
    buf, slot, _, _ = uz.compress_chunked_table(x, bb, bb * per_chunk, mode, dtype=dtype)
    y = torch.empty_like(x)

    def decode(s):
        return uz.decompress_chunked(s, slot, dtype, n, bb, bb * per_chunk, out=y, shared=mode == "sampled")

    chunk = blocks // per_chunk // 2
    check_damage(decode, buf, chunk * slot, per_chunk, (e - 1) * per_chunk * be, x, f"{dtype} {mode} {blocks} blocks", uz,
                 mode == "sampled")


# two waves per block; the same kernel, one wave per block; ring of entries;
# two launches: plain words, entries
@pytest.mark.parametrize("dtype,mode,size,block", [("bf16", "per_block", 2 << 20, 65536), ("bf16", "per_block", 8 << 20, 4096),
                                                   ("fp16", "sampled", 2 << 20, 16384), ("fp32", "per_block", 16 << 20, 16384),
                                                   ("bf16", "per_block", 200 << 20, 65536),
                                                   ("bf16", "per_block", 200 << 20, 262144),
                                                   ("fp16", "sampled", 200 << 20, 65536),
                                                   ("fp16", "sampled", 200 << 20, 262144)])
def test_streams(uz, dtype, mode, size, block):
    e = EB[dtype]
    n = size // e - 5
    x = tensor(dtype, n, seed=block)
    s, got = uz.compress_table(x, block, mode, dtype=dtype)
    s = s[: int(got.item())].clone()
    y = torch.empty_like(x)

    def decode(buf, in_bytes=None):
        call = uz.decompress if mode == "per_block" else uz.decompress_table
        return call(buf, dtype, n, out=y, in_bytes=in_bytes)

    nb = -(-n * e // block)
    check_damage(decode, s, 0, nb, (e - 1) * n, x, f"{dtype} {mode} {size >> 20} MiB of {block}", uz, mode == "sampled")
    for nbytes in (s.numel() - 16, 32, 8):
        say(f"[damage] {dtype} {mode} {size >> 20} MiB of {block}: {nbytes} bytes given")
        _, status = decode(s, nbytes)
        torch.cuda.synchronize()
        assert int(status.item()) == uz.ECORRUPT, nbytes
