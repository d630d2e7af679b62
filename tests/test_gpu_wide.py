"""GPU: calls of few blocks, coded by a workgroup per block, and the line to
the encoder of one wave per block (512 blocks on a chip of 256 compute
units), against the oracle byte for byte.

The other encoder tests use small tensors, which the workgroup encoder
takes; the cases past the line here are what holds the one-wave encoder to
the same edges: staging windows that slide, STORED blocks, partial last
blocks, the XCD-local producer."""
import numpy as np
import pytest
import torch

from oracle import ref
import workloads as W

pytestmark = pytest.mark.gpu

EB = {"bf16": 2, "fp16": 2, "fp32": 4, "e4m3fn": 2, "e5m2": 2}
LINE = 512


@pytest.fixture(scope="module")
def uz():
    import paper_2604_17172_amd as m
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16 if a.itemsize == 2 else np.int32)).cuda()


def dev_bytes(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def values(dtype, n, seed):
    """Ordinary values with stretches of random bits (STORED blocks) and of
    one value (a table of one symbol)."""
    if dtype in ("e4m3fn", "e5m2"):
        x = W.normal_fp8_pairs(n, dtype, seed=seed)
    elif dtype == "bf16":
        x = W.normal_bf16(n, seed=seed)
    elif dtype == "fp16":
        x = W.grad_fp16(n, seed=seed)
    else:
        x = W.grad_fp32(n, seed=seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    for _ in range(3):
        a, m = int(rng.integers(0, n)), int(rng.integers(1, n // 6 + 2))
        x[a:a + m] = rng.integers(0, 1 << (8 * x.itemsize), x[a:a + m].size, dtype=np.uint64).astype(x.dtype)
        a = int(rng.integers(0, n))
        x[a:a + m] = x[a]
    return x


def check(uz, x, dtype, bb):
    xt = dev(x)
    out, size = uz.compress(xt, bb, dtype=dtype, check=True)
    assert np.array_equal(out[: int(size.item())].cpu().numpy(), ref.compress(x, dtype, bb)), (dtype, bb, x.size)
    out, size = uz.compress_table(xt, bb, "sampled", dtype=dtype)
    torch.cuda.synchronize()
    assert np.array_equal(out[: int(size.item())].cpu().numpy(), ref.compress_table(x, dtype, bb, "sampled")), \
        (dtype, bb, x.size, "sampled")


def check_chunks(uz, x, dtype, bb, cb):
    for mode in ("per_block", "sampled"):
        out, slot, sizes, flags = uz.compress_chunked_table(dev(x), bb, cb, mode, dtype=dtype, epoch=3)
        torch.cuda.synchronize()
        assert bool((flags == 3).all())
        buf, sz = out.cpu().numpy(), sizes.cpu().numpy()
        for c, want in enumerate(ref.compress_chunked(x, dtype, bb, cb, mode)):
            assert np.array_equal(buf[c * slot:c * slot + sz[c]], want), (dtype, bb, cb, x.size, mode, c)


# elements of the last block: the rounds' (512), the waves' (8 rounds) and the
# largest block's edges
@pytest.mark.parametrize("tail", [1, 511, 513, 8 * 512 - 1, 8 * 512 + 1, 9 * 512, 63 * 512 + 7, 64 * 512 - 1])
@pytest.mark.parametrize("dtype", sorted(EB))
def test_block_edges(uz, dtype, tail):
    bb = 32768 * EB[dtype]
    check(uz, values(dtype, tail, seed=tail), dtype, bb)
    check(uz, values(dtype, 2 * 32768 + tail, seed=tail), dtype, bb)
    check_chunks(uz, values(dtype, 3 * 32768 + tail, seed=tail), dtype, bb, 2 * bb)


@pytest.mark.parametrize("blocks", [LINE - 1, LINE, LINE + 1])
@pytest.mark.parametrize("dtype", sorted(EB))
def test_blocks_around_the_line(uz, dtype, blocks):
    be = 4096 // EB[dtype]
    x = values(dtype, (blocks - 1) * be + be // 3, seed=blocks)
    check(uz, x, dtype, 4096)
    # 16 KiB chunks: past 64 chunks (and 512 blocks) coded XCD by XCD
    check_chunks(uz, x, dtype, 4096, 16384)
    check_chunks(uz, x, dtype, 4096, 4096 * 100)


# fp32 chunks of two and more blocks of 64 KiB, their number a multiple of 8:
# past one block per compute unit coded XCD by XCD, else by workgroups.
@pytest.mark.parametrize("blocks,per_chunk", [(256, 4), (258, 4), (285, 4), (272, 2), (272, 1), (512, 16)])
def test_large_fp32_chunks(uz, blocks, per_chunk):
    x = values("fp32", (blocks - 1) * 16384 + 999, seed=blocks + per_chunk)
    check_chunks(uz, x, "fp32", 65536, 65536 * per_chunk)


@pytest.mark.parametrize("dtype", ["bf16", "fp16", "fp32", "e4m3fn"])
def test_one_wave_per_block_spills_and_stores(uz, dtype):
    """Past the line in the largest blocks that keep their symbols in
    registers: words beyond the staging window, STORED blocks."""
    be = 32768
    n = (LINE + 3) * be + 777
    x = np.tile(values(dtype, 37 * be + 11, seed=5), n // (37 * be) + 1)[:n].copy()
    if dtype in ("bf16", "fp16"):
        # exponents spread until a block needs more than the window holds
        rng = np.random.Generator(np.random.PCG64(9))
        m = 40 * be
        e = rng.integers(95, 159, m) << 7 if dtype == "bf16" else rng.integers(1, 31, m) << 10
        low = rng.integers(0, 1 << (7 if dtype == "bf16" else 10), m)
        x[: m] = (e | low | rng.integers(0, 2, m) << 15).astype(x.dtype)
    check(uz, x, dtype, be * EB[dtype])


# The most inputs whose decoders' tables and rings, slabs and symbols fit the
# fused reduce's LDS in the largest blocks it takes (six and five), one fewer,
# and one more, which the two kernels take.
@pytest.mark.parametrize("dtype,bb,n_in", [("bf16", 131072, k) for k in (5, 6, 7)] +
                         [("fp32", 262144, k) for k in (4, 5, 6)])
def test_fused_reduce_lds_edge(uz, dtype, bb, n_in):
    n = 2 * bb // EB[dtype] + 4321
    streams = [ref.compress(W.normal_bf16(n, seed=i) if dtype == "bf16" else W.grad_fp32(n, seed=i), dtype, bb)
               for i in range(n_in)]
    out, size, raw, status = uz.reduce_fused([dev_bytes(s) for s in streams], dtype, n, bb)
    torch.cuda.synchronize()
    want_s, want_y = ref.reduce(streams, dtype, n, bb)
    assert int(status.item()) == 0
    assert np.array_equal(raw.cpu().numpy().view(want_y.dtype), want_y)
    assert np.array_equal(out[: int(size.item())].cpu().numpy(), want_s)


# FP8 pairs and 16-bit types under a stream's table stay with the decoder's
# ring of plain words past 4096 blocks too.
@pytest.mark.parametrize("blocks", [3072, 3073, 4097])
@pytest.mark.parametrize("dtype,mode", [("e4m3fn", "per_block"), ("e5m2", "sampled"), ("bf16", "sampled"),
                                        ("fp16", "sampled")])
def test_wordy_chunks_decode(uz, dtype, mode, blocks):
    n = (blocks - 1) * 4096 + 1234
    x = values(dtype, n, seed=blocks)
    buf, slot, sizes, _ = uz.compress_chunked_table(dev(x), 8192, 8192 * 16, mode, dtype=dtype)
    y, status = uz.decompress_chunked(buf, slot, dtype, n, 8192, 8192 * 16, shared=mode == "sampled")
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and bool((sizes > 0).all())
    assert np.array_equal(y.cpu().numpy().view(x.dtype), x)


# One stream: its header says whether the plain ring (more than 3072 blocks)
# or the ring of entries decodes.
@pytest.mark.parametrize("block_bytes", [16384, 65536, 1 << 20])
@pytest.mark.parametrize("dtype,mode", [("e4m3fn", "per_block"), ("e5m2", "sampled"), ("bf16", "sampled")])
def test_wordy_stream_decode(uz, dtype, mode, block_bytes):
    part = values(dtype, 3 * (1 << 20) + 77, seed=21)
    n = 140 << 20
    x = dev(part).repeat(n // part.size + 1)[:n].contiguous()
    s, size = uz.compress_table(x, block_bytes, mode, dtype=dtype)
    torch.cuda.synchronize()
    s = s[: int(size.item())]
    y, status = uz.decompress_table(s, dtype, n) if mode == "sampled" else uz.decompress(s, dtype, n)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert bool((y.view(torch.int16) == x).all())


# A stream under a weak table (of its first 256 KiB, another distribution's):
# past 192 MiB and from 1281 blocks on more than 0.35 words per element, which
# its header gives, take it to the plain ring.
@pytest.mark.parametrize("blocks", [1280, 1281])
def test_weak_table_stream_decode(uz, blocks):
    bb = 262144
    n = (blocks - 1) * (bb // 2) + 777
    x = dev(W.normal_bf16(1 << 20, sigma=0.02, seed=3)).repeat(-(-n >> 20))[:n].contiguous()
    x[: 1 << 17] = dev(W.normal_bf16(1 << 17, sigma=1.0, seed=4))
    s, size = uz.compress_table(x, bb, "sampled", dtype="bf16")
    torch.cuda.synchronize()
    size = int(size.item())
    assert 10 * (size - n) > 7 * n
    y, status = uz.decompress_table(s[:size], "bf16", n)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and bool((y.view(torch.int16) == x).all())
