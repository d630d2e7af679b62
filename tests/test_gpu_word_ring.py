"""GPU: the decoders' word ring at its limits.

A block is coded when its words average less than 256 a round (512
elements); a stretch of rare symbols inside it takes up to 512, which drains
the chunks a decoding wave holds ready and makes it load one on the spot.
Blocks here hold stretches of one symbol and of all 256, in every order, at
lengths around the four rounds of the decoder's loop, so that the ring runs
low at the start, in the middle and at the end of a block, over full rounds
and partial ones.  The decoded values must equal the input bit for bit, and
the fused reduce of such streams the oracle's."""
import numpy as np
import pytest
import torch

from oracle import ref

pytestmark = pytest.mark.gpu

BITS = {"bf16": np.uint16, "fp16": np.uint16, "fp32": np.uint32}


def tensor(dtype, n, pattern, block_elems, seed):
    """Bit patterns whose coded symbols are 126 in the quiet stretches and
    uniform over all 256 in the loud ones (the symbol is the top byte of the
    element rotated left by one)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    at = np.arange(n) % block_elems
    loud = {"spike": at < block_elems // 12, "head": at < block_elems * 3 // 10, "tail": at >= block_elems * 7 // 10,
            "waves": (at // 3072) % 3 == 1, "flat": np.ones(n, bool)}[pattern]
    sym = np.where(loud, rng.integers(0, 256, n), 126).astype(np.uint64)
    bits = 16 if BITS[dtype] is np.uint16 else 32
    v = sym << (bits - 8) | rng.integers(0, 1 << (bits - 8), n).astype(np.uint64)
    return ((v >> 1) | ((v & 1) << (bits - 1))).astype(BITS[dtype])


def dev(a):
    signed = np.int16 if a.dtype == np.uint16 else np.int32 if a.dtype == np.uint32 else a.dtype
    return torch.from_numpy(np.ascontiguousarray(a).view(signed)).cuda()


@pytest.mark.parametrize("pattern", ["spike", "head", "tail", "waves", "flat"])
@pytest.mark.parametrize("dtype", ["bf16", "fp16", "fp32"])
def test_bursts_of_words(dtype, pattern):
    import paper_2604_17172_amd as uz
    e = 2 if BITS[dtype] is np.uint16 else 4
    # whole rounds 0-3 past the loop's four, one element more and one less
    for block_bytes, n in [(65536, 65536 // e + 2048 + 1), (65536, 3 * 65536 // e + 1536 - 1), (8192, 5 * 8192 // e + 513),
                           (262144, 262144 // e + 512 * 7)]:
        x = tensor(dtype, n, pattern, block_bytes // e, seed=n)
        s = ref.compress(x, dtype, block_bytes)
        out, size = uz.compress(dev(x), block_bytes, dtype=dtype, check=True)
        assert np.array_equal(out[: int(size.item())].cpu().numpy(), s), (dtype, pattern, block_bytes, n)
        y, status = uz.decompress(dev(s), dtype, n)
        torch.cuda.synchronize()
        assert int(status.item()) == 0, (dtype, pattern, block_bytes, n)
        assert np.array_equal(y.cpu().numpy().view(BITS[dtype]), x), (dtype, pattern, block_bytes, n)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_bursts_in_the_fused_reduce(dtype):
    import paper_2604_17172_amd as uz
    e = 2 if BITS[dtype] is np.uint16 else 4
    n = 2 * 65536 // e + 1000
    xs = [tensor(dtype, n, p, 65536 // e, seed=i) for i, p in enumerate(["head", "tail", "waves"])]
    streams = [ref.compress(x, dtype, 65536) for x in xs]
    out, size, raw, status = uz.reduce_fused([dev(s) for s in streams], dtype, n, 65536)
    torch.cuda.synchronize()
    want_s, want_y = ref.reduce(streams, dtype, n, 65536)
    assert int(status.item()) == 0
    assert np.array_equal(raw.cpu().numpy().view(BITS[dtype]), want_y)
    assert np.array_equal(out[: int(size.item())].cpu().numpy(), want_s)


# Which decoder takes a call goes by its number of blocks on 256 compute units:
# two waves per block up to 768, one wave per block with the ring of table
# entries up to 3072, with the ring of plain words up to 4096, then with the
# ring of entries again; 16-bit types under a stream's table (here "sampled")
# and FP8 stay with the plain ring past 4096, and fp32 has it from 1409 on
# (for up to 256 MiB).  Chunk streams state their blocks, so small ones reach
# every line.
@pytest.mark.parametrize("pattern", ["head", "waves"])
@pytest.mark.parametrize("blocks", [768, 769, 1408, 1409, 3072, 3073, 4096, 4097])
@pytest.mark.parametrize("dtype", ["bf16", "fp16", "fp32"])
def test_chunk_decoders_by_blocks(dtype, blocks, pattern):
    import paper_2604_17172_amd as uz
    e = 2 if BITS[dtype] is np.uint16 else 4
    be = 8192 // e
    n = (blocks - 1) * be + be // 2 + 3
    x = tensor(dtype, n, pattern, be, seed=blocks)
    for mode in ("per_block", "sampled"):
        buf, slot, sizes, _ = uz.compress_chunked_table(dev(x), 8192, 8192 * 16, mode, dtype=dtype)
        y, status = uz.decompress_chunked(buf, slot, dtype, n, 8192, 8192 * 16, shared=mode == "sampled")
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and bool((sizes > 0).all()), (dtype, blocks, pattern, mode)
        assert np.array_equal(y.cpu().numpy().view(BITS[dtype]), x), (dtype, blocks, pattern, mode)


# One stream of up to 12 MiB goes to the kernel of two waves per block, which
# decodes more blocks than it has workgroups (768) one wave per block.
@pytest.mark.parametrize("mode", ["per_block", "sampled"])
@pytest.mark.parametrize("blocks", [767, 768, 769, 1537, 3072])
@pytest.mark.parametrize("dtype", ["bf16", "fp32", "e4m3fn"])
def test_stream_of_small_blocks(dtype, blocks, mode):
    import paper_2604_17172_amd as uz
    bits = "bf16" if dtype == "e4m3fn" else dtype
    be = 4096 // (4 if dtype == "fp32" else 2)
    n = (blocks - 1) * be + be // 2 + 3
    x = tensor(bits, n, "waves", be, seed=blocks)
    x[3 * be:5 * be] = np.random.Generator(np.random.PCG64(blocks)).integers(0, 1 << 16, 2 * be)  # STORED blocks
    s = ref.compress(x, dtype, 4096) if mode == "per_block" else ref.compress_table(x, dtype, 4096, mode)
    y, status = uz.decompress(dev(s), dtype, n) if mode == "per_block" else uz.decompress_table(dev(s), dtype, n)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert np.array_equal(y.cpu().numpy().view(BITS[bits]), x)


# One stream does not state its block size: where the plain ring may have its
# blocks (192 to 256 MiB, 16-bit types also twice, four times .. as much) two
# kernels are launched and its header says which decodes.
@pytest.mark.parametrize("block_bytes", [16384, 32768, 65536, 131072, 262144])
@pytest.mark.parametrize("dtype", ["bf16", "fp16", "fp32"])
def test_stream_decoders_by_size(dtype, block_bytes):
    import paper_2604_17172_amd as uz
    e = 2 if BITS[dtype] is np.uint16 else 4
    for size in (70 << 20, 200 << 20, 300 << 20, 400 << 20):
        n = size // e - 1234
        piece = tensor(dtype, 1 << 20, "waves", 65536 // e, seed=size)
        x = dev(np.tile(piece, n // piece.size + 1)[:n])
        out, _ = uz.compress(x, block_bytes, dtype=dtype, check=True)
        y, status = uz.decompress(out, dtype, n)
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and torch.equal(y, x), (dtype, block_bytes, size)
