"""More than 2^32 elements in one tensor: every element offset, value position and bitmap
word index in the kernels has to be 64-bit.  The tensor (8.6 GB of fp16) is made on the GPU
and checked there against definitions that PyTorch's own routines state independently:
nnz = count_nonzero, values = x[x != 0] (boolean indexing keeps index order), the bitmap's
bits by sampling words, and the round trip bit for bit.  The CPU oracle is applied to slices
(the first, the last and one across the 2^32 boundary)."""
import numpy as np
import pytest
import torch

from paper_2110_15362_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_tensor_of_more_than_2_to_32_elements(oracle):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (they never fall back to the CPU)")
    import paper_2110_15362_amd.bittrain as bt
    dev = "cuda"
    n = (1 << 32) + 3 * 16384 + 5
    g = torch.Generator(device=dev).manual_seed(99)
    x = torch.empty(n, dtype=torch.float16, device=dev)
    chunk = 1 << 28
    for lo in range(0, n, chunk):
        hi = min(n, lo + chunk)
        v = torch.randn(hi - lo, generator=g, device=dev)
        v[torch.rand(hi - lo, generator=g, device=dev) < 0.8] = 0.0          # 80 % zeros
        x[lo:hi] = v.to(torch.float16)
        del v
    words = (n + 31) // 32
    bitmap = torch.empty(words, dtype=torch.int32, device=dev)
    nnz_true = int(torch.count_nonzero(x.view(torch.int16)))
    values = torch.empty(nnz_true + 8, dtype=torch.float16, device=dev)
    values.view(torch.uint8).fill_(0x5A)
    nnz = torch.zeros(1, dtype=torch.int64, device=dev)
    tiles = bt.bt_index_bytes(n, torch.float16) // 8
    index = torch.empty(tiles, dtype=torch.int64, device=dev)
    ws = bt.new_workspace(n, torch.float16)
    bt.bt_compress_indexed(x, bitmap, values[:nnz_true], nnz, index, ws)
    torch.cuda.synchronize()
    assert int(nnz.item()) == nnz_true
    assert int((values[nnz_true:].view(torch.int16) != 0x5A5A).sum()) == 0, "wrote past values[nnz)"
    # values in index order, in slices to bound the temporaries
    pos = 0
    for lo in range(0, n, chunk):
        xs = x[lo:min(n, lo + chunk)].view(torch.int16)
        want = xs[xs != 0]
        assert torch.equal(values[pos:pos + want.numel()].view(torch.int16), want), lo
        pos += want.numel()
        del want
    assert pos == nnz_true
    # the tile index: cumulative counts at tile starts, at a sample of tiles including the last ones
    tile = bt.bt_tile_elems(torch.float16)
    idx = index.cpu().numpy()
    assert idx[0] == 0
    for t in (1, 2, 1000, (1 << 32) // tile - 1, (1 << 32) // tile, (1 << 32) // tile + 1, tiles - 2, tiles - 1):
        lo = max(0, t - 64)
        seg = int(torch.count_nonzero(x[lo * tile:t * tile].view(torch.int16)))
        assert idx[t] - idx[lo] == seg, t
    assert nnz_true - idx[tiles - 1] == int(torch.count_nonzero(x[(tiles - 1) * tile:].view(torch.int16)))
    # bitmap and values against the CPU oracle on three slices
    for lo, hi in ((0, 70016), ((1 << 32) - 32 * 1000, (1 << 32) + 32 * 1000), (n - 50021 - (n - 50021) % 32, n)):
        assert lo % 32 == 0
        xb = wl.bits(x[lo:hi].cpu())
        o_bitmap, o_values, o_nnz = oracle.compress(xb)
        got = bitmap[lo // 32:(hi + 31) // 32].cpu().numpy().view(np.uint32)
        assert np.array_equal(got, o_bitmap), (lo, hi)
        before = int(torch.count_nonzero(x[:lo].view(torch.int16))) if lo else 0
        assert np.array_equal(wl.bits(values[before:before + o_nnz].cpu()), o_values), (lo, hi)
    # both restorations, bit for bit
    out = torch.empty_like(x)
    bt.bt_decompress(bitmap, values[:nnz_true], out, ws)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), x.view(torch.int16))
    out.zero_()
    bt.bt_decompress_indexed(bitmap, values[:nnz_true], index, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), x.view(torch.int16))
    # ReLU backward in place on the big tensor: out = bit ? out : 0 leaves it unchanged where bits are set
    bt.bt_relu_backward_from_bitmap(bitmap, out, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), x.view(torch.int16))
    assert int(ws[8:12].cpu().numpy().view(np.uint32)[0]) == 0, "a bounded wait ran out"


def test_streams_of_more_than_one_launch():
    """ReLU with its bitmap and its backward, in place, on a little more than 32 GiB, which is where a second launch begins: every
    element against torch, in slices made again from their seeds."""
    import paper_2110_15362_amd.bittrain as bt
    n, chunk = (1 << 34) + 4101, 1 << 28
    bounds = [(lo, min(n, lo + chunk)) for lo in range(0, n, chunk)]

    def bits(seed, lo, hi):
        g = torch.Generator(device="cuda").manual_seed(seed + lo // chunk)
        return torch.randint(-(1 << 15), 1 << 15, (hi - lo,), generator=g, device="cuda", dtype=torch.int16)
    x = torch.empty(n, dtype=torch.int16, device="cuda")
    bitmap = torch.full(((n + 31) // 32 + 1,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    for lo, hi in bounds:
        x[lo:hi] = bits(1000, lo, hi)
    h = x.view(torch.bfloat16)
    bt.bt_relu_forward(h, h, bitmap[:-1])
    for lo, hi in bounds:
        assert torch.equal(x[lo:hi], torch.relu(bits(1000, lo, hi).view(torch.bfloat16)).view(torch.int16)), lo
        x[lo:hi] = bits(5000, lo, hi)
    bt.bt_relu_backward_from_bitmap(bitmap[:-1], h, h)
    for lo, hi in bounds:
        kept = torch.relu(bits(1000, lo, hi).view(torch.bfloat16)).view(torch.int16) != 0
        assert torch.equal(x[lo:hi], torch.where(kept, bits(5000, lo, hi), 0)), lo
    assert int(bitmap[-1].item()) == 0x5A5A5A5A
