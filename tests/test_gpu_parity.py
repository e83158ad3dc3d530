"""GPU parity: libbittrain (through its C ABI) against the CPU oracle, byte for byte.

Integer / bit work throughout, so the bar is exact equality of the bitmap, the
value array [0, nnz), nnz, the restored tensor and the ReLU-backward output."""
import numpy as np
import pytest
import torch

from paper_2110_15362_amd import workloads as wl

pytestmark = pytest.mark.gpu

DTYPES = ["f32", "f16", "bf16", "f64"]
# tile of eight rows = 8192 fp32 / 16384 16-bit / 4096 fp64 elements (small tensors: of two or four); wave strip = a quarter of it;
# row = 256 / 512 / 128
SIZES = [1, 3, 4, 5, 7, 8, 9, 31, 32, 33, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2049,
         4095, 4096, 4097, 8191, 8192, 8193, 12305, 16384, 3 * 8192 + 17, 100003, 5 * 8192, 1000000 + 37]


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (they never fall back to the CPU)")
    import paper_2110_15362_amd.bittrain as bt
    bt.lib()
    from tests import gpu_util
    return gpu_util


def _check_compress(gpu, oracle, x, **kw):
    xb = wl.bits(x)
    o_bitmap, o_values, o_nnz = oracle.compress(xb)
    bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, **kw)
    assert nnz == o_nnz
    assert np.array_equal(bitmap, o_bitmap)
    cap = kw.get("cap")
    written = o_nnz if cap is None else min(o_nnz, cap)
    assert np.array_equal(values[:written], o_values[:written])
    assert tail_ok, "wrote outside bitmap[0,W) or values[0,min(nnz,cap))"
    return o_bitmap, o_values, o_nnz


def _check_decompress(gpu, oracle, o_bitmap, o_values, n, dtype, expect_bits, **kw):
    out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, dtype, **kw)
    assert np.array_equal(out, oracle.decompress(o_bitmap, o_values, n))
    assert np.array_equal(out, expect_bits)
    assert guard_ok, "wrote past out[n)"


@pytest.mark.parametrize("dt", DTYPES)
def test_compress_sizes_and_tails(gpu, oracle, dt):
    for i, n in enumerate(SIZES):
        for zf in (0.5, 0.0, 1.0, 0.93):
            x = wl.random_sparse(n, dt, zf, seed=1000 + i)
            _check_compress(gpu, oracle, x)


@pytest.mark.parametrize("dt", DTYPES)
def test_decompress_sizes_and_tails(gpu, oracle, dt):
    for i, n in enumerate(SIZES):
        for zf in (0.5, 0.0, 1.0, 0.93):
            x = wl.random_sparse(n, dt, zf, seed=2000 + i)
            xb = wl.bits(x)
            o_bitmap, o_values, _ = oracle.compress(xb)
            _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, xb)


@pytest.mark.parametrize("dt", DTYPES)
def test_relu_backward_sizes_and_tails(gpu, oracle, dt):
    for i, n in enumerate(SIZES):
        x = torch.relu(wl.random_sparse(n, dt, 0.2, seed=3000 + i))
        g = wl.random_sparse(n, dt, 0.0, seed=4000 + i)
        o_bitmap, _, _ = oracle.compress(wl.bits(x))
        expect = oracle.relu_backward(o_bitmap, wl.bits(g))
        for inplace in (False, True):
            out, guard_ok = gpu.gpu_relu_backward(o_bitmap, g, inplace=inplace)
            assert np.array_equal(out, expect)
            assert guard_ok


@pytest.mark.parametrize("dt", DTYPES)
def test_special_bit_patterns(gpu, oracle, dt):
    """-0.0, denormals, NaN payloads and infinities are values; the round trip is bit exact."""
    base = wl.special_values(dt)
    x = base.repeat(700)[:11111]
    o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x)
    _check_decompress(gpu, oracle, o_bitmap, o_values, x.numel(), x.dtype, wl.bits(x))
    # ReLU backward is a select: NaN / Inf gradients under a cleared bit give +0
    g = base.flip(0).repeat(700)[:11111]
    out, guard_ok = gpu.gpu_relu_backward(o_bitmap, g)
    assert np.array_equal(out, oracle.relu_backward(o_bitmap, wl.bits(g))) and guard_ok


def test_single_nonzero_first_and_last(gpu, oracle):
    for n in (4096, 4097, 50000):
        for pos in (0, n - 1, n // 2):
            x = torch.zeros(n)
            x[pos] = -3.25
            o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x)
            assert o_nnz == 1
            _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x))


def test_values_capacity_is_respected(gpu, oracle):
    """nnz > values_cap: nothing beyond the capacity is written, bitmap and nnz are complete."""
    x = wl.random_sparse(70001, "f32", 0.5, seed=5)
    for cap in (0, 1, 1000, 17000, 34999):
        _check_compress(gpu, oracle, x, cap=cap)
    xh = wl.random_sparse(70001, "f16", 0.3, seed=6)
    for cap in (0, 3, 8191, 30001):
        _check_compress(gpu, oracle, xh, cap=cap)


@pytest.mark.parametrize("dt", DTYPES)
def test_values_pointer_only_element_aligned(gpu, oracle, dt):
    for off in (1, 2, 3, 5, 7):
        x = wl.random_sparse(40000 + off, dt, 0.4, seed=70 + off)
        o_bitmap, o_values, _ = _check_compress(gpu, oracle, x, values_offset=off)
        _check_decompress(gpu, oracle, o_bitmap, o_values, x.numel(), x.dtype, wl.bits(x), values_offset=off)


def test_workspace_reuse_across_calls_and_sizes(gpu, oracle):
    """One workspace, initialised once, serves many calls of different sizes and kinds
    (the kernels leave it ready for the next call)."""
    import paper_2110_15362_amd.bittrain as bt
    ws = bt.new_workspace(300000, torch.float32)
    for rep, n in enumerate([300000, 17, 4096, 250001, 8192, 1, 300000, 123457]):
        x = wl.random_sparse(n, "f32", 0.6, seed=900 + rep)
        o_bitmap, o_values, _ = _check_compress(gpu, oracle, x, ws=ws)
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x), ws=ws)
        xh = wl.random_sparse(n, "bf16", 0.6, seed=950 + rep)
        o_bitmap, o_values, _ = _check_compress(gpu, oracle, xh, ws=ws)
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, xh.dtype, wl.bits(xh), ws=ws)
    hdr = ws[:16].cpu().numpy().view(np.uint32)
    assert hdr[0] == 32          # calls completed on this workspace (8 sizes x 4 calls)
    assert hdr[2] == 0           # no tile ever gave up waiting for another tile's count


@pytest.mark.parametrize("dt", ["f32", "bf16", "f64"])
def test_tile_record_and_scan_window_boundaries(gpu, oracle, dt):
    """Sizes around the bookkeeping granularities: a tile (8192 fp32 / 16384 16-bit / 4096 fp64 elements), a scanner row (128
    tiles), the workspace's blocks and the launches without a scanner (256), the scanner's passes (256 and 384), and some between."""
    tile = {"f32": 8192, "bf16": 16384, "f64": 4096}[dt]
    sizes = []
    for tiles in (1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 383, 384, 385, 447, 448, 449, 511, 512, 513, 897, 1025):
        sizes += [tiles * tile - 1, tiles * tile, tiles * tile + 1]
    for i, n in enumerate(sizes):
        x = wl.random_sparse(n, dt, 0.5 if i % 3 else 0.97, seed=6000 + i)
        o_bitmap, o_values, _ = _check_compress(gpu, oracle, x)
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x))


def test_workspace_reuse_large_small_large(gpu, oracle):
    """What a call leaves in the workspace must never be mistaken for the next call's
    counts, whatever the order of sizes (more tiles, fewer tiles, more again)."""
    import paper_2110_15362_amd.bittrain as bt
    ws = bt.new_workspace(8192 * 1300, torch.float32)
    for rep, tiles in enumerate([1300, 3, 700, 1, 1299, 64, 65, 1300, 513]):
        n = 8192 * tiles - 5 * rep
        x = wl.random_sparse(n, "f32", 0.3 + 0.07 * rep, seed=7000 + rep)
        o_bitmap, o_values, _ = _check_compress(gpu, oracle, x, ws=ws)
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x), ws=ws)
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x), ws=ws)
    assert ws[:16].cpu().numpy().view(np.uint32)[2] == 0


def test_all_zero_and_all_nonzero_large(gpu, oracle):
    n = 8192 * 700 + 123
    for x in (torch.zeros(n), torch.full((n,), -1.5), torch.zeros(n, dtype=torch.float16),
              torch.full((n,), 0.25, dtype=torch.bfloat16)):
        o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x)
        assert o_nnz in (0, n)
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x))


def test_empty_tensor(gpu):
    import paper_2110_15362_amd.bittrain as bt
    dev = "cuda"
    x = torch.empty(0, device=dev)
    nnz = torch.full((1,), 99, dtype=torch.int64, device=dev)
    bitmap = torch.empty(0, dtype=torch.int32, device=dev)
    ws = bt.new_workspace(0, torch.float32)
    bt.bt_compress(x, bitmap, x, nnz, ws)
    bt.bt_decompress(bitmap, x, x, ws)
    bt.bt_relu_backward_from_bitmap(bitmap, x, x)
    torch.cuda.synchronize()
    assert int(nnz.item()) == 0


def test_config1(gpu, oracle):
    cfg = wl.config1()
    x, g = cfg["x"], cfg["grad"]
    o_bitmap, o_values, _ = _check_compress(gpu, oracle, x)
    _check_decompress(gpu, oracle, o_bitmap, o_values, x.numel(), x.dtype, wl.bits(x))
    out, ok = gpu.gpu_relu_backward(o_bitmap, g)
    assert np.array_equal(out, oracle.relu_backward(o_bitmap, wl.bits(g))) and ok


@pytest.mark.parametrize("z", [0.5, 0.7, 0.9])
def test_config2_full_size(gpu, oracle, z):
    x = wl.config2(z)["x"]
    o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x)
    assert abs(1 - o_nnz / x.numel() - z) < 1e-3
    _check_decompress(gpu, oracle, o_bitmap, o_values, x.numel(), x.dtype, wl.bits(x))
    g = torch.randn(x.numel(), generator=torch.Generator().manual_seed(12))
    out, ok = gpu.gpu_relu_backward(o_bitmap, g)
    assert np.array_equal(out, oracle.relu_backward(o_bitmap, wl.bits(g))) and ok


@pytest.mark.parametrize("variant", ["a", "b"])
def test_config3_full_size(gpu, oracle, variant):
    x = wl.config3(variant)["x"]
    o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x)
    assert abs(1 - o_nnz / x.numel() - 0.65) < 5e-3
    _check_decompress(gpu, oracle, o_bitmap, o_values, x.numel(), x.dtype, wl.bits(x))
    g = torch.randn(x.numel(), generator=torch.Generator().manual_seed(13)).to(torch.bfloat16)
    out, ok = gpu.gpu_relu_backward(o_bitmap, g)
    assert np.array_equal(out, oracle.relu_backward(o_bitmap, wl.bits(g))) and ok


def test_config4_resnet50_set_full_size(gpu, oracle):
    """All 49 tensors compressed in forward order with one workspace on one stream, then
    restored in reverse order; every bitmap, value array, nnz and restored tensor is compared."""
    import paper_2110_15362_amd.bittrain as bt
    dev = "cuda"
    shapes = wl.config4_shapes()
    n_max = max(int(np.prod(s)) for s in shapes)
    ws = bt.new_workspace(n_max, torch.float32)
    scratch = torch.empty(n_max, dtype=torch.float32, device=dev)      # worst-case value buffer
    nnz_d = torch.zeros(1, dtype=torch.int64, device=dev)
    stash, dense_bytes, comp_bytes = [], 0, 0
    for cfg in wl.config4_tensors():
        x = cfg["x"].reshape(-1)
        n = x.numel()
        o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x))
        xd = x.to(dev)
        bitmap = torch.empty((n + 31) // 32, dtype=torch.int32, device=dev)
        bt.bt_compress(xd, bitmap, scratch[:n], nnz_d, ws)
        nnz = int(nnz_d.item())
        assert nnz == o_nnz
        values = scratch[:nnz].clone()                                 # right-sized stash
        assert np.array_equal(bitmap.cpu().numpy().view(np.uint32), o_bitmap), cfg["name"]
        assert np.array_equal(wl.bits(values.cpu()), o_values), cfg["name"]
        stash.append((bitmap, values, n, o_nnz))
        dense_bytes += 4 * n
        comp_bytes += bt.bt_compressed_size(n, nnz, torch.float32)
        assert bt.bt_compressed_size(n, nnz, torch.float32) == oracle.compressed_size(n, o_nnz, 4)
    # backward sweep: regenerate the inputs (same seed) and walk them in reverse
    xs = [c["x"].reshape(-1) for c in wl.config4_tensors()]
    out = torch.empty(n_max, dtype=torch.float32, device=dev)
    for (bitmap, values, n, _), x in zip(reversed(stash), reversed(xs)):
        bt.bt_decompress(bitmap, values, out[:n], ws)
        assert np.array_equal(wl.bits(out[:n].cpu()), wl.bits(x))
    assert dense_bytes == 4 * 614957056
    saved = 1 - comp_bytes / dense_bytes
    assert 0.66 < saved < 0.68, saved        # 70 % zeros: 1 - (0.3 + 1/32)


@pytest.mark.parametrize("p", [0.05, 0.95])
def test_config5_full_size(gpu, oracle, p):
    x = wl.config5(p)["x"]
    n = x.numel()
    o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x)
    if p == 0.05:
        assert oracle.compressed_size(n, o_nnz, 2) > 2 * n      # the compressed form is larger
    _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x))


def test_repeated_calls_are_identical(gpu, oracle):
    """The grid scan is the only place where tiles talk to each other: 300 back-to-back
    calls on inputs with whole empty tiles must give the same bytes every time."""
    import paper_2110_15362_amd.bittrain as bt
    dev = "cuda"
    x = wl.config3("b", batch=1)["x"].reshape(-1)
    n = x.numel()
    o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x))
    xd = x.to(dev)
    ws = bt.new_workspace(n, x.dtype)
    bitmap = torch.empty((n + 31) // 32, dtype=torch.int32, device=dev)
    values = torch.empty(n, dtype=x.dtype, device=dev)
    out = torch.empty_like(xd)
    nnz = torch.zeros(1, dtype=torch.int64, device=dev)
    ref_bitmap = torch.from_numpy(o_bitmap.view(np.int32)).to(dev)
    ref_values = torch.from_numpy(o_values.view(np.int16)).to(dev)
    for it in range(300):
        bitmap.zero_(); values.zero_(); out.fill_(1.0)
        bt.bt_compress(xd, bitmap, values, nnz, ws)
        bt.bt_decompress(bitmap, values, out, ws)
        assert int(nnz.item()) == o_nnz
        assert torch.equal(bitmap, ref_bitmap)
        assert torch.equal(values[:o_nnz].view(torch.int16), ref_values)
        assert torch.equal(out.view(torch.int16), xd.view(torch.int16))


@pytest.mark.parametrize("dt", DTYPES)
def test_compress_tiles_around_the_staging_limit(gpu, oracle, dt):
    """A tile whose values fit the staging area is compacted into one run before its prefix is known, a fuller one in
    two phases per wave: numbers of kept elements around that limit, at every alignment of the value array, in front of and
    behind tiles of the other kind, whole and cut off by the capacity."""
    width = {"f32": 4, "f16": 2, "bf16": 2, "f64": 8}[dt]
    tile = 32768 // width
    limit = (160 * 1024 // 8 - 64 - 16) // width
    rng = np.random.RandomState(31 + width)

    def one(kept):
        x = torch.zeros(tile, dtype=wl.DTYPES[dt])
        at = torch.from_numpy(rng.permutation(tile)[:kept].copy())
        x[at] = wl.random_sparse(kept, dt, 0.0, seed=kept) if kept else x[at]
        return x
    for i, kept in enumerate([(limit,), (limit + 1,), (limit - 1, tile), (tile, limit), (tile - 1, limit + 1, 3, limit), (0, limit + 2)]):
        x = torch.cat([one(k) for k in kept] + [wl.random_sparse(777, dt, 0.5, seed=i)])
        nnz = int((torch.from_numpy(wl.bits(x).astype(np.int64)) != 0).sum())
        for offset in range(16 // width):
            _check_compress(gpu, oracle, x, values_offset=offset)
        for cap in (nnz // 2 + 1, nnz - 3, 5):
            _check_compress(gpu, oracle, x, cap=cap, values_offset=1)


def _plan_edges(width):
    """Numbers of elements around which the library changes how it launches a call on a small tensor: compression at 64 tiles
    of two rows, 256 of four and 256 of eight (a row is 4 KiB a tile), restoration at 256 of two and of four."""
    row = 4096 // width
    return sorted({tiles * rows * row + d for tiles, rows in ((1, 2), (64, 2), (256, 2), (256, 4), (256, 8)) for d in (-1, 0, 1)})


@pytest.mark.parametrize("dt", DTYPES)
def test_small_launches_at_the_edges_of_their_plans(gpu, oracle, dt):
    """Both directions on either side of every change of plan, all on one workspace and in an order that mixes the plans, so
    that each finds what another left there; misaligned values; pruning; the calls are counted."""
    import paper_2110_15362_amd.bittrain as bt
    sizes = _plan_edges({"f32": 4, "f16": 2, "bf16": 2, "f64": 8}[dt])
    ws = bt.new_workspace(max(sizes), wl.DTYPES[dt])
    calls = 0
    for i, n in enumerate(sizes[::2] + sizes[1::2][::-1]):
        x = wl.random_sparse(n, dt, (0.5, 0.1, 0.93)[i % 3], seed=600 + i)
        o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x, ws=ws, values_offset=i % 4)
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x), ws=ws, values_offset=(i + 1) % 4)
        p_bitmap, p_values, p_nnz = oracle.compress(oracle.prune(wl.bits(x), dt, 0.2))
        bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, ws=ws, threshold=0.2, cap=p_nnz // 2)
        assert tail_ok and nnz == p_nnz and np.array_equal(bitmap, p_bitmap) and np.array_equal(values, p_values[:p_nnz // 2])
        calls += 3
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    bt.bt_workspace_status(ws, status)
    assert status.tolist() == [0, calls]


def _small_plans(dt):
    """name -> a number of elements that takes it: the launches of compression without a scanner, and one with it."""
    row = 4096 // wl.DTYPES[dt].itemsize
    return {"two_rows": 40 * 2 * row - 5, "four_rows": 100 * 4 * row + 77, "eight_rows": 200 * 8 * row + 1, "scanner": 300 * 8 * row + 4321}


def _refused(gpu, x, o_bitmap, o_values, ws):
    """Both directions on a workspace that has failed: every output keeps the fill pattern."""
    n = x.numel()
    bitmap, values, nnz, _ = gpu.gpu_compress(x, ws=ws)
    assert nnz == -7 and (bitmap == 0x5A5A5A5A).all() and (values.view(np.uint8) == 0x5A).all(), n
    out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, x.dtype, ws=ws)
    assert guard_ok and (out.view(np.uint8) == 0x5A).all(), n


@pytest.mark.parametrize("dt", DTYPES)
@pytest.mark.parametrize("plan", ["two_rows", "four_rows", "eight_rows"])
def test_a_small_launch_whose_wait_runs_out_ends(gpu, oracle, dt, plan):
    """Forced from the host: the last tile of a launch without a scanner is told nothing and has one poll.  The call must end
    inside its buffers and say that it gave up; until bt_workspace_init nothing on that workspace writes anything, in either
    direction and at any size; afterwards it works again."""
    import paper_2110_15362_amd.bittrain as bt
    n = _small_plans(dt)[plan]
    x = wl.random_sparse(n, dt, 0.5, seed=77)
    ws = bt.new_workspace(max(_small_plans(dt).values()), x.dtype)
    words = ws.view(torch.int32)
    words[bt.BT_WS_MUTE_WORD], words[bt.BT_WS_WAIT_LIMIT_WORD], words[bt.BT_WS_PATIENCE_WORD] = 2, 1, 1
    with gpu.instrumented():
        bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, ws=ws)
    assert tail_ok and nnz == -7, "nnz of a failed call is not written"
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 1
    # (the error word is all that a refused call looks at: from here on the library's own build)
    for m in _small_plans(dt).values():
        y = wl.random_sparse(m, dt, 0.5, seed=78)
        o_bitmap, o_values, _ = oracle.compress(wl.bits(y))
        _refused(gpu, y, o_bitmap, o_values, ws)
    bt.bt_workspace_init(ws)
    assert not bool(words.any())
    o_bitmap, o_values, _ = _check_compress(gpu, oracle, x, ws=ws)
    _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x), ws=ws)


def _dense_moves():
    """(dtype, number of tiles) around the sizes where the dense output moves, and well beyond them."""
    edges = {"f32": 1000, "f64": 1000, "f16": 1280, "bf16": 1280}
    return [(dt, e + d) for dt, e in edges.items() for d in (-1, 0, 1)] + [("f64", 1279), ("f64", 1280), ("f64", 1281), ("f32", 1500)]


@pytest.mark.parametrize("dt,tiles", _dense_moves())
def test_activation_compress_around_the_size_where_the_dense_output_moves(gpu, oracle, dt, tiles):
    """Launches of up to 1000 tiles (16-bit elements: 1280) store the dense output before the prefixes are there, larger ones
    after: every type on both sides, with tiles that fit the staging area and tiles that don't."""
    import paper_2110_15362_amd.bittrain as bt
    tile = bt.bt_tile_elems(wl.DTYPES[dt])
    n = tiles * tile - 5
    x = wl.random_sparse(n, dt, 0.3, seed=tiles)
    x[5 * tile:9 * tile].abs_()                      # all of it survives: more than the staging area holds
    want = oracle.prune(wl.bits(x), dt, 0.0)
    o_bitmap, o_values, o_nnz = oracle.compress(want)
    for inplace in (False, True):
        xd = x.cuda()
        dense = xd if inplace else torch.empty_like(xd)
        bitmap = torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda")
        values, nnz = torch.empty_like(xd), torch.zeros(1, dtype=torch.int64, device="cuda")
        bt.bt_activation_compress(xd, 0.0, dense, bitmap, values, nnz, bt.new_workspace(n, x.dtype))
        torch.cuda.synchronize()
        assert int(nnz.item()) == o_nnz
        assert np.array_equal(wl.bits(dense.cpu()), want)
        assert np.array_equal(bitmap.cpu().numpy().view(np.uint32), o_bitmap)
        assert np.array_equal(wl.bits(values[:o_nnz].cpu()), o_values)


# ---- activation pruning fused into compression (Section 4.3) ------------------------------


def _check_compress_pruned(gpu, oracle, x, dt, thr, **kw):
    o_bitmap, o_values, o_nnz = oracle.compress_pruned(wl.bits(x), dt, thr)
    bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, threshold=thr, **kw)
    assert nnz == o_nnz
    assert np.array_equal(bitmap, o_bitmap)
    assert np.array_equal(values[:o_nnz], o_values)
    assert tail_ok
    return o_bitmap, o_values, o_nnz


@pytest.mark.parametrize("dt", DTYPES)
def test_compress_pruned_thresholds_and_tails(gpu, oracle, dt):
    """The paper's thresholds (0, 0.01, 0.05, 0.1) plus a negative and an infinite one, on
    pre-activation tensors (no ReLU applied), at sizes that cover tiles and ragged tails."""
    for i, n in enumerate([1, 7, 33, 4097, 8192, 8193, 16385, 3 * 16384 + 5, 100003, 600001]):
        x = wl.random_sparse(n, dt, 0.1, seed=8000 + i)      # N(0,1) with a few exact zeros
        for thr in (0.0, 0.01, 0.05, 0.1, -0.5, float("inf")):
            o_bitmap, o_values, o_nnz = _check_compress_pruned(gpu, oracle, x, dt, thr)
        # decompressing the threshold-0 form gives ReLU(x) bit for bit (ReLU(-0.0) = +0 here)
        o_bitmap, o_values, o_nnz = oracle.compress_pruned(wl.bits(x), dt, 0.0)
        relu_bits = wl.bits(torch.where(x.double() > 0, x, torch.zeros_like(x)))
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, relu_bits)


@pytest.mark.parametrize("dt", DTYPES)
def test_compress_pruned_special_values(gpu, oracle, dt):
    """Denormals, -0.0, infinities and NaNs against thresholds that are themselves tiny:
    the comparison is the IEEE single-precision one on both sides."""
    x = wl.special_values(dt).repeat(1100)[:17000]
    tiny = {"f32": 1e-45, "f16": 6e-8, "bf16": 1e-40, "f64": 1e-45}[dt]
    for thr in (0.0, tiny, -tiny, 1.0, float("-inf"), float("nan")):
        _check_compress_pruned(gpu, oracle, x, dt, thr)


def test_compress_pruned_config2_full_size(gpu, oracle):
    x = wl.config2(0.5)["base"]                      # the pre-activation draw: N(0,1), no zeros
    for thr in (0.0, 0.1):
        o_bitmap, o_values, o_nnz = _check_compress_pruned(gpu, oracle, x, "f32", thr)
        assert abs(o_nnz / x.numel() - (0.5 if thr == 0.0 else 0.4602)) < 2e-3


@pytest.mark.parametrize("dt", DTYPES)
def test_mask_apply_with_a_foreign_bitmap(gpu, oracle, dt):
    """Double mask: the bitmap of one tensor (a normalisation layer's input) applied to another
    (its output); out of place and in place; the result compresses to the same bitmap."""
    import paper_2110_15362_amd.bittrain as bt
    for k, n in enumerate((1, 33, 8191, 8193, 3 * 16384 + 5, 1000003)):
        src = wl.random_sparse(n, dt, 0.6, 900 + k)
        y = torch.randn(n, generator=torch.Generator().manual_seed(950 + k)).to(src.dtype)   # dense, like a BN output
        bitmap, _, nnz = oracle.compress(wl.bits(src))
        want = oracle.mask_apply(bitmap, wl.bits(y))
        for inplace in (False, True):
            out, ok = gpu.gpu_relu_backward(bitmap, y, inplace=inplace, call=bt.bt_mask_apply)
            assert ok and np.array_equal(out, want), (n, inplace)
        got_bitmap, _, got_nnz, ok = gpu.gpu_compress(torch.from_numpy(want.view({2: np.int16, 4: np.int32, 8: np.int64}[want.itemsize])).view(src.dtype))
        y_nonzero_under_mask = int(((wl.bits(y) != 0) & (wl.bits(src) != 0)).sum())
        assert ok and got_nnz == y_nonzero_under_mask and got_nnz <= nnz


def test_a_wait_that_runs_out_ends_the_kernel_and_raises_the_flag(gpu, oracle):
    """Failure path, forced from the host: with the wait limit of the workspace set to one pass, the grid scan
    gives up on a tensor that needs two.  The kernels must still end, stay inside their buffers and leave the
    error word set; after bt_workspace_init the workspace works again."""
    import paper_2110_15362_amd.bittrain as bt
    n = 600 * 8192 + 77
    x = wl.random_sparse(n, "f32", 0.5, seed=31337)
    ws = bt.new_workspace(n, torch.float32)
    words = ws.view(torch.int32)
    words[bt.BT_WS_WAIT_LIMIT_WORD] = 1            # one pass of the scan
    bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, ws=ws)          # synchronises; returns at all
    assert tail_ok, "wrote outside bitmap[0,W) or values[0,min(nnz,cap))"
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 1
    status = torch.zeros(2, dtype=torch.int32, device="cuda")
    bt.bt_workspace_status(ws, status)
    assert int(status[0].item()) == 1
    o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x))
    # a later call on the failed workspace writes nothing: the output keeps the test's fill pattern
    out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, torch.float32, ws=ws)
    assert guard_ok and int(words[bt.BT_WS_ERROR_WORD].item()) == 1
    assert (out == 0x5A5A5A5A).all()
    # whatever a failing call reports as nnz, nothing at or beyond the capacity is written
    bt.bt_workspace_init(ws)
    words[bt.BT_WS_WAIT_LIMIT_WORD] = 1
    cap, guard = n // 8, 4096
    xd = x.cuda()
    vbuf = torch.full((cap + guard,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    bm = torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda")
    nnz_d = torch.zeros(1, dtype=torch.int64, device="cuda")
    bt.bt_compress(xd, bm, vbuf[:cap].view(torch.float32), nnz_d, ws)
    torch.cuda.synchronize()
    assert bool((vbuf[cap:] == 0x5A5A5A5A).all()), "wrote at or beyond the capacity"
    bt.bt_workspace_init(ws)
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 0 and int(words[bt.BT_WS_WAIT_LIMIT_WORD].item()) == 0
    _check_compress(gpu, oracle, x, ws=ws)
    _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x), ws=ws)
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 0


@pytest.mark.parametrize("dt", DTYPES)
@pytest.mark.parametrize("plan", ["two_rows", "four_rows", "eight_rows", "scanner"])
def test_compression_that_stops_waiting_counts_the_input_itself(gpu, oracle, dt, plan):
    """Forced from the host: no tile but the one that ends the call is told anything and their patience is a poll (looked at
    every 256th), so every workgroup stops waiting and counts the kept elements before its tile itself, with its values already
    compacted: in launches with and without a scanner, in tiles that fit the staging area and tiles that don't, with pruning and
    with a dense output on top of the input.  Every output must be right all the same, and nothing has failed."""
    with gpu.instrumented():
        _stops_waiting(gpu, oracle, dt, plan)


def _stops_waiting(gpu, oracle, dt, plan):
    import paper_2110_15362_amd.bittrain as bt
    n = _small_plans(dt)[plan]
    tile = bt.bt_tile_elems(wl.DTYPES[dt])
    x = wl.random_sparse(n, dt, 0.6, seed=98)
    full = slice(n // 3, n // 3 + min(3 * tile, n // 3))
    x[full] = wl.random_sparse(full.stop - full.start, dt, 0.0, seed=97).abs()
    ws = bt.new_workspace(n, x.dtype)
    words = ws.view(torch.int32)
    words[bt.BT_WS_MUTE_WORD], words[bt.BT_WS_PATIENCE_WORD] = 1, 1
    _check_compress(gpu, oracle, x, ws=ws)
    want = oracle.prune(wl.bits(x), dt, 0.25)
    o_bitmap, o_values, o_nnz = oracle.compress(want)
    bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, ws=ws, threshold=0.25)
    assert tail_ok and nnz == o_nnz
    assert np.array_equal(bitmap, o_bitmap) and np.array_equal(values[:o_nnz], o_values)
    for inplace in (False, True):
        xd = x.cuda()
        dense = xd if inplace else torch.empty_like(xd)
        bitmap, values = torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda"), torch.empty_like(xd)
        nnz = torch.zeros(1, dtype=torch.int64, device="cuda")
        bt.bt_activation_compress(xd, 0.25, dense, bitmap, values, nnz, ws)
        assert int(nnz.item()) == o_nnz and np.array_equal(wl.bits(dense.cpu()), want)
        assert np.array_equal(bitmap.cpu().numpy().view(np.uint32), o_bitmap)
        assert np.array_equal(wl.bits(values[:o_nnz].cpu()), o_values)
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 0 and int(words[0].item()) == 4
    assert words[[bt.BT_WS_MUTE_WORD, bt.BT_WS_PATIENCE_WORD]].tolist() == [1, 1]      # the kernels leave the caller's words alone


@pytest.mark.parametrize("dt", DTYPES)
def test_restoration_that_stops_waiting_counts_the_bitmap_itself(gpu, oracle, dt):
    """Forced from the host: no tile is told its offset and their patience is a poll (looked at every 256th), so every restoring
    workgroup stops waiting and counts the set bits before its tile itself.  The output must be right all the same, and nothing
    has failed.  (More than 256 tiles of four rows: smaller tensors are restored without waiting for anything.)"""
    import paper_2110_15362_amd.bittrain as bt
    n = 150 * bt.bt_tile_elems(wl.DTYPES[dt]) + 4321
    x = wl.random_sparse(n, dt, 0.6, seed=99)
    o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x))
    ws = bt.new_workspace(n, x.dtype)
    words = ws.view(torch.int32)
    words[bt.BT_WS_MUTE_WORD], words[bt.BT_WS_PATIENCE_WORD] = 1, 1
    with gpu.instrumented():
        for _ in range(2):
            out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, x.dtype, ws=ws)
            assert guard_ok
            assert np.array_equal(out, wl.bits(x))
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 0 and int(words[0].item()) == 2


@pytest.mark.parametrize("dt", DTYPES)
def test_wide_prefix_entries_give_the_same_results(gpu, oracle, dt):
    """Forced from the host: the scanner of a call on one tensor writes 8-byte entries (what it does by itself only
    once the offsets reach 2^32) instead of pairs of lower halves.  Several passes of the scanner, a ragged last tile;
    compression and restoration, two calls in a row on the same workspace."""
    import paper_2110_15362_amd.bittrain as bt
    n = 1100 * bt.bt_tile_elems(wl.DTYPES[dt]) + 77
    x = wl.random_sparse(n, dt, 0.55, seed=123)
    ws = bt.new_workspace(n, x.dtype)
    ws.view(torch.int32)[bt.BT_WS_WIDE_WORD] = 1
    o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x))
    for _ in range(2):
        bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, ws=ws)
        assert tail_ok and nnz == o_nnz
        assert np.array_equal(bitmap, o_bitmap) and np.array_equal(values[:o_nnz], o_values)
        out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, x.dtype, ws=ws)
        assert guard_ok and np.array_equal(out, wl.bits(x))
    assert int(ws.view(torch.int32)[bt.BT_WS_ERROR_WORD].item()) == 0
    assert int(ws.view(torch.int32)[bt.BT_WS_WIDE_WORD].item()) == 1      # the kernels leave the caller's words alone


def test_stream_probe_stays_inside_its_buffers(gpu):
    """The benchmark's plain stream reads tiles * read_rows * 4 KiB and writes tiles * write_rows * 4 KiB, no more."""
    from paper_2110_15362_amd import bench_aids as bt
    tiles = 777
    for r, w in ((8, 4), (4, 8), (8, 8), (8, 0), (0, 8)):
        src = torch.arange(tiles * max(r, 1) * 1024, dtype=torch.int32, device="cuda")
        guard = 4096
        dst = torch.full((max(tiles * w * 1024, 4 * tiles) + guard,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        bt.bt_stream_probe(src, dst[:dst.numel() - guard], tiles, r, w)
        torch.cuda.synchronize()
        assert bool((dst[dst.numel() - guard:] == 0x5A5A5A5A).all()), (r, w)
        if w:
            assert not bool((dst[:tiles * w * 1024] == 0x5A5A5A5A).all()), (r, w)


@pytest.mark.parametrize("dt", DTYPES)
def test_activation_compress_dense_and_stash_in_one_pass(gpu, oracle, dt):
    """bt_activation_compress: the dense pruned tensor equals the oracle's pruning, the compressed form
    equals Algorithm 1 on it; out of place and in place; ReLU for threshold 0."""
    import paper_2110_15362_amd.bittrain as bt
    dev = "cuda"
    for i, n in enumerate([1, 33, 4097, 8193, 3 * 16384 + 5, 100003, 600001]):
        x = wl.random_sparse(n, dt, 0.1, seed=8500 + i)
        if n > 100:
            x[:16] = wl.special_values(dt)
        xb = wl.bits(x)
        for thr in (0.0, 0.05, -0.5):
            want_dense = oracle.prune(xb, dt, thr)
            o_bitmap, o_values, o_nnz = oracle.compress(want_dense)
            for inplace in (False, True):
                pad = 16 // x.element_size()
                xd = x.to(dev)
                dbuf = xd if inplace else torch.empty(n + pad, dtype=x.dtype, device=dev)
                if not inplace:
                    dbuf.view(torch.uint8).fill_(0x5A)
                dense = xd if inplace else dbuf[:n]
                words = (n + 31) // 32
                bitmap = torch.full((words + 4,), 0x5A5A5A5A, dtype=torch.int32, device=dev)
                values = torch.empty(n + 8, dtype=x.dtype, device=dev)
                values.view(torch.uint8).fill_(0x5A)
                nnz = torch.full((1,), -7, dtype=torch.int64, device=dev)
                ws = bt.new_workspace(n, x.dtype)
                bt.bt_activation_compress(xd, thr, dense, bitmap[:words], values[:n], nnz, ws)
                torch.cuda.synchronize()
                assert int(nnz.item()) == o_nnz, (n, thr, inplace)
                assert np.array_equal(wl.bits(dense.cpu()), want_dense), (n, thr, inplace)
                assert np.array_equal(bitmap[:words].cpu().numpy().view(np.uint32), o_bitmap)
                assert np.array_equal(wl.bits(values[:o_nnz].cpu()), o_values)
                sent = np.frombuffer(bytes([0x5A] * x.element_size()), dtype=wl.bits(values.cpu()).dtype)[0]
                assert (wl.bits(values[o_nnz:].cpu()) == sent).all() and bool((bitmap[words:] == 0x5A5A5A5A).all())
                if not inplace:
                    assert (wl.bits(dbuf[n:].cpu()) == sent).all(), "wrote past dense[n)"
    # threshold 0 on pre-activations is ReLU
    x = wl.random_sparse(50000, "f32", 0.0, seed=8600)
    xd = x.to(dev)
    y = torch.empty_like(xd)
    bitmap = torch.empty((50000 + 31) // 32, dtype=torch.int32, device=dev)
    values = torch.empty(50000, device=dev)
    nnz = torch.zeros(1, dtype=torch.int64, device=dev)
    bt.bt_activation_compress(xd, 0.0, y, bitmap, values, nnz, bt.new_workspace(50000, torch.float32))
    torch.cuda.synchronize()
    assert torch.equal(y, torch.relu(xd))


@pytest.mark.parametrize("dt", ["f32", "bf16", "f64"])
def test_bitmap_bits_beyond_n_are_ignored(gpu, oracle, dt):
    """A bitmap whose last word carries set bits at positions >= n (not what bt_compress writes, but allowed
    on input): Algorithm 2 and the select run over the n valid bits only."""
    import paper_2110_15362_amd.bittrain as bt
    # the last two: restored in tiles of four rows, and of eight behind the scanner
    for n in (5, 33, 8191, 3 * 16384 + 7, 100001, 70 * bt.bt_tile_elems(wl.DTYPES[dt]) + 9, 300 * bt.bt_tile_elems(wl.DTYPES[dt]) + 7):
        x = wl.random_sparse(n, dt, 0.5, seed=9100 + n % 97)
        o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x))
        dirty = o_bitmap.copy()
        dirty[-1] |= np.uint32((0xFFFFFFFF << (n % 32)) & 0xFFFFFFFF)          # n % 32 != 0 for these sizes
        assert not np.array_equal(dirty, o_bitmap)
        out, ok = gpu.gpu_decompress(dirty, o_values, n, x.dtype)
        assert ok and np.array_equal(out, wl.bits(x))
        g = torch.randn(n, generator=torch.Generator().manual_seed(n)).to(x.dtype)
        got, ok = gpu.gpu_relu_backward(dirty, g)
        assert ok and np.array_equal(got, oracle.relu_backward(o_bitmap, wl.bits(g)))
        # the indexed restoration too
        tile = bt.bt_tile_elems(x.dtype)
        index = torch.from_numpy(oracle.tile_index(o_bitmap, n, tile).view(np.int64).copy()).cuda()
        bm = torch.from_numpy(dirty.view(np.int32).copy()).cuda()
        vals = x[x.view({2: torch.int16, 4: torch.int32, 8: torch.int64}[x.element_size()]) != 0].cuda()
        outd = torch.empty(n, dtype=x.dtype, device="cuda")
        bt.bt_decompress_indexed(bm, vals, index, outd)
        torch.cuda.synchronize()
        assert np.array_equal(wl.bits(outd.cpu()), wl.bits(x))


def test_two_streams_with_their_own_workspaces(gpu, oracle):
    """Calls that use distinct workspaces are independent: two streams (default priority) compress and
    restore different tensors at the same time, several times over."""
    import paper_2110_15362_amd.bittrain as bt
    dev = "cuda"
    xs = [wl.random_sparse(n, "f32", z, seed=9300 + k) for k, (n, z) in enumerate(((300 * 8192 + 5, 0.5), (170 * 8192 + 9, 0.8)))]
    want = [oracle.compress(wl.bits(x)) for x in xs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    bufs = []
    for x in xs:
        n = x.numel()
        bufs.append(dict(x=x.to(dev), bitmap=torch.empty((n + 31) // 32, dtype=torch.int32, device=dev),
                         values=torch.empty(n, device=dev), out=torch.empty(n, device=dev),
                         nnz=torch.zeros(1, dtype=torch.int64, device=dev), ws=bt.new_workspace(n, torch.float32)))
    torch.cuda.synchronize()
    for rep in range(5):
        for b in bufs:
            b["values"].fill_(7); b["out"].fill_(7); b["bitmap"].fill_(-1)
        torch.cuda.synchronize()
        for s, b in zip(streams, bufs):
            with torch.cuda.stream(s):
                for _ in range(3):
                    bt.bt_compress(b["x"], b["bitmap"], b["values"], b["nnz"], b["ws"])
                    bt.bt_decompress(b["bitmap"], b["values"], b["out"], b["ws"])
        torch.cuda.synchronize()
        for b, x, (o_bitmap, o_values, o_nnz) in zip(bufs, xs, want):
            assert int(b["nnz"].item()) == o_nnz
            assert np.array_equal(b["bitmap"].cpu().numpy().view(np.uint32), o_bitmap)
            assert np.array_equal(wl.bits(b["values"][:o_nnz].cpu()), o_values)
            assert np.array_equal(wl.bits(b["out"].cpu()), wl.bits(x))
            assert int(b["ws"].view(torch.int32)[2].item()) == 0


def _pattern_masks(n, tile):
    """Zero / non-zero layouts whose run lengths sit on, just before and just after the sizes the kernels
    work in: a 16-byte vector, a bitmap word, a wave row, a wave's strip and a tile of eight rows, and those of two
    (a sixteenth and a quarter of the large tile, the latter also the strip of eight rows)."""
    i = np.arange(n)
    row, small_strip, strip = tile // 32, tile // 16, tile // 4
    masks = {"alternate": i % 2 == 0, "every_32nd": i % 32 == 31, "every_33rd": i % 33 == 0,
             "first_of_each_word_missing": i % 32 != 0, "dense_then_empty": i < n // 2, "empty_then_dense": i >= n // 2,
             "only_the_last_tile": i >= (n // tile) * tile, "only_the_last_element": i == n - 1}
    for name, period in (("row", row), ("small_strip", small_strip), ("strip", strip), ("tile", tile)):
        masks["every_other_%s" % name] = (i // period) % 2 == 0
        masks["runs_of_%s_minus_1" % name] = (i // (period - 1)) % 2 == 1
        masks["runs_of_%s_plus_1" % name] = (i // (period + 1)) % 2 == 1
        masks["one_per_%s" % name] = i % period == period - 1
    rng = np.random.default_rng(17)
    for block in (3, 64, 1000):
        masks["random_blocks_of_%d" % block] = np.repeat(rng.random(n // block + 1) < 0.4, block)[:n]
    return masks


@pytest.mark.parametrize("tiles", [3, 70, 200, 260])
@pytest.mark.parametrize("dt", ["f32", "f16", "f64"])
def test_structured_zero_patterns(gpu, oracle, dt, tiles):
    """The ranks, the scatter through LDS and the tile offsets depend on where the zeros are, not
    only on how many there are: run lengths on and around every internal size, in tensors that are compressed in tiles of two, four
    and eight rows and in eight with the scanner, and restored in two, four and (twice) in eight."""
    tile = {"f32": 8192, "f16": 16384, "f64": 4096}[dt]
    n = tiles * tile + tile // 4 + 37
    base = wl.random_sparse(n, dt, 0.0, 23)                    # no zeros: every kept element is distinct enough
    base[base == 0] = 0.5                                      # (a draw can be too small for a half)
    g = wl.random_sparse(n, dt, 0.0, 24)
    assert int((wl.bits(base) == 0).sum()) == 0
    for name, keep in _pattern_masks(n, tile).items():
        x = base.clone()
        x[torch.from_numpy(~keep)] = 0
        o_bitmap, o_values, o_nnz = _check_compress(gpu, oracle, x)
        assert o_nnz == int(keep.sum()), name
        _check_decompress(gpu, oracle, o_bitmap, o_values, n, x.dtype, wl.bits(x))
        out, guard_ok = gpu.gpu_relu_backward(o_bitmap, g)
        assert np.array_equal(out, oracle.relu_backward(o_bitmap, wl.bits(g))) and guard_ok, name


@pytest.mark.parametrize("dt", ["f32", "bf16", "f64"])
def test_relu_backward_around_the_largest_gradient_read_through_the_caches(gpu, dt):
    """Gradients of up to 48 MiB are read with plain loads, larger ones past the caches: the last of the one kind and the first
    of the other, with ragged ends, against torch on the device."""
    from paper_2110_15362_amd import bittrain as bt
    dtype = wl.DTYPES[dt]
    wide = {2: torch.int16, 4: torch.int32, 8: torch.int64}[dtype.itemsize]
    last = (48 << 20) // dtype.itemsize
    g = torch.Generator(device="cuda").manual_seed(9)
    words = torch.randint(-(1 << 31), 1 << 31, ((last + 5) // 32 + 1,), generator=g, device="cuda").to(torch.int32)
    grad = torch.randint(-(1 << 15), 1 << 15, (last + 5,), generator=g, device="cuda").to(wide)
    keep = ((words[:, None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1).reshape(-1).bool()
    for n in (last - 3, last, last + 1, last + 5):
        out = torch.full((n + 4,), 0x5A, dtype=wide, device="cuda")
        bt.bt_relu_backward_from_bitmap(words, grad[:n].view(dtype), out[:n].view(dtype))
        assert torch.equal(out[:n], torch.where(keep[:n], grad[:n], 0)), n
        assert bool((out[n:] == 0x5A).all()), n


def test_binding_sees_the_same_in_every_kind_of_tensor(gpu, oracle):
    """Ordinary tensors and parameters are read through the tensor object, everything else through Python: the same results on
    the same stream, the same refusals, and a function mode still sees what is asked of the tensors."""
    from torch.overrides import TorchFunctionMode

    from paper_2110_15362_amd import bittrain as bt

    class Sub(torch.Tensor):
        pass

    class Mode(TorchFunctionMode):
        def __init__(self):
            super().__init__()
            self.seen = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.seen += 1
            return func(*args, **(kwargs or {}))
    n = 70001
    x = wl.random_sparse(n, "f32", 0.5, 77).cuda()
    o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x.cpu()))
    bitmap = torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda")
    values, out = torch.empty_like(x), torch.empty_like(x)
    nnz = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = bt.new_workspace(n, x.dtype)
    side, mode = torch.cuda.Stream(), Mode()

    def both(t, o, stream=None):
        bitmap.zero_(), values.zero_(), out.zero_(), nnz.zero_()
        torch.cuda.synchronize()
        bt.bt_compress(t, bitmap, values, nnz, ws, stream=stream)
        bt.bt_decompress(bitmap, values, o, ws, stream=stream)
        torch.cuda.synchronize()
        assert int(nnz.item()) == o_nnz and np.array_equal(bitmap.cpu().numpy().view(np.uint32), o_bitmap)
        assert np.array_equal(wl.bits(values.cpu())[:o_nnz], o_values) and torch.equal(out, x)
    both(x, out)
    both(torch.nn.Parameter(x), out)
    both(x.as_subclass(Sub), out.as_subclass(Sub))
    both(x, out, side)
    with torch.cuda.stream(side):
        both(x, out)
    with torch.inference_mode():
        both(x.clone(), out)
    with mode:
        bt.bt_relu_backward_from_bitmap(bitmap, x, out)
    assert mode.seen >= 18      # six looks at each of three tensors
    for kind in (lambda t: t, lambda t: t.as_subclass(Sub)):
        for bad, error in ((x[::2], "contiguous"), (x.cpu(), "device memory"), (x.half(), "dtype"), (x.to(torch.int32), "dtype")):
            with pytest.raises((ValueError, TypeError), match=error):
                bt.bt_decompress(bitmap, values, kind(bad), ws)
        with pytest.raises(TypeError, match="not torch.int32"):
            bt.bt_compress(kind(x.to(torch.int32)), bitmap, kind(values.to(torch.int32)), nnz, ws)
    with pytest.raises(RuntimeError):      # a batched tensor has no address
        torch.func.vmap(lambda t: (bt.bt_relu_backward_from_bitmap(bitmap, t, t), t)[1])(x.reshape(1, -1))


@pytest.mark.parametrize("dt", DTYPES)
@pytest.mark.parametrize("rows,tiles", [(2, 3), (4, 70), (8, 200), (8, 261)])
def test_last_tiles_that_end_anywhere(gpu, oracle, dt, rows, tiles):
    """The last tile of a tensor, in every plan (tiles of two and four rows, of eight without and with a grid scan), ending around
    vectors, rows, waves' quarters and the tile: compressed, pruned with a threshold below zero (nothing beyond the end is kept,
    although what lies there in memory would be), with a dense output beside, restored."""
    import paper_2110_15362_amd.bittrain as bt
    dtype = wl.DTYPES[dt]
    vec, row = 16 // dtype.itemsize, 1024 // dtype.itemsize
    quarter, tile = rows * row, 4 * rows * row
    whole = tiles * tile
    ws = bt.new_workspace(whole + tile, dtype)
    for i, r in enumerate((1, vec - 1, vec, vec + 1, 2 * vec + 1, row - 1, row, row + 1, quarter - 1, quarter, quarter + vec + 1, 3 * quarter + 5, tile - 1)):
        n = whole + r
        x = wl.random_sparse(n, dt, 0.4, seed=9100 + i)
        buf = torch.ones(n + 64, dtype=dtype, device="cuda")      # what a read beyond the end would find
        buf[:n] = x.cuda()
        want = wl.bits(x)
        for call in ("compress", "pruned", "activation"):
            if call == "pruned":
                want = oracle.prune(want, dt, -0.5)
            o_bitmap, o_values, o_nnz = oracle.compress(want)
            bitmap = torch.full((o_bitmap.size + 2,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            values, dense = torch.zeros(n, dtype=dtype, device="cuda"), torch.full((n + 64,), 7, dtype=dtype, device="cuda")
            nnz = torch.zeros(1, dtype=torch.int64, device="cuda")
            if call == "compress":
                bt.bt_compress(buf[:n], bitmap[:o_bitmap.size], values, nnz, ws)
            elif call == "pruned":
                bt.bt_compress_pruned(buf[:n], -0.5, bitmap[:o_bitmap.size], values, nnz, ws)
            else:
                bt.bt_activation_compress(buf[:n], -0.5, dense[:n], bitmap[:o_bitmap.size], values, nnz, ws)
            if call != "activation":
                bt.bt_decompress(bitmap[:o_bitmap.size], values, dense[:n], ws)
            torch.cuda.synchronize()
            assert int(nnz.item()) == o_nnz, (n, call)
            assert np.array_equal(bitmap.cpu().numpy().view(np.uint32)[:-2], o_bitmap) and bool((bitmap[-2:] == 0x5A5A5A5A).all()), (n, call)
            assert np.array_equal(wl.bits(values[:o_nnz].cpu()), o_values[:o_nnz]), (n, call)
            assert np.array_equal(wl.bits(dense[:n].cpu()), want) and bool((dense[n:] == 7).all()), (n, call)
