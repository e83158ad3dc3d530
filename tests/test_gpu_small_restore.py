"""bt_decompress at the sizes where its launches change (tiles of two rows, eight waves a tile, the scanner), with values off every
16-byte boundary and ragged ends, against the CPU oracle, byte for byte; and tiles of the scanner's launches that stop waiting for it."""
import numpy as np
import pytest
import torch

from paper_2110_15362_amd import workloads as wl
from tests import gpu_util as gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bt():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (they never fall back to the CPU)")
    import paper_2110_15362_amd.bittrain as bt
    bt.lib()
    return bt


def _check(bt, oracle, dt, n, zeros, seed, ws, offset):
    x = wl.random_sparse(n, dt, zeros, seed)
    o_bitmap, o_values, _ = oracle.compress(wl.bits(x))
    out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, x.dtype, ws=ws, values_offset=offset)
    assert guard_ok and np.array_equal(out, wl.bits(x)), (dt, n)


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16", "f64"])
def test_sizes_on_both_sides_of_every_line(bt, oracle, dt):
    width = wl.DTYPES[dt].itemsize
    two, eight = 320 * 2 * 4096 // width, 32768 // width      # elements of 320 tiles of two rows; of a tile of eight waves
    last = 1 << 21 if width == 2 else 7 << 18
    sizes = [two - 1, two, two + 1, two + eight - 3, (two // eight + 5) * eight, 3 * two // 2 + 31, last - eight, last - 1, last, last + 1, last + 2 * eight + 77]
    ws = bt.new_workspace(max(sizes), wl.DTYPES[dt])
    for i, n in enumerate(sizes):
        _check(bt, oracle, dt, n, (0.5, 0.03, 0.97, 1.0, 0.0)[i % 5], 700 + i, ws, i % 5)
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    bt.bt_workspace_status(ws, status)
    assert status.tolist() == [0, len(sizes)]


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16", "f64"])
def test_launches_whose_waves_read_a_quarter_of_the_counts(bt, oracle, dt):
    tile = bt.bt_tile_elems(wl.DTYPES[dt])
    sizes = [257 * tile, 256 * tile, 512 * tile, 256 * tile + 1, 512 * tile + 1, 511 * tile + 3, 384 * tile - 29]
    ws = bt.new_workspace(max(sizes), wl.DTYPES[dt])
    for i, n in enumerate(sizes):
        _check(bt, oracle, dt, n, (0.5, 0.03, 0.97)[i % 3], 800 + i, ws, i % 4)
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    bt.bt_workspace_status(ws, status)
    assert status.tolist() == [0, len(sizes)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_a_launch_whose_last_tile_gives_up_says_so(bt, oracle, dt):
    """The limit of one poll fails every such call; what it writes stays inside its buffers, and the workspace works again once initialised."""
    n = 260 * bt.bt_tile_elems(wl.DTYPES[dt]) + 5
    x = wl.random_sparse(n, dt, 0.5, 4)
    o_bitmap, o_values, _ = oracle.compress(wl.bits(x))
    ws = bt.new_workspace(n, x.dtype)
    words = ws.view(torch.int32)
    words[bt.BT_WS_WAIT_LIMIT_WORD] = 1
    _, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, x.dtype, ws=ws)
    assert guard_ok and int(words[bt.BT_WS_ERROR_WORD].item()) == 1
    out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, x.dtype, ws=ws)
    assert guard_ok and (out.view(np.uint8) == gpu.SENTINEL).all()
    bt.bt_workspace_init(ws)
    _check(bt, oracle, dt, n, 0.5, 5, ws, 1)


# without a scanner (of doubles no launch that waits is) and with one
@pytest.mark.parametrize("dt,tiles", [("f32", 300), ("bf16", 300), ("f32", 600), ("bf16", 600), ("f64", 460), ("f64", 600)])
def test_tiles_that_stop_waiting_count_the_bitmap_themselves(bt, oracle, dt, tiles):
    n = tiles * bt.bt_tile_elems(wl.DTYPES[dt]) + 4321
    ws = bt.new_workspace(n, wl.DTYPES[dt])
    words = ws.view(torch.int32)
    words[bt.BT_WS_MUTE_WORD], words[bt.BT_WS_PATIENCE_WORD] = 1, 1
    with gpu.instrumented():
        _check(bt, oracle, dt, n, 0.6, 99, ws, 0)
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 0 and int(words[0].item()) == 1


@pytest.mark.parametrize("n", [500 * 1000, 1300 * 1000])
def test_a_small_restoration_on_a_failed_workspace_writes_nothing(bt, oracle, n):
    x = wl.random_sparse(n, "f32", 0.5, 3)
    o_bitmap, o_values, _ = oracle.compress(wl.bits(x))
    ws = bt.new_workspace(n, x.dtype)
    ws.view(torch.int32)[bt.BT_WS_ERROR_WORD] = 1
    out, guard_ok = gpu.gpu_decompress(o_bitmap, o_values, n, x.dtype, ws=ws)
    assert guard_ok and (out.view(np.uint8) == gpu.SENTINEL).all()
