"""Compression in launches of a few hundred tiles, where all four waves of a tile wait for the counts before it: the first and last
sizes that go there and the neighbours that do not, against the CPU oracle, byte for byte."""
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


def _check(bt, oracle, x, dt, ws):
    """compress, prune into half the room, index and activation call of x on one workspace."""
    n, dev = x.numel(), "cuda"
    o_bitmap, o_values, o_nnz = oracle.compress(wl.bits(x))
    bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, ws=ws, values_offset=n % 3)
    assert tail_ok and nnz == o_nnz and np.array_equal(bitmap, o_bitmap) and np.array_equal(values[:o_nnz], o_values)
    want = oracle.prune(wl.bits(x), dt, 0.2)
    p_bitmap, p_values, p_nnz = oracle.compress(want)
    bitmap, values, nnz, tail_ok = gpu.gpu_compress(x, ws=ws, threshold=0.2, cap=p_nnz // 2)
    assert tail_ok and nnz == p_nnz and np.array_equal(bitmap, p_bitmap) and np.array_equal(values, p_values[:p_nnz // 2])
    tile = bt.bt_tile_elems(x.dtype)
    bm, vals = torch.empty((n + 31) // 32, dtype=torch.int32, device=dev), torch.empty(n, dtype=x.dtype, device=dev)
    cnt, index = torch.zeros(1, dtype=torch.int64, device=dev), torch.zeros((n + tile - 1) // tile, dtype=torch.int64, device=dev)
    xd = x.to(dev)
    bt.bt_compress_indexed(xd, bm, vals, cnt, index, ws)
    assert int(cnt) == o_nnz and np.array_equal(wl.bits(vals[:o_nnz].cpu()), o_values)
    assert np.array_equal(index.cpu().numpy().view(np.uint64), oracle.tile_index(o_bitmap, n, tile))
    bt.bt_activation_compress(xd, 0.2, xd, bm, vals, cnt, ws)
    assert int(cnt) == p_nnz and np.array_equal(bm.cpu().numpy().view(np.uint32), p_bitmap)
    assert np.array_equal(wl.bits(xd.cpu()), want) and np.array_equal(wl.bits(vals[:p_nnz].cpu()), p_values)


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16", "f64"])
def test_sizes_on_both_sides_of_every_line(bt, oracle, dt):
    t = bt.bt_tile_elems(wl.DTYPES[dt])
    sizes = [257 * t, 448 * t + 1, 256 * t + 1, 448 * t, 512 * t, 449 * t - 7, 512 * t + 3, 300 * t - 1]
    ws = bt.new_workspace(max(sizes), wl.DTYPES[dt])
    for i, n in enumerate(sizes):
        _check(bt, oracle, wl.random_sparse(n, dt, (0.5, 0.05, 0.95)[i % 3], seed=40 + i), dt, ws)
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    bt.bt_workspace_status(ws, status)
    assert status.tolist() == [0, 4 * len(sizes)]


@pytest.mark.parametrize("dt", ["f32", "bf16", "f64"])
@pytest.mark.parametrize("tiles", [300, 600])      # without and with a scanner
def test_tiles_that_stop_waiting_count_the_input_themselves(bt, oracle, dt, tiles):
    n = tiles * bt.bt_tile_elems(wl.DTYPES[dt]) - 11
    x = wl.random_sparse(n, dt, 0.5, seed=90)
    ws = bt.new_workspace(n, x.dtype)
    words = ws.view(torch.int32)
    words[bt.BT_WS_MUTE_WORD], words[bt.BT_WS_PATIENCE_WORD] = 1, 1
    with gpu.instrumented():
        _check(bt, oracle, x, dt, ws)
    assert int(words[bt.BT_WS_ERROR_WORD].item()) == 0 and int(words[0].item()) == 4


@pytest.mark.parametrize("dt", ["f32", "bf16", "f64"])
def test_a_launch_whose_last_tile_gives_up_says_so(bt, oracle, dt):
    n = 270 * bt.bt_tile_elems(wl.DTYPES[dt]) + 5
    x = wl.random_sparse(n, dt, 0.5, seed=91)
    ws = bt.new_workspace(n, x.dtype)
    words = ws.view(torch.int32)
    words[bt.BT_WS_MUTE_WORD], words[bt.BT_WS_WAIT_LIMIT_WORD], words[bt.BT_WS_PATIENCE_WORD] = 2, 1, 1
    with gpu.instrumented():
        if dt == "f64":                    # (only its activation call has such launches)
            xd, nnz = x.cuda(), torch.full((1,), -7, dtype=torch.int64, device="cuda")
            bm, vals = torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=x.dtype, device="cuda")
            bt.bt_activation_compress(xd, 0.0, torch.empty_like(xd), bm, vals, nnz, ws)
            nnz = int(nnz.item())
        else:
            _, _, nnz, tail_ok = gpu.gpu_compress(x, ws=ws)
            assert tail_ok
    assert nnz == -7 and int(words[bt.BT_WS_ERROR_WORD].item()) == 1
    bt.bt_workspace_init(ws)
    _check(bt, oracle, x, dt, ws)


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16", "f64"])
def test_few_tiles_on_one_xcd_and_on_all(bt, oracle, dt):
    """One workgroup in eight works in the smallest launches, of up to 28 tiles of two rows, without a dense output."""
    two = 8192 // wl.DTYPES[dt].itemsize
    sizes = [1, two - 1, two, two + 1, 8 * two, 8 * two + 1, 27 * two + 5, 28 * two, 28 * two + 1, 29 * two, 64 * two, 64 * two + 1]
    ws = bt.new_workspace(max(sizes), wl.DTYPES[dt])
    for i, n in enumerate(sizes):
        _check(bt, oracle, wl.random_sparse(n, dt, (0.5, 0.05, 0.95)[i % 3], seed=140 + i), dt, ws)
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    bt.bt_workspace_status(ws, status)
    assert status.tolist() == [0, 4 * len(sizes)]
