"""The autograd steps on ordinary tensors, which one call in C++ takes with its allocations, against the same steps on a subclass, which
go the general way call by call: the same bytes, the same decisions and the same statistics."""
import time

import pytest
import torch

pytestmark = pytest.mark.gpu
DTYPES = [torch.float32, torch.float16, torch.bfloat16, torch.float64]


class _Sub(torch.Tensor):
    pass


@pytest.fixture(scope="module")
def ag():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (they never fall back to the CPU)")
    from paper_2110_15362_amd import autograd
    return autograd


def _bytes(t):
    return t.as_subclass(torch.Tensor).contiguous().reshape(-1).view(torch.uint8)


@pytest.mark.parametrize("deferred", [False, True])
@pytest.mark.parametrize("dtype", DTYPES)
def test_packing(ag, dtype, deferred):
    g = torch.Generator(device="cuda").manual_seed(5)
    for shape, zeros, nan in (((4096,), 0.5, True), ((3, 7, 411), 0.9, True), ((260 * 8192 + 13,), 0.5, True), ((64, 64), 1.0, True),
                              ((10, 1000), 0.0, True), ((1001, 1003), 0.02, True), ((64, 64), 1.0, False), ((260 * 8192 + 13,), 1.0, False)):
        x = torch.randn(shape, generator=g, device="cuda").to(dtype)
        x[torch.rand(shape, generator=g, device="cuda") < zeros] = 0
        if nan:
            x.view(-1)[7] = float("nan")
        else:
            assert not x.any()             # no value at all
        got = []
        for t in (x, x.as_subclass(_Sub)):
            stash = ag.BitmapStash(deferred=deferred)
            packed = stash._pack(t)
            stash._finish_waiting(block=True)
            got.append((stash, packed, packed if packed is t else stash._unpack(packed)))
        (s0, p0, u0), (s1, p1, u1) = got
        assert s0.stats == s1.stats and u0.shape == x.shape and u0.dtype == dtype
        assert torch.equal(_bytes(u0), _bytes(x)) and torch.equal(_bytes(u1), _bytes(x))
        assert isinstance(p0, ag._Packed) == isinstance(p1, ag._Packed) and (nan or (isinstance(p0, ag._Packed) and p0.dense is None))
        if isinstance(p0, ag._Packed) and p0.dense is None:
            assert nan or (p0.values.numel() == 0 and s0.stats["compressed"] == 1)
            assert p0.values.untyped_storage().nbytes() == p1.values.untyped_storage().nbytes()
            assert torch.equal(p0.bitmap, p1.bitmap) and torch.equal(p0.index, p1.index) and torch.equal(_bytes(p0.values), _bytes(p1.values))


@pytest.mark.parametrize("dtype", DTYPES)
def test_relu(ag, dtype):
    special = torch.tensor([0.0, -0.0, 1.0, -1.0, float("nan"), float("inf"), -float("inf"), 1e-8, -1e-8], device="cuda")
    for n in (0, 1, 9, 33, 4097, 100003):
        x = torch.cat([special, torch.randn(n, device="cuda")])[:n].to(dtype).reshape(1, n)
        grad = torch.randn(n, device="cuda").to(dtype).reshape(1, n)
        out = []
        for t in (x.clone(), x.clone().as_subclass(_Sub)):
            t.requires_grad_()
            y = ag.bitmap_relu(t)
            y.backward(grad if type(t) is torch.Tensor else grad.as_subclass(_Sub))
            out.append((y.detach(), t.grad))
        assert out[0][0].shape == x.shape and type(out[0][0]) is torch.Tensor
        for a, b in zip(*out):
            assert torch.equal(_bytes(a), _bytes(b))
        assert torch.equal(_bytes(out[0][0]), _bytes(torch.relu(x)))


def test_what_is_refused_stays_refused(ag):
    x = torch.ones(64, 64, device="cuda")
    for bad in (x.t()[:, 1:], x.int(), x.cpu()):
        with pytest.raises(TypeError):
            ag.bitmap_relu(bad)
    stash = ag.BitmapStash(min_numel=1)
    for t in (x.t()[:, 1:], x.int(), x.cpu(), x.view(-1)[1:], torch.nn.Parameter(x)):
        assert stash._pack(t) is t
    assert stash.stats["tensors"] == 0


@pytest.mark.parametrize("deferred", [False, True])
def test_a_refused_packing_gives_its_place_back(ag, deferred, monkeypatch):
    """The library's host checks refuse the workspace: nothing is queued, and no place on the host is lost."""
    from paper_2110_15362_amd import bittrain as bt
    x = torch.randn(5000, device="cuda").relu()
    st = ag._state(x.device)
    assert ag.BitmapStash(min_numel=1)._pack(x) is not None
    places = len(st.places)
    with monkeypatch.context() as m:
        m.setattr(st, "workspace", lambda n, dtype: torch.empty(128, dtype=torch.uint8, device="cuda"))
        with pytest.raises(bt.BitTrainError, match="workspace"):
            ag.BitmapStash(deferred=deferred)._pack(x)
    assert len(st.places) == places and len({p.address for p in st.places}) == places
    stash = ag.BitmapStash()
    assert torch.equal(stash._unpack(stash._pack(x)), x)


def test_a_host_that_looks_at_nnz_sees_it_change_once(ag):
    """In pinned memory that held -1, without waiting for the stream, from every way to end a compression: no elements, the last of
    two-row, four-row and eight-row tiles and of those whose four waves read the counts, the scanner, and a batch with an empty tensor."""
    from paper_2110_15362_amd import bittrain as bt
    g = torch.Generator(device="cuda").manual_seed(6)
    tile, L = bt.bt_tile_elems(torch.float32), bt.lib()
    sizes = [0, 1, 5 * tile + 3, 100 * tile, 250 * tile, 300 * tile, 1000 * tile + 1]
    xs = [torch.randn(n, generator=g, device="cuda").relu() for n in sizes]
    bitmaps = [torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda") for n in sizes]
    values = [torch.empty_like(x) for x in xs]
    word = torch.empty(len(sizes), dtype=torch.int64, pin_memory=True)
    ws, wsb = bt.new_workspace(max(sizes), torch.float32), bt.new_batch_workspace(sizes, torch.float32)
    want = [int(torch.count_nonzero(x)) for x in xs]
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream().cuda_stream

    def seen(count):
        end = time.monotonic() + 10
        while (word[:count] == -1).any() and time.monotonic() < end:
            pass
        got = word[:count].tolist()
        torch.cuda.synchronize()
        assert word[:count].tolist() == got
        return got
    for x, b, v, k in zip(xs, bitmaps, values, want):
        word.fill_(-1)
        bt._check("bt_compress", L.bt_compress(x.data_ptr(), x.numel(), bt.BT_F32, b.data_ptr(), v.data_ptr(), v.numel(), word.data_ptr(),
                                               ws.data_ptr(), ws.numel(), stream))
        assert seen(1) == [k]
    word.fill_(-1)
    items = (bt.CompressItem * len(sizes))(*[bt.CompressItem(x.data_ptr(), x.numel(), b.data_ptr(), v.data_ptr(), v.numel(), word[i:].data_ptr(), None, None)
                                             for i, (x, b, v) in enumerate(zip(xs, bitmaps, values))])
    bt.bt_compress_batch(items, len(sizes), torch.float32, wsb)
    assert seen(len(sizes)) == want
