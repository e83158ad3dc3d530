"""What BitmapStash does on the host around its compressions, without a GPU: the compressions, the events behind them and
pinned memory are stand-ins, so every order of events and every failure can be had."""
import contextlib
import gc
import threading
import weakref

import pytest
import torch

N = 4096
NNZ = 100


class _Stream(str):
    def wait_stream(self, other):
        self.__dict__.setdefault("waited", []).append(other)


@pytest.fixture
def ag(monkeypatch):
    """The module, with ordinary host memory for pinned memory and names for streams."""
    from paper_2110_15362_amd import autograd, bittrain
    bittrain.lib()
    empty, current = torch.empty, [_Stream("default")]

    @contextlib.contextmanager
    def stream(other):
        current.append(other)
        yield
        current.pop()
    monkeypatch.setattr(torch, "empty", lambda *a, pin_memory=False, **k: empty(*a, **k))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: current[-1])
    monkeypatch.setattr(torch.cuda, "stream", stream)
    return autograd


class _Event:
    """A compression that is over once somebody waits for it."""

    def __init__(self, wait=None):
        self.wait = wait

    def query(self):
        return False

    def synchronize(self):
        if self.wait is not None:
            self.wait()


class _Values:
    """The worst-case buffer of a packing, which is cut to size by a copy."""

    def __init__(self, failures=0, on_copy=None):
        self.failures, self.on_copy = failures, on_copy

    def __getitem__(self, cut):
        self.length = cut.stop
        return self

    def clone(self):
        if self.failures:
            self.failures -= 1
            raise torch.OutOfMemoryError("out of memory")
        if self.on_copy is not None:
            self.on_copy()
        return torch.zeros(self.length)


def _waiting(ag, stash, st, values, event=None, stream="default"):
    """A packing of N elements, of which NNZ are stored, that `stash` has not settled yet."""
    p = ag._Packed(torch.zeros(N // 32, dtype=torch.int32), values, torch.zeros(1, dtype=torch.int64), torch.Size([N]), torch.float32, st.device)
    p.pending = True
    place = st.place()
    place.word[0] = NNZ
    stash._waiting.append(ag._Pending(p, torch.ones(N), place, event or _Event(), None, stream))
    return p


def _distinct(places):
    return len({id(p) for p in places}) == len(places)


def test_a_place_is_given_back_once_though_settling_failed(ag):
    """The copy that cuts a packing to size runs out of memory: the tensor stays dense, the packings after it are settled as
    ever, and no two of the compressions that follow write their nnz to the same word."""
    st = ag._StreamState(torch.device("cpu"))
    stash = ag.BitmapStash(deferred=True)
    first = _waiting(ag, stash, st, _Values(failures=1))
    second = _waiting(ag, stash, st, _Values())
    with pytest.raises(torch.OutOfMemoryError):
        stash._finish_waiting(block=True)
    stash._finish_waiting(block=True)
    assert len(st.places) == 8 and _distinct(st.places)
    taken = [st.place() for _ in range(12)]
    assert _distinct(taken) and len({p.address for p in taken}) == 12
    assert not first.pending and torch.equal(stash._unpack(first), torch.ones(N))
    assert not second.pending and second.dense is None and second.values.numel() == NNZ
    assert stash.stats["compressed"] == 1


def test_two_threads_settle_a_packing_once(ag):
    """One thread packs and another unpacks: the second comes while the first waits for the event."""
    st = ag._StreamState(torch.device("cpu"))
    stash = ag.BitmapStash(deferred=True)
    waits, both = [], threading.Event()

    def wait():      # up to half a second for the other thread to get here too
        waits.append(threading.get_ident())
        if len(waits) > 1:
            both.set()
        both.wait(0.5)
    p = _waiting(ag, stash, st, _Values(), _Event(wait))
    threads = [threading.Thread(target=stash._finish_waiting, kwargs={"only": p}) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(10)
    assert len(waits) == 1 and stash._waiting == []
    assert not p.pending and p.values.numel() == NNZ and stash.stats["compressed"] == 1
    assert len(st.places) == 8 and _distinct(st.places)


@pytest.mark.parametrize("gave_up", [False, True])
def test_a_packing_is_settled_on_the_stream_it_was_packed_on(ag, monkeypatch, gave_up):
    """Wherever the host is by then (leaving the stash, packing on another stream): its values are read there in the backward pass,
    which nothing else orders behind their copy, and so is its workspace used by the next call.  Work here is ordered behind it too."""
    st = ag._StreamState(torch.device("cpu"))
    stash, used = ag.BitmapStash(deferred=True), []

    def note(*args):
        used.append(torch.cuda.current_stream())
    monkeypatch.setattr(ag.bt, "bt_workspace_init", note)
    for stream in ("side", "default", "other"):
        _waiting(ag, stash, st, _Values(on_copy=note), stream=_Stream(stream))
        if gave_up:
            stash._waiting[-1].place.word[0] = -1
    with pytest.warns(UserWarning) if gave_up else contextlib.nullcontext():
        stash._finish_waiting(block=True)
    here = torch.cuda.current_stream()
    assert used == ["side", "default", "other"] and here == "default" and here.waited == ["side", "other"]


def test_leaving_the_stash_takes_its_hooks_off_though_settling_failed(ag):
    class Stash(ag.BitmapStash):
        packed = 0

        def _pack(self, t):
            Stash.packed += 1
            return t
    x = torch.ones(4, requires_grad=True)
    stash = Stash(deferred=True)
    with pytest.raises(torch.OutOfMemoryError):
        with stash:
            (x * x).sum()
            _waiting(ag, stash, ag._StreamState(torch.device("cpu")), _Values(failures=1))
    inside = Stash.packed
    try:
        (x * x).sum()
        assert inside > 0 and Stash.packed == inside
    finally:
        if Stash.packed != inside:      # (not for the tests after this one)
            torch.autograd.graph.saved_tensors_hooks.__exit__(stash)


def test_a_place_that_nobody_gives_back_keeps_its_memory(ag):
    """Its compression may still be on the way (the host was interrupted while it waited, a packing was let go of unsettled),
    and what it writes to must not have become something else's memory by then."""
    st = ag._StreamState(torch.device("cpu"))
    place = st.place()
    address, memory = place.address, weakref.ref(place.memory)
    del place
    gc.collect()
    assert memory() is not None and memory().data_ptr() == address
    assert all(p.address != address for p in [st.place() for _ in range(20)])


class _OnDevice(torch.Tensor):
    is_cuda = True


@pytest.fixture
def packing(ag, monkeypatch):
    """`packing(values)` has a new stash pack a tensor of them as if it were on a device; the compression is done by torch at
    once.  `packing.wait`: called while the host waits for the stream."""
    st = ag._StreamState(torch.device("cpu"))

    def compress(t, packed, values, st, ws, stream):
        kept = t[t != 0].as_subclass(torch.Tensor)
        values[:kept.numel()] = kept
        place = st.place()
        place.word[0] = kept.numel()
        return place

    class Stream:
        cuda_stream = 0

        def synchronize(self):
            wait, pack.wait = pack.wait, None
            if wait is not None:
                wait()

    def pack(values):
        return ag.BitmapStash()._pack(values.as_subclass(_OnDevice))
    pack.wait, pack.state = None, st
    monkeypatch.setattr(ag, "_state", lambda device: st)
    monkeypatch.setattr(ag.bt, "bt_workspace_init", lambda ws: None)
    monkeypatch.setattr(ag.BitmapStash, "_compress", staticmethod(compress))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream())
    return pack


def _sparse(n, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(n, generator=g).relu()


def test_another_thread_packs_on_the_same_stream_before_the_values_are_copied(ag, packing):
    """The second compression is queued between the end of the first and the copy that cuts it to size: larger, smaller and of
    the same size."""
    x = _sparse(N, 1)
    for n in (N // 2 + 4096, N, 2 * N):
        y, inner = _sparse(n, n), []
        packing.wait = lambda: inner.append(packing(y))
        p = packing(x)
        assert torch.equal(p.values, x[x != 0])
        assert torch.equal(inner[0].values, y[y != 0])
    assert packing.state.scratch[torch.float32].numel() == 2 * N      # the larger one is kept


def test_a_new_workspace_is_seen_by_others_only_once_it_is_initialised(ag, packing, monkeypatch):
    st, seen = packing.state, []
    monkeypatch.setattr(ag.bt, "bt_workspace_init", lambda ws: seen.append(st.ws is ws))
    st.workspace(N, torch.float32)
    st.workspace(1 << 30, torch.float32)
    assert seen == [False, False]


def test_a_workspace_that_another_thread_replaces_meanwhile_is_not_the_small_one(ag, packing):
    """The larger one is there between this thread's two looks, at what the workspace serves and at the workspace."""
    st = packing.state
    st.workspace(N, torch.float32)
    large = torch.empty(ag.bt.bt_workspace_bytes(1 << 28, torch.float32), dtype=torch.uint8)

    class Fits(dict):
        def get(self, dtype, default):
            st.ws = large
            return 1 << 28
    st.fits = Fits()
    assert st.workspace(1 << 28, torch.float32) is large


@pytest.mark.parametrize("last", ["small", "large"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_of_two_new_workspaces_the_larger_one_stays(ag, packing, monkeypatch, dtype, last):
    """Two threads on one stream find no workspace, both make one, and whichever is through last puts its own there.  From then on
    everything that either has asked for is served."""
    st, both, first_is_through = packing.state, threading.Barrier(2), threading.Event()
    asked = {"small": (N, dtype), "large": (1 << 28, torch.float32)}

    def init(ws):
        both.wait(10)
        if threading.current_thread().name == last:
            first_is_through.wait(10)
    monkeypatch.setattr(ag.bt, "bt_workspace_init", init)

    def ask(who):
        got[who] = st.workspace(*asked[who])
        if who != last:
            first_is_through.set()
    got = {}
    threads = [threading.Thread(target=ask, args=(who,), name=who) for who in asked]
    for t in threads:
        t.start()
    for t in threads:
        t.join(20)
    monkeypatch.setattr(ag.bt, "bt_workspace_init", lambda ws: None)
    for who, (n, dtype) in asked.items():
        need = ag.bt.bt_workspace_bytes(n, dtype)
        assert got[who].numel() >= need and st.workspace(n, dtype).numel() >= need


def test_a_larger_workspace_that_comes_while_a_smaller_one_is_initialised_stays(ag, packing, monkeypatch):
    st = packing.state

    def init(ws):
        if ws.numel() == 1 << 16:
            st.workspace(1 << 28, torch.float32)
    monkeypatch.setattr(ag.bt, "bt_workspace_init", init)
    st.workspace(N, torch.bfloat16)
    assert st.workspace(1 << 28, torch.float32).numel() >= ag.bt.bt_workspace_bytes(1 << 28, torch.float32)


@pytest.mark.parametrize("deferred", [False, True])
@pytest.mark.parametrize("started", [False, True])
def test_a_packing_that_raises_gives_its_place_back_unless_its_compression_may_still_write_to_it(ag, packing, monkeypatch, deferred, started):
    """Out of memory for the bitmap, or a refused call, before anything is queued; and an error met while the host waits."""
    import ctypes
    import types

    def pack(t, scratch, ws, place, wait):
        if started:
            ctypes.c_int64.from_address(place).value = -1
        raise torch.OutOfMemoryError("out of memory")
    st = packing.state
    monkeypatch.setattr(ag, "_native", lambda: types.SimpleNamespace(pack=pack))
    for lost in range(1, 4):
        with pytest.raises(torch.OutOfMemoryError):
            ag.BitmapStash(deferred=deferred)._pack_plain(_sparse(N, 1))
        assert len(st.places) == (8 - lost if started else 8) and _distinct(st.places)
    assert len(st.words) == 8


def test_a_refused_compression_gives_its_place_back(ag, monkeypatch):
    """The general way: the library refuses (here, a workspace that is none), so nothing is queued that could write to the place."""
    st = ag._StreamState(torch.device("cpu"))
    x = _sparse(N, 1)
    packed = ag._Packed(torch.zeros(N // 32, dtype=torch.int32), None, torch.zeros(1, dtype=torch.int64), x.shape, x.dtype, st.device)

    class Stream:
        cuda_stream = 0
    with pytest.raises(ag.bt.BitTrainError):
        ag.BitmapStash._compress(x, packed, torch.empty(N), st, torch.empty(0, dtype=torch.uint8), Stream())
    assert len(st.places) == 8 and _distinct(st.places)


@pytest.fixture
def relu_backward(ag, monkeypatch):
    """bitmap_relu's backward with the kernel's work done by torch on what it is handed: the memory at an address."""
    import ctypes
    import types

    def kernel(bitmap, grad_out, grad_in):
        n = grad_out.numel()
        assert grad_out.is_contiguous() and grad_out.data_ptr() % 16 == 0 and grad_in.data_ptr() % 16 == 0
        held = (ctypes.c_float * n).from_address(grad_out.data_ptr())
        kept = (bitmap.repeat_interleave(32) >> torch.arange(32).repeat(bitmap.numel()))[:n] & 1
        grad_in.copy_(torch.where(kept.bool(), torch.frombuffer(held, dtype=torch.float32), torch.zeros(n)))
    monkeypatch.setattr(ag.bt, "bt_relu_backward_from_bitmap", kernel)
    ctx = types.SimpleNamespace(bitmap=torch.tensor([0x35A5A5A5], dtype=torch.int32))
    kept = (ctx.bitmap >> torch.arange(32)) & 1
    return lambda grad: (ag._BitmapReLU.backward(ctx, grad)[0], kept)


@pytest.mark.parametrize("start", [0, 1, 2, 3, 4])
def test_relu_backward_takes_gradients_off_a_16_byte_boundary(relu_backward, start):
    """What a concatenation hands back to its parts: a contiguous view that begins anywhere."""
    grad = torch.randn(40)[start:start + 32]
    got, kept = relu_backward(grad)
    assert torch.equal(got, grad * kept)


def test_tensors_whose_memory_does_not_hold_their_values(ag, packing, relu_backward, monkeypatch):
    """Negated views and zero tensors (which have no memory at all): the stash leaves them alone, and bitmap_relu hands the
    kernels memory that holds what they are, also in one pass with the compression and as gradients."""
    for t in (torch._neg_view(_sparse(N, 1)), torch._efficientzerotensor(N)):
        t = t.as_subclass(_OnDevice)
        assert ag.BitmapStash()._pack(t) is t
    grad = torch.randn(33)
    for g, want in ((torch._neg_view(grad[:32]), -grad[:32]), (torch._neg_view(grad[1:]), -grad[1:]),
                    (torch._efficientzerotensor(32), torch.zeros(32))):
        got, kept = relu_backward(g)
        assert torch.equal(got, want * kept)

    handed = []
    monkeypatch.setattr(ag.bt, "bt_activation_compress", lambda x, *rest: handed.append(x))
    x = torch._neg_view(grad[:32])
    ag._BitmapReLU.forward(torch.autograd.function.FunctionCtx(), x.as_subclass(_OnDevice), True)
    assert not handed[0].is_neg() and torch.equal(handed[0], -grad[:32])


class _Elsewhere(torch.Tensor):
    """A tensor of the second of two devices, as far as one can ask it."""
    is_cuda = True
    device = torch.device("cuda", 1)


@pytest.fixture
def two_devices(ag, monkeypatch):
    """The first of two devices is the current one.  `calls`: (what was called, the device that was current then)."""
    current, calls = [0], []
    empty, empty_like = torch.empty, torch.empty_like

    @contextlib.contextmanager
    def device(d):
        current.append(torch.device(d).index)
        yield
        current.pop()

    class Stream(_Stream):
        cuda_stream = 0

        def synchronize(self):
            note("wait")

    def note(name):
        calls.append((name, current[-1]))

    def compress(t, packed, values, st, ws, stream):
        note("compress")
        assert stream == "stream of %d" % current[-1]
        place = st.place()
        place.word[0] = NNZ
        return place

    class Event(_Event):
        def record(self, stream):
            note("record")
    monkeypatch.setattr(torch, "empty", lambda *a, pin_memory=False, device=None, **k: empty(*a, **k))
    monkeypatch.setattr(torch, "empty_like", lambda t: empty_like(t.as_subclass(torch.Tensor)))
    monkeypatch.setattr(torch.cuda, "device", device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: current[-1])
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: Stream("stream of %d" % current[-1]))
    monkeypatch.setattr(torch.cuda, "Event", Event)
    states = {}
    monkeypatch.setattr(ag, "_state", lambda device: states.setdefault(device, ag._StreamState(torch.device("cpu"))))
    monkeypatch.setattr(ag.BitmapStash, "_compress", staticmethod(compress))
    for name in ("bt_workspace_init", "bt_decompress_indexed", "bt_relu_forward", "bt_relu_backward_from_bitmap", "bt_activation_compress"):
        monkeypatch.setattr(ag.bt, name, lambda *a, name=name: note(name))
    return calls


@pytest.mark.parametrize("deferred", [False, True])
def test_a_tensor_off_the_current_device_is_packed_on_its_own(ag, two_devices, deferred):
    """Its values are copied, and it is unpacked and used, on its device's stream, which nothing else orders behind a compression on
    another device's."""
    stash = ag.BitmapStash(deferred=deferred)
    packed = stash._pack(_sparse(N, 1).as_subclass(_Elsewhere))
    assert isinstance(packed, ag._Packed)
    stash._unpack(packed)
    assert {"compress", "bt_workspace_init", "bt_decompress_indexed"} <= {name for name, _ in two_devices}
    assert {device for _, device in two_devices} == {1} and torch.cuda.current_device() == 0


@pytest.mark.parametrize("fused", [False, True])
def test_bitmap_relu_off_the_current_device(ag, two_devices, fused):
    ctx = torch.autograd.function.FunctionCtx()
    ag._BitmapReLU.forward(ctx, _sparse(N, 1).as_subclass(_Elsewhere), fused)
    ag._BitmapReLU.backward(ctx, _sparse(N, 2).as_subclass(_Elsewhere))
    assert {"bt_activation_compress" if fused else "bt_relu_forward", "bt_relu_backward_from_bitmap"} <= {name for name, _ in two_devices}
    assert {device for _, device in two_devices} == {1} and torch.cuda.current_device() == 0
