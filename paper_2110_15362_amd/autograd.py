"""BitTrain as PyTorch autograd plumbing (the integration the paper describes in its
implementation details and names as future work): activations saved for backward are
kept in the bitmap format between the forward and the backward pass.

Two pieces, both thin: every byte of codec work is done by libbittrain's kernels.

* ``BitmapStash`` -- a ``torch.autograd.graph.saved_tensors_hooks`` context.  Packing a
  saved activation runs ``bt_compress_indexed`` into a reusable worst-case scratch buffer, waits for
  nnz, which the kernel writes straight to the host (one wait per tensor: the price of right-sizing), and keeps
  only ``values[:nnz]`` and the bitmap; if that is not smaller than the dense tensor the
  tensor is kept as it is.  Packing also keeps the tile index (8 bytes per 32 KiB of
  dense data) that compression produces on the way, so unpacking runs
  ``bt_decompress_indexed``, which needs no scan over the bitmap.  The round trip is
  bit-exact, so gradients are identical to those of the unhooked graph.
* ``bitmap_relu`` -- a ReLU whose backward is served by
  ``bt_relu_backward_from_bitmap`` and which saves nothing but the bitmap of its output
  (1/32 of an fp32 activation): output and bitmap from one pass, bt_relu_forward.
"""
import math
import threading
import warnings

import torch

from . import bittrain as bt

_SUPPORTED = (torch.float32, torch.float16, torch.bfloat16, torch.float64)


def _native():
    """The steps in C++ (csrc/call.cpp)."""
    if bt._lib is None:
        bt.lib()
    return bt._call


def _elsewhere(device):
    """Whether a tensor on `device` needs it made the current one: calls and allocations go to the current device's stream."""
    return device.index is not None and device.index != torch.cuda.current_device()


class _StreamState:
    """Reusable buffers of one (device, stream): workspace, worst-case value scratch, and places in pinned host memory
    that compressions write their nnz to (a call that gave up a wait, or found a workspace on which one was given up, writes
    none).  Work on different streams must not share them: a workspace serves one call at a time.  Threads on one stream may: their
    calls are in its order, and a value scratch and a place are one packing's until it gives them back."""

    def __init__(self, device):
        self.device = device
        self.ws = None        # replaced by a larger one only
        self.fits = {}        # dtype -> elements that `ws`, and so whatever replaces it, is known to serve
        self.lock = threading.RLock()
        self.scratch = {}
        self.nnz = torch.zeros(1, dtype=torch.int64, device=device)
        self.places = []      # free ones
        self.words = []       # the memory of all, kept: a place that is never given back (the host was interrupted in its wait)
                              # may still be written to, and not be something else by then

    def place(self):
        """A place for one compression's nnz, holding -2 until that compression is queued and -1 from then on; back to `places` when it
        is over."""
        try:
            p = self.places.pop()
        except IndexError:                # (not asked before: another thread may take the last one)
            self.places += [_Place(self) for _ in range(7)]
            p = _Place(self)
        p.word[0] = -2
        return p

    def workspace(self, n, dtype):
        fits = self.fits.get(dtype, -1)
        ws = self.ws                          # (after `fits`: another thread may replace it between the two)
        if n <= fits:
            return ws
        need = bt.bt_workspace_bytes(n, dtype)
        if ws is None or ws.numel() < need:
            ws = torch.empty(max(need, 1 << 16), dtype=torch.uint8, device=self.device)
            bt.bt_workspace_init(ws)
            with self.lock:                   # (only now: another thread on this stream may look for one in between, or make one too)
                if self.ws is None or self.ws.numel() < ws.numel():
                    self.ws = ws
        self.fits[dtype] = n                  # (behind a workspace that serves them: this one, or a larger one)
        return ws

    def take_scratch(self, n, dtype):
        """A value buffer for n elements that is nobody else's until it comes back: another thread that packs on this stream takes
        another one, or its values would land in this one before they are copied out of it."""
        buf = self.scratch.pop(dtype, None)
        if buf is None or buf.numel() < n:
            buf = torch.empty(n, dtype=dtype, device=self.device)
        return buf

    def give_scratch(self, buf):
        """Back, once its last use is on the stream; the largest is kept."""
        other = self.scratch.get(buf.dtype)
        if other is None or other.numel() < buf.numel():
            self.scratch[buf.dtype] = buf


class _Place:
    """64 bits of pinned host memory, as the device and as the host address them."""
    __slots__ = ("state", "memory", "word", "address")

    def __init__(self, state):
        self.state = state
        self.memory = torch.empty(1, dtype=torch.int64, pin_memory=True)
        self.word, self.address = self.memory.numpy(), self.memory.data_ptr()
        state.words.append(self.memory)

    def read(self):
        """nnz, or -1 from a compression that failed; only after the compression is over, or -2 if none has been queued."""
        return int(self.word[0])

    def give_back(self):
        """After the compression is over, and once: whoever takes the place next shares it with nobody."""
        self.state.places.append(self)


_states = {}


def _state(device):
    key = (device, torch._C._cuda_getCurrentRawStream(device.index))
    st = _states.get(key)
    if st is None:
        st = _states[key] = _StreamState(device)
    return st


class _Packed:
    """A saved activation in the bitmap format.  `dense` is set instead when the tensor turned out not to be
    worth compressing (or its compression failed); `pending` while that is not known yet (deferred mode)."""
    __slots__ = ("bitmap", "values", "index", "shape", "dtype", "device", "dense", "pending")

    def __init__(self, bitmap, values, index, shape, dtype, device):
        self.bitmap, self.values, self.index = bitmap, values, index
        self.shape, self.dtype, self.device = shape, dtype, device
        self.dense, self.pending = None, None


class _Pending:
    """What a deferred packing still waits for: nnz on its way to pinned host memory, the event behind the
    compression on its stream, and the dense tensor, kept until the result is known to be good."""
    __slots__ = ("packed", "dense", "place", "event", "ws", "stream", "lock", "taken")

    def __init__(self, packed, dense, place, event, ws, stream):
        self.packed, self.dense, self.place, self.event, self.ws, self.stream = packed, dense, place, event, ws, stream
        self.lock, self.taken = threading.RLock(), False       # one thread may pack while another unpacks: the first settles it


class BitmapStash(torch.autograd.graph.saved_tensors_hooks):
    """``with BitmapStash(): loss = model(x)`` keeps saved activations compressed.

    min_numel: smaller tensors are left alone (a call costs a few microseconds).
    deferred: False (default) reads nnz back right after the compression, which makes the host wait for the
    device once per saved tensor, and stores exactly nnz values at once.  True never waits: the compression
    writes into a buffer of worst-case size and nnz to pinned host memory, and
    the buffer is cut down to nnz values (and the dense tensor let go) at the next packing or unpacking after
    the event has passed; until then the tensor costs more memory than it did dense, so at most
    `max_waiting` packings are left in that state (the host waits for the oldest one beyond that).
    ``stats`` counts dense and stored bytes of everything that went through the hooks.
    """

    def __init__(self, min_numel=4096, deferred=False, max_waiting=2):
        self.min_numel = min_numel
        self.deferred = deferred
        self.max_waiting = max(1, max_waiting)
        self.stats = {"tensors": 0, "compressed": 0, "failed": 0, "dense_bytes": 0, "stored_bytes": 0}
        self._waiting = []
        super().__init__(self._pack, self._unpack)

    def _settle(self, p, nnz, values_full, ws):
        """The compression of `p` (a _Packed) is over: keep it, cut to size, or go back to the dense tensor."""
        n, width = math.prod(p.shape), p.dtype.itemsize
        gave_up = nnz < 0
        if gave_up:
            bt.bt_workspace_init(ws)                               # what the kernel wrote is not valid; make the workspace usable again
            self.stats["failed"] += 1
            warnings.warn("BitmapStash: a compression gave up a wait; the tensor is kept dense")
        stored = 0 if gave_up else bt.bt_compressed_size(n, nnz, p.dtype) + 8 * p.index.numel()      # M_b plus the tile index
        if gave_up or stored >= n * width:
            self.stats["stored_bytes"] += n * width
            return False                                           # too dense (the bitmap form would be larger), or no good
        p.values = values_full[:nnz].clone()
        self.stats["compressed"] += 1
        self.stats["stored_bytes"] += stored
        return True

    def _finish_waiting(self, only=None, block=False, most=None):
        """Deferred mode: settle every packing whose result has arrived; wait for `only`'s (for all, if `block`; for the oldest
        of more than `most`)."""
        for w in list(self._waiting):
            if block or w.packed is only or w.event.query():
                self._finish(w)
        if most is not None:
            for w in self._waiting[:max(0, len(self._waiting) - most)]:
                self._finish(w)

    def _finish(self, w):
        """Wait for the packing `w` (a _Pending) and settle it, once, whatever becomes of that; if it fails, the tensor stays dense."""
        with w.lock:
            if w.taken:
                return
            w.taken = True
            kept = False
            try:
                w.event.synchronize()
                nnz = w.place.read()
                w.place.give_back()
                here = torch.cuda.current_stream()
                if here == w.stream:
                    kept = self._settle(w.packed, nnz, w.packed.values, w.ws)
                else:                     # where backward unpacks it, and where the next call on the workspace is
                    with torch.cuda.stream(w.stream):
                        kept = self._settle(w.packed, nnz, w.packed.values, w.ws)
                    here.wait_stream(w.stream)      # (who unpacks it here is behind the copy too)
            finally:
                if not kept:
                    w.packed.dense, w.packed.bitmap, w.packed.values, w.packed.index = w.dense, None, None, None
                w.packed.pending = None
                self._waiting.remove(w)

    def __exit__(self, *exc):
        try:
            self._finish_waiting(block=True)  # leaves nothing behind that still holds a dense tensor
        finally:
            super().__exit__(*exc)

    def _pack_plain(self, t):
        """_pack of an ordinary tensor, around one call that allocates, compresses and, unless deferred, waits and copies (see
        csrc/call.cpp); None if it is no such tensor after all.  (A packing of fp32 [500, 1024], waiting included, 35 -> 19 us; a step of four
        layers of 1024 features, on fp32 with 8192 rows 1915 -> 1830 us, with 500 rows 850 -> 675, on bf16 with 8192 rows 960 -> 820, deferred
        865 -> 770.)"""
        st = _state(t.device)
        n, dtype = t.numel(), t.dtype
        ws = st.workspace(n, dtype)
        if self.deferred:
            self._finish_waiting(most=self.max_waiting - 1)        # bounds what the unsettled packings hold
            values = torch.empty(n, dtype=dtype, device=t.device)  # its own: it outlives this call
        else:
            values = st.take_scratch(n, dtype)
        place = st.place()
        try:
            got = _native().pack(t, values, ws, place.address, not self.deferred)
        except BaseException:
            if place.read() != -1:            # (not queued at all, or over as far as the place is concerned: it was the copy that failed)
                place.give_back()
            raise
        finally:
            if not self.deferred:
                st.give_scratch(values)
        if got is None:
            place.give_back()
            return None
        self.stats["tensors"] += 1
        self.stats["dense_bytes"] += n * t.element_size()
        packed = _Packed(got[0], None, got[1], t.shape, dtype, t.device)
        if self.deferred:
            packed.values = values
            self._defer(packed, t, place, ws, torch.cuda.current_stream())
            return packed
        nnz, kept = got[2], got[3]
        place.give_back()
        if nnz < 0:
            self._settle(packed, nnz, None, ws)
            return t
        if kept is None:
            self.stats["stored_bytes"] += n * t.element_size()
            return t
        packed.values = kept
        self.stats["compressed"] += 1
        self.stats["stored_bytes"] += 4 * got[0].numel() + nnz * t.element_size() + 8 * got[1].numel()
        return packed

    def _defer(self, packed, t, place, ws, stream):
        """`packed` is settled later (see _finish_waiting)."""
        event = torch.cuda.Event()
        event.record(stream)
        packed.pending = True
        self._waiting.append(_Pending(packed, t.detach(), place, event, ws, stream))

    def _pack(self, t):
        if (not t.is_cuda or t.dtype not in _SUPPORTED or t.numel() < self.min_numel or not t.is_contiguous()
                or isinstance(t, torch.nn.Parameter) or t.is_neg() or t._is_zerotensor() or t.data_ptr() % 16 != 0):
            return t                      # (the library takes memory from a 16-byte boundary on that holds the values)
        if _elsewhere(t.device):
            with torch.cuda.device(t.device):
                return self._pack(t)
        if type(t) is torch.Tensor:
            packed = self._pack_plain(t)
            if packed is not None:
                return packed
        st = _state(t.device)
        n = t.numel()
        self.stats["tensors"] += 1
        self.stats["dense_bytes"] += n * t.element_size()
        bitmap = torch.empty((n + 31) // 32, dtype=torch.int32, device=t.device)
        index = torch.empty(bt.bt_index_bytes(n, t.dtype) // 8, dtype=torch.int64, device=t.device)
        ws = st.workspace(n, t.dtype)
        stream = torch.cuda.current_stream()
        packed = _Packed(bitmap, None, index, t.shape, t.dtype, t.device)
        if self.deferred:
            self._finish_waiting(most=self.max_waiting - 1)        # bounds what the unsettled packings hold
            packed.values = torch.empty(n, dtype=t.dtype, device=t.device)     # its own: it outlives this call
            place = self._compress(t, packed, packed.values, st, ws, stream)
            self._defer(packed, t, place, ws, stream)
            return packed
        scratch = st.take_scratch(n, t.dtype)
        try:
            place = self._compress(t, packed, scratch[:n], st, ws, stream)
            stream.synchronize()                                   # nnz is needed to right-size
            nnz = place.read()
            place.give_back()
            return packed if self._settle(packed, nnz, scratch, ws) else t
        finally:
            st.give_scratch(scratch)

    @staticmethod
    def _compress(t, packed, values, st, ws, stream):
        """bt_compress_indexed of `t`, nnz to a place on the host, which is returned.  (Through device memory it took a kernel for
        the status and a copy.)"""
        place = st.place()
        place.word[0] = -1
        status = bt.lib().bt_compress_indexed(
            t.data_ptr(), t.numel(), bt.dtype_code(t.dtype), packed.bitmap.data_ptr(), values.data_ptr(), values.numel(), place.address,
            packed.index.data_ptr(), ws.data_ptr(), ws.numel(), stream.cuda_stream)
        if status not in (bt.BT_OK, bt.BT_ERR_HIP):                # refused: nothing is queued that could write to it
            place.give_back()
        bt._check("bt_compress_indexed", status)
        return place

    def _unpack(self, obj):
        if not isinstance(obj, _Packed):
            return obj
        if _elsewhere(obj.device):
            with torch.cuda.device(obj.device):
                return self._unpack(obj)
        if obj.pending:
            self._finish_waiting(only=obj)
        if obj.dense is not None:
            return obj.dense
        out = _native().unpack(obj.bitmap, obj.values, obj.index, obj.shape)
        if out is None:
            out = torch.empty(obj.shape, dtype=obj.dtype, device=obj.device)
            bt.bt_decompress_indexed(obj.bitmap, obj.values, obj.index, out)
        return out


def _held(t):
    """`t`, or a copy of it if its memory does not hold its values (a negated view, a zero tensor)."""
    return torch.zeros_like(t) if t._is_zerotensor() else t.resolve_neg()


class _BitmapReLU(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, fused):
        if not fused:
            done = _native().relu(x)
            if done is not None:
                y, ctx.bitmap = done
                return y
        if not (x.is_cuda and x.dtype in _SUPPORTED and x.is_contiguous()):
            raise TypeError("bitmap_relu needs a contiguous float64/float32/float16/bfloat16 device tensor")
        if _elsewhere(x.device):
            with torch.cuda.device(x.device):
                return _BitmapReLU.forward(ctx, x, fused)
        n = x.numel()
        bitmap = torch.empty((n + 31) // 32, dtype=torch.int32, device=x.device)
        if fused:
            # y = x where x > 0 else +0 (a NaN input gives 0 here, NaN in torch.relu); capacity 0: no value is written
            x = _held(x)
            y = torch.empty_like(x)
            st = _state(x.device)
            bt.bt_activation_compress(x, 0.0, y, bitmap, torch.empty(0, dtype=x.dtype, device=x.device), st.nnz, st.workspace(n, x.dtype))
        elif not (x.is_neg() or x._is_zerotensor()) and x.data_ptr() % 16 == 0:
            y = torch.empty_like(x)
            bt.bt_relu_forward(x, y, bitmap)
        else:                             # (a view off a 16-byte boundary, or whose memory does not hold its values; y is neither)
            y = torch.relu(x)
            bt.bt_relu_forward(y, y, bitmap)
        ctx.bitmap = bitmap
        return y

    @staticmethod
    def backward(ctx, grad_out):
        grad_in = _native().relu_gradient(ctx.bitmap, grad_out)
        if grad_in is not None:
            return grad_in, None
        if _elsewhere(grad_out.device):
            with torch.cuda.device(grad_out.device):
                return _BitmapReLU.backward(ctx, grad_out)
        grad_out = _held(grad_out.contiguous())
        if grad_out.data_ptr() % 16 != 0:      # (a part of a concatenation's gradient)
            grad_out = grad_out.clone()
        grad_in = torch.empty_like(grad_out)
        bt.bt_relu_backward_from_bitmap(ctx.bitmap, grad_out, grad_in)
        return grad_in, None


def bitmap_relu(x, fused=False):
    """ReLU that keeps only the 1-bit-per-element mask of its output for backward, both from one pass over x.
    fused=True takes bt_activation_compress for it, which differs for NaN inputs only (0 instead of NaN)."""
    return _BitmapReLU.apply(x, fused)
