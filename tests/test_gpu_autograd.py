"""The codec inside a PyTorch graph (GPU): because the round trip is bit-exact, gradients
with compressed saved activations are identical to those of the plain graph."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ag():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2110_15362_amd import autograd
    return autograd


def _mlp(seed, dtype):
    g = torch.Generator().manual_seed(seed)
    w1 = (torch.randn(1024, 512, generator=g) * 0.05).to(dtype).cuda().requires_grad_()
    w2 = (torch.randn(768, 1024, generator=g) * 0.05).to(dtype).cuda().requires_grad_()
    w3 = (torch.randn(64, 768, generator=g) * 0.05).to(dtype).cuda().requires_grad_()
    x = torch.randn(2048, 512, generator=g).to(dtype).cuda().requires_grad_()
    return x, (w1, w2, w3)


def _forward(x, ws, relu):
    h = relu(torch.nn.functional.linear(x, ws[0]))
    h = relu(torch.nn.functional.linear(h, ws[1]))
    return torch.nn.functional.linear(h, ws[2]).float().pow(2).mean()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_saved_tensor_hooks_give_identical_gradients(ag, dtype):
    x, ws = _mlp(1, dtype)
    _forward(x, ws, torch.relu).backward()
    ref = [t.grad.clone() for t in (x,) + ws]
    for t in (x,) + ws:
        t.grad = None
    stash = ag.BitmapStash(min_numel=1024)
    with stash:
        loss = _forward(x, ws, torch.relu)
    loss.backward()
    for r, t in zip(ref, (x,) + ws):
        assert torch.equal(r, t.grad)
    # the two ReLU outputs (about half zeros) were compressed; the dense input was not worth it
    assert stash.stats["compressed"] >= 2
    assert stash.stats["stored_bytes"] < 0.8 * stash.stats["dense_bytes"]


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_bitmap_relu_backward_matches_torch(ag, dtype, fused):
    x, ws = _mlp(2, dtype)
    ref_loss = _forward(x, ws, torch.relu)
    ref_loss.backward()
    ref = [t.grad.clone() for t in (x,) + ws]
    for t in (x,) + ws:
        t.grad = None
    loss = _forward(x, ws, lambda t: ag.bitmap_relu(t, fused=fused))
    loss.backward()
    assert torch.equal(loss, ref_loss)
    for r, t in zip(ref, (x,) + ws):
        assert torch.equal(r, t.grad)


def _relu_mlp_step(ag, stash, layers, batch, hidden, seed=0, deferred=False):
    """Forward and backward of y = relu(... relu(x W_0) ... W_{L-1}), sum as loss.  Returns the gradients, the
    peak of allocated device memory above what was allocated before the step, and the stash's counters."""
    import contextlib
    g = torch.Generator(device="cuda").manual_seed(seed)
    ws = [(torch.randn(hidden, hidden, device="cuda", generator=g) / hidden ** 0.5).requires_grad_() for _ in range(layers)]
    x = torch.randn(batch, hidden, device="cuda", generator=g)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    ctx = ag.BitmapStash(deferred=deferred) if stash else contextlib.nullcontext()
    with ctx:
        y = x
        for w in ws:
            y = ag.bitmap_relu(y @ w) if stash else torch.relu(y @ w)
        loss = y.sum()
    loss.backward()
    torch.cuda.synchronize()
    peak = torch.cuda.max_memory_allocated() - before
    return [w.grad for w in ws], peak, (ctx.stats if stash else None)


def test_stash_lowers_peak_memory_of_a_step(ag):
    """16 layers whose saved activations are 32 MiB each (512 MiB dense, about half of the elements zero): with the
    stash the step's peak of allocated memory is clearly lower, and the gradients are the same bits."""
    layers, batch, hidden = 16, 8192, 1024
    grads_off, peak_off, _ = _relu_mlp_step(ag, False, layers, batch, hidden)
    grads_on, peak_on, stats = _relu_mlp_step(ag, True, layers, batch, hidden)
    assert stats["dense_bytes"] >= 100 * 1000 * 1000 and stats["compressed"] >= layers - 1 and stats["failed"] == 0
    assert stats["stored_bytes"] < 0.65 * stats["dense_bytes"]
    assert peak_on < 0.85 * peak_off, (peak_on, peak_off)
    for a, b in zip(grads_on, grads_off):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    print("peak MiB without / with the stash: %.0f / %.0f; stored %.0f of %.0f MiB" % (
        peak_off / 2**20, peak_on / 2**20, stats["stored_bytes"] / 2**20, stats["dense_bytes"] / 2**20))


def test_deferred_stash_gives_the_same_gradients_without_waiting_for_the_device(ag):
    layers, batch, hidden = 8, 4096, 1024
    grads_off, peak_off, _ = _relu_mlp_step(ag, False, layers, batch, hidden, seed=3)
    grads_on, peak_on, stats = _relu_mlp_step(ag, True, layers, batch, hidden, seed=3, deferred=True)
    assert stats["tensors"] >= layers and stats["compressed"] >= layers - 1 and stats["failed"] == 0
    assert stats["stored_bytes"] < 0.75 * stats["dense_bytes"]        # (the dense input and the weights pass through too)
    for a, b in zip(grads_on, grads_off):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16, torch.float16, torch.float64])
def test_relu_forward_is_torch_relu_with_its_bitmap(ag, dt):
    """Every 16-bit pattern, and for wider elements the borders between kinds of numbers and random bits: torch's ReLU bit by
    bit (NaNs keep theirs, -0 becomes +0); sizes around words, vectors and workgroups (4 KiB) and on both sides of the change to
    loads past the caches (48 MiB); in place and not; nothing beyond the ends."""
    from paper_2110_15362_amd import bittrain as bt
    width = dt.itemsize
    iv = {2: torch.int16, 4: torch.int32, 8: torch.int64}[width]
    last = (48 << 20) // width
    g = torch.Generator(device="cuda").manual_seed(4)
    if width == 2:
        special = torch.arange(-(1 << 15), 1 << 15, device="cuda").to(iv)
    else:
        inf = {4: 0x7F800000, 8: 0x7FF0000000000000}[width]
        top = -(1 << (8 * width - 1))      # the sign
        special = torch.tensor([0, 1, inf - 1, inf, inf + 1, top - 1 & 0x7FFFFFFF, top, top + 1, top + inf - 1, top + inf, top + inf + 1, -1],
                               dtype=torch.int64, device="cuda").to(iv)
    bits = torch.randint(torch.iinfo(iv).min, torch.iinfo(iv).max, (last + 5 + 16,), generator=g, device="cuda", dtype=iv)
    bits[:special.numel()] = special
    block = 4096 // width
    for n in (1, 31, 33, block - 1, block, block + 1, 65 * block + 7, 70000, last, last + 5):
        words = (n + 31) // 32
        for inplace in (False, True):
            x = bits[:n + 16].clone()
            out = x if inplace else torch.full_like(x, 0x5A)
            guard = out[n:].clone()
            assert guard.numel() == 16
            bitmap = torch.full((words + 2,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
            want = torch.relu(x[:n].clone().view(dt)).view(iv)
            bt.bt_relu_forward(x[:n].view(dt), out[:n].view(dt), bitmap[:words])
            assert torch.equal(out[:n], want), (n, inplace)
            assert torch.equal(out[n:], guard) and bool((bitmap[words:] == 0x5A5A5A5A).all()), (n, inplace)
            kept = torch.zeros(words * 32, dtype=torch.int64, device="cuda")
            kept[:n] = want != 0
            packed = (kept.view(-1, 32) << torch.arange(32, device="cuda")).sum(1)
            assert torch.equal(bitmap[:words].to(torch.int64) & 0xFFFFFFFF, packed), (n, inplace)


def test_bitmap_relu_takes_views_off_a_16_byte_boundary_and_empty_tensors(ag):
    base = torch.randn(4097, device="cuda")
    for x in (base[1:], base[:0], base[:1], torch._neg_view(base)):      # (the last one's memory holds what it is not)
        x = x.clone().detach() if x.numel() < 2 else x.detach()
        x.requires_grad_()
        y = ag.bitmap_relu(x)
        assert torch.equal(y, torch.relu(x.detach()))
        y.sum().backward()
        assert torch.equal(x.grad, (x.detach() > 0).float())


@pytest.mark.parametrize("deferred", [False, True])
def test_stash_keeps_what_a_failed_compression_was_given(ag, deferred, monkeypatch):
    """The grid scan of every compression gives up at once (a limit of one pass): no nnz reaches the host, the tensors are kept
    dense with a warning, the workspace serves the next step, and no place on the host is lost."""
    from paper_2110_15362_amd import bittrain as bt
    n = 300 * bt.bt_tile_elems(torch.float32)
    w = torch.ones(n, device="cuda", requires_grad=True)
    h = torch.relu(torch.randn(n, device="cuda"))
    st = ag._state(h.device)
    words = st.workspace(n, h.dtype).view(torch.int32)

    def step(limit):
        words[bt.BT_WS_WAIT_LIMIT_WORD] = limit
        stash = ag.BitmapStash(deferred=deferred)
        with stash:
            loss = (h * w).sum()
        loss.backward()
        assert torch.equal(w.grad, h)
        w.grad = None
        return stash.stats
    assert step(0)["compressed"] == 1
    places = len(st.places)

    def distinct():
        return len({p.address for p in st.places}) == len(st.places)
    with pytest.warns(UserWarning, match="gave up"):
        assert step(1)["failed"] == 1
    assert len(st.places) == places and distinct()
    stats = step(0)
    assert stats["compressed"] == 1 and stats["failed"] == 0 and len(st.places) == places and distinct()


def test_deferred_packings_of_another_stream(ag):
    """Packed on one stream, settled where the host leaves the stash, on another, and unpacked on the first."""
    x, ws = _mlp(4, torch.float32)
    _forward(x, ws, torch.relu).backward()
    ref = [t.grad.clone() for t in (x,) + ws]
    for t in (x,) + ws:
        t.grad = None
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    stash = ag.BitmapStash(min_numel=1024, deferred=True)
    with stash:
        with torch.cuda.stream(side):
            loss = _forward(x, ws, torch.relu)
    loss.backward()
    torch.cuda.synchronize()
    for r, t in zip(ref, (x,) + ws):
        assert torch.equal(r, t.grad)
    assert stash.stats["compressed"] >= 2 and stash.stats["failed"] == 0


def test_bitmap_relu_in_a_concatenation(ag):
    """Its gradient is a view that begins where the other part ends, off every 16-byte boundary."""
    x = torch.randn(4099, device="cuda", requires_grad=True)
    w = torch.randn(3 + 4099, device="cuda")
    (torch.cat([torch.ones(3, device="cuda"), ag.bitmap_relu(x)]) * w).sum().backward()
    assert torch.equal(x.grad, torch.where(x.detach() > 0, w[3:], 0))


@pytest.mark.parametrize("fused", [False, True])
def test_negated_views_are_what_they_look_like(ag, fused):
    """In the stash (saved by a product), through bitmap_relu, and as the gradient that comes back to it."""
    h = torch.relu(torch.randn(8192, device="cuda"))
    w = torch.ones(8192, device="cuda", requires_grad=True)
    with ag.BitmapStash():
        loss = (torch._neg_view(h) * w).sum()
    loss.backward()
    assert torch.equal(w.grad, -h)
    x = torch.randn(8192, device="cuda").requires_grad_()
    y = ag.bitmap_relu(torch._neg_view(x), fused=fused)
    assert torch.equal(y, torch.relu(-x))
    y.backward(torch._neg_view(h))
    assert torch.equal(x.grad, torch.where(x < 0, h, 0))
