"""The autograd steps on ordinary tensors, which one call in C++ takes with its allocations, against the same steps on a subclass, which
go the general way call by call: the same bytes, the same decisions and the same statistics."""
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
    for shape, zeros in (((4096,), 0.5), ((3, 7, 411), 0.9), ((260 * 8192 + 13,), 0.5), ((64, 64), 1.0), ((10, 1000), 0.0), ((1001, 1003), 0.02)):
        x = torch.randn(shape, generator=g, device="cuda").to(dtype)
        x[torch.rand(shape, generator=g, device="cuda") < zeros] = 0
        x.view(-1)[7] = float("nan")
        got = []
        for t in (x, x.as_subclass(_Sub)):
            stash = ag.BitmapStash(deferred=deferred)
            packed = stash._pack(t)
            stash._finish_waiting(block=True)
            got.append((stash, packed, packed if packed is t else stash._unpack(packed)))
        (s0, p0, u0), (s1, p1, u1) = got
        assert s0.stats == s1.stats and u0.shape == x.shape and u0.dtype == dtype
        assert torch.equal(_bytes(u0), _bytes(x)) and torch.equal(_bytes(u1), _bytes(x))
        assert isinstance(p0, ag._Packed) == isinstance(p1, ag._Packed)
        if isinstance(p0, ag._Packed) and p0.dense is None:
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
