"""The cache object of block prompt processing (Sec. 2.2): what it holds, and
what torch follows of its appends."""
import pytest
import torch
from torch.autograd import forward_ad
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2609_23314_amd import vd
from paper_2609_23314_amd.driver import EvictingCache


def test_cache_keeps_no_scratch(monkeypatch):
    """A cache holds what its constructor made and nothing of a pass: one made (or
    pickled) with these attributes alone evicts, and is left with them."""
    names = {"k", "v", "units", "n", "seen", "budget", "variant", "num_q_heads", "running_sum", "pos", "capacity"}
    made = EvictingCache(1, 1, 1, 64, 8, [4], dtype=torch.float32, device="cpu")
    cache = EvictingCache.__new__(EvictingCache)
    cache.__dict__.update({a: getattr(made, a) for a in names})
    monkeypatch.setattr(vd, "vd_evict_step", lambda *a, **kw: None)
    cache.n = [6]
    cache.evict()
    assert cache.n == [4] and set(vars(cache)) == names == set(vars(made))


# ---- what torch does around the copies of an append reaches the cache on either device

DEVICES = ["cpu", pytest.param("cuda", marks=pytest.mark.gpu)]


def _cache(device):
    return EvictingCache(1, 2, 3, 64, 40, [40], dtype=torch.float32, device=device)


def _new_rows(device, seed=0):
    g = torch.Generator().manual_seed(seed)
    return torch.randn((2, 3, 6, 64), generator=g).to(device)


@pytest.mark.parametrize("device", DEVICES)
def test_append_carries_forward_mode_tangents(device):
    rows, tangent, cache = _new_rows(device), _new_rows(device, 1), _cache(device)
    with forward_ad.dual_level():
        cache.append(0, forward_ad.make_dual(rows, tangent), rows)
        got = forward_ad.unpack_dual(cache.k).tangent
        assert got is not None and torch.equal(got[0, :, :, :6], tangent) and not got[0, :, :, 6:].any()
        assert torch.equal(forward_ad.unpack_dual(cache.k).primal[0, :, :, :6], rows)


@pytest.mark.parametrize("device", DEVICES)
def test_append_under_functorch(device):
    rows, tangent = _new_rows(device), _new_rows(device, 1)

    def kept(x):
        cache = _cache(device)
        cache.append(0, x, rows)
        return cache.k

    value, out = torch.func.jvp(kept, (rows,), (tangent,))
    assert torch.equal(value[0, :, :, :6], rows) and torch.equal(out[0, :, :, :6], tangent)
    with pytest.raises(RuntimeError, match="vmap: inplace"):
        torch.func.vmap(kept)(torch.stack([rows, rows]))


class _Ops(TorchDispatchMode):
    def __init__(self):
        super().__init__()
        self.names = []

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        self.names.append(func.__name__)
        return func(*args, **(kwargs or {}))


class _Functions(TorchFunctionMode):
    def __init__(self):
        super().__init__()
        self.names = []

    def __torch_function__(self, func, types, args=(), kwargs=None):
        self.names.append(getattr(func, "__name__", ""))
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("mode", [_Ops, _Functions])
@pytest.mark.parametrize("device", DEVICES)
def test_append_shows_its_copies_to_modes(device, mode):
    rows, cache = _new_rows(device), _cache(device)
    with mode() as seen:
        cache.append(0, rows, rows)
    assert sum(name.startswith("copy_") for name in seen.names) >= 2, seen.names
    assert torch.equal(cache.k[0, :, :, :6], rows) and torch.equal(cache.v[0, :, :, :6], rows)


@pytest.mark.parametrize("device", DEVICES)
def test_append_compiles_whole(device):
    rows, cache = _new_rows(device), _cache(device)
    torch.compile(cache.append, fullgraph=True, backend="eager")(0, rows, rows)
    assert cache.n == [6] and torch.equal(cache.k[0, :, :, :6], rows) and torch.equal(cache.v[0, :, :, :6], rows)


@pytest.mark.gpu
def test_append_takes_a_default_device():
    """A default device alone is no reason to copy with torch."""
    rows, cache = _new_rows("cuda"), _cache("cuda")
    with torch.device("cuda"):
        assert vd.vd_append(cache.k, cache.v, 0, 0, rows, rows, cache.pos, 0)
    assert torch.equal(cache.k[0, :, :, :6], rows)


@pytest.mark.parametrize("device", DEVICES)
def test_append_counts_as_an_inplace_change(device):
    """Each append moves the version counters as torch's copies do, so that a backward
    through rows saved before it is refused instead of reading the changed ones."""
    rows, cache = _new_rows(device), _cache(device)
    cache.append(0, rows, rows)
    w = torch.ones((), device=device, requires_grad=True)
    products = [(x * w).sum() for x in (cache.k, cache.v)]
    before = [x._version for x in (cache.k, cache.v, cache.pos)]
    cache.append(0, rows, rows)
    assert all(x._version > b for x, b in zip((cache.k, cache.v, cache.pos), before))
    for y in products:
        with pytest.raises(RuntimeError, match="modified by an inplace operation"):
            y.backward()


@pytest.mark.parametrize("device", DEVICES)
def test_append_and_inference_tensors(device):
    rows = _new_rows(device)
    with torch.inference_mode():
        cache = _cache(device)
        cache.append(0, rows, rows)
        assert torch.equal(cache.v[0, :, :, :6], rows)
    with pytest.raises(RuntimeError, match="[Ii]nference"):
        cache.append(0, rows, rows)
    made = _cache(device)
    with torch.inference_mode():
        made.append(0, rows, rows)
    assert torch.equal(made.k[0, :, :, :6], rows)
