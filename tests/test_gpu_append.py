"""Appending rows (Sec. 2.2, Eq. block_processing): the one-launch append
against plain copies, bit for bit, at the edges of its tiles (a workgroup
takes 1024 16-byte chunks of one unit, or several units with at most 128),
and the rows and caches it leaves to torch's copies."""
import ctypes

import pytest
import torch

from paper_2609_23314_amd import vd
from paper_2609_23314_amd.driver import EvictingCache

gpu = pytest.mark.gpu
DEV = "cuda"


def _rows(L, H, t, D, dtype, seed, device=DEV):
    g = torch.Generator(device=device).manual_seed(seed)
    return torch.randn((L, H, t, D), generator=g, device=device).to(dtype)


def _check(cache, k0, v0, p0, seq, n0, k_rows, v_rows, seen):
    t, per = k_rows.shape[2], cache.k.shape[1] * cache.k.shape[2]
    k0[seq, :, :, n0:n0 + t] = k_rows
    v0[seq, :, :, n0:n0 + t] = v_rows
    p0[seq * per:(seq + 1) * per, n0:n0 + t] = torch.arange(seen, seen + t, device=p0.device)
    assert torch.equal(cache.k, k0) and torch.equal(cache.v, v0) and torch.equal(cache.pos, p0)


@gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("L,H", [(1, 1), (3, 5)])
def test_append_matches_copies(dtype, D, L, H):
    per_tile = 1024 // (D * dtype.itemsize // 16)          # rows of a full workgroup
    sizes = [1, 2, 7, 8, 9, per_tile - 1, per_tile, per_tile + 1, 2 * per_tile + 3]
    cache = EvictingCache(2, L, H, D, sum(sizes) + 5, [10 ** 6] * 2, dtype=dtype, device=DEV)
    k0, v0, p0 = cache.k.clone(), cache.v.clone(), cache.pos.clone()
    long = _rows(L, H, 2 * per_tile + 20, D, dtype, 7)
    for i, t in enumerate(sizes):
        for seq in (1, 0):
            n0, seen = cache.n[seq], cache.seen[seq]
            k_rows = long[:, :, i:i + t]                                    # a part of a longer prompt
            v_rows = _rows(H, L, t, D, dtype, i).transpose(0, 1)            # heads before layers
            assert vd.vd_append(cache.k, cache.v, seq, n0, k_rows, v_rows, cache.pos, seen)
            cache.append(seq, k_rows, v_rows)
            _check(cache, k0, v0, p0, seq, n0, k_rows, v_rows, seen)


@gpu
def test_append_leaves_other_rows_to_copies():
    """Rows of another type, device, layout or gradient, and rows of the cache
    itself, give what torch's copies give."""
    L, H, D, t = 2, 3, 64, 6
    good = _rows(L, H, t, D, torch.float32, 1)
    offset = torch.empty(good.numel() + 1, device=DEV)[1:].view(good.shape).copy_(good)   # not 16-byte aligned
    for k_rows in (good.to(torch.bfloat16), good.cpu(), good.transpose(2, 3).contiguous().transpose(2, 3),
                   offset, good[:, :1], good.double()):
        cache = EvictingCache(1, L, H, D, 40, [40], dtype=torch.float32, device=DEV)
        k0, v0, p0 = cache.k.clone(), cache.v.clone(), cache.pos.clone()
        assert not vd.vd_append(cache.k, cache.v, 0, 0, k_rows, good, cache.pos, 0)
        cache.append(0, k_rows, good)
        _check(cache, k0, v0, p0, 0, 0, k_rows, good, 0)
    cache = EvictingCache(1, L, H, D, 40, [40], dtype=torch.float32, device=DEV)
    cache.append(0, good, good + 1)
    assert not vd.vd_append(cache.k, cache.v, 0, t, cache.v[0, :, :, :t], good, cache.pos, t)
    assert not vd.vd_append(cache.k, cache.v, 0, t, good.clone().requires_grad_(), good, cache.pos, t)
    cache.append(0, cache.v[0, :, :, :t], good)
    assert torch.equal(cache.k[0, :, :, t:2 * t], good + 1) and torch.equal(cache.v[0, :, :, t:2 * t], good)


@pytest.mark.parametrize("k_rows", [torch.ones(2, 3, 4, 64), torch.ones(1, 1, 4, 64, dtype=torch.float64)])
def test_append_on_the_cpu(k_rows):
    cache = EvictingCache(2, 2, 3, 64, 10, [4, 4], dtype=torch.float32, device="cpu")
    cache.append(1, k_rows, torch.full((2, 3, 4, 64), 2.0))
    assert cache.n == [0, 4] and cache.seen == [0, 4]
    assert cache.k[1, :, :, :4].eq(1).all() and cache.v[1, :, :, :4].eq(2).all() and not cache.k[0].any()
    assert cache.pos[6:, :4].eq(torch.arange(4)).all() and cache.pos[:6].eq(-1).all()


def test_append_rejects_bad_arguments():
    d = vd.VdCacheDesc()
    d.k, d.v = 0x7F0000000000, 0x7F0100000000
    d.dtype, d.head_dim, d.capacity = vd.VD_DTYPE_BF16, 64, 32
    d.num_seqs, d.num_layers, d.num_kv_heads, d.num_q_heads = 2, 3, 4, 4
    d.stride_slot, d.stride_head, d.stride_layer, d.stride_seq = 64, 2048, 8192, 24576
    good = dict(seq=1, n_old=4, rows=8, k=0x7E0000000000, ks=(4096, 1024, 64), v=0x7E0100000000, vs=(4096, 1024, 64),
                pos=None, pos0=0)

    def call(**kw):
        a = {**good, **kw}
        s = ctypes.c_int64 * 3
        return vd.load().vd_append(ctypes.byref(d), a["seq"], a["n_old"], a["rows"], a["k"], s(*a["ks"]), a["v"],
                                   s(*a["vs"]), a["pos"], a["pos0"], None)

    for bad in (dict(seq=2), dict(seq=-1), dict(n_old=-1), dict(rows=0), dict(rows=29), dict(k=None), dict(v=None),
                dict(k=0x7E0000000008), dict(ks=(4096, 1024, 63)), dict(vs=(-8, 1024, 64)), dict(pos0=-1),
                dict(pos0=2 ** 31 - 8), dict(pos=0x7D0000000002), dict(ks=(2 ** 60, 0, 0)),
                dict(k=0x7F0000000000 + 2 * 49152 - 128),    # the cache's last row
                dict(v=0x7F0000000000 - 64), dict(k=0x7F0100000000)):
        assert call(**bad) == vd.VD_ERR_INVALID_ARG, bad
    d.head_dim = 96
    assert call() == vd.VD_ERR_UNSUPPORTED


@pytest.mark.parametrize("stride", ["stride_layer", "stride_head"])
def test_append_rejects_units_that_share_memory(stride):
    d = vd.VdCacheDesc()
    d.k, d.v = 0x7F0000000000, 0x7F0100000000
    d.dtype, d.head_dim, d.capacity = vd.VD_DTYPE_BF16, 64, 32
    d.num_seqs, d.num_layers, d.num_kv_heads, d.num_q_heads = 2, 3, 4, 4
    d.stride_slot, d.stride_head, d.stride_layer, d.stride_seq = 64, 2048, 8192, 24576
    setattr(d, stride, 0)
    s = (ctypes.c_int64 * 3)(4096, 1024, 64)
    assert vd.load().vd_append(ctypes.byref(d), 0, 0, 8, 0x7E0000000000, s, 0x7E0100000000, s, None, 0,
                               None) == vd.VD_ERR_INVALID_ARG


@pytest.mark.parametrize("device", ["cpu", pytest.param("cuda", marks=gpu)])
@pytest.mark.parametrize("shape", [(1, 1, 3), (1, 2, 1)])
def test_append_to_an_expanded_cache_is_refused(device, shape):
    """As torch refuses to copy into memory that several units share."""
    cache = EvictingCache(1, 2, 3, 64, 40, [40], dtype=torch.float32, device=device)
    cache.k, cache.v = [torch.zeros((*shape, 40, 64), device=device).expand(1, 2, 3, 40, 64) for _ in range(2)]
    rows = torch.ones((2, 3, 4, 64), device=device)
    with pytest.raises(RuntimeError, match="single memory location"):
        cache.append(0, rows, rows)
    assert cache.n == [0] and cache.seen == [0] and not cache.k.any() and not cache.v.any()
