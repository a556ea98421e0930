"""The pass with several workgroups per unit (``vd_evict_step_split``) against
the one with a single workgroup, on the same inputs.  The column sums are added
in the same order, so everything agrees bit for bit.  Sizes sit where
the split count changes, at shares of less than a row group and of no row, at
the edges of the staging (all, some and none of the new rows in LDS), at a
single eviction, at units that do not evict, and at the slot limit."""
import ctypes
import os

import pytest
import torch

from paper_2609_23314_amd import build as lib_build
from paper_2609_23314_amd import synth, vd
from paper_2609_23314_amd.driver import EvictingCache
from test_gpu_half_block import cancelling_rows, last_pass

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(params=["release", "debug"])
def library(request):
    saved = (vd._lib, vd.LIB_PATH)
    if request.param == "debug":
        assert os.path.exists(lib_build.DEBUG_LIB), "build the debug library first"
        vd._lib, vd.LIB_PATH = None, lib_build.DEBUG_LIB
    lib = vd.load()
    yield lib if request.param == "debug" else None
    vd._lib, vd.LIB_PATH = saved


def lds_word(library):
    if library is None:
        return 0
    word = ctypes.c_uint32(0)
    library.vd_debug_take_error_word.argtypes = [ctypes.c_void_p]
    assert library.vd_debug_take_error_word(ctypes.byref(word)) == vd.VD_OK
    return word.value


# units as (L, H); n, N and what the state covers, per sequence, from the rows R
# that the longest unit has to have for a split, at least
SHAPES = [lambda R: ((1, 1), [R + 5], [R - 95], [R - 95]),
          lambda R: ((3, 5), [R + 300, R // 2, 0], [R, R // 2 + 100, 4], [R, R // 2 - 50, 0]),
          lambda R: ((4, 5), [R + 1, R // 2 + 1, 40], [R, R // 2, 40], [R, R // 2, 39]),
          lambda R: ((2, 4), [R, R - 299, 900], [400, R - 300, 899], [0, R - 299, 700]),
          lambda R: ((8, 8), [2 * R + 1], [R + R // 2], [R + R // 2]),
          lambda R: ((1, 3), [16384], [16383], [16383]), lambda R: ((1, 2), [16384], [8000], [8000])]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("variant", ["l2", "dir", "norm", "key_norm"])
@pytest.mark.parametrize("D,shape,ties,state", [(D, i, False, True) for D in (64, 128, 256) for i in range(7)] +
                         [(128, 1, True, True)] + [(D, i, False, False) for D in (64, 256) for i in range(5)])
def test_split_matches_whole(library, dtype, variant, D, shape, ties, state):
    (L, H), n, N, count = SHAPES[shape](768 * 1024 // (D * dtype.itemsize))
    S, C = len(n), min(max(n) + 3, 16384)
    U = S * L * H
    k, v = [synth.random_rows((S, L, H, C, D), dtype, 17 + i, DEV) for i in range(2)]
    if ties:
        k, v = [x[:, :, :, :1].expand(-1, -1, -1, C, -1).contiguous() for x in (k, v)]
        v[:, :, :, 5::40] *= 2
        k[:, :, :, 7::50] *= 2
    scored = k if variant.startswith("key") else v
    sums = torch.zeros((S, L, H, D + 1), dtype=torch.float64, device=DEV) if state else None
    for s in range(S if state else 0):
        sums[s, ..., :D] = scored[s, :, :, :count[s]].double().sum(2)
        sums[s, ..., D] = count[s]
    size = vd.vd_evict_step_split_size(v, k)
    assert size > 0
    scratch = torch.full((size,), 0xFF, dtype=torch.uint8, device=DEV)
    runs = []
    for use in (None, scratch):
        a = dict(k=k.clone(), v=v.clone(), pos=torch.arange(C, dtype=torch.int32, device=DEV).repeat(U, 1),
                 scores=torch.zeros((U, C), device=DEV), keep=torch.zeros((U, C), dtype=torch.uint8, device=DEV))
        a["sums"] = sums.clone().view(U, -1) if state else None
        vd.vd_evict_step(a["k"], a["v"], n, N, variant, running_sum=a["sums"], pos=a["pos"], scores_out=a["scores"],
                         keep_out=a["keep"], scratch=use)
        assert lds_word(library) == 0
        if library is not None:  # each of the 256 compute units' share of the units, 64 at most and 64 KB of rows
            most = min(64, 256 // U, max(a for a, b in zip(n, N) if a > b) * D * dtype.itemsize // 65536)
            assert last_pass(library) == (1024, 0 if use is None else most)
        runs.append(a)
    ref, got = runs
    for x in ("k", "v", "pos", "scores", "keep") + (("sums",) if state else ()):
        assert torch.equal(got[x], ref[x]), x


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("variant", ["l2", "dir"])
def test_split_sums_in_the_whole_pass_order(dtype, D, variant):
    """Rows whose sums depend on the order they are added in, without a running sum:
    the scores of the split pass, of the whole one and of vd_score agree."""
    R = 768 * 1024 // (D * dtype.itemsize)
    n = [R + 6, R // 2, 2 * 1024 // dtype.itemsize + 2]
    k, v = [cancelling_rows((3, 2, 3, R + 6, D), dtype, 5 + i) for i in range(2)]
    scratch = torch.full((vd.vd_evict_step_split_size(v, k),), 0xFF, dtype=torch.uint8, device=DEV)
    runs = []
    for use in (None, scratch):
        a = [k.clone(), v.clone(), torch.zeros((18, R + 6), device=DEV)]
        vd.vd_evict_step(*a[:2], n, [m - 100 for m in n], variant, scores_out=a[2], scratch=use)
        runs.append(a)
    for x, y in zip(*runs):
        assert torch.equal(x, y)
    alone = vd.vd_score(v, n, variant, scores=torch.zeros((18, R + 6), device=DEV))[0]
    assert torch.equal(alone, runs[0][2])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("variant,scores,summed", [("norm", True, []), ("key_norm", False, []), ("l2", False, [0]),
                                                   ("l2", True, [0, 1]), ("dir", False, [0])])
def test_columns_are_summed_only_for_a_mean(dtype, variant, scores, summed):
    """Without a running sum: the norms need no column sums, nor does a unit that
    neither evicts nor reports scores (their place in the scratch is left alone)."""
    D, L, H = 128, 1, 3
    n = [768 * 1024 // (D * dtype.itemsize) + 40, 300, 0]
    C, U = n[0], 3 * L * H
    k, v = [synth.random_rows((3, L, H, C, D), dtype, 31 + i, DEV) for i in range(2)]
    scratch = torch.full((vd.vd_evict_step_split_size(v, k),), 0xFF, dtype=torch.uint8, device=DEV)
    part = U * ((C + 3) // 4 * 4) * 4 + U * D * 8
    out = torch.zeros((U, C), device=DEV) if scores else None
    vd.vd_evict_step(k, v, n, [n[0] - 40, 300, 5], variant, scores_out=out, scratch=scratch)
    sums = scratch[part:].view(3, -1)
    assert sums.numel() == U * 16 * D * 8
    assert [s for s in range(3) if bool((sums[s] != 0xFF).any())] == summed


def test_scratch_is_checked():
    k, v = torch.zeros((2, 1, 1, 2, 4096, 128), dtype=torch.bfloat16, device=DEV)  # 1 MB a unit
    size = vd.vd_evict_step_split_size(v, k)
    assert size > 0
    for scratch in (torch.zeros(size - 1, dtype=torch.uint8, device=DEV),
                    torch.zeros(size + 16, dtype=torch.uint8, device=DEV)[1:]):
        with pytest.raises(vd.VdError, match="workspace"):
            vd.vd_evict_step(k, v, [4000], [3000], scratch=scratch)
    k, v = torch.zeros((2, 1, 16, 16, 512, 64), dtype=torch.bfloat16, device=DEV)
    assert vd.vd_evict_step_split_size(v, k) == 0


def test_cache_across_streams():
    """A cache's passes on two streams, ordered by the caller, share its scratch."""
    def run(streams):
        cache = EvictingCache(1, 2, 2, 128, 3328, [3072])
        for b in range(16):
            rows = [synth.random_rows((2, 2, 256, 128), torch.bfloat16, 2 * b + i, DEV) for i in range(2)]
            cache.append(0, *rows)
            s = streams[b % len(streams)]
            if s is not None:
                s.wait_stream(torch.cuda.current_stream())
            cache.evict(stream=s)
            if s is not None:
                torch.cuda.current_stream().wait_stream(s)
        return cache
    a, b = run([None]), run([torch.cuda.Stream(), None, torch.cuda.Stream()])
    for x, y in ((a.k, b.k), (a.v, b.v), (a.pos, b.pos), (a.running_sum, b.running_sum)):
        assert torch.equal(x, y)


def test_graph_outlives_its_cache():
    """A captured pass writes to the cache's tensors and to memory of the graph's
    own: with the cache object gone and the freed memory given to other tensors,
    replays leave those alone and give the eager results."""
    L, H, D, N, n = 2, 2, 128, 8000, 8192
    cache = EvictingCache(1, L, H, D, n, [N], device=DEV)
    size = vd.vd_evict_step_split_size(cache.v, cache.k)
    assert size > 0
    for x, seed in ((cache.k, 5), (cache.v, 6)):
        x.copy_(synth.random_rows((1, L, H, n, D), torch.bfloat16, seed, DEV))
    cache.running_sum.view(L * H, D + 1)[:, :D] = cache.v[0, :, :, :N].double().sum(2).view(L * H, D)
    cache.running_sum.view(L * H, D + 1)[:, D] = N
    cache.pos.copy_(torch.arange(n, dtype=torch.int32, device=DEV).expand(L * H, -1))
    held = [cache.k, cache.v, cache.running_sum, cache.pos]
    start = [x.clone() for x in held]
    cache.n = [n]
    cache.evict()                               # eager
    want = [x.clone() for x in held]
    cache.n = [n]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cache.evict()
    del cache
    others = [torch.full((size,), 7, dtype=torch.uint8, device=DEV) for _ in range(4)]
    for rep in range(3):
        for x, y in zip(held, start):
            x.copy_(y)
        work = torch.randn(1 << 20, device=DEV).sum()   # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(held, want)), (rep, float(work))
        assert all(bool((x == 7).all()) for x in others), rep


class _Handle:
    """A stream known by its handle alone, as another library hands it over."""
    def __init__(self, stream):
        self.cuda_stream = stream.cuda_stream


@pytest.mark.parametrize("wrap", [lambda s: s, _Handle], ids=["stream", "handle"])
@pytest.mark.parametrize("which", ["current", "side", "default"])
def test_scratch_belongs_to_the_stream_of_its_call(which, wrap):
    """What a call takes from torch goes back to the stream that the call ran on."""
    s = {"current": torch.cuda.current_stream, "side": torch.cuda.Stream, "default": torch.cuda.default_stream}[which]()
    size = 64 << 20  # a segment of its own
    buf = vd._call_scratch(size, torch.device("cuda", torch.cuda.current_device()), wrap(s))
    owner = [x["stream"] for x in torch.cuda.memory_snapshot()
             if x["address"] <= buf.data_ptr() < x["address"] + x["total_size"]]
    assert owner == [s.cuda_stream]
    with torch.cuda.stream(s):
        own = vd._call_scratch(size, buf.device, None)
    owner = [x["stream"] for x in torch.cuda.memory_snapshot()
             if x["address"] <= own.data_ptr() < x["address"] + x["total_size"]]
    assert owner == [s.cuda_stream]


@pytest.mark.parametrize("wrap", [lambda s: s, _Handle], ids=["stream", "handle"])
def test_call_takes_its_own_scratch(wrap):
    k, v = [synth.random_rows((1, 2, 2, 6150, 64), torch.bfloat16, 3 + i, DEV) for i in range(2)]
    ref = [k.clone(), v.clone()]
    vd.vd_evict_step(*ref, [6150], [6000])
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    vd.vd_evict_step(k, v, [6150], [6000], scratch=True, stream=wrap(s))
    torch.cuda.current_stream().wait_stream(s)
    assert torch.equal(k, ref[0]) and torch.equal(v, ref[1])


def test_pass_without_memory_for_its_scratch(monkeypatch):
    """Where torch has no memory for the scratch the pass runs with one workgroup per unit."""
    k, v = [synth.random_rows((1, 2, 2, 6150, 64), torch.bfloat16, 3 + i, DEV) for i in range(2)]
    ref = [k.clone(), v.clone()]
    vd.vd_evict_step(*ref, [6150], [6000])

    def none_left(*a, **kw):
        raise torch.OutOfMemoryError("no memory")

    with monkeypatch.context() as m:
        m.setattr(torch, "empty", none_left)
        vd.vd_evict_step(k, v, [6150], [6000], scratch=True)
    assert torch.equal(k, ref[0]) and torch.equal(v, ref[1])
