"""The pass with two workgroups per CU (launches of more than 256 units whose
rows to stage fit half the LDS, or are 128 bytes each) against the same sequences one at a time, which
take the full workgroup: scores, kept sets, rows, positions and state bit for bit.
Cases sit at the edges of the row tiles (512 threads take 256 to 32
rows per chunk column), of the staging, and of the selection (no eviction, one
row, a crossing fill, all keys equal).

The fp64 column sums are added in one order whatever the workgroup's size, which
the last test asks with rows whose sums depend on it."""
import ctypes
import os

import pytest
import torch

from paper_2609_23314_amd import build as lib_build
from paper_2609_23314_amd import synth, vd

pytestmark = pytest.mark.gpu
DEV = "cuda"
S, L, H = 3, 12, 8                    # 288 units in one launch, 96 in each of three

SIZES = [([130, 97, 64], [100, 96, 64]), ([67, 2, 1], [3, 1, 1]), ([1030, 700, 513], [1000, 690, 512]),
         ([300, 290, 80], [256, 257, 70])]


@pytest.fixture(params=["release", "debug"])
def library(request):
    saved = (vd._lib, vd.LIB_PATH)
    if request.param == "debug":
        assert os.path.exists(lib_build.DEBUG_LIB), "build the debug library first"
        vd._lib, vd.LIB_PATH = None, lib_build.DEBUG_LIB
    lib = vd.load()
    yield lib if request.param == "debug" else None
    vd._lib, vd.LIB_PATH = saved


def last_pass(library):
    """Threads per workgroup and splits of this thread's last pass (debug build)."""
    threads, splits = ctypes.c_int32(-1), ctypes.c_int32(-1)
    assert library.vd_debug_last_pass(ctypes.byref(threads), ctypes.byref(splits)) == vd.VD_OK
    return threads.value, splits.value


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("variant", ["l2", "dir", "norm", "key_norm"])
@pytest.mark.parametrize("D,n,N,ties", [(D, n, N, False) for D in (64, 128, 256) for n, N in SIZES] +
                         [(128, *SIZES[3], True), (64, [2300, 2100, 2050], [1300, 1500, 2050], False),
                          (64, [2300, 2100, 2050], [2200, 2060, 2050], False), (256, [40, 2, 1], [3, 1, 1], False)])
def test_half_block_matches_full(library, dtype, D, variant, n, N, ties):
    C, U = max(n) + 3, S * L * H
    k, v = [synth.random_rows((S, L, H, C, D), dtype, 91 + i, DEV) for i in range(2)]
    if ties:
        k, v = [x[:, :, :, :1].expand(-1, -1, -1, C, -1).contiguous() for x in (k, v)]
        v[:, :, :, 5::40] *= 2
        k[:, :, :, 7::50] *= 2
    scored = k if variant.startswith("key") else v
    count = [min(a, b) for a, b in zip(n, N)]
    count[2] = max(0, count[2] - 5)   # one sequence's state lags behind
    sums = torch.zeros((S, L, H, D + 1), dtype=torch.float64, device=DEV)
    for s in range(S):
        sums[s, ..., :D] = scored[s, :, :, :count[s]].double().sum(2)
        sums[s, ..., D] = count[s]
    pos = torch.arange(C, dtype=torch.int32, device=DEV).repeat(U, 1)
    one = [x.clone() for x in (k, v, sums, pos)]
    got = dict(scores=torch.zeros((U, C), device=DEV), keep=torch.zeros((U, C), dtype=torch.uint8, device=DEV))
    ref = {a: x.clone() for a, x in got.items()}
    vd.vd_evict_step(k, v, n, N, variant, running_sum=sums.view(U, -1), pos=pos, scores_out=got["scores"],
                     keep_out=got["keep"])
    if library is not None:  # fp32 rows that half the LDS cannot stage take the full workgroup here too
        full = dtype == torch.float32 and ((D == 256 and n[0] == 67) or (D == 64 and N[0] == 1300))
        assert last_pass(library) == (1024 if full else 512, 0)
    for s in range(S):
        u = slice(s * L * H, (s + 1) * L * H)
        vd.vd_evict_step(one[0][s:s + 1], one[1][s:s + 1], n[s:s + 1], N[s:s + 1], variant,
                         running_sum=one[2][s].view(L * H, -1), pos=one[3][u], scores_out=ref["scores"][u],
                         keep_out=ref["keep"][u])
        assert library is None or last_pass(library) == (1024, 0)
    for a, b in zip((k, v, pos), (one[0], one[1], one[3])):
        assert torch.equal(a, b)
    assert torch.equal(got["keep"], ref["keep"]) and torch.equal(got["scores"], ref["scores"])
    assert torch.equal(sums, one[2])
    if library is not None:
        word = ctypes.c_uint32(0)
        library.vd_debug_take_error_word.argtypes = [ctypes.c_void_p]
        assert library.vd_debug_take_error_word(ctypes.byref(word)) == vd.VD_OK and word.value == 0


def cancelling_rows(shape, dtype, seed):
    """Rows of three scales 2^0, 2^30 and 2^55 whose large ones cancel exactly, so
    that what an fp64 sum of them keeps of the small ones depends on its order."""
    x = synth.random_rows(shape, torch.float32, seed, DEV)
    g = torch.Generator(device=DEV).manual_seed(seed)
    C, half = shape[-2], shape[-2] // 2
    scale = 2.0 ** torch.tensor([0.0, 30.0, 55.0], device=DEV)[torch.randint(3, (half, 1), generator=g, device=DEV)]
    x = x.to(dtype).float()
    x[..., :half, :] *= scale
    at = half + torch.randperm(half, generator=g, device=DEV)
    x[..., at, :] = torch.where(scale > 1, -x[..., :half, :], x[..., at, :])
    return x[..., torch.randperm(C, generator=g, device=DEV), :].to(dtype).contiguous()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("variant", ["l2", "dir"])
@pytest.mark.parametrize("n", [40, 130, 333])
def test_sums_do_not_depend_on_the_launch(dtype, D, variant, n):
    U, N = S * L * H, n - 9
    k, v = [cancelling_rows((S, L, H, n, D), dtype, 7 * n + i) for i in range(2)]

    def evict(s0, s1, N, state, rows=n):
        a = [x[s0:s1].clone() for x in (k, v)]
        u = (s1 - s0) * L * H
        sums = torch.zeros((u, D + 1), dtype=torch.float64, device=DEV) if state else None
        scores = torch.zeros((u, n), device=DEV)
        vd.vd_evict_step(*a, [rows] * (s1 - s0), [N] * (s1 - s0), variant, running_sum=sums, scores_out=scores)
        if state:  # a second pass on the state of the first: the old rows from the state, new ones behind them
            vd.vd_evict_step(*a, [rows] * (s1 - s0), [N] * (s1 - s0), variant, running_sum=sums)
        return [*a, scores] + ([sums] if state else [])

    for state in (False, True):
        whole, parts = evict(0, S, N, state), [evict(s, s + 1, N, state) for s in range(S)]
        for i, x in enumerate(whole):
            assert torch.equal(x, torch.cat([p[i] for p in parts])), (state, i)
    alone = vd.vd_score(v, [n] * S, variant)[0]
    for N2 in (N, n - 1, n):  # half workgroups, a decode step's full ones, nothing to evict
        assert torch.equal(alone, evict(0, S, N2, False)[2]), N2


@pytest.mark.parametrize("units,n,D,threads", [(256, 80, 64, 1024), (257, 80, 64, 512), (288, 480, 64, 512),
                                               (288, 700, 64, 1024), (512, 700, 64, 1024), (513, 700, 64, 512),
                                               (288, 1400, 64, 512), (288, 200, 128, 512), (288, 300, 128, 1024)])
def test_workgroup_of_the_scores(units, n, D, threads):
    """Scores alone: half workgroups where half the LDS stages the bf16 rows, and for
    rows of 128 bytes that it does not, unless a whole one does and there are at most
    two units per CU."""
    saved = (vd._lib, vd.LIB_PATH)
    vd._lib, vd.LIB_PATH = None, lib_build.DEBUG_LIB
    try:
        v = synth.random_rows((1, 1, units, n, D), torch.bfloat16, n, DEV)
        scores = vd.vd_score(v, [n])[0]
        assert last_pass(vd.load()) == (threads, 0)
        assert torch.equal(scores, torch.cat([vd.vd_score(v[:, :, a:a + 200], [n])[0] for a in range(0, units, 200)]))
        assert last_pass(vd.load()) == (1024, 0)
    finally:
        vd._lib, vd.LIB_PATH = saved
