"""GPU tests of the two bulk encode kernels against each other (a workgroup per tile for short inputs, a wavefront per tile
for long ones: the same products in the same order) and of the power of two that fp32 inputs are scaled by."""
import numpy as np
import pytest
import torch

from paper_2502_02617_amd import Context, PQ_KEY, PQ_VALUE, synth
from tests.test_gpu_parity import DEV, say

pytestmark = pytest.mark.gpu
LONG = 25600                                       # tokens of 8 heads: 3200 tiles, the long kernel of every variant
PIECES = (1, 62, 1, 64, 65, 700, 12347, 12360)     # single slots, parts of tiles, whole ones; 8 to 1552 tiles per call


def context(pre, depth):
    ctx = {"dense": lambda: Context(seed=5), "hadamard": lambda: Context(seed=5, hadamard=True),
           "identity": lambda: Context(S=np.eye(128))}[pre]()
    if depth == 7:
        ctx.set_recursion_depth(7, (3, 1, 2))
    return ctx


def encoded(ctx, kind, x, calls, first=0):
    codes, radii = ctx.alloc_cache_for(x.shape[1], LONG + 64, DEV)
    codes.zero_(), radii.zero_()
    at = 0
    for n in calls:
        ctx.encode_kv(x[at:at + n], kind, codes, radii, dst_token0=first + at)
        at += n
    return codes, radii


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("pre", ["dense", "hadamard", "identity"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_short_calls_write_the_same_bits(dtype, pre, depth):
    say(f"encode in pieces, {dtype}, S {pre}, depth {depth}")
    ctx = context(pre, depth)
    assert sum(PIECES) == LONG
    x = synth.kv_stream(LONG, 8, seed=7).permute(1, 0, 2).contiguous().to(DEV)
    x = (x.float() * 1.01234567).to(dtype)
    for kind, first in ((PQ_KEY, 0), (PQ_VALUE, 29)):
        whole, parts = encoded(ctx, kind, x, (LONG,), first), encoded(ctx, kind, x, PIECES, first)
        assert all(torch.equal(a, b) for a, b in zip(whole, parts))
        # keys and values in one launch
        n = 1500
        kc, vc = (ctx.alloc_cache_for(8, 1536, DEV) for _ in range(2))
        for t in (*kc, *vc):
            t.zero_()
        ctx.encode_kv_pair(x[:n], x[:n], *kc, *vc, dst_token0=first)
        one = encoded(ctx, kind, x, (n,), first)
        assert all(torch.equal(a, b[:, :a.shape[1]]) for a, b in zip(kc if kind == PQ_KEY else vc, one))


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("pre", ["dense", "hadamard", "identity"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_a_workgroup_takes_several_tiles(dtype, pre, depth):
    """Calls that give each workgroup of the short kernel three to six tiles: the third is the first to reuse its buffers, the eighth
    wavefront in turn is the last to store.  The dispatch draws the line at six tiles per CU (twelve for bf16 and four levels)."""
    say(f"encode, several tiles per workgroup, {dtype}, S {pre}, depth {depth}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ctx, pieces = context(pre, depth), (6272, 12288, 7040)
    assert sum(pieces) == LONG and all(3 * cus <= 8 * n // 64 <= 6 * cus for n in pieces)
    assert 8 * LONG // 64 > 12 * cus                       # the long kernel
    x = synth.kv_stream(LONG, 8, seed=17).permute(1, 0, 2).contiguous().to(DEV)
    x = (x.float() * 1.01234567).to(dtype)
    n = 6144                                               # both kinds on half of the workgroups each: six tiles again
    assert 2 * 8 * n // 64 <= 6 * cus and 8 * n // 64 >= 3 * (cus // 2)
    for first in (0, 29):                                  # whole tiles; the first and the last of a call in part
        whole = {}
        for kind in (PQ_KEY, PQ_VALUE):
            whole[kind], parts = encoded(ctx, kind, x, (LONG,), first), encoded(ctx, kind, x, pieces, first)
            assert all(torch.equal(a, b) for a, b in zip(whole[kind], parts))
        kc, vc = (ctx.alloc_cache_for(8, n, DEV) for _ in range(2))
        for t in (*kc, *vc):
            t.zero_()
        m = n - 64 if first else n
        ctx.encode_kv_pair(x[:m], x[:m], *kc, *vc, dst_token0=first)
        full = (first + m) // 64                           # tiles that the call fills
        for kind, got in ((PQ_KEY, kc), (PQ_VALUE, vc)):
            assert all(torch.equal(a[:, :full], b[:, :full]) for a, b in zip(got, whole[kind]))


def radii_of(cache, n):
    """Key tiles hold [token][block]: -> [n, heads, 8], 64 bits"""
    return cache[1].view(torch.float16).flatten(1).unflatten(1, (-1, 8))[:, :n].transpose(0, 1).double()


@pytest.mark.parametrize("calls,H", [((900,), 1), ((LONG,), 1), ((12000,), 8), ((LONG,), 8)])
@pytest.mark.parametrize("pre", ["dense", "hadamard"])
def test_the_scale_of_an_fp32_vector_reaches_its_radii_only(pre, calls, H):
    """One head: the short kernel, one tile per workgroup or two; eight: six of its tiles per workgroup, and the long kernel."""
    say(f"fp32 vectors of many sizes, S {pre}, {calls} tokens of {H} heads")
    ctx, n = context(pre, 4), calls[0]
    x = synth.kv_stream(n, H, seed=9).permute(1, 0, 2).contiguous().to(DEV).float() * 1.01234567
    ref = encoded(ctx, PQ_KEY, x, calls)
    # the factor that is taken out is 2^103 at most, so a vector's largest coordinate stays above 2^-88 here
    k = torch.randint(-84, 116, (n, H, 1), generator=torch.Generator().manual_seed(1)).to(DEV)
    assert (x.abs().amax(2, keepdim=True) * torch.exp2(k.float())).min() >= 2.0 ** -88
    y = x * torch.exp2(k.float())
    got = encoded(ctx, PQ_KEY, y, calls)
    assert torch.equal(got[0], ref[0])                                     # every product is scaled by a power of two
    r = radii_of(ref, n)
    want = r * torch.exp2(k.double())
    have = radii_of(got, n)
    normal = (want >= 2.0 ** -14) & (want <= 65504) & (r >= 2.0 ** -14)
    assert torch.equal(have[normal], want[normal])
    assert torch.all(have[want > 65504] == 65504)
    assert torch.all(have[want < 2.0 ** -25] == 0)
    # a vector of zeros, of infinities or of NaN does not reach its neighbours
    for bad in (0.0, float("inf"), float("nan")):
        z = x.clone()
        z[3] = bad
        got = encoded(ctx, PQ_KEY, z, calls)
        keep = torch.arange(n, device=DEV) != 3
        assert torch.equal(radii_of(got, n)[keep], r[keep])
