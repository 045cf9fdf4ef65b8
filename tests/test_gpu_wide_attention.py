"""GPU test of the attention kernel for more than four (query token, head) pairs per kv head against the one for up to four:
the same cache, the pairs taken four at a time by calls of one query token and at most four heads."""
import pytest
import torch

from paper_2502_02617_amd import Context, PQ_KEY, PQ_VALUE, synth
from tests.test_gpu_parity import DEV, say

pytestmark = pytest.mark.gpu
SCALE = 128 ** -0.5


def attend(ctx, q, caches, start, lens, max_ctx):
    """q [B, M, Hq, 128] -> fp32 [B, M, Hq, 128]"""
    B, M, Hq = q.shape[:3]
    out = torch.empty(q.shape, dtype=torch.float32, device=DEV)
    ws = torch.empty(Context.attn_mq_workspace_bytes(B, M, Hq, caches[0].shape[0], max_ctx), dtype=torch.uint8, device=DEV)
    ctx.attn_decode_polar_mq(q, out, *caches, start, lens, max_ctx, SCALE, ws)
    return out


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("G,M", [(5, 1), (2, 4), (7, 1), (3, 3), (16, 1), (4, 4), (1, 16)])
def test_wide_pairs_are_those_of_four_at_a_time(G, M, depth):
    say(f"wide attention, {G} heads, {M} query tokens, depth {depth}")
    B, H, n = 16, 8, 3300                                  # some three tiles per wavefront: pieces cross streams
    ctx = Context(seed=2)
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    lens = torch.tensor([n - 37 * b for b in range(B)], dtype=torch.int32)
    lens[3], lens[4], lens[5] = M, 64, 65                  # every query token sees one token at least
    start = torch.arange(B) * (-(-n // 64) * 64)
    pool = B * (-(-n // 64) * 64)
    caches = []
    for kind in (PQ_KEY, PQ_VALUE):
        codes, radii = ctx.alloc_cache_for(H, pool, DEV)
        x = synth.kv_stream(pool, H, seed=20 + kind).permute(1, 0, 2).contiguous().to(DEV)
        ctx.encode_kv(x, kind, codes, radii)
        caches += [codes, radii]
    q = torch.randn((B, M, H * G, 128), generator=torch.Generator().manual_seed(5)).bfloat16().to(DEV)
    start_d = start.to(DEV)
    got = attend(ctx, q, caches, start_d, lens.to(DEV), n)
    ref = torch.empty_like(got)
    for m in range(M):
        seen = (lens - (M - 1 - m)).clamp(min=0).to(DEV)
        by_head = q[:, m].unflatten(1, (H, G))
        for g in range(0, G, 4):
            part = by_head[:, :, g:g + 4].flatten(1, 2)[:, None].contiguous()
            ref[:, m].unflatten(1, (H, G))[:, :, g:g + 4] = attend(ctx, part, caches, start_d, seen, n)[:, 0].unflatten(1, (H, -1))
    # the two differ by the rounding of weights and values to binary16 against other references: each is 7e-4 off 64 bits,
    # rows that rest on few tokens up to five times that
    assert (got - ref).norm() <= 1.4e-3 * ref.norm()
    assert ((got - ref).norm(dim=-1) <= 2e-2 * torch.maximum(ref.norm(dim=-1), ref.norm(dim=-1).square().mean().sqrt())).all()
    again = attend(ctx, q, caches, start_d, lens.to(DEV), n)
    assert torch.equal(got, again)                         # the split of the work is fixed: the same bits


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("G,M", [(5, 1), (8, 1), (2, 4), (1, 7)])
def test_long_calls_of_five_to_eight_pairs(G, M, depth):
    """More than 18 tiles for each of the 3072 wavefronts, which then take the pairs in two groups of four; the sequences share
    their tiles."""
    say(f"long attention, {G} heads, {M} query tokens, depth {depth}")
    B, H, n = 64, 8, 7000
    ctx = Context(seed=2)
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    lens = torch.tensor([n - 11 * b for b in range(B)], dtype=torch.int32)
    pool = -(-n // 64) * 64
    assert B * H * (pool // 64) > 18 * 3072
    caches = []
    for kind in (PQ_KEY, PQ_VALUE):
        codes, radii = ctx.alloc_cache_for(H, pool, DEV)
        x = synth.kv_stream(pool, H, seed=20 + kind).permute(1, 0, 2).contiguous().to(DEV)
        ctx.encode_kv(x, kind, codes, radii)
        caches += [codes, radii]
    q = torch.randn((B, M, H * G, 128), generator=torch.Generator().manual_seed(5)).bfloat16().to(DEV)
    start = torch.zeros(B, dtype=torch.int64, device=DEV)
    got = attend(ctx, q, caches, start, lens.to(DEV), n)
    ref = torch.empty_like(got)
    for m in range(M):
        seen = (lens - (M - 1 - m)).to(DEV)
        by_head = q[:, m].unflatten(1, (H, G))
        for g in range(0, G, 4):
            part = by_head[:, :, g:g + 4].flatten(1, 2)[:, None].contiguous()
            ref[:, m].unflatten(1, (H, G))[:, :, g:g + 4] = attend(ctx, part, caches, start, seen, n)[:, 0].unflatten(1, (H, -1))
    # as above
    assert (got - ref).norm() <= 1.4e-3 * ref.norm()
    assert ((got - ref).norm(dim=-1) <= 2e-2 * torch.maximum(ref.norm(dim=-1), ref.norm(dim=-1).square().mean().sqrt())).all()
    assert torch.equal(got, attend(ctx, q, caches, start, lens.to(DEV), n))


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("G", [5, 16])
def test_small_keys_are_scored_as_large_ones(G, depth):
    """Key radii times 2^-shift and queries times 2^shift, both exactly: the same scores but for their rounding, which is some 6e-8
    of |q'| |k| = 16 each.  A weight moves to the next binary16 number, by 2^-10.5 of itself, where that makes it cross the
    middle between two: a share of 2^11 4e-6 of them does if the scores differ by 4e-6."""
    say(f"wide attention, {G} heads, keys of several sizes, depth {depth}")
    B, H, n = 16, 8, 64
    ctx = Context(seed=2)
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    caches = []
    for kind in (PQ_KEY, PQ_VALUE):
        codes, radii = ctx.alloc_cache_for(H, B * n, DEV)
        x = torch.randn((B * n, H, 128), generator=torch.Generator().manual_seed(20 + kind)).to(DEV)
        ctx.encode_kv(x, kind, codes, radii)
        caches += [codes, radii]
    radii = caches[1].clone()
    small = caches[1].view(torch.float16)[..., 1::2] if depth == 7 else caches[1].view(torch.float16)
    large = small.clone()
    assert 1.0 < large.min() and large.max() < 32.0            # normal numbers at every shift
    q = torch.randn((B, 1, H * G, 128), generator=torch.Generator().manual_seed(5)).bfloat16().to(DEV)
    start, lens = torch.arange(B, device=DEV) * n, torch.full((B,), n, dtype=torch.int32, device=DEV)
    lens[1::2] -= torch.arange(0, 56, 7, dtype=torch.int32, device=DEV)
    ref = attend(ctx, q, caches, start, lens, n)
    for shift in (4, 8, 12, 14):
        small.copy_(large * 2.0 ** -shift)
        got = attend(ctx, q * 2.0 ** shift, caches, start, lens, n)
        rel = float((got - ref).norm() / ref.norm())
        print(f"2^-{shift}: relative difference {rel:.2e}")
        assert rel <= 2 ** -10.5 * (2 ** 11 * 4e-6) ** 0.5
    assert not torch.equal(radii, caches[1])
