"""GPU test of the unquantised window of hybrid attention: rows beyond a sequence's window do not enter its sums."""
import numpy as np
import pytest
import torch

from paper_2502_02617_amd import Context, PQ_KEY, PQ_VALUE
from tests import helpers
from tests.test_gpu_parity import DEV, say

pytestmark = pytest.mark.gpu


# G = 4 with 288 sequences: 1728 items of two heads, more than are taken one head at a time
@pytest.mark.parametrize("G,times", [(1, 1), (2, 1), (4, 1), (7, 1), (4, 16)])
def test_an_infinity_in_the_last_row_of_the_window_stays_in_its_coordinate(G, times):
    wins, Hkv, cap = [1, 7, 8, 9, 40, 63, 64, 65, 100] * times, 2, 130
    say(f"window with an infinity, lengths {wins}, {G} query heads per kv head")
    B, g = len(wins), torch.Generator().manual_seed(G)
    ctx = Context(seed=2)
    caches = [t.zero_() for kind in (PQ_KEY, PQ_VALUE) for t in ctx.alloc_cache_for(Hkv, 64 * B, DEV)]
    q = torch.randn((B, Hkv * G, 128), generator=g).bfloat16()
    k, v = (torch.randn((B, Hkv, cap, 128), generator=g).bfloat16() for _ in range(2))
    for b, n in enumerate(wins):
        k[b, :, n:] = float("nan")
        v[b, :, n:] = float("nan")
        v[b, :, n - 1, 5] = float("inf")
        v[b, :, n - 1, 70] = float("-inf")
    out = torch.zeros((B, Hkv * G, 128), dtype=torch.float32, device=DEV)
    ws = torch.empty(Context.attn_hybrid_workspace_bytes(B, Hkv * G, Hkv, 64, cap), dtype=torch.uint8, device=DEV)
    ctx.attn_decode_hybrid(q.to(DEV), out, *caches, torch.arange(B, device=DEV) * 64, torch.zeros(B, dtype=torch.int32, device=DEV),
                           k.to(DEV), v.to(DEV), torch.tensor(wins, dtype=torch.int32, device=DEV), 64, helpers.softmax_scale(), ws)
    got = out.cpu().double().numpy().reshape(B, Hkv, G, 128)
    rest = [c for c in range(128) if c not in (5, 70)]
    for b, n in enumerate(wins):
        assert np.all(got[b, :, :, 5] == np.inf) and np.all(got[b, :, :, 70] == -np.inf), n
        qb, kb, vb = q[b].double().view(Hkv, G, 128), k[b, :, :n].double(), v[b, :, :n].double()
        p = torch.softmax(torch.stack([qb[h] @ kb[h].T for h in range(Hkv)]) * helpers.softmax_scale(), dim=-1)
        ref = torch.stack([p[h] @ vb[h][:, rest] for h in range(Hkv)]).numpy()
        # fp32 sums of up to 128 products, twice
        assert helpers.rel_l2(got[b][:, :, rest], ref) <= 1e-5, n


# Items of two heads (B * Hq / 2 * chunks of 64) up to which a wavefront takes one head: 512, 514 and far more; groups of four, six and
# eight, one, two, three and eight chunks
@pytest.mark.parametrize("B,Hkv,G,cap", [(256, 1, 4, 64), (257, 1, 4, 64), (16, 8, 4, 128), (17, 8, 4, 128), (32, 8, 4, 130), (32, 2, 6, 130),
                                         (40, 1, 8, 200), (4, 8, 4, 512), (5, 8, 4, 500), (9, 8, 4, 256)])
def test_window_items_of_one_and_of_two_heads(B, Hkv, G, cap):
    g = torch.Generator().manual_seed(B + cap)
    wins = [int(n) for n in torch.randint(0, cap + 1, (B,), generator=g)]
    wins[:3] = [cap, 0, max(1, cap - 1)]
    say(f"window of {B} sequences, {Hkv} kv heads, {G} query heads each, up to {cap} rows, "
        f"{B * Hkv * G // 2 * ((cap + 63) // 64)} items of two heads")
    ctx = Context(seed=2)
    caches = [t.zero_() for kind in (PQ_KEY, PQ_VALUE) for t in ctx.alloc_cache_for(Hkv, 64 * B, DEV)]
    q = torch.randn((B, Hkv * G, 128), generator=g).bfloat16()
    k, v = (torch.randn((B, Hkv, cap, 128), generator=g).bfloat16() for _ in range(2))
    for b, n in enumerate(wins):
        k[b, :, n:] = float("nan")
        v[b, :, n:] = float("nan")
    out = torch.full((B, Hkv * G, 128), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(Context.attn_hybrid_workspace_bytes(B, Hkv * G, Hkv, 64, cap), dtype=torch.uint8, device=DEV)
    ctx.attn_decode_hybrid(q.to(DEV), out, *caches, torch.arange(B, device=DEV) * 64, torch.zeros(B, dtype=torch.int32, device=DEV),
                           k.to(DEV), v.to(DEV), torch.tensor(wins, dtype=torch.int32, device=DEV), 64, helpers.softmax_scale(), ws)
    got = out.cpu().double().view(B, Hkv, G, 128)
    for b, n in enumerate(wins):
        if n == 0:
            assert bool((got[b] == 0).all())
            continue
        p = torch.softmax(torch.matmul(q[b].double().view(Hkv, G, 128), k[b, :, :n].double().transpose(1, 2).contiguous())
                          * helpers.softmax_scale(), dim=-1)
        # fp32 sums of up to 128 products for a score and 512 for a value
        assert helpers.rel_l2(got[b].numpy(), torch.matmul(p, v[b, :, :n].double()).numpy()) <= 1e-5, (b, n)
