"""DeQuant of ranges that give a wavefront more than one half tile, its first one outside the range."""
import pytest
import torch

from paper_2502_02617_amd import Context, PQ_KEY, PQ_VALUE, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("kind", [PQ_KEY, PQ_VALUE])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("hadamard", [False, True])
def test_a_range_behind_its_first_half_tile(kind, dtype, hadamard):
    ctx, H, pool = Context(seed=5, hadamard=hadamard), 8, 16640           # 4160 half tiles, 4096 wavefronts
    codes, radii = Context.alloc_cache(H, pool, DEV)
    x = synth.kv_stream(pool, 1, seed=9)[0].to(DEV)
    ctx.encode_kv(x[:, None, :].expand(pool, H, 128), kind, codes, radii, ld_token=128, ld_head=0, n_tokens=pool, n_heads=H)
    whole = torch.empty((pool, H, 128), dtype=dtype, device=DEV)
    ctx.decode_kv(kind, codes, radii, 0, pool, whole)
    assert torch.equal(whole[:, 0], whole[:, H - 1])                      # the same vectors in every head
    for first, n in ((33, pool - 33), (32, pool - 64), (63, 16500)):
        part = torch.full((n, H, 128), float("nan"), dtype=dtype, device=DEV)
        ctx.decode_kv(kind, codes, radii, first, n, part)
        assert torch.equal(part, whole[first:first + n])
