"""GPU tests of pq_decode_kv on the oracle's own records: half tiles cut at either end, odd strides, both kinds of S."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_02617_amd import Context, PQ_KEY, PQ_VALUE, synth
from tests import helpers
from tests.test_gpu_deep import make
from tests.test_gpu_parity import DEV, say

pytestmark = pytest.mark.gpu

# slots [token0, token0 + n): one slot, the edges of half tiles and tiles, a range over several tiles
RANGES = [(0, 1), (31, 1), (32, 1), (0, 32), (31, 2), (5, 59), (0, 64), (63, 66), (37, 300)]


@pytest.mark.parametrize("kind", [PQ_KEY, PQ_VALUE])
@pytest.mark.parametrize("which", ["dense", "hadamard", "deep"])
def test_dequant_ranges_and_strides(which, kind):
    say(f"DeQuant {which} kind={kind}")
    H, pool = 3, 384
    x = synth.kv_stream(pool, H, seed=71 + kind)                                   # [H, pool, 128]
    x[1, 100:110] *= 2.0 ** -18                                                    # subnormal radii
    x[2, 40:50] *= 2.0 ** 6
    x[0, 7] = 0.0
    xs = x.double().numpy().reshape(-1, 128)
    if which == "deep":
        ctx, S, cb, cbt = make((2, 2, 2))
        rec = oracle.encode_deep(xs, S, cb, (2, 2, 2), cbt).reshape(H, pool, 50)
    else:
        ctx = Context(seed=3, hadamard=which == "hadamard")
        S, cb = ctx.preconditioner(), oracle.default_codebooks()
        rec = oracle.encode(xs, S, cb).reshape(H, pool, 62)
    codes, radii = ctx.alloc_cache_for(H, pool, DEV)
    (helpers.upload_records_deep if which == "deep" else helpers.upload_records)(kind, rec, codes, radii, 0)
    for rotated in (False, True):
        flat = rec.reshape(H * pool, -1)
        ref_all = oracle.decode_deep(flat, S, cb, (2, 2, 2), cbt, rotated=rotated) if which == "deep" \
            else oracle.decode(flat, S, cb, rotated=rotated)
        ref_all = ref_all.reshape(H, pool, 128)
        for token0, n in RANGES:
            ref = ref_all[:, token0:token0 + n].transpose(1, 0, 2)
            for dtype, width in ((torch.float32, 128), (torch.float32, 131), (torch.bfloat16, 128), (torch.bfloat16, 131)):
                buf = torch.full((n, H, width), 7.0, dtype=dtype, device=DEV)      # 131: rows at odd element offsets
                ctx.decode_kv(kind, codes, radii, token0, n, buf[:, :, :128], rotated=rotated)
                torch.cuda.synchronize()
                assert torch.all(buf[:, :, 128:] == 7.0)
                got = buf[:, :, :128].double().cpu().numpy()
                # fp32: two binary16 terms per factor carry 22 bits and a sign, 2^-22 of a vector's norm at most, and the
                # sums of 128 products round in fp32 (measured 1.5e-7); bf16 adds half a unit of its 8 bits
                bound = 1e-6 if dtype == torch.float32 else 2.0 ** -8
                norm = np.linalg.norm(ref, axis=2)
                err = np.linalg.norm(got - ref, axis=2)
                assert np.all(err <= bound * norm), (rotated, token0, n, dtype, width, float(np.max(err / np.maximum(norm, 1e-30))))


@pytest.mark.parametrize("which", ["dense", "hadamard", "deep"])
def test_a_long_range_is_its_pieces(which):
    say(f"DeQuant of a long range, {which}")
    ctx = make((2, 2, 2))[0] if which == "deep" else Context(seed=3, hadamard=which == "hadamard")
    H, n, first = 8, 20000, 37                             # 5008 half tiles: more than one per wavefront; the pieces take one
    pool = -(-(first + n) // 64) * 64
    x = synth.kv_stream(pool, H, seed=4).permute(1, 0, 2).contiguous().to(DEV)
    for kind in (PQ_KEY, PQ_VALUE):
        codes, radii = ctx.alloc_cache_for(H, pool, DEV)
        ctx.encode_kv(x, kind, codes, radii)
        whole = torch.empty((n, H, 128), dtype=torch.float32, device=DEV)
        parts = torch.empty_like(whole)
        ctx.decode_kv(kind, codes, radii, first, n, whole)
        for at in range(0, n, 5000):
            ctx.decode_kv(kind, codes, radii, first + at, 5000, parts[at:at + 5000])
        assert torch.equal(whole, parts)
