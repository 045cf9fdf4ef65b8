"""GPU test of pq_decode_kv without its trailing S^T: the fp32 products of procedure DeQuant, top level first, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_02617_amd import Context, PQ_KEY, PQ_VALUE, synth
from tests import helpers
from tests.test_gpu_parity import DEV, say

pytestmark = pytest.mark.gpu


def products(rec, ctx):
    """Canonical records [n, 62] -> [n, 128] float32: radius times the (cos, sin) of levels 4, 3, 2, 1, one rounding each."""
    cs = [np.stack([np.cos(c), np.sin(c)], axis=1).astype(np.float32) for c in (ctx.codebook(l)[0] for l in (1, 2, 3, 4))]
    codes = [np.stack([rec[:, :32] >> 4, rec[:, :32] & 15], axis=2).reshape(len(rec), 64)]
    for lo, hi in ((32, 40), (40, 44), (44, 46)):
        codes.append(np.stack([(rec[:, lo:hi] >> s) & 3 for s in (6, 4, 2, 0)], axis=2).reshape(len(rec), -1))
    r = np.ascontiguousarray(rec[:, 46:62]).view(np.float16).astype(np.float32)
    for level in (4, 3, 2, 1):
        r = (r[:, :, None] * cs[level - 1][codes[level - 1]]).reshape(len(rec), -1)
    return r


@pytest.mark.parametrize("kind", [PQ_KEY, PQ_VALUE])
def test_rotated_vectors_are_the_products_in_order(kind):
    say(f"DeQuant in the rotated domain, kind={kind}")
    H, pool = 3, 384
    ctx = Context(seed=3)
    x = synth.kv_stream(pool, H, seed=81 + kind)
    x[1, 100:110] *= 2.0 ** -18                                    # subnormal radii
    rec = oracle.encode(x.double().numpy().reshape(-1, 128), ctx.preconditioner(), oracle.default_codebooks())
    codes, radii = ctx.alloc_cache_for(H, pool, DEV)
    helpers.upload_records(kind, rec.reshape(H, pool, 62), codes, radii, 0)
    ref = torch.from_numpy(products(rec, ctx).reshape(H, pool, 128).transpose(1, 0, 2).copy())
    for token0, n in ((0, 1), (15, 1), (16, 17), (37, 300), (0, 384)):
        for dtype, width in ((torch.float32, 128), (torch.float32, 131), (torch.bfloat16, 128), (torch.bfloat16, 131)):
            buf = torch.full((n, H, width), 7.0, dtype=dtype, device=DEV)
            ctx.decode_kv(kind, codes, radii, token0, n, buf[:, :, :128], rotated=True)
            assert torch.all(buf[:, :, 128:] == 7.0)
            assert torch.equal(buf[:, :, :128].cpu(), ref[token0:token0 + n].to(dtype)), (token0, n, dtype, width)
