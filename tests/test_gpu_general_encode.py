"""General format: the encoder at the ends of its groups of sixteen vectors."""
import pytest
import torch

import oracle
from paper_2502_02617_amd import Context, GeneralFormat, general_encode

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n", [1, 15, 16, 17, 65])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("L,bits", [(4, [3, 3, 2, 3]), (7, [4, 3, 2, 2, 1, 2, 3])])
def test_encode_at_the_ends_of_a_group_of_vectors(n, dtype, L, bits):
    """Rows with a stride and an offset, records on an odd address; the byte behind the last record stays."""
    ctx, fmt = Context(seed=4), GeneralFormat(L, bits)
    cbg, rb = oracle.general_codebooks(L, bits), fmt.record_bytes()
    x = torch.randn((n, 131), generator=torch.Generator().manual_seed(n)).to(dtype)
    rec = torch.full((n * rb + 2,), 0x5A, dtype=torch.uint8, device=DEV)
    general_encode(ctx, fmt, cbg, x.to(DEV)[:, 1:129], rec[1:])
    torch.cuda.synchronize()
    got = rec.cpu().numpy()
    assert got[0] == 0x5A and got[-1] == 0x5A
    want = oracle.encode_general(x[:, 1:129].double().numpy(), ctx.preconditioner(), L, bits, cbg)
    # a radius next to a rounding boundary of binary16 or an angle next to a cell's may go either way: at most one of some 10^4
    assert (got[1:-1].reshape(n, rb) != want).sum() <= 2
