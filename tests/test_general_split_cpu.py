"""General format: which calls the split attention takes, seen from the size of their workspace (no GPU)."""
import pytest

from paper_2502_02617_amd import library

MOST = 1 << 30  # tokens of a pool: the split kernels count them in 32 bits, and 64 sequences may all be as long as the pool


@pytest.mark.parametrize("B,Hq,Hkv", [(1, 1, 1), (1, 8, 2), (4, 32, 8), (64, 2, 1)])
def test_no_split_where_32_bits_could_overflow(B, Hq, Hkv):
    size = library().pq_general_attn_workspace_bytes
    assert size(B, Hq, Hkv, 65536) > 0
    assert size(B, Hq, Hkv, MOST) > 0
    # what the kernels form in 32 bits at that bound: chunks of all sequences plus the slots they are dealt to, a token plus a chunk
    assert 64 * (MOST // 64) + 256 < 1 << 31 and MOST + 64 < 1 << 31
    for pool in (MOST + 1, (1 << 31) - 64, (1 << 31) - 1, 1 << 31, 1 << 40):
        assert size(B, Hq, Hkv, pool) == 0
