"""The workspace of a larger problem holds that of a smaller one: a program may size it once, for its longest context and
largest batch, and a smaller call then splits its work as with a workspace of its own size."""
import pytest

from paper_2502_02617_amd import Context

CTX = [0, 1, 64, 100, 300, 500, 512, 700, 800, 960, 1024, 1500, 2048, 3000, 4096, 8192, 16384, 32768, 65536, 131072, 1 << 20]
BATCH = [1, 2, 3, 4, 7, 8, 16, 31, 32, 64, 100, 128, 256, 600]


@pytest.mark.parametrize("Hkv", [1, 2, 8])
@pytest.mark.parametrize("G", [1, 4, 7, 8, 16])
def test_workspace_sizes_never_shrink_with_context_or_batch(G, Hkv):
    for M in [m for m in (1, 2, 4) if m * G <= 16]:
        size = {(B, n): Context.attn_mq_workspace_bytes(B, M, Hkv * G, Hkv, n) for B in BATCH for n in CTX}
        check(size)
        if M == 1:
            assert all(Context.attn_workspace_bytes(B, Hkv * G, Hkv, n) == s for (B, n), s in size.items())
    for cap in (1, 64, 300, 512):
        check({(B, n): Context.attn_hybrid_workspace_bytes(B, Hkv * G, Hkv, n, cap) for B in BATCH for n in CTX})


def check(size):
    for B in BATCH:
        assert all(size[B, a] <= size[B, b] for a, b in zip(CTX, CTX[1:])), B
    for n in CTX:
        assert all(size[a, n] <= size[b, n] for a, b in zip(BATCH, BATCH[1:])), n
