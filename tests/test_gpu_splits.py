"""GPU tests of how the attention calls divide their work: shares of the partial kernel, output rows and appended
vectors per workgroup, each at the sizes where a rule changes sides and at its remainders."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_02617_amd import (Context, GeneralFormat, PQ_KEY, PQ_VALUE, PolarQuantError, general_attn_decode,
                                  general_encode, synth)
from tests import helpers
from tests.test_gpu_parity import DEV, build_cache, env, gpu_attention, say  # noqa: F401

pytestmark = pytest.mark.gpu


# rows per workgroup of the combine kernel: 1 up to 256 rows, 2 up to 1024, then 4; the last group is incomplete
@pytest.mark.parametrize("B,Hq,Hkv,hi", [(64, 4, 1, 80), (37, 7, 1, 200), (79, 13, 1, 150), (147, 7, 1, 130)])
def test_combine_row_groups(env, B, Hq, Hkv, hi):  # noqa: F811
    ctx, S, cb = env
    rng = np.random.default_rng(B)
    lens = [int(n) for n in rng.integers(0, hi + 1, size=B)]
    lens[B - 1] = 1000                      # the last row group merges sixteen pieces
    say(f"combine row groups: {B * Hq} rows")
    caches, starts, _, k_rec, v_rec = build_cache(ctx, S, cb, lens, Hkv, seed=31000 + B)
    q = synth.queries(B, Hq, seed=31000 + B)
    got = gpu_attention(ctx, q, caches, starts, lens)
    ref = oracle.attention(q.double().numpy(), k_rec, v_rec, starts, np.array(lens, np.int32), S, cb, helpers.softmax_scale())
    assert all(np.all(got[b] == 0.0) for b in range(B) if lens[b] == 0)
    rows = [helpers.rel_l2(got[b], ref[b]) for b in range(B) if lens[b]]
    say(f"  rel L2 {helpers.rel_l2(got, ref):.2e}, worst sequence {max(rows):.2e}")
    assert helpers.rel_l2(got, ref) <= 2e-3 and max(rows) <= 4e-3


@pytest.mark.parametrize("lens", [[64], [1, 64, 65], [2000, 3, 129]])
def test_a_smaller_workspace_takes_larger_shares(env, lens):  # noqa: F811
    """The workspace of shares of one tile is what the size function returns; one that only holds the pieces of
    four-tile shares is accepted too, anything below that refused."""
    ctx, S, cb = env
    B, Hq, Hkv = len(lens), 8, 2
    say(f"workspace sizes, lens={lens}")
    caches, starts, _, k_rec, v_rec = build_cache(ctx, S, cb, lens, Hkv, seed=32000 + B)
    q = synth.queries(B, Hq, seed=32000 + B)
    ref = oracle.attention(q.double().numpy(), k_rec, v_rec, starts, np.array(lens, np.int32), S, cb, helpers.softmax_scale())

    def up(n):
        return (n + 255) & ~255

    tiles = B * Hkv * ((max(lens) + 63) // 64)
    pieces = (-(-tiles // 4) + 15) // 16 * 16 + B * Hkv
    coarse = up(up(up(B * Hq * 256) + 4 * (2 + B + 1 + 2 * B * Hkv)) + pieces * 4 * 8) + pieces * 4 * 512
    out = torch.empty((B, Hq, 128), dtype=torch.float32, device=DEV)
    args = (torch.from_numpy(starts).to(DEV), torch.tensor(lens, dtype=torch.int32, device=DEV), max(lens), helpers.softmax_scale())
    assert coarse <= Context.attn_workspace_bytes(B, Hq, Hkv, max(lens))
    for nbytes in (Context.attn_workspace_bytes(B, Hq, Hkv, max(lens)), coarse):
        out.fill_(float("nan"))
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)
        ctx.attn_decode_polar(q.to(DEV), out, *caches, *args, ws)
        torch.cuda.synchronize()
        assert helpers.rel_l2(out.cpu().numpy(), ref) <= 2e-3
    with pytest.raises(PolarQuantError, match="PQ_ENOMEM"):
        ctx.attn_decode_polar(q.to(DEV), out, *caches, *args, ws[:coarse - 1])


# the prologue of a decode step appends one vector per workgroup up to 512 vectors in all, then four
@pytest.mark.parametrize("hadamard", [False, True])
@pytest.mark.parametrize("B,Hkv,depth", [(32, 8, 4), (43, 6, 4), (87, 3, 4), (87, 3, 7)])
def test_step_append_equals_bulk_append(B, Hkv, depth, hadamard):
    say(f"decode step appends {2 * B * Hkv} vectors, depth {depth}, hadamard {hadamard}")
    ctx = Context(seed=5, hadamard=hadamard)
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    lens = [1 + (b % 64) for b in range(B)]
    g = torch.Generator().manual_seed(B)
    xk, xv = (torch.randn((B, Hkv, 128), generator=g).bfloat16().to(DEV) for _ in range(2))
    start = torch.arange(B, dtype=torch.int64, device=DEV) * 64
    ln = torch.tensor(lens, dtype=torch.int32, device=DEV)
    slot = start + ln.long() - 1
    slot[3] = -1                            # a slot outside the pool: nothing is written
    caches = []
    for _ in range(2):
        pair = [ctx.alloc_cache_for(Hkv, 64 * B, DEV) for _ in (PQ_KEY, PQ_VALUE)]
        for codes, radii in pair:
            codes.fill_(0x5A)
            radii.fill_(0x1234)
        caches.append([t for p in pair for t in p])
    q = torch.randn((B, Hkv, 128), generator=g).bfloat16().to(DEV)
    out = torch.empty((B, Hkv, 128), dtype=torch.float32, device=DEV)
    ws = torch.empty(Context.attn_workspace_bytes(B, Hkv, Hkv, 64), dtype=torch.uint8, device=DEV)
    ctx.decode_step_polar(xk, xv, slot, q, out, *caches[0], start, ln, 64, helpers.softmax_scale(), ws)
    ctx.append_kv_pair(xk, xv, *caches[1], slot)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*caches))


# the general format: heads per workgroup 1, 2 (512 rows) and 4 (1024 rows); lengths around the 128 tokens of a round
@pytest.mark.parametrize("B,Hq,Hkv,bits", [(6, 7, 1, (4, 2, 2, 2, 2)), (130, 4, 2, (3, 3, 2, 3)), (130, 8, 2, (4, 3, 3, 3)),
                                           (33, 32, 8, (3, 2, 3, 2, 3, 1))])
def test_general_attention_heads_per_workgroup(B, Hq, Hkv, bits):
    say(f"general attention, {B * Hq} rows, {Hq // Hkv} heads per kv head, bits {bits}")
    ctx = Context(seed=14)
    S, L = ctx.preconditioner(), len(bits)
    fmt = GeneralFormat(L, bits)
    cbg = oracle.general_codebooks(L, bits)
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 70, size=B)
    lens[:6] = [127, 128, 129, 256, 1, 0]
    starts = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int64)
    pool = int(lens.sum())
    recs = []
    for part in (0, 1):
        x = synth.kv_stream(pool, Hkv, seed=600 + part).double().numpy().reshape(-1, 128)
        recs.append(oracle.encode_general(x, S, L, bits, cbg).reshape(Hkv, pool, -1))
    q = synth.queries(B, Hq, seed=78)
    out = torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device=DEV)
    # the records end where their allocation ends, and start one byte into it
    dev = [torch.zeros(r.size + 1, dtype=torch.uint8, device=DEV)[1:].view(*r.shape) for r in recs]
    for d, r in zip(dev, recs):
        d.copy_(torch.from_numpy(r))
    general_attn_decode(ctx, fmt, cbg, q.to(DEV), out, *dev, torch.from_numpy(starts).to(DEV),
                        torch.from_numpy(lens.astype(np.int32)).to(DEV), helpers.softmax_scale())
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    ref = oracle.attention_general(q.double().numpy(), *recs, starts, lens.astype(np.int32), S, L, bits, cbg, helpers.softmax_scale())
    assert np.all(np.isfinite(got)) and np.all(got[5] == 0.0)
    err = helpers.rel_l2(got, ref)
    say(f"  rel L2 {err:.2e}")
    # fp32 throughout: an element of a key carries five roundings of 2^-24, a score of up to some 30 its product with them
    assert err <= 5e-6


@pytest.mark.parametrize("n,ld,shift", [(1, 128, 0), (15, 131, 1), (16, 128, 2), (17, 256, 3), (100, 129, 0)])
def test_general_encode_groups(n, ld, shift):
    """Sixteen vectors per workgroup: incomplete groups, rows at any stride, records at any byte."""
    say(f"general encode of {n} vectors, stride {ld}")
    ctx = Context(seed=15)
    bits = (4, 2, 2, 2)
    fmt = GeneralFormat(4, bits)
    cbg = fmt.codebooks()
    x = torch.randn((n, ld), generator=torch.Generator().manual_seed(n))
    rec_or = oracle.encode_general(x[:, :128].double().numpy(), ctx.preconditioner(), 4, bits, oracle.general_codebooks(4, bits))
    rb = fmt.record_bytes()
    buf = torch.full((shift + n * rb + 5,), 0xA5, dtype=torch.uint8, device=DEV)
    general_encode(ctx, fmt, cbg, x.to(DEV)[:, :128], buf[shift:])
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert np.all(got[:shift] == 0xA5) and np.all(got[shift + n * rb:] == 0xA5)
    # at most one tie (an angle or a radius on a boundary) among these few values
    assert np.count_nonzero(got[shift:shift + n * rb].reshape(n, rb) != rec_or) <= 1


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("n,H,dtype", [(1, 1, torch.float32), (63, 1, torch.bfloat16), (65, 3, torch.float32), (64, 255, torch.bfloat16),
                                       (64, 257, torch.bfloat16), (2100, 130, torch.bfloat16)])
def test_fit_counts(n, H, dtype, depth):
    """Every angle is counted once whatever the spread of the tiles over the workgroups, and the histograms have the mean
    of the exact angles to half a bin."""
    say(f"angle counts of {n} x {H} vectors, depth {depth}")
    ctx = Context(seed=6)
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    x = torch.randn((n, H, 128), generator=torch.Generator().manual_seed(n + H)).to(dtype)
    ws = torch.full((Context.fit_workspace_bytes(),), 0xFF, dtype=torch.uint8, device=DEV)
    ctx.fit_count_angles(x.to(DEV), ws)
    torch.cuda.synchronize()
    hist = ws.cpu().numpy().view(np.uint32)
    r = x.reshape(-1, 128).double().numpy() @ ctx.preconditioner()
    off = 0
    for level in range(1, 8):
        bins, per = (8192, 2048) if level == 1 else (2048, 2048)
        h = hist[off:off + bins].astype(np.float64)
        off += bins
        assert h.sum() == (n * H * (128 >> level) if level <= depth else 0)
        psi = np.arctan2(r[:, 1::2], r[:, 0::2])
        if level == 1:
            psi = np.where(psi < 0, psi + 2 * np.pi, psi)
        r = np.hypot(r[:, 0::2], r[:, 1::2])
        if level <= depth:
            k = np.arange(bins + 1)
            e = (k // per) * (np.pi / 2) + np.arctan2(k % per, per - k % per)
            # half of the widest bin (9.8e-4 rad); the two-term product with S moves an angle by some 1e-5
            assert abs((h * 0.5 * (e[1:] + e[:-1])).sum() / h.sum() - psi.mean()) <= 5.1e-4


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("T,H,dtype", [(1, 1, torch.float32), (64, 127, torch.bfloat16), (64, 257, torch.float32), (130, 90, torch.bfloat16),
                                       (64, 2050, torch.bfloat16)])
def test_encode_spread_over_workgroups(T, H, dtype, depth):
    """Whatever the number of tiles against the number of workgroups (and 256 x 8 wavefronts), a head's tiles are what a call
    with that head alone writes; keys and values, single and paired calls."""
    say(f"encode {T} tokens x {H} heads, depth {depth}")
    ctx = Context(seed=7)
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    g = torch.Generator().manual_seed(T + H)
    xk, xv = (torch.randn((T, H, 128), generator=g).to(dtype).to(DEV) for _ in range(2))
    first, pool = 5, (5 + T + 63) // 64 * 64

    def cache(heads):
        c, r = ctx.alloc_cache_for(heads, pool, DEV)
        return c.fill_(0x5A), r.fill_(0x1234)

    single = [cache(H), cache(H)]
    pair = [cache(H), cache(H)]
    for (c, r), x, kind in zip(single, (xk, xv), (PQ_KEY, PQ_VALUE)):
        ctx.encode_kv(x, kind, c, r, dst_token0=first)
    ctx.encode_kv_pair(xk, xv, *pair[0], *pair[1], dst_token0=first)
    torch.cuda.synchronize()
    for (c, r), (c2, r2), x, kind in zip(single, pair, (xk, xv), (PQ_KEY, PQ_VALUE)):
        assert torch.equal(c, c2) and torch.equal(r, r2)
        for h in {0, H // 2, H - 1}:
            c1, r1 = cache(1)
            ctx.encode_kv(x[:, h:h + 1].contiguous(), kind, c1, r1, dst_token0=first)
            torch.cuda.synchronize()
            assert torch.equal(c[h], c1[0]) and torch.equal(r[h], r1[0])


# shares of exactly four tiles with wavefronts to spare (a workspace that holds no smaller shares), in each variant of the partial
# kernel: 16, 12 and 8 wavefronts per workgroup
@pytest.mark.parametrize("M,G,waves", [(1, 4, 16), (2, 4, 12), (4, 4, 8)])
def test_four_tile_shares_of_a_full_batch(env, M, G, waves):  # noqa: F811
    ctx, S, cb = env
    B, Hkv, n = 1, 2, 2 * waves * 64
    say(f"shares of four tiles: {B * Hkv * n // 64} tiles, {M} x {G} pairs")
    caches, starts, _, k_rec, v_rec = build_cache(ctx, S, cb, [n], Hkv, seed=33000 + M)
    q = synth.queries(B * M, Hkv * G, seed=33000 + M).reshape(B, M, Hkv * G, 128).contiguous()

    def up(k):
        return (k + 255) & ~255

    pieces = waves + B * Hkv
    coarse = up(up(up(B * M * Hkv * G * 256) + 4 * (2 + B + 1 + 2 * B * Hkv)) + pieces * M * G * 8) + pieces * M * G * 512
    fine = Context.attn_mq_workspace_bytes(B, M, Hkv * G, Hkv, n)
    assert coarse < fine
    for nbytes in (coarse, fine):
        out = torch.full((B, M, Hkv * G, 128), float("nan"), dtype=torch.float32, device=DEV)
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)
        ctx.attn_decode_polar_mq(q.to(DEV), out, *caches, torch.from_numpy(starts).to(DEV),
                                 torch.tensor([n], dtype=torch.int32, device=DEV), n, helpers.softmax_scale(), ws)
        got = out.cpu().double().numpy()
        for m in range(M):
            ref = oracle.attention(q[:, m].double().numpy(), k_rec, v_rec, starts, np.array([n - (M - 1 - m)], np.int32), S, cb,
                                   helpers.softmax_scale())
            assert helpers.rel_l2(got[:, m], ref) <= 2e-3
    with pytest.raises(PolarQuantError, match="PQ_ENOMEM"):
        ctx.attn_decode_polar_mq(q.to(DEV), out, *caches, torch.from_numpy(starts).to(DEV),
                                 torch.tensor([n], dtype=torch.int32, device=DEV), n, helpers.softmax_scale(), ws[:coarse - 1])


# one head per workgroup: sixteen wavefronts up to 256 rows, then eight
@pytest.mark.parametrize("B,Hq,Hkv,bits", [(256, 1, 1, (4, 2, 2, 2, 2)), (257, 1, 1, (3, 3, 2, 3)), (40, 7, 1, (4, 3, 3, 3)),
                                           (73, 7, 1, (4, 2, 2, 2, 2))])
def test_general_attention_one_head_per_workgroup(B, Hq, Hkv, bits):
    test_general_attention_heads_per_workgroup(B, Hq, Hkv, bits)
