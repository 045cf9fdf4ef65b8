"""General format: a sequence worked on by several workgroups (a workspace is there) against one workgroup per row."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2502_02617_amd import Context, GeneralFormat, general_attn_decode, general_encode, library, synth
from tests import helpers

pytestmark = pytest.mark.gpu
DEV, D = "cuda", 128


def _rows_only(ctx, fmt, cbg, q, out, k, v, st, ln, scale):
    """The same call without a workspace."""
    cb = np.ascontiguousarray(cbg)
    rc = library().pq_general_attn_decode(ctx._h, ctypes.byref(fmt), cb.ctypes.data, q.data_ptr(), out.data_ptr(), k.data_ptr(),
                                          v.data_ptr(), st.data_ptr(), ln.data_ptr(), q.shape[0], q.shape[1], k.shape[0], k.shape[1],
                                          scale, torch.cuda.current_stream().cuda_stream)
    assert rc == 0


# lengths around the chunk (64 tokens), two chunks (nothing is split in a call whose sequences have no more), and pieces of several
# chunks; empty sequences and one that leaves the pool (its row is zeros); sixty-four sequences, one more than which are never split
@pytest.mark.parametrize("G,Hkv,lens,L,bits", [
    (4, 2, [1, 64, 65, 0, 128], 4, [3, 3, 2, 3]),
    (4, 2, [129, 63, 2049, 700], 5, [4, 2, 2, 2, 2]),
    (2, 1, [3000, 1, 193], 7, [4, 3, 2, 2, 1, 2, 3]),
    (3, 1, [1025, 0, 64], 6, [3, 2, 3, 2, 3, 1]),
    (4, 2, [0, 0, 700, 0, 1, 0, 0, 65, 0], 5, [4, 2, 2, 2, 2]),
    (4, 2, [0, 0, 0], 5, [4, 2, 2, 2, 2]),
    (1, 1, [5 * k for k in range(63)] + [4000], 4, [4, 3, 3, 3]),
    (1, 1, [5 * k for k in range(64)] + [4000], 4, [4, 3, 3, 3]),
])
def test_split_attention_equals_one_workgroup_per_row(G, Hkv, lens, L, bits):
    ctx, fmt = Context(seed=3), GeneralFormat(L, bits)
    cbg = oracle.general_codebooks(L, bits)
    B, Hq = len(lens), G * Hkv
    starts = np.concatenate([[0], np.cumsum(lens)[:-1]]) + 3 * np.arange(B)
    pool = max(int(starts[-1] + lens[-1]) + 5, 520 * B)          # above eight chunks per sequence: long enough to be split
    lens = list(lens)
    if B == 4:                                                   # a range that ends one token beyond the pool
        starts[0] = pool - lens[0] + 1
    n_bytes = library().pq_general_attn_workspace_bytes(B, Hq, Hkv, pool)
    assert (n_bytes > 0) == (B <= 64)
    k, v = (torch.zeros((Hkv, pool, fmt.record_bytes()), dtype=torch.uint8, device=DEV) for _ in range(2))
    for i, t in enumerate((k, v)):
        for h in range(Hkv):
            general_encode(ctx, fmt, cbg, synth.kv_stream(pool, 1, seed=10 * i + h).reshape(pool, D).to(DEV), t[h])
    q = synth.queries(B, Hq, seed=5).to(DEV)
    st = torch.tensor(starts, dtype=torch.int64, device=DEV)
    ln = torch.tensor(lens, dtype=torch.int32, device=DEV)
    out, ref = (torch.full((B, Hq, D), float("nan"), device=DEV) for _ in range(2))
    print(f"[gpu-test] general attention G={G} Hkv={Hkv} B={B} depth {L}", flush=True)
    general_attn_decode(ctx, fmt, cbg, q, out, k, v, st, ln, helpers.softmax_scale())
    _rows_only(ctx, fmt, cbg, q, ref, k, v, st, ln, helpers.softmax_scale())
    torch.cuda.synchronize()
    got, want = out.double().cpu().numpy(), ref.double().cpu().numpy()
    assert np.all(np.isfinite(got))
    for b, n in enumerate(lens):
        if n == 0 or starts[b] + n > pool:
            assert np.all(got[b] == 0.0)
    if not want.any():
        return
    # both are within 6e-7 of the 64-bit result (fp32 products and sums); the largest of any row 4e-6
    assert helpers.rel_l2(got, want) <= 2e-6
    if B <= 5:
        ln_ref = np.array([n if starts[b] + n <= pool else 0 for b, n in enumerate(lens)], np.int32)
        full = oracle.attention_general(q.double().cpu().numpy(), k.cpu().numpy(), v.cpu().numpy(), np.minimum(starts, pool), ln_ref,
                                        ctx.preconditioner(), L, bits, cbg, helpers.softmax_scale())
        assert helpers.rel_l2(got, full) <= 2e-6


def test_captured_attention_takes_no_workspace():
    """A graph outlives the allocator's workspace: the captured call is the one without, on every replay."""
    ctx, fmt = Context(seed=3), GeneralFormat(5, [4, 2, 2, 2, 2])
    cbg, pool, B, Hq = oracle.general_codebooks(5, [4, 2, 2, 2, 2]), 4096, 2, 4
    rec = torch.zeros((1, pool, fmt.record_bytes()), dtype=torch.uint8, device=DEV)
    general_encode(ctx, fmt, cbg, synth.kv_stream(pool, 1, seed=1).reshape(pool, D).to(DEV), rec[0])
    q, out, ref = synth.queries(B, Hq, seed=5).to(DEV), torch.zeros((B, Hq, D), device=DEV), torch.zeros((B, Hq, D), device=DEV)
    st = torch.tensor([0, 2000], dtype=torch.int64, device=DEV)
    ln = torch.tensor([1900, 77], dtype=torch.int32, device=DEV)
    general_attn_decode(ctx, fmt, cbg, q, out, rec, rec, st, ln, helpers.softmax_scale())
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        general_attn_decode(ctx, fmt, cbg, q, out, rec, rec, st, ln, helpers.softmax_scale())
    for r in range(4):
        out.zero_()
        ln.fill_(300 * r + 1)
        graph.replay()
        _rows_only(ctx, fmt, cbg, q, ref, rec, rec, st, ln, helpers.softmax_scale())
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def _split(ctx, fmt, cbg, q, out, k, v, st, ln, scale, ws):
    cb = np.ascontiguousarray(cbg)
    rc = library().pq_general_attn_decode_ws(ctx._h, ctypes.byref(fmt), cb.ctypes.data, q.data_ptr(), out.data_ptr(), k.data_ptr(),
                                             v.data_ptr(), st.data_ptr(), ln.data_ptr(), q.shape[0], q.shape[1], k.shape[0], k.shape[1],
                                             scale, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0


@pytest.mark.parametrize("G,Hkv", [(4, 2), (1, 3)])
def test_the_workspace_may_hold_anything(G, Hkv):
    """The arrivals of the pieces are counted in it: zeros, ones, noise and what an earlier call left, in eager calls on two streams
    and in a replayed graph whose lengths change; the same bits every time."""
    L, bits, pool, B = 5, [4, 2, 2, 2, 2], 16384, 3
    ctx, fmt, cbg, Hq = Context(seed=3), GeneralFormat(L, bits), oracle.general_codebooks(L, bits), G * Hkv
    rec = torch.zeros((Hkv, pool, fmt.record_bytes()), dtype=torch.uint8, device=DEV)
    for h in range(Hkv):
        general_encode(ctx, fmt, cbg, synth.kv_stream(pool, 1, seed=h).reshape(pool, D).to(DEV), rec[h])
    q, scale = synth.queries(B, Hq, seed=5).to(DEV), helpers.softmax_scale()
    st = torch.tensor([0, 5000, 9000], dtype=torch.int64, device=DEV)
    n_bytes = library().pq_general_attn_workspace_bytes(B, Hq, Hkv, pool)
    lengths = [[4000, 700, 0], [1, 128, 64], [300, 65, 7000], [4000, 3900, 7300]]
    g = torch.Generator(device=DEV).manual_seed(1)
    want = []
    for n in lengths:
        ln = torch.tensor(n, dtype=torch.int32, device=DEV)
        ref = torch.zeros((B, Hq, D), device=DEV)
        _rows_only(ctx, fmt, cbg, q, ref, rec, rec, st, ln, scale)
        want.append(torch.full((B, Hq, D), float("nan"), device=DEV))
        _split(ctx, fmt, cbg, q, want[-1], rec, rec, st, ln, scale, torch.zeros(n_bytes, dtype=torch.uint8, device=DEV))
        assert helpers.rel_l2(want[-1].double().cpu().numpy(), ref.double().cpu().numpy()) <= 2e-6
    fills = [torch.full((n_bytes,), 255, dtype=torch.uint8, device=DEV)] + \
            [torch.randint(0, 256, (n_bytes,), dtype=torch.uint8, device=DEV, generator=g) for _ in range(2)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in fills]
    outs = [[torch.full((B, Hq, D), float("nan"), device=DEV) for _ in lengths] for _ in fills]
    lns = [torch.tensor(n, dtype=torch.int32, device=DEV) for n in lengths]
    torch.cuda.synchronize()
    for _ in range(4):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                for j in range(len(lengths)):
                    _split(ctx, fmt, cbg, q, outs[i][j], rec, rec, st, lns[j], scale, fills[i])
        torch.cuda.synchronize()
        assert all(torch.equal(outs[i][j], want[j]) for i in range(len(fills)) for j in range(len(lengths)))
    ln, out, ws = lns[0].clone(), torch.zeros((B, Hq, D), device=DEV), fills[1]
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        _split(ctx, fmt, cbg, q, out, rec, rec, st, ln, scale, ws)
    for r in range(8):
        out.fill_(float("nan"))
        ln.copy_(lns[r % len(lengths)])
        if r == 5:
            ws.fill_(77)
        graph.replay()
        _split(ctx, fmt, cbg, q, outs[0][0], rec, rec, st, lns[0], scale, fills[0])
        torch.cuda.synchronize()
        assert torch.equal(out, want[r % len(lengths)]) and torch.equal(outs[0][0], want[0])


@pytest.mark.parametrize("pool", [512, 8192])                    # one workgroup per row, and split
def test_a_start_near_the_largest_number_gives_a_zero_row(pool):
    ctx, fmt, B, Hq = Context(seed=3), GeneralFormat(5, [4, 2, 2, 2, 2]), 3, 2
    cbg = oracle.general_codebooks(5, [4, 2, 2, 2, 2])
    rec = torch.zeros((1, pool, fmt.record_bytes()), dtype=torch.uint8, device=DEV)
    general_encode(ctx, fmt, cbg, synth.kv_stream(pool, 1, seed=1).reshape(pool, D).to(DEV), rec[0])
    assert (library().pq_general_attn_workspace_bytes(B, Hq, 1, pool) > 0) == (pool == 8192)
    st = torch.tensor([0, (1 << 63) - 5, (1 << 63) - 1], dtype=torch.int64, device=DEV)
    ln = torch.tensor([100, 100, 1], dtype=torch.int32, device=DEV)
    out = torch.full((B, Hq, D), float("nan"), device=DEV)
    general_attn_decode(ctx, fmt, cbg, synth.queries(B, Hq, seed=5).to(DEV), out, rec, rec, st, ln, helpers.softmax_scale())
    torch.cuda.synchronize()
    assert bool(out[0].any()) and bool((out[1:] == 0).all())
