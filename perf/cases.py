"""What the speed of this library is judged on: the calls that a serving program makes, through the Python binding.

    listed()             twelve cases, from one short conversation to a full serving batch
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  what a program has in hand before the call, on the GPU
    run(state)           one pass, as a program calls it
    work(case)           bytes and operations that a pass cannot do without
    tolerance(case)      how far another correct implementation may be off
    exact(case, seed)    the same numbers in 64 bits with plain torch

The caches that the attention cases read are made here, in torch and without the library: random keys and values with a
few outlier channels per head, rotated, polar-transformed, quantised and laid out as tiles by the definitions in
csrc/pq_layout.h.  A bank of tiles is quantised per head and the cache is filled with tiles picked from it at random, so
that codes and radii have the distribution of real vectors and a gigabyte of cache is made in milliseconds.
"""
import functools
import math

import numpy as np
import torch

from paper_2502_02617_amd import (Context, GeneralFormat, PQ_KEY, PQ_VALUE, general_attn_decode, general_encode)

D = 128
TILE = 64
BANK_TILES = 48                       # distinct tiles per head plane
SCALE = 1.0 / math.sqrt(D)
BITS4 = (4, 2, 2, 2)                  # Section 4.1
BITS7 = (4, 2, 2, 2, 2, 2, 2)         # full recursion depth, 50 bytes per vector
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
DEV = "cuda"

# The shapes are those of this library's configurations (32 query heads on 8 key / value heads, contexts of 32768 and
# 131072, 64 ragged sequences of 1k-64k, 32768-token prompts) and smaller and odd ones next to them.
LISTED = [
    # one conversation, short context: what a single user waits for per token
    {"name": "step_single_1k", "op": "step", "batch": 1, "lo": 1000, "hi": 1000, "kv_heads": 8, "group": 4,
     "pre": "dense", "depth": 4, "x": "bf16", "out": "bf16", "lens_seed": 0},
    # an ordinary batch of conversations of mixed length
    {"name": "step_chat_b32_4k", "op": "step", "batch": 32, "lo": 200, "hi": 4096, "kv_heads": 8, "group": 4,
     "pre": "dense", "depth": 4, "x": "bf16", "out": "bf16", "lens_seed": 1},
    # the benchmark's own decode step: 16 sequences of 32768 tokens
    {"name": "step_b16_32k", "op": "step", "batch": 16, "lo": 32768, "hi": 32768, "kv_heads": 8, "group": 4,
     "pre": "dense", "depth": 4, "x": "bf16", "out": "bf16", "lens_seed": 2},
    # one layer of a full serving batch: 64 sequences of 1k to 64k tokens
    {"name": "step_ragged_b64_64k", "op": "step", "batch": 64, "lo": 1024, "hi": 65536, "kv_heads": 8, "group": 4,
     "pre": "dense", "depth": 4, "x": "bf16", "out": "bf16", "lens_seed": 4},
    # the smaller cache format (full recursion depth), middle-sized contexts
    {"name": "step_deep_b16_16k", "op": "step", "batch": 16, "lo": 12000, "hi": 16384, "kv_heads": 8, "group": 4,
     "pre": "dense", "depth": 7, "x": "bf16", "out": "bf16", "lens_seed": 5},
    # verification of four draft tokens per sequence
    {"name": "draft4_b16_16k", "op": "multi", "batch": 16, "lo": 9000, "hi": 16384, "kv_heads": 8, "group": 4, "queries": 4,
     "pre": "dense", "depth": 4, "out": "bf16", "lens_seed": 6},
    # quantised long prompts plus the generated tokens in 16 bits (the evaluation protocol of Section 5.3)
    {"name": "hybrid_b4_128k", "op": "hybrid", "batch": 4, "lo": 131072, "hi": 131072, "kv_heads": 8, "group": 4,
     "window": 256, "pre": "hadamard", "depth": 4, "out": "f32", "lens_seed": 7},
    # prefill of one layer: keys and values of a 32768-token prompt
    {"name": "encode_prompt_32k", "op": "encode", "kind": "pair", "tokens": 32768, "first": 0, "kv_heads": 8, "x": "bf16",
     "pre": "dense", "depth": 4},
    # a chunk of a prompt behind tokens that are already cached, keys in 32 bits
    {"name": "encode_chunk_f32", "op": "encode", "kind": "key", "tokens": 3001, "first": 37, "kv_heads": 8, "x": "f32",
     "pre": "dense", "depth": 4},
    # the cache back as vectors, for a program that attends with its own kernels
    {"name": "dequant_32k", "op": "dequant", "kind": "value", "tokens": 32768, "first": 0, "kv_heads": 8, "out": "bf16",
     "pre": "dense"},
    # codebooks fitted to a prompt's own angles (Section 4.1's online variant)
    {"name": "fit_32k", "op": "fit", "tokens": 32768, "kv_heads": 8, "x": "bf16", "pre": "dense", "rounds": 10},
    # a format outside Section 4.1: a new sequence's prompt is encoded, four others take a decode step
    {"name": "general_d5_b4_2k", "op": "general", "batch": 4, "lo": 2048, "hi": 2048, "tokens": 2048, "kv_heads": 2, "group": 4,
     "bits": "4,2,2,2,2", "x": "bf16", "pre": "dense", "lens_seed": 8},
]

GENERAL_BITS = ("4,2,2,2,2", "3,3,2,3", "4,3,3,3", "3,2,3,2,3,1", "4,3,2,2,1,2,2")


def listed():
    return [dict(c) for c in LISTED]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "multi", "hybrid", "encode", "encode", "dequant", "fit", "general"])
    kv_heads, group = rng.choice([1, 2, 4, 8, 8]), rng.choice([1, 2, 4, 4, 7, 8])
    pre = rng.choice(["dense", "dense", "hadamard"])
    x, out = rng.choice(["bf16", "bf16", "f32"]), rng.choice(["bf16", "f32"])
    c = {"op": op, "kv_heads": kv_heads, "pre": pre}
    if op in ("step", "multi", "hybrid"):
        c["batch"] = _log(rng, 1, 64)
        c["hi"] = min(_log(rng, 100, 131072), 1000000 // c["batch"])
        c["lo"] = c["hi"] if rng.random() < 0.3 else max(1, c["hi"] // rng.randint(2, 64))
        c["group"], c["out"], c["lens_seed"] = group, out, rng.randrange(1 << 20)
        c["depth"] = rng.choice([4, 4, 7])
    if op == "step":
        c["x"] = x
    if op == "multi":
        c["group"] = rng.choice([1, 2, 4, 4])
        c["queries"] = rng.randint(2, 16 // c["group"])
    if op == "hybrid":
        c["window"] = _log(rng, 16, 512)
    if op == "encode":
        c["kind"], c["x"], c["depth"] = rng.choice(["pair", "pair", "key", "value"]), x, rng.choice([4, 4, 7])
        c["tokens"], c["first"] = _log(rng, 100, 32768), rng.choice([0, 0, rng.randrange(1, 200)])
    if op == "dequant":
        c["kind"], c["out"] = rng.choice(["key", "value"]), out
        c["tokens"], c["first"] = _log(rng, 100, 32768), rng.choice([0, rng.randrange(1, 200)])
    if op == "fit":
        c["tokens"], c["x"], c["rounds"] = _log(rng, 1000, 32768), x, rng.randint(5, 20)
    if op == "general":
        c["batch"], c["group"], c["bits"], c["x"] = rng.randint(1, 6), rng.choice([1, 2, 4]), rng.choice(GENERAL_BITS), x
        c["kv_heads"] = rng.choice([1, 2, 4])
        c["hi"] = min(_log(rng, 100, 8000), 65536 // (c["batch"] * c["kv_heads"] * c["group"]))
        c["lo"] = c["hi"] if rng.random() < 0.3 else max(1, c["hi"] // rng.randint(2, 16))
        c["tokens"], c["lens_seed"] = _log(rng, 50, 4096 // c["kv_heads"]), rng.randrange(1 << 20)
    return c


def _lengths(case):
    return np.random.default_rng(case["lens_seed"]).integers(case["lo"], case["hi"] + 1, size=case["batch"])


# ---- the method in torch, 64 bits -------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _preconditioner(pre):
    """The model's rotation S: the Q factor of a Gaussian matrix, or a randomised Hadamard matrix."""
    rng = np.random.default_rng(2024)
    if pre == "hadamard":
        i = np.arange(D)
        parity = np.array([bin(v).count("1") & 1 for v in range(D)])[i[:, None] & i[None, :]]
        return np.where(rng.random(D) < 0.5, -1.0, 1.0)[:, None] * (1.0 - 2.0 * parity) / math.sqrt(D)
    q, r = np.linalg.qr(rng.standard_normal((D, D)))
    return q * np.sign(np.diag(r))[None, :]


@functools.lru_cache(maxsize=None)
def _codebooks(bits):
    """Centroids of levels 1..len(bits): equal cells at level 1, the optimal quantiser of sin^m(2 psi) above (Lemma 2)."""
    books = [2.0 * math.pi * (np.arange(1 << bits[0]) + 0.5) / (1 << bits[0])]
    t = np.linspace(0.0, 0.5 * math.pi, 400001)
    for level in range(2, len(bits) + 1):
        f = np.sin(2.0 * t) ** ((1 << (level - 1)) - 1)
        step = t[1] - t[0]
        mass = np.concatenate([[0.0], np.cumsum(0.5 * (f[1:] + f[:-1])) * step])
        g = f * t
        moment = np.concatenate([[0.0], np.cumsum(0.5 * (g[1:] + g[:-1])) * step])
        c = 0.5 * math.pi * (np.arange(1 << bits[level - 1]) + 0.5) / (1 << bits[level - 1])
        for _ in range(20000):
            edge = np.concatenate([[0.0], 0.5 * (c[1:] + c[:-1]), [0.5 * math.pi]])
            new = np.diff(np.interp(edge, t, moment)) / np.diff(np.interp(edge, t, mass))
            done = np.max(np.abs(new - c)) < 1e-13
            c = new
            if done:
                break
        books.append(c)
    return tuple(tuple(b) for b in books)


def _f64(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device=DEV)


def _angles(x, depth, pre):
    """x [..., 128] -> the angles of levels 1..depth, and the radii left at the top."""
    r = x.double() @ _f64(_preconditioner(pre))
    angles = []
    for level in range(depth):
        a, b = r[..., 0::2], r[..., 1::2]
        psi = torch.atan2(b, a)
        angles.append(torch.where(psi < 0, psi + 2.0 * math.pi, psi) if level == 0 else psi)
        r = torch.sqrt(a * a + b * b)
    return angles, r


def _quantise(x, bits, pre):
    """-> codes of each level (int64 [..., 128 >> level]) and binary16 radii."""
    angles, r = _angles(x, len(bits), pre)
    codes = []
    for psi, book in zip(angles, _codebooks(bits)):
        c = _f64(book)
        codes.append(torch.bucketize(psi.contiguous(), 0.5 * (c[1:] + c[:-1])))
    return codes, r.clamp(max=65504.0).to(torch.float16)


def _dequantise(codes, radii, bits):
    """-> the vectors in the rotated domain, float64 [..., 128]."""
    r = radii.double()
    for level in range(len(bits), 0, -1):
        theta = _f64(_codebooks(bits)[level - 1])[codes[level - 1]]
        r = torch.stack([r * torch.cos(theta), r * torch.sin(theta)], dim=-1).flatten(-2)
    return r


def _bytes(fields, widths):
    """Fields [..., n] of the given widths, one after another in a little-endian bit stream -> bytes [..., ceil / 8]."""
    bits = torch.cat([(f[..., None] >> torch.arange(w, device=DEV)) & 1 for f, w in zip(fields, widths)], dim=-1) \
        if isinstance(fields, (list, tuple)) else ((fields[..., None] >> torch.arange(widths, device=DEV)) & 1).flatten(-2)
    pad = -bits.shape[-1] % 8
    if pad:
        bits = torch.nn.functional.pad(bits, (0, pad))
    bits = bits.unflatten(-1, (-1, 8))
    return (bits << torch.arange(8, device=DEV)).sum(-1).to(torch.uint8)


def _tiles(kind, codes, radii, depth):
    """codes / radii of [H, T * 64] vectors -> tile codes uint8 [H, T, 2944] and radius planes int16 [H, T, 512 or 128]."""
    c1, c2, c3, c4 = [c.unflatten(1, (-1, TILE)) for c in codes[:4]]
    c1, c2, c3 = c1.unflatten(-1, (8, 4, 2)), c2.unflatten(-1, (8, 4)), c3.unflatten(-1, (8, 2))
    quarter = (c1[..., 1] << 6) | (c2 << 4) | c1[..., 0]                     # [H, T, 64, 8, 4]
    block = (c4 << 4) | (c3[..., 0] << 2) | c3[..., 1]                       # [H, T, 64, 8]
    if kind == "key":
        fields = [f for b in range(8) for f in [*quarter[..., b, :].unbind(-1), block[..., b]]]
        s = _bytes(fields, [10, 10, 10, 10, 6] * 8)                          # [H, T, 64, 46]
        planes = [s[..., 0:16], s[..., 16:32], s[..., 32:44], s[..., 44:46]]
    else:                                                                    # token 16 i + 4 g + e, slot 4 i + e of lane (g, 2 b + h)
        q = quarter.unflatten(2, (4, 4, 4)).unflatten(-1, (2, 2))            # [H, T, i, g, e, b, h, 2]
        q = q.permute(0, 1, 3, 5, 6, 2, 4, 7).flatten(5).flatten(2, 4)       # [H, T, 64 lanes, 32 fields]
        s = _bytes(q, 10)
        bi = block.unflatten(2, (4, 4, 4)).permute(0, 1, 3, 5, 2, 4).flatten(4).flatten(2, 3)
        planes = [s[..., 0:16], s[..., 16:32], s[..., 32:40], _bytes(bi, 6)]
    tile_codes = torch.cat([p.flatten(2) for p in planes], dim=-1)
    if depth == 7:
        words, shift = torch.zeros_like(c4[..., 0]), 0
        for c in codes[4:]:
            for f in c.unflatten(1, (-1, TILE)).unbind(-1):
                words, shift = words | (f << shift), shift + 2
        r = radii.unflatten(1, (-1, TILE))[..., 0].view(torch.int16)
        return tile_codes, torch.stack([words.to(torch.int16), r], dim=-1).flatten(2)
    r = radii.unflatten(1, (-1, TILE))                                       # [H, T, 64, 8]
    if kind == "value":
        r = r.unflatten(2, (4, 4, 4)).permute(0, 1, 3, 5, 2, 4)
    return tile_codes, r.flatten(2).contiguous().view(torch.int16)


# ---- inputs -----------------------------------------------------------------------------------------------------------

def _gen(seed, part):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + part)
    return g


def _vectors(shape, g):
    """[..., heads, tokens, 128] float32: N(0, 1), four channels per head scaled by exp(N(2, 0.5^2))."""
    heads = shape[-3]
    scale = torch.ones(heads, D, device=DEV)
    pick = torch.rand(heads, D, generator=g, device=DEV).argsort(dim=1)[:, :4]
    scale.scatter_(1, pick, torch.exp(2.0 + 0.5 * torch.randn(heads, 4, generator=g, device=DEV)))
    return torch.randn(shape, generator=g, device=DEV) * scale[:, None, :]


def _bits(case):
    return BITS7 if case.get("depth") == 7 else BITS4


def _context(case):
    ctx = Context(S=_preconditioner(case["pre"]))
    if case.get("depth") == 7:
        ctx.set_recursion_depth(7, BITS7[4:])
    return ctx


def _bank(case, seed, part):
    """Quantised vectors of one stream: codes and radii of [kv_heads, BANK_TILES * 64] vectors."""
    x = _vectors((case["kv_heads"], BANK_TILES * TILE, D), _gen(seed, part)).bfloat16()
    return _quantise(x, _bits(case), case["pre"])


def _picks(n_tiles, seed, part):
    return torch.randint(0, BANK_TILES, (n_tiles,), generator=_gen(seed, part), device=DEV)


def _sequences(case):
    lens = _lengths(case)
    tiles = (lens + TILE - 1) // TILE
    start = np.concatenate([[0], np.cumsum(tiles)[:-1]]) * TILE
    return lens, start, int(tiles.sum())


def _new_tokens(case, seed, part):
    x = _vectors((case["kv_heads"], case["batch"], D), _gen(seed, part))
    return x.transpose(0, 1).contiguous().to(DTYPES[case.get("x", "bf16")])


def _query(case, seed, *more):
    shape = (case["batch"], *more, case["kv_heads"] * case["group"], D)
    return torch.randn(shape, generator=_gen(seed, 9), device=DEV).bfloat16()


def _window(case, seed):
    shape = (case["batch"], case["kv_heads"], case["window"], D)
    return _vectors(shape, _gen(seed, 7)).bfloat16(), _vectors(shape, _gen(seed, 8)).bfloat16()


def _window_lengths(case):
    """How far each sequence has generated: between half of the window and all of it."""
    return np.random.default_rng(case["lens_seed"] + 1).integers((case["window"] + 1) // 2, case["window"] + 1, size=case["batch"])


def _stream(case, seed, part):
    """Vectors to encode, [kv_heads, tokens, 128]: what a projection leaves behind, head-major."""
    return _vectors((case["kv_heads"], case["tokens"], D), _gen(seed, part)).to(DTYPES[case["x"]])


def _attention_state(case, seed):
    lens, start, n_tiles = _sequences(case)
    st = {"op": case["op"], "ctx": _context(case), "max_ctx": int(lens.max()),
          "start": torch.from_numpy(start).to(DEV), "len": torch.from_numpy(lens.astype(np.int32)).to(DEV)}
    for i, kind in enumerate(("key", "value")):
        codes, radii = _tiles(kind, *_bank(case, seed, i), case["depth"])
        at = _picks(n_tiles, seed, 2 + i)
        st[kind] = (codes[:, at], radii[:, at])
    B, Hq, Hkv = case["batch"], case["kv_heads"] * case["group"], case["kv_heads"]
    if case["op"] == "multi":
        st["q"] = _query(case, seed, case["queries"])
        n = Context.attn_mq_workspace_bytes(B, case["queries"], Hq, Hkv, st["max_ctx"])
    elif case["op"] == "hybrid":
        st["q"], st["window"] = _query(case, seed), _window(case, seed)
        st["win_len"] = torch.from_numpy(_window_lengths(case).astype(np.int32)).to(DEV)
        n = Context.attn_hybrid_workspace_bytes(B, Hq, Hkv, st["max_ctx"], case["window"])
    else:
        st["q"] = _query(case, seed)
        st["xk"], st["xv"] = _new_tokens(case, seed, 5), _new_tokens(case, seed, 6)
        st["slot"] = st["start"] + st["len"].long() - 1      # the context counts the new token
        n = Context.attn_workspace_bytes(B, Hq, Hkv, st["max_ctx"])
    st["out"] = torch.empty(st["q"].shape, dtype=DTYPES[case["out"]], device=DEV)
    st["workspace"] = torch.empty(n, dtype=torch.uint8, device=DEV)
    return st


def _general_bits(case):
    return tuple(int(b) for b in case["bits"].split(","))


def _general_records(codes, radii, bits):
    stream = torch.cat([(c[..., None] >> torch.arange(w, device=DEV)).bitwise_and(1).flatten(-2) for c, w in zip(codes, bits)], dim=-1)
    return torch.cat([_bytes(stream, 1), radii.contiguous().view(torch.uint8)], dim=-1)


def _general_bank(case, seed, part, n):
    x = _vectors((case["kv_heads"], n, D), _gen(seed, part)).bfloat16()
    return _quantise(x, _general_bits(case), case["pre"])


def _general_state(case, seed):
    lens = _lengths(case)
    start = np.concatenate([[0], np.cumsum(lens)[:-1]])
    n, bits = int(lens.sum()), _general_bits(case)
    fmt = GeneralFormat(len(bits), bits)
    st = {"op": "general", "ctx": _context(case), "fmt": fmt, "books": np.concatenate([np.asarray(b) for b in _codebooks(bits)]),
          "start": torch.from_numpy(start).to(DEV), "len": torch.from_numpy(lens.astype(np.int32)).to(DEV), "q": _query(case, seed)}
    for i, kind in enumerate(("key", "value")):
        st[kind] = _general_records(*_general_bank(case, seed, i, n), bits).contiguous()
        st["x_" + kind] = _stream(case, seed, 5 + i).flatten(0, 1)
        st["new_" + kind] = torch.zeros((case["kv_heads"] * case["tokens"], fmt.record_bytes()), dtype=torch.uint8, device=DEV)
    st["out"] = torch.empty(st["q"].shape, dtype=torch.float32, device=DEV)
    return st


def _cache(case):
    pool = -(-(case["first"] + case["tokens"]) // TILE) * TILE
    codes, radii = Context.alloc_cache(case["kv_heads"], pool, DEV, 128 if case.get("depth") == 7 else 512)
    return codes.zero_(), radii.zero_()


def prepare(case, seed):
    op = case["op"]
    if op in ("step", "multi", "hybrid"):
        return _attention_state(case, seed)
    if op == "general":
        return _general_state(case, seed)
    st = {"op": op, "ctx": _context(case)}
    if op == "encode":
        st["kind"] = case["kind"]
        st["x"] = [_stream(case, seed, p).transpose(0, 1) for p in ((0, 1) if case["kind"] == "pair" else (0,))]
        st["cache"], st["first"] = [_cache(case) for _ in st["x"]], case["first"]
    elif op == "dequant":
        n_tiles = -(-(case["first"] + case["tokens"]) // TILE)
        codes, radii = _tiles(case["kind"], *_bank(case, seed, 0), 4)
        at = _picks(n_tiles, seed, 2)
        st["kind"], st["cache"], st["first"], st["tokens"] = case["kind"], (codes[:, at], radii[:, at]), case["first"], case["tokens"]
        st["out"] = torch.empty((case["tokens"], case["kv_heads"], D), dtype=DTYPES[case["out"]], device=DEV)
    else:
        st["x"], st["rounds"] = _stream(case, seed, 0).transpose(0, 1), case["rounds"]
        st["workspace"] = torch.empty(Context.fit_workspace_bytes(), dtype=torch.uint8, device=DEV)
    return st


# ---- one pass ---------------------------------------------------------------------------------------------------------

def run(st):
    op, ctx = st["op"], st["ctx"]
    if op == "step":
        ctx.decode_step_polar(st["xk"], st["xv"], st["slot"], st["q"], st["out"], *st["key"], *st["value"], st["start"], st["len"],
                              st["max_ctx"], SCALE, st["workspace"])
        return {"out": st["out"], "key": st["key"], "value": st["value"]}
    if op == "multi":
        ctx.attn_decode_polar_mq(st["q"], st["out"], *st["key"], *st["value"], st["start"], st["len"], st["max_ctx"], SCALE,
                                 st["workspace"])
        return {"out": st["out"]}
    if op == "hybrid":
        ctx.attn_decode_hybrid(st["q"], st["out"], *st["key"], *st["value"], st["start"], st["len"], *st["window"], st["win_len"],
                               st["max_ctx"], SCALE, st["workspace"])
        return {"out": st["out"]}
    if op == "encode":
        if st["kind"] == "pair":
            ctx.encode_kv_pair(*st["x"], *st["cache"][0], *st["cache"][1], dst_token0=st["first"])
        else:
            ctx.encode_kv(st["x"][0], PQ_KEY if st["kind"] == "key" else PQ_VALUE, *st["cache"][0], dst_token0=st["first"])
        return {"cache": st["cache"]}
    if op == "dequant":
        ctx.decode_kv(PQ_KEY if st["kind"] == "key" else PQ_VALUE, *st["cache"], st["first"], st["tokens"], st["out"])
        return {"out": st["out"]}
    if op == "fit":
        return {"centroids": ctx.fit_codebooks(st["x"], st["rounds"], workspace=st["workspace"])}
    general_encode(ctx, st["fmt"], st["books"], st["x_key"], st["new_key"])
    general_encode(ctx, st["fmt"], st["books"], st["x_value"], st["new_value"])
    general_attn_decode(ctx, st["fmt"], st["books"], st["q"], st["out"], st["key"], st["value"], st["start"], st["len"], SCALE)
    return {"out": st["out"], "new_key": st["new_key"], "new_value": st["new_value"]}


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def work(case):
    op, H = case["op"], case["kv_heads"]
    size = {"bf16": 2, "f32": 4}
    rotate = 2 * D * D                                        # one vector times S
    record = 50 if case.get("depth") == 7 else 62
    if op in ("step", "multi", "hybrid"):
        lens, rows = _lengths(case), case["batch"] * case.get("queries", 1) * H * case["group"]
        cached = int(lens.sum()) * H
        n_bytes = 2 * record * cached + rows * D * (2 + size[case["out"]])
        flops = 4 * D * cached * case["group"] * case.get("queries", 1) + 2 * rotate * rows
        if op == "step":
            n_bytes += 2 * case["batch"] * H * D * size[case["x"]]
            flops += 2 * rotate * case["batch"] * H
        if op == "hybrid":
            window = int(_window_lengths(case).sum()) * H
            n_bytes += 2 * window * D * 2
            flops += 4 * D * window * case["group"]
        return {"bytes": n_bytes, "flops": flops}
    if op == "general":
        bits = _general_bits(case)
        record = (sum((D >> (l + 1)) * b for l, b in enumerate(bits)) + 7) // 8 + 2 * (D >> len(bits))
        cached, rows, new = int(_lengths(case).sum()) * H, case["batch"] * H * case["group"], 2 * case["tokens"] * H
        return {"bytes": 2 * record * cached + rows * D * 6 + new * (D * size[case["x"]] + record),
                "flops": 4 * D * cached * case["group"] + 2 * rotate * rows + rotate * new}
    n = case["tokens"] * H * (2 if case.get("kind") == "pair" else 1)
    if op == "encode":
        return {"bytes": n * (D * size[case["x"]] + record), "flops": rotate * n}
    if op == "dequant":
        return {"bytes": n * (62 + D * size[case["out"]]), "flops": rotate * n}
    return {"bytes": n * D * size[case["x"]], "flops": rotate * n}


def tolerance(case):
    op = case["op"]
    if op in ("step", "multi", "hybrid"):
        # binary16 matrix operands: 8e-4 off the 64-bit result; a bfloat16 output adds its own 1.7e-3.  The largest
        # difference is that of a row whose softmax rests on few tokens.  The appended records: see below.
        return {"rel": 8e-3 if case["out"] == "bf16" else 4e-3, "max": 0.2, "differ": 1e-4}
    if op == "encode":
        # a binary16 radius next to a rounding boundary (1e-4 of them) or an angle next to a cell boundary (3e-7) may go either way
        return {"rel": 0.0, "differ": 5e-4}
    if op == "dequant":
        return {"rel": 8e-3, "max": 0.02} if case["out"] == "bf16" else {"rel": 1e-6, "max": 1e-5}
    if op == "fit":
        # counts in bins of 5e-4 to 1e-3 rad: up to 1e-4 rad off the k-means on the angles themselves
        return {"rel": 2e-4, "max": 1e-3}
    return {"rel": 4e-6, "max": 4e-5, "differ": 5e-4}          # plain 32-bit sums; records as in encode


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------

def _attend(q, k, v):
    """q [rows, 128], k and v [tokens, 128], float64."""
    return torch.softmax((q @ k.T) * SCALE, dim=1) @ v


def _exact_attention(case, seed):
    bits, S = _bits(case), _f64(_preconditioner(case["pre"]))
    lens, start, n_tiles = _sequences(case)
    G, M = case["group"], case.get("queries", 1)
    banks = [_dequantise(*_bank(case, seed, i), bits) for i in (0, 1)]                     # [H, bank tokens, 128]
    picks = [_picks(n_tiles, seed, 2 + i) for i in (0, 1)]
    q = (_query(case, seed, M) if case["op"] == "multi" else _query(case, seed)[:, None]).double() @ S  # [B, M, Hq, 128]
    new = [_dequantise(*_quantise(_new_tokens(case, seed, p), bits, case["pre"]), bits) for p in (5, 6)] if case["op"] == "step" else None
    if case["op"] == "hybrid":
        window = [w.double() @ S for w in _window(case, seed)]
        win_len = _window_lengths(case)
    out = torch.zeros_like(q)
    for b, n in enumerate(lens):
        n, t0 = int(n), int(start[b]) // TILE
        for h in range(case["kv_heads"]):
            kv = [bank[h].view(BANK_TILES, TILE, D)[at[t0:t0 + -(-n // TILE)]].reshape(-1, D)[:n] for bank, at in zip(banks, picks)]
            if new:
                kv = [torch.cat([x[:-1], y[b, h][None]]) for x, y in zip(kv, new)]
            if case["op"] == "hybrid":
                kv = [torch.cat([x, w[b, h, :int(win_len[b])]]) for x, w in zip(kv, window)]
            for m in range(M):
                seen = max(n - (M - 1 - m), 0) if case["op"] == "multi" else len(kv[0])
                if seen:
                    rows = slice(h * G, (h + 1) * G)
                    out[b, m, rows] = _attend(q[b, m, rows], kv[0][:seen], kv[1][:seen])
    out = out @ S.T
    return {"out": out if case["op"] == "multi" else out[:, 0]}


def _exact_general(case, seed):
    bits, S, G = _general_bits(case), _f64(_preconditioner(case["pre"])), case["group"]
    lens = _lengths(case)
    kd, vd = [_dequantise(*_general_bank(case, seed, i, int(lens.sum())), bits) for i in (0, 1)]
    q = _query(case, seed).double() @ S
    out, at = torch.zeros_like(q), 0
    for b, n in enumerate(lens):
        for h in range(case["kv_heads"]):
            rows = slice(h * G, (h + 1) * G)
            out[b, rows] = _attend(q[b, rows], kd[h, at:at + int(n)], vd[h, at:at + int(n)])
        at += int(n)
    return {"out": out @ S.T, "new_key": None, "new_value": None}


def _exact_fit(case, seed):
    """k-means rounds on the angles themselves, from the analytic codebook."""
    angles, _ = _angles(_stream(case, seed, 0), 4, case["pre"])
    fitted = []
    for psi, book in zip(angles, _codebooks(BITS4)):
        psi, c = psi.reshape(-1).sort().values, _f64(book)
        total = torch.cat([psi.new_zeros(1), psi.cumsum(0)])
        for _ in range(case["rounds"]):
            cut = torch.searchsorted(psi, 0.5 * (c[1:] + c[:-1]))
            cut = torch.cat([cut.new_zeros(1), cut, cut.new_full((1,), psi.numel())])
            count = cut[1:] - cut[:-1]
            c = torch.where(count > 0, (total[cut[1:]] - total[cut[:-1]]) / count.clamp(min=1), c)
        fitted.append(c)
    return {"centroids": torch.cat(fitted)}


def exact(case, seed):
    op = case["op"]
    if op in ("step", "multi", "hybrid"):
        out = _exact_attention(case, seed)
        return {**out, "key": None, "value": None} if op == "step" else out
    if op == "general":
        return _exact_general(case, seed)
    if op == "fit":
        return _exact_fit(case, seed)
    if op == "dequant":
        n_tiles = -(-(case["first"] + case["tokens"]) // TILE)
        bank = _dequantise(*_bank(case, seed, 0), BITS4).unflatten(1, (BANK_TILES, TILE))
        v = bank[:, _picks(n_tiles, seed, 2)].flatten(1, 2)[:, case["first"]:case["first"] + case["tokens"]]
        return {"out": (v @ _f64(_preconditioner(case["pre"])).T).transpose(0, 1)}
    return None                                              # encode: bytes only
