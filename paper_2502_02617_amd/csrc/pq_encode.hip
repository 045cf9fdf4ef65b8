/*
 * pq_encode.hip -- pq_encode_kv / pq_encode_kv_pair / pq_append_kv: Algorithm 1
 * lines 2 and 4 (precondition with S, procedure Polar, procedure Quant) plus
 * bit-packing into the tile layout, for gfx950.
 *
 * Bulk kernels (pq_encode_kv, and for keys and values in one launch
 * pq_encode_kv_pair; the append kernel lives in pq_polar.h):
 * one wavefront owns one destination tile (64 token slots of one head plane);
 * where there are few tiles, a workgroup does.
 *   1. y = x * S on the matrix cores.  S is held as three bf16 terms
 *      S1 + S2 + S3 (24 significant bits) so that bf16 MFMAs with fp32
 *      accumulation reproduce an fp32-accurate rotation; bf16 inputs are
 *      exact operands.  fp32 inputs and S are two binary16 terms each and three
 *      products are accumulated, all but that of the two second terms, 2^-22 of
 *      the whole at most (three bf16 terms and six products where S leaves
 *      coordinates unmixed).
 *      The product is computed transposed, D = S^T-tile (32 rotated
 *      coordinates) x X^T (32 vectors), with the rows of each S^T tile
 *      ordered so that a lane ends up with complete blocks of 16 consecutive
 *      rotated coordinates of one vector in its accumulator registers: the
 *      whole polar recursion of a block is then register-local.
 *   2. Four polar levels per block; every angle is quantised by comparing
 *      in the tangent domain (v > tan(t) * u for each inner boundary t, on
 *      squared radii above level 1), which is the nearest-centroid rule of
 *      procedure Quant without evaluating an arctangent or, but for the
 *      block radius, a square root.
 *   3. Whole tiles: the blocks' indices go through LDS to the lanes that own the
 *      tile's bit strings, which join them in registers and store them.
 *      Partially written tiles: the fields are scattered with LDS atomics into an
 *      image of the tile, and the image is written out.
 *   At recursion depth 7 the recursion goes on over the block radii of a vector
 *   (levels 5, 6, 7) and one word per token replaces the block radii.
 */
#include <type_traits>

#include "pq_common.h"
#include "pq_polar.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

/* wavefronts per workgroup (two per SIMD: the kernel uses the whole register file).  Sixteen
   wavefronts working on one 32-vector half at a time in 128 registers measured slower: every
   A-operand fetch then feeds one matrix instruction instead of two. */
template <int XT> struct EncodeShape { static constexpr int waves = 8; };
/* tile image in LDS: the code bytes, then the radius plane (512 binary16 block radii, or at
   depth 7 the 64 words of radius and upper-level codes) */
template <bool DEEP> struct TileImage {
    static constexpr int radii_halves = DEEP ? PQ_DEEP_RADII_HALVES : PQL_RADII;
    static constexpr int dwords = (PQL_CODE_BYTES + radii_halves * 2) / 4; /* 992 or 800 */
};

struct EncodeArgs {
    const void *x;
    int64_t ld_token, ld_head;
    uint8_t *codes;
    uint16_t *radii;
    int64_t pool_tiles;
    int64_t pool_tokens;
    /* tokens [dst0, dst0 + n) of every head plane */
    int64_t dst0, n_tokens;
    int64_t first_tile, n_tiles; /* tiles spanned by the range */
    int n_heads;
    int64_t n_items;
    const uint4 *S_bf16x3;
    const PqDeviceConsts *consts;
};

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ uint32_t bf16_rne_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

union BOperand {
    bf16x8 v;
    f16x8 h;
    uint4 q;
    uint32_t w[4];
};

/* ---- partially written tiles: an image of the tile's present contents in LDS, into which the fields of block b of slot
 * tau are scattered without branches: every field's bits are cleared and the field, shifted to its place inside a pair of
 * dwords, is OR-ed in.  The image is shared by the lanes of one wavefront and the fields of different slots share
 * dwords: LDS atomics.  The positions are those of pq_layout.h, written out per plane. ---- */
__device__ __forceinline__ void put_pair(uint32_t *img, uint32_t at0, uint32_t at1, uint32_t field, uint32_t width, uint32_t sh)
{
    const uint64_t m = (uint64_t)((1u << width) - 1u) << sh;
    atomicAnd(&img[at0], ~(uint32_t)m);
    atomicAnd(&img[at1], ~(uint32_t)(m >> 32));
    const uint64_t w = (uint64_t)field << sh;
    atomicOr(&img[at0], (uint32_t)w);
    atomicOr(&img[at1], (uint32_t)(w >> 32));
}

template <int KIND, bool DEEP>
__device__ __forceinline__ void emit_block(uint32_t *img, int tau, int b, const BlockCodes &bc)
{
    const uint32_t q0 = bc.q[0], q1 = bc.q[1], q2 = bc.q[2], q3 = bc.q[3], bi = bc.bi;
    uint32_t radius_half;
    if (KIND == PQ_KEY) {
        /* dword d of the token's string: planes of 4, 4, 3 dwords per token, then one half per token */
        auto at = [&](uint32_t d) {
            return d < 4u ? 4u * tau + d : d < 8u ? (PQL_OFF_P1 / 4 - 4) + 4u * tau + d
                 : d < 11u ? (PQL_OFF_P2 / 4 - 8) + 3u * tau + d : PQL_OFF_KP3 / 4 + ((uint32_t)tau >> 1);
        };
        const uint32_t bit = PQL_BLOCK_BITS * (uint32_t)b, d = bit >> 5, sh = bit & 31u;
        /* the string's last half sits in a dword shared by two tokens */
        const uint32_t sh1 = (d + 1u == 11u) ? 16u * ((uint32_t)tau & 1u) : 0u;
        /* 46 bits reach into a third dword when they start above bit 18 (never in the string's last dwords) */
        const bool third = sh > 18u;
        const uint32_t a0 = at(d), a1 = at(d + 1u), a2 = at(third ? d + 2u : d);
        const uint64_t m = ((1ull << PQL_BLOCK_BITS) - 1ull) << sh;
        atomicAnd(&img[a0], ~(uint32_t)m);
        atomicAnd(&img[a1], ~((uint32_t)(m >> 32) << sh1));
        if (third) atomicAnd(&img[a2], ~(0x3FFFu >> (32u - sh)));
        const uint32_t lo = q0 | (q1 << 10) | (q2 << 20) | (q3 << 30), hi = (q3 >> 2) | (bi << 8); /* 32 + 14 bits */
        const uint64_t w = (((uint64_t)hi << 32) | lo) << sh;
        atomicOr(&img[a0], (uint32_t)w);
        atomicOr(&img[a1], (uint32_t)(w >> 32) << sh1);
        if (third) atomicOr(&img[a2], hi >> (32u - sh));
        radius_half = 8u * tau + b;
    } else {
        const uint32_t i = (uint32_t)tau >> 4, g = ((uint32_t)tau >> 2) & 3u, e = (uint32_t)tau & 3u, s = 4u * i + e;
        /* dword d of lane lam's string: planes of 4, 4, 2 dwords per lane */
        auto at = [&](uint32_t lam, uint32_t d) {
            return d < 4u ? 4u * lam + d : d < 8u ? (PQL_OFF_P1 / 4 - 4) + 4u * lam + d : (PQL_OFF_P2 / 4 - 8) + 2u * lam + d;
        };
        const uint32_t bit = PQL_SLOT_BITS * s, d = bit >> 5, sh = bit & 31u;
        /* the dword after a string's last one belongs to the next lane (or the next plane): it gets zeros */
        const uint32_t lam0 = 16u * g + 2u * b;
        put_pair(img, at(lam0, d), at(lam0, d + 1u), q0 | (q1 << 10), PQL_SLOT_BITS, sh);
        put_pair(img, at(lam0 + 1u, d), at(lam0 + 1u, d + 1u), q2 | (q3 << 10), PQL_SLOT_BITS, sh);
        const uint32_t bbit = 6u * s, base = PQL_OFF_VB / 4 + 3u * (8u * g + b) + (bbit >> 5);
        put_pair(img, base, base + 1u, bi, 6u, bbit & 31u);
        radius_half = 16u * (8u * g + b) + s;
    }
    if (!DEEP) reinterpret_cast<uint16_t *>(img)[PQL_CODE_BYTES / 2 + radius_half] = bc.radius;
}

/* ---- whole tiles: every block leaves its indices and radius in LDS at a place of its own (plain writes, compile-time
 * shifts), and once the tile is complete a lane reads the blocks of its strings, joins them and stores
 * full-width dwords.  An image for whole tiles too, with its addresses and atomics, made the keys and values of 32768
 * tokens 64.1 us against 57.6 (235 against 219 at four times as many; one-term S 43.3 against 41.8; value tiles
 * gain most: 34.9 against 30.6 for 262144 vectors, keys 30.7 against 30.2).
 *   keys:   [block][token] of two dwords: Q0 | Q1 << 10 | Q2 << 20 | Q3 << 30, then Q3 >> 2 | B << 8 | radius << 16
 *   values: [half-block][token] of one dword: its two indices, for the first half also B << 20; behind them the
 *           radii [block][token].  Rows of 68 dwords and 68 halves: the reads of 16 half-blocks (8 blocks) at one token
 *           then fall on different banks. ---- */
constexpr int kRow = 68, kRadiiAt = 16 * kRow /* dwords */, kWaveDwords = kRadiiAt + 8 * kRow / 2;

template <int KIND, bool DEEP>
__device__ __forceinline__ void leave_block(uint32_t *buf, int tau, int b, const BlockCodes &bc)
{
    if (KIND == PQ_KEY) {
        const uint32_t lo = bc.q[0] | (bc.q[1] << 10) | (bc.q[2] << 20) | (bc.q[3] << 30);
        uint32_t hi = (bc.q[3] >> 2) | (bc.bi << 8);
        if (!DEEP) hi |= (uint32_t)bc.radius << 16;
        *reinterpret_cast<uint2 *>(buf + 2 * (64 * b + tau)) = make_uint2(lo, hi);
    } else {
        buf[(2 * b) * kRow + tau] = bc.q[0] | (bc.q[1] << 10) | (bc.bi << 20);
        buf[(2 * b + 1) * kRow + tau] = bc.q[2] | (bc.q[3] << 10);
        if (!DEEP) reinterpret_cast<uint16_t *>(buf + kRadiiAt)[b * kRow + tau] = bc.radius;
    }
}

/* `width` bits of v (the others zero) to bit BIT of the string w, whose bits from there on are zero */
template <int BIT, int WIDTH>
__device__ __forceinline__ void put_field(uint32_t *w, uint32_t v)
{
    constexpr int d = BIT >> 5, s = BIT & 31;
    if constexpr (s == 0) w[d] = v;
    else {
        w[d] |= v << s;
        if constexpr (s + WIDTH > 32) w[d + 1] = v >> (32 - s);
    }
}

template <bool DEEP, int B>
__device__ __forceinline__ void join_key_block(uint32_t (&w)[12], uint32_t (&rad)[4], const uint32_t *buf, int lane)
{
    const uint2 f = *reinterpret_cast<const uint2 *>(buf + 2 * (64 * B + lane));
    put_field<PQL_BLOCK_BITS * B, 32>(w, f.x);
    put_field<PQL_BLOCK_BITS * B + 32, 14>(w, DEEP ? f.y : f.y & 0x3FFFu);
    if (!DEEP) rad[B / 2] = (B & 1) ? __builtin_amdgcn_perm(f.y, rad[B / 2], 0x07060100u) : f.y >> 16;
}

template <int I, bool DEEP>
__device__ __forceinline__ void join_value_slots(uint32_t (&w)[10], uint32_t (&vb)[3], uint32_t (&rad)[4], const uint32_t *buf, int lane)
{
    const int g = lane >> 4, n = lane & 15;
    const uint4 f = *reinterpret_cast<const uint4 *>(buf + n * kRow + 16 * I + 4 * g); /* slots 4 I .. 4 I + 3 */
    put_field<PQL_SLOT_BITS * (4 * I), 20>(w, f.x & 0xFFFFFu);
    put_field<PQL_SLOT_BITS * (4 * I + 1), 20>(w, f.y & 0xFFFFFu);
    put_field<PQL_SLOT_BITS * (4 * I + 2), 20>(w, f.z & 0xFFFFFu);
    put_field<PQL_SLOT_BITS * (4 * I + 3), 20>(w, f.w & 0xFFFFFu);
    put_field<6 * (4 * I), 6>(vb, f.x >> 20);
    put_field<6 * (4 * I + 1), 6>(vb, f.y >> 20);
    put_field<6 * (4 * I + 2), 6>(vb, f.z >> 20);
    put_field<6 * (4 * I + 3), 6>(vb, f.w >> 20);
    if (!DEEP && I < 2) { /* half n & 1 of the block stores slots 8 (n & 1) .. + 7 of its radii */
        const uint2 r = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(buf + kRadiiAt) + (n >> 1) * kRow +
                                                         16 * (2 * (n & 1) + I) + 4 * g);
        rad[2 * I] = r.x;
        rad[2 * I + 1] = r.y;
    }
}

/* the strings and radii of a whole tile, one lane per token (keys) or half-block of 16 tokens (values) */
template <int KIND, bool DEEP>
__device__ __forceinline__ void store_tile(const uint32_t *buf, uint8_t *gcodes, uint16_t *gradii, int lane)
{
    struct Three { uint32_t x, y, z; };
    uint32_t rad[4];
    if (KIND == PQ_KEY) {
        uint32_t w[12];
        join_key_block<DEEP, 0>(w, rad, buf, lane); join_key_block<DEEP, 1>(w, rad, buf, lane);
        join_key_block<DEEP, 2>(w, rad, buf, lane); join_key_block<DEEP, 3>(w, rad, buf, lane);
        join_key_block<DEEP, 4>(w, rad, buf, lane); join_key_block<DEEP, 5>(w, rad, buf, lane);
        join_key_block<DEEP, 6>(w, rad, buf, lane); join_key_block<DEEP, 7>(w, rad, buf, lane);
        reinterpret_cast<uint4 *>(gcodes + PQL_OFF_P0)[lane] = make_uint4(w[0], w[1], w[2], w[3]);
        reinterpret_cast<uint4 *>(gcodes + PQL_OFF_P1)[lane] = make_uint4(w[4], w[5], w[6], w[7]);
        reinterpret_cast<Three *>(gcodes + PQL_OFF_P2)[lane] = Three{w[8], w[9], w[10]};
        reinterpret_cast<uint16_t *>(gcodes + PQL_OFF_KP3)[lane] = (uint16_t)w[11];
    } else {
        uint32_t w[10], vb[3];
        join_value_slots<0, DEEP>(w, vb, rad, buf, lane); join_value_slots<1, DEEP>(w, vb, rad, buf, lane);
        join_value_slots<2, DEEP>(w, vb, rad, buf, lane); join_value_slots<3, DEEP>(w, vb, rad, buf, lane);
        reinterpret_cast<uint4 *>(gcodes + PQL_OFF_P0)[lane] = make_uint4(w[0], w[1], w[2], w[3]);
        reinterpret_cast<uint4 *>(gcodes + PQL_OFF_P1)[lane] = make_uint4(w[4], w[5], w[6], w[7]);
        reinterpret_cast<uint2 *>(gcodes + PQL_OFF_P2)[lane] = make_uint2(w[8], w[9]);
        if ((lane & 1) == 0) reinterpret_cast<Three *>(gcodes + PQL_OFF_VB)[lane >> 1] = Three{vb[0], vb[1], vb[2]};
    }
    if (!DEEP) reinterpret_cast<uint4 *>(gradii)[lane] = make_uint4(rad[0], rad[1], rad[2], rad[3]);
}

/* lanes 0..31: the value of lane + 32; lanes 32..63: the value of lane - 32 */
__device__ __forceinline__ uint32_t from_other_half(uint32_t x, int upper_half)
{
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return upper_half ? r[0] : r[1];
}

/* NTERMS = 3: S as three bf16 terms.  NTERMS = 1: every entry of S is +-1/sqrt(128), the
   operand is sqrt(128) * S (exactly +-1), one product per k-step replaces three and
   the common factor is taken out of the block radius (the angles do not see it).
   NTERMS = 2: S as two binary16 terms of 2^15 S, 23 significant bits.

   fp32 input with NTERMS = 1 or 2 is two binary16 terms as well, after a power of two has brought the vector's
   largest coordinate to [2^14, 2^15) (the factor comes out of the radius, the angles do not see it): three products
   (two for a +-1 S) instead of the six (three) that three bf16 terms of 8 bits take, and a third of the vector
   instructions to split an input: keys and values of 32768 tokens of 8 heads 116 -> 82 us, 89 -> 72 with a +-1 S.
   Operands: two terms leave up to 2^-23 of a number (three bf16 terms 2^-25), or 2^-39 of the vector's largest coordinate where that
   is more, and the product that is left out is 2^-22 of its whole at most; rms 7e-8 of a product, ten times that of three bf16 terms.
   The fp32 sums, which are half as many, round by more: of 268 M radii of vectors with outlier channels 7.2e-5 differ by a last
   bit from 64 bits (three bf16 terms 8.0e-5), of coordinates spread over 2^12 4.7e-5 (5.1e-5); with a Hadamard S, whose entries
   are exact, 7.0e-5 (7.2e-5) and, spread, 4.68e-5 (4.53e-5: there it is larger, by 3 %).
   2^-39 of the largest coordinate per coordinate is 2^-40 of it rms in a rotated one (the columns of S have norm 1).  Sums that pass
   2^-16 of it round by 2^-41 rms at each of the products behind, a dozen on average of 24: 2^-39.  So an S that
   spreads every coordinate over all pairs of the result by 2^-16 at least (pq_ctx::mixing) does not see it; any other keeps
   NTERMS = 3. */
template <int XT, int NTERMS> struct Operands {
    static constexpr bool half = XT == PQ_F32 && NTERMS <= 2;             /* binary16 terms, else bf16 */
    static constexpr int x_terms = XT == PQ_BF16 ? 1 : (half ? 2 : 3);
    static constexpr int top = NTERMS == 3 ? 2 : 1;                       /* products of terms x + s <= top take part */
    static constexpr int products = x_terms == 1 ? NTERMS : (NTERMS == 3 ? 6 : NTERMS + 1); /* of a k-step */
    static constexpr int s_chunks = NTERMS * 4 * 8 * 64;                  /* 16-byte chunks of S in LDS */
};

template <int XT, int NTERMS>
__device__ __forceinline__ f32x16 multiply(const BOperand &s, const BOperand &x, const f32x16 &c)
{
    if constexpr (Operands<XT, NTERMS>::half) return __builtin_amdgcn_mfma_f32_32x32x16_f16(s.h, x.h, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(s.v, x.v, c, 0, 0, 0);
}

/* Chunk of S as the matrix instructions take it, from the chunks of its bf16 terms (t[1], t[2]: NTERMS > 1). */
template <int XT, int NTERMS>
__device__ __forceinline__ void s_operand(BOperand (&out)[NTERMS], const uint4 *t)
{
    if constexpr (NTERMS == 2) {
        BOperand b[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) b[k].q = t[k];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float f[3];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                f[k] = 32768.f * __uint_as_float((e & 1) ? b[k].w[e / 2] & 0xFFFF0000u : b[k].w[e / 2] << 16);
            const _Float16 hi = (_Float16)(f[0] + f[1]);
            out[0].h[e] = hi;
            out[1].h[e] = (_Float16)((f[0] - (float)hi) + f[1] + f[2]);
        }
    } else {
#pragma unroll
        for (int k = 0; k < NTERMS; ++k) out[k].q = t[k];
        if constexpr (Operands<XT, NTERMS>::half) { /* +-1 */
#pragma unroll
            for (int k = 0; k < 4; ++k) out[0].w[k] = (out[0].w[k] & 0x80008000u) | 0x3C003C00u;
        }
    }
}

/* Eight coordinates as three bf16 terms. */
__device__ __forceinline__ void split_bf16(const float (&f)[8], BOperand (&out)[3])
{
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        uint32_t b[3][2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            float rest = f[e + z];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                b[k][z] = bf16_rne_bits(rest);
                rest -= __uint_as_float(b[k][z] << 16);
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) out[k].w[e / 2] = b[k][0] | (b[k][1] << 16);
    }
}

/* The power of two that brings a vector with largest coordinate m to [2^14, 2^15), as a biased exponent: at least 13 (an
   infinity among the inputs), and 2^103 at most. */
__device__ __forceinline__ uint32_t half_exponent(float m) { return min(268u - (__float_as_uint(m) >> 23), 230u); }

/* What the rotated coordinates have to be multiplied with: the power of two and, with two terms of S, its 2^15. */
template <int NTERMS>
__device__ __forceinline__ float half_unscale(uint32_t e) { return __uint_as_float(((NTERMS == 1 ? 254u : 239u) - e) << 23); }

/* Eight coordinates times the power of two of exponent e as two binary16 terms. */
__device__ __forceinline__ void split_half(const float (&f)[8], uint32_t e, BOperand (&out)[2])
{
    const float scale = __uint_as_float(e << 23);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const _Float16 hi = (_Float16)(f[i] * scale);
        out[0].h[i] = hi;
        out[1].h[i] = (_Float16)__builtin_fmaf(f[i], scale, -(float)hi);
    }
}

__device__ __forceinline__ float max_abs(float m, const float4 &a)
{
    return fmaxf(fmaxf(m, fmaxf(fabsf(a.x), fabsf(a.y))), fmaxf(fabsf(a.z), fabsf(a.w)));
}

/* GENERAL: codebooks set by the caller; level 1 goes through the pseudo-angle cell table (staged
   in LDS), the upper levels compare against three free boundaries. */
/* DEEP: recursion to level 7.  The squared radii of a vector's blocks are kept as the row tiles
   complete (a lane half holds blocks 4H..4H+3 of its vectors); levels 5 and 6 then run inside the
   lane, level 7 joins the two halves with one lane exchange, and the vector's radius and upper
   codes go into its word of the radius plane. */
/* LDS of the encode kernels, shared by all their variants (a workgroup runs alone on its CU):
   S in A-operand order, 32 KB per bf16 term; a tile's blocks, or the image of a partially written tile, per wavefront;
   the level-1 cell table of caller-set codebooks. */
__shared__ uint4 sS[3 * 4 * 8 * 64];
__shared__ __align__(16) uint32_t sImg[8][kWaveDwords];
__shared__ PqDeviceConsts::Lut1Cell sLut[512];

/* The tiles of one launch share: wavefront w of workgroup `block` takes items w * n_blocks + block and then every
 * (8 n_blocks)-th (an item = one destination tile of one head plane). */
template <int XT, int KIND, int NTERMS, bool GENERAL, bool DEEP>
__device__ __forceinline__ void encode_tiles(const EncodeArgs &a, int block, int n_blocks)
{
    constexpr int kImgDwords = TileImage<DEEP>::dwords, kRadiiHalves = TileImage<DEEP>::radii_halves;
    constexpr int kWaves = EncodeShape<XT>::waves, kThreads = kWaves * 64;
    typedef Operands<XT, NTERMS> Op;
    static_assert(kWaves == 8 && kImgDwords <= kWaveDwords && 8 * 64 * 2 <= kWaveDwords, "sImg: eight wavefronts, an image or the blocks of a tile");
    const int lane = threadIdx.x & 63;
    /* same value in all lanes: keeps the item geometry and the tile pointers in scalar registers */
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 31, H = lane >> 5; /* vector within the 32-vector group, lane half */

    /* bf16 input: both 32-vector halves of the tile share every A-operand fetch (halves the
       LDS traffic); fp32 input carries two or three terms per value and goes one half at a time */
    constexpr int NXT = Op::x_terms;
    constexpr int NVT = (XT == PQ_BF16) ? 2 : 1; /* 32-vector halves per pass */
    /* The operand registers of a pass are dead once its last row tile has been multiplied,
       so the next pass's rows are requested then, under the last quantisation stage, and the first
       one's before S is staged (not with three terms of fp32 input: twelve products' operands leave no room) */
    constexpr bool kPipelined = XT == PQ_BF16 || Op::half;
    BOperand xb[NVT][NXT][8];
    float4 raw[XT == PQ_BF16 ? 1 : 16]; /* fp32 input: the rows requested ahead */

    /* which tile and which source rows an item covers */
    struct Geometry {
        int head;
        int64_t tile;       /* tile index inside the head plane */
        int tau_lo, tau_hi; /* slots [tau_lo, tau_hi) of the tile are written */
        int64_t src_t0;     /* source token index of slot tau_lo */
    };
    /* Item = head * n_tiles + tile.  The 64-bit division happens once per wavefront; from then on the position
       advances by the (head, tile) parts of the stride between a wavefront's items. */
    struct Position {
        int head;
        int64_t tile_in; /* tile within the range, below n_tiles */
    };
    const int64_t item_stride = (int64_t)n_blocks * (EncodeShape<XT>::waves);
    /* consecutive tiles go to different workgroups: a short input occupies every CU, one wavefront per SIMD first (3001 fp32
       tokens of 8 heads: 22.4 us with eight consecutive tiles per workgroup on 47 CUs, 15.6 on all; 1000 bf16 tokens, keys
       and values: 18.6 -> 10.9; 32768: 69.4 -> 68.4) */
    const int64_t item0 = (int64_t)wave * n_blocks + block;
    const int stride_heads = (int)(item_stride / a.n_tiles);
    const int64_t stride_tiles = item_stride % a.n_tiles;
    auto advance = [&](Position p) {
        p.head += stride_heads;
        p.tile_in += stride_tiles;
        if (p.tile_in >= a.n_tiles) {
            p.tile_in -= a.n_tiles;
            ++p.head;
        }
        return p;
    };
    auto geometry = [&](const Position &p) {
        Geometry g;
        g.head = p.head;
        g.tile = a.first_tile + p.tile_in;
        const int64_t lo = g.tile * 64 > a.dst0 ? g.tile * 64 : a.dst0;
        const int64_t hi = (g.tile + 1) * 64 < a.dst0 + a.n_tokens ? (g.tile + 1) * 64 : a.dst0 + a.n_tokens;
        g.tau_lo = (int)(lo - g.tile * 64);
        g.tau_hi = (int)(hi - g.tile * 64);
        g.src_t0 = lo - a.dst0;
        return g;
    };
    /* element offset of the input row that feeds slot tau_ of the item; a lane without a slot
       to write reads the first row of the range again: its results are never emitted, and
       every address stays inside the input */
    auto source_row = [&](const Geometry &g, int tau_) {
        const bool ok = tau_ >= g.tau_lo && tau_ < g.tau_hi;
        const int64_t t_src = g.src_t0 + (ok ? tau_ - g.tau_lo : 0);
        return t_src * a.ld_token + (int64_t)g.head * a.ld_head;
    };
    /* B operands of a pass: this lane's 8-coordinate slices of its vectors, every k-step
       (coordinates 64 H + 8 ks .. + 7: one contiguous half row per lane); fp32 rows as they are */
    auto load_rows = [&](const Geometry &g, int half0) {
#pragma unroll
        for (int v = 0; v < NVT; ++v) {
            const int64_t row = source_row(g, 32 * (half0 + v) + j);
            if constexpr (XT == PQ_BF16) {
                const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(a.x) + row);
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) xb[v][0][ks].q = xr[8 * H + ks];
            } else {
                const float4 *xr = reinterpret_cast<const float4 *>(static_cast<const float *>(a.x) + row);
#pragma unroll
                for (int k = 0; k < 16; ++k) raw[k] = xr[16 * H + k];
            }
        }
    };
    /* the first pass of a tile that has something to write */
    auto first_half = [&](const Geometry &g) { return NVT == 1 && g.tau_lo >= 32 ? 1 : 0; };
    auto load_item = [&](const Position &p) {
        const Geometry g = geometry(p);
        load_rows(g, first_half(g));
    };
    Position pos{(int)(item0 / a.n_tiles), item0 % a.n_tiles};
    if (kPipelined && item0 < a.n_items) load_item(pos);

    {   /* all of a thread's chunks are requested before the first one is stored: one round trip to L2
           instead of one per chunk */
        constexpr int kChunks = 4 * 8 * 64, kPerThread = kChunks / kThreads, kIn = NTERMS == 1 ? 1 : 3;
        static_assert(kChunks % kThreads == 0, "S chunks must divide evenly over the workgroup");
        uint4 stage[kPerThread][kIn];
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
#pragma unroll
            for (int k = 0; k < kIn; ++k) stage[i][k] = a.S_bf16x3[k * kChunks + threadIdx.x + i * kThreads];
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            BOperand s[NTERMS];
            s_operand<XT, NTERMS>(s, stage[i]);
#pragma unroll
            for (int k = 0; k < NTERMS; ++k) sS[k * kChunks + threadIdx.x + i * kThreads] = s[k].q;
        }
    }
    __syncthreads();

    Thresholds th0 = load_thresholds(*a.consts, NTERMS == 1 ? PQ_INV_SQRT_D : 1.0f);
    if (GENERAL) {
        for (int c = threadIdx.x; c < 512; c += kThreads) sLut[c] = a.consts->lut1[c];
        th0.lut1 = sLut;
        __syncthreads();
    }

    UpperTables ut = {};
    if (DEEP) ut = load_upper_tables(*a.consts);

    uint32_t *img = sImg[wave];

    /* The hardware prefers the older of the two wavefronts of a SIMD, which then finishes well before the other
       and leaves it to run alone; each wavefront lowers its issue priority as it works through its items, so
       that the one behind catches up. */
    const int my_items = item0 < a.n_items ? (int)((a.n_items - item0 + item_stride - 1) / item_stride) : 0;
    int items_done = 0;
    for (int64_t item = item0; item < a.n_items; item += item_stride, pos = advance(pos)) {
        {
            const int q4 = 4 * items_done; /* prio = 3 - floor(4 items_done / my_items) */
            const int prio = 3 - (q4 >= my_items) - (q4 >= 2 * my_items) - (q4 >= 3 * my_items);
            if (prio >= 3) __builtin_amdgcn_s_setprio(3);
            else if (prio == 2) __builtin_amdgcn_s_setprio(2);
            else if (prio == 1) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
            ++items_done;
        }
        const Geometry geo = geometry(pos);
        const int head = geo.head, tau_lo = geo.tau_lo, tau_hi = geo.tau_hi;
        const int64_t tile = geo.tile;
        const bool full = (tau_lo == 0 && tau_hi == 64);
        uint8_t *gcodes = a.codes + ((int64_t)head * a.pool_tiles + tile) * PQL_CODE_BYTES;
        uint16_t *gradii = a.radii + ((int64_t)head * a.pool_tiles + tile) * kRadiiHalves;

        if (!full) { /* ---- image of a partially written tile: its present contents ---- */
            const uint32_t *gc = reinterpret_cast<const uint32_t *>(gcodes);
            const uint32_t *gr = reinterpret_cast<const uint32_t *>(gradii);
            for (int c = lane; c < PQL_CODE_BYTES / 4; c += 64) img[c] = gc[c];
            for (int c = lane; c < kRadiiHalves / 2; c += 64) img[PQL_CODE_BYTES / 4 + c] = gr[c];
            wave_lds_sync();
        }

        for (int vt0 = 0; vt0 < 2; vt0 += NVT) {
            /* wave-uniform skip of a pass with nothing to write */
            if (32 * (vt0 + NVT) <= tau_lo || 32 * vt0 >= tau_hi) continue;

            bool valid[NVT];
            int tau[NVT];
            Thresholds th = th0;
#pragma unroll
            for (int v = 0; v < NVT; ++v) {
                tau[v] = 32 * (vt0 + v) + j;
                valid[v] = tau[v] >= tau_lo && tau[v] < tau_hi;
                /* ---- B operands: this lane's 8-coordinate slices of its vector, every k-step
                   (coordinates 64 H + 8 ks .. + 7: one contiguous half row per lane) ---- */
                if constexpr (XT != PQ_BF16) {
                    uint32_t e = 0;
                    if constexpr (Op::half) {
                        float m = 0.f; /* of the vector: its other half is in the lane 32 further on */
#pragma unroll
                        for (int k = 0; k < 16; ++k) m = max_abs(m, raw[k]);
                        e = half_exponent(fmaxf(m, __uint_as_float(from_other_half(__float_as_uint(m), H))));
                        th.radius_scale = th0.radius_scale * half_unscale<NTERMS>(e);
                    } else {
                        load_rows(geo, vt0);
                    }
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        const float4 p0 = raw[2 * ks], p1 = raw[2 * ks + 1];
                        const float f[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
                        BOperand t[NXT];
                        if constexpr (Op::half) split_half(f, e, t);
                        else split_bf16(f, t);
#pragma unroll
                        for (int k = 0; k < NXT; ++k) xb[v][k][ks] = t[k];
                        if (Op::half) __builtin_amdgcn_sched_barrier(0); /* a k-step after the other: all at once spills */
                    }
                }
            }

            /* D[i][j] = sum_k S[k][col(rt,i)] * x[j][k]: 32 rotated coordinates x 32 vectors per row
               tile rt.  The products of row tile rt+1 are issued between the steps of the polar
               recursion of row tile rt, in a fixed interleaving: each pair of matrix instructions
               is followed by a slice of vector work that does not depend on them, so the matrix
               cores run while the vector ALU quantises.  Stage -1 only multiplies, stage 3 only
               quantises. */
            f32x16 acc_even[NVT], acc_odd[NVT];
            float q4[NVT][4]; /* DEEP: squared radii of blocks 4H .. 4H+3 */
#pragma unroll
            for (int st = -1; st < 4; ++st) {
                f32x16 (&cur)[NVT] = (st & 1) ? acc_odd : acc_even;   /* row tile st: quantised now */
                f32x16 (&nxt)[NVT] = (st & 1) ? acc_even : acc_odd;   /* row tile st+1: accumulated now */
                const bool mul = st < 3, quant = st >= 0;
                if (kPipelined && st == 3) {
                    if (NVT == 1 && vt0 == 0 && tau_hi > 32) load_rows(geo, 1);
                    else if (item + item_stride < a.n_items) load_item(advance(pos));
                }
                PolarState ps[NVT];
                BOperand sa_next;
                if (mul) sa_next.q = sS[(((NTERMS - 1) * 4 + (st + 1)) * 8 + 0) * 64 + lane];
                /* The vector work that goes with k-step ks comes in U units (level-1 pair ks in two parts
                   and the upper-level nodes it completes, per vector); they are spread evenly behind the
                   NM matrix instructions of the k-step. */
                constexpr int NM = NVT * Op::products;
                constexpr int U = 3 * NVT;
                auto unit = [&](int ks, int u) {
                    const int v = NVT == 2 ? (u < 4 ? u >> 1 : u - 4) : 0;
                    const int part = NVT == 2 ? (u < 4 ? (u & 1) : 2) : u;
                    if (part == 0) polar_level1_a<GENERAL>(ps[v], cur[v], ks, th);
                    if (part == 1) polar_level1_b<GENERAL>(ps[v], cur[v], ks);
                    if (part == 2) polar_upper<GENERAL>(ps[v], ks, th);
                };
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    int m = 0;
#pragma unroll
                    for (int term = NTERMS - 1; term >= 0; --term) { /* smallest terms first */
                        if (mul) {
                            /* A operand of this step; the next one is requested from LDS right away */
                            const BOperand sa = sa_next;
                            const int nterm = term > 0 ? term - 1 : NTERMS - 1, nks = term > 0 ? ks : ks + 1;
                            if (nks < 8) sa_next.q = sS[((nterm * 4 + (st + 1)) * 8 + nks) * 64 + lane];
#pragma unroll
                            for (int v = 0; v < NVT; ++v)
#pragma unroll
                                for (int xt = 0; xt < NXT; ++xt) {
                                    if (xt + term > Op::top) continue; /* Operands: what is left out */
                                    /* the first product of a row tile starts from a zero accumulator operand */
                                    const bool first = (ks == 0 && term == NTERMS - 1 && xt == 0);
                                    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                                    nxt[v] = multiply<XT, NTERMS>(sa, xb[v][xt][ks], first ? zero : nxt[v]);
                                    if (quant) {
#pragma unroll
                                        for (int u = m * U / NM; u < (m + 1) * U / NM; ++u) unit(ks, u);
                                        __builtin_amdgcn_sched_barrier(0);
                                    }
                                    ++m;
                                }
                        }
                    }
                    if (!mul) {
#pragma unroll
                        for (int u = 0; u < U; ++u) unit(ks, u);
                    }
                }
                if (quant) {
                    /* lane (H, j): cur[v][r] = rotated coordinate 16*(4H + st) + r of vector tau[v] */
                    const int b = 4 * H + st;
                    if (DEEP) {
#pragma unroll
                        for (int v = 0; v < NVT; ++v) q4[v][st < 0 ? 0 : st] = ps[v].out.q4;
                    }
                    /* a full tile has a slot for every lane: no per-lane branch there.  (Around a
                       single vector's fields it would let the optimiser move that vector's whole
                       recursion behind the branch and undo the interleaving above.) */
                    if (full) {
#pragma unroll
                        for (int v = 0; v < NVT; ++v) leave_block<KIND, DEEP>(img, tau[v], b, ps[v].out);
                    } else {
#pragma unroll
                        for (int v = 0; v < NVT; ++v)
                            if (valid[v]) emit_block<KIND, DEEP>(img, tau[v], b, ps[v].out);
                    }
                }
            }
            if (DEEP) {
#pragma unroll
                for (int v = 0; v < NVT; ++v) {
                    const UpperHalf mine = polar_upper_half(q4[v], H, ut);
                    UpperHalf other;
                    other.codes = from_other_half(mine.codes, H);
                    other.q6 = __uint_as_float(from_other_half(__float_as_uint(mine.q6), H));
                    const uint32_t word = H == 0 ? polar_upper_join(mine, other, th.radius_scale, ut)
                                                 : polar_upper_join(other, mine, th.radius_scale, ut);
                    if (H == 0 && valid[v]) {
                        if (full) reinterpret_cast<uint32_t *>(gradii)[tau[v]] = word;
                        else img[PQL_CODE_BYTES / 4 + tau[v]] = word;
                    }
                }
            }
        }
        wave_lds_sync();

        if (full) {
            store_tile<KIND, DEEP>(img, gcodes, gradii, lane);
        } else { /* ---- image -> global, 16 bytes per lane per store ---- */
            const uint4 *src = reinterpret_cast<const uint4 *>(img);
            uint4 *dc = reinterpret_cast<uint4 *>(gcodes);
            uint4 *dr = reinterpret_cast<uint4 *>(gradii);
            for (int c = lane; c < PQL_CODE_BYTES / 16; c += 64) dc[c] = src[c];
            for (int c = lane; c < kRadiiHalves * 2 / 16; c += 64) dr[c] = src[PQL_CODE_BYTES / 16 + c];
        }
        wave_lds_sync();
    }
}

/* Short inputs: the eight wavefronts of a workgroup share a tile.  The tile's rows are fetched once, eight threads per vector,
 * and left in LDS as matrix operands; wavefront (v, rt) rotates the 32 vectors of half v into row tile rt -- blocks rt and
 * 4 + rt -- with its part of S in registers, straight from memory.  No wavefront does more than an eighth of a tile's
 * chain, and a workgroup's next rows are under way meanwhile.  Bound by the latency of that chain and the launch: 3001 fp32
 * tokens of 8 heads 15.2 -> 10.8 us (13.3 with a wavefront per tile and two binary16 terms), 2000 bf16 tokens, keys and values, 12.0 -> 9.6
 * (then the host's calls).  Issuing the next tile's products between the steps of this one's recursion, as the long kernel
 * does, gave nothing (14.4 against 14.1 us for 3000 fp32 tokens, keys and values). */
__shared__ float sQ4[2][2][4][64]; /* DEEP: squared radii of the tile's blocks */
__shared__ float sUnscale[2][64];

template <int XT, int KIND, int NTERMS, bool GENERAL, bool DEEP>
__device__ __forceinline__ void encode_tiles_together(const EncodeArgs &a, int block, int n_blocks)
{
    typedef Operands<XT, NTERMS> Op;
    constexpr int kImgDwords = TileImage<DEEP>::dwords, kRadiiHalves = TileImage<DEEP>::radii_halves;
    constexpr int kIn = NTERMS == 1 ? 1 : 3, kThreads = 512, NXT = Op::x_terms;
    constexpr int kRows = NXT * 8 * 2 * 64; /* a tile's rows, [term][k-step][half][lane]: two buffers where the long kernels keep S */
    static_assert(2 * kRows <= 3 * 4 * 8 * 64, "the rows of two tiles");
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, H = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), v = wave & 1, rt = wave >> 1;
    struct Place {
        int head, tau_lo, tau_hi; /* slots [tau_lo, tau_hi) of the tile are written */
        int64_t tile, src_t0;     /* tile inside the head plane; source token of slot tau_lo */
    };
    auto place = [&](int64_t item) {
        Place p;
        p.head = (int)(item / a.n_tiles);
        p.tile = a.first_tile + item % a.n_tiles;
        const int64_t lo = max(p.tile * 64, a.dst0), hi = min((p.tile + 1) * 64, a.dst0 + a.n_tokens);
        p.tau_lo = (int)(lo - p.tile * 64);
        p.tau_hi = (int)(hi - p.tile * 64);
        p.src_t0 = lo - a.dst0;
        return p;
    };
    /* this thread's sixteen coordinates 16 part .. + 15 of vector vec; eight vectors on neighbouring lanes, so that their operands
       go to neighbouring places.  A slot that is not written gets the first row of the range, and its results are not emitted. */
    const int vec = 8 * wave + (lane & 7), part = lane >> 3;
    u32x4 raw[XT == PQ_BF16 ? 2 : 4];
    auto load_row = [&](const Place &p) {
        const bool valid = vec >= p.tau_lo && vec < p.tau_hi;
        const int64_t row = (p.src_t0 + (valid ? vec - p.tau_lo : 0)) * a.ld_token + (int64_t)p.head * a.ld_head + 16 * part;
        constexpr int kBytes = XT == PQ_BF16 ? 2 : 4;
        const u32x4 *xr = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.x) + row * kBytes);
#pragma unroll
        for (int k = 0; k < kBytes; ++k) raw[k] = xr[k];
    };
    auto leave_row = [&](int buffer) {
        /* k-steps 2 (part & 3), + 1 of lane half part >> 2 */
        uint4 *dst = sS + buffer * kRows + (4 * (part & 3) + (vec >> 5)) * 64 + 32 * (part >> 2) + (vec & 31);
        if constexpr (XT == PQ_BF16) {
            dst[0] = make_uint4(raw[0].x, raw[0].y, raw[0].z, raw[0].w);
            dst[2 * 64] = make_uint4(raw[1].x, raw[1].y, raw[1].z, raw[1].w);
        } else {
            uint32_t e = 0;
            if constexpr (Op::half) {
                float m = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) m = max_abs(m, __builtin_bit_cast(float4, raw[k]));
#pragma unroll
                for (int d = 8; d < 64; d <<= 1) m = fmaxf(m, __shfl_xor(m, d)); /* the vector's eight parts */
                e = half_exponent(m);
                if (part == 0) sUnscale[buffer][vec] = half_unscale<NTERMS>(e);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float4 p0 = __builtin_bit_cast(float4, raw[2 * k]), p1 = __builtin_bit_cast(float4, raw[2 * k + 1]);
                const float f[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
                BOperand t[NXT];
                if constexpr (Op::half) split_half(f, e, t);
                else split_bf16(f, t);
#pragma unroll
                for (int x = 0; x < NXT; ++x) dst[(8 * x + k) * 2 * 64] = t[x].q;
            }
        }
    };
    if (block >= a.n_items) return;
    Place p = place(block);
    load_row(p);
    BOperand sa[8][NTERMS];
    { /* requested behind the first rows: everything the first tile needs is in flight at once */
        uint4 stage[8][kIn];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
#pragma unroll
            for (int k = 0; k < kIn; ++k) stage[ks][k] = a.S_bf16x3[((k * 4 + rt) * 8 + ks) * 64 + lane];
        leave_row(0);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            if (NTERMS == 2) __builtin_amdgcn_sched_barrier(0); /* one chunk after the other: all at once spills */
            s_operand<XT, NTERMS>(sa[ks], stage[ks]);
        }
    }
    Thresholds th = load_thresholds(*a.consts, NTERMS == 1 ? PQ_INV_SQRT_D : 1.0f);
    const float base_scale = th.radius_scale;
    UpperTables ut = {};
    if (DEEP) ut = load_upper_tables(*a.consts);
    if (GENERAL) {
        sLut[tid] = a.consts->lut1[tid];
        th.lut1 = sLut;
    }
    const int tau = 32 * v + j;
    int64_t next = (int64_t)block + n_blocks;
    Place p_next = p;
    if (next < a.n_items) {
        p_next = place(next);
        load_row(p_next);
    }
    __syncthreads();
    /* buffers are used in turn and a tile has one barrier: what a wavefront writes for the tile after the next is behind the
       next tile's barrier, which nobody reaches before having read this tile's */
    for (int turn = 0, storer = 0;; turn ^= 1, storer = (storer + 1) & 7) {
        const int tau_lo = p.tau_lo, tau_hi = p.tau_hi;
        const bool full = tau_lo == 0 && tau_hi == 64, valid = tau >= tau_lo && tau < tau_hi;
        uint8_t *gcodes = a.codes + ((int64_t)p.head * a.pool_tiles + p.tile) * PQL_CODE_BYTES;
        uint16_t *gradii = a.radii + ((int64_t)p.head * a.pool_tiles + p.tile) * kRadiiHalves;
        uint32_t *img = sImg[turn];
        if (!full) { /* the tile's present contents */
            const uint32_t *gc = reinterpret_cast<const uint32_t *>(gcodes);
            const uint32_t *gr = reinterpret_cast<const uint32_t *>(gradii);
            for (int c = tid; c < PQL_CODE_BYTES / 4; c += kThreads) img[c] = gc[c];
            for (int c = tid; c < kRadiiHalves / 2; c += kThreads) img[PQL_CODE_BYTES / 4 + c] = gr[c];
            __syncthreads();
        }
        if (Op::half) th.radius_scale = base_scale * sUnscale[turn][tau];
        if (32 * v < tau_hi && 32 * v + 32 > tau_lo) {
            f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                BOperand xb[NXT];
#pragma unroll
                for (int x = 0; x < NXT; ++x) xb[x].q = sS[turn * kRows + ((x * 8 + ks) * 2 + v) * 64 + lane];
#pragma unroll
                for (int term = NTERMS - 1; term >= 0; --term)
#pragma unroll
                    for (int x = 0; x < NXT; ++x)
                        if (x + term <= Op::top) acc = multiply<XT, NTERMS>(sa[ks][term], xb[x], acc);
            }
            const BlockCodes bc = polar_quant_block<GENERAL>(acc, th);
            if (full) leave_block<KIND, DEEP>(img, tau, 4 * H + rt, bc);
            else if (valid) emit_block<KIND, DEEP>(img, tau, 4 * H + rt, bc);
            if (DEEP) sQ4[turn][v][rt][lane] = bc.q4;
        }
        const bool more = next < a.n_items;
        const int64_t after = next + n_blocks;
        Place p_after = p_next;
        if (more) {
            leave_row(turn ^ 1);
            if (after < a.n_items) {
                p_after = place(after);
                load_row(p_after);
            }
        }
        __syncthreads();
        if (DEEP && rt == 3) {
            float q4[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) q4[k] = sQ4[turn][v][k][lane];
            const UpperHalf mine = polar_upper_half(q4, H, ut);
            UpperHalf other;
            other.codes = from_other_half(mine.codes, H);
            other.q6 = __uint_as_float(from_other_half(__float_as_uint(mine.q6), H));
            const uint32_t word = H == 0 ? polar_upper_join(mine, other, th.radius_scale, ut)
                                         : polar_upper_join(other, mine, th.radius_scale, ut);
            if (H == 0 && valid) {
                if (full) reinterpret_cast<uint32_t *>(gradii)[tau] = word;
                else img[PQL_CODE_BYTES / 4 + tau] = word;
            }
        }
        if (full) {
            if (wave == storer) store_tile<KIND, DEEP>(img, gcodes, gradii, lane);
        } else {
            if (DEEP) __syncthreads();
            const uint4 *src = reinterpret_cast<const uint4 *>(img);
            for (int c = tid; c < kImgDwords / 4; c += kThreads) {
                if (c < PQL_CODE_BYTES / 16) reinterpret_cast<uint4 *>(gcodes)[c] = src[c];
                else reinterpret_cast<uint4 *>(gradii)[c - PQL_CODE_BYTES / 16] = src[c];
            }
        }
        if (!more) break;
        p = p_next;
        p_next = p_after;
        next = after;
    }
}

template <int XT, int KIND, int NTERMS, bool GENERAL, bool DEEP>
__global__ __launch_bounds__(512) void pq_encode_short_kernel(EncodeArgs a)
{
    encode_tiles_together<XT, KIND, NTERMS, GENERAL, DEEP>(a, (int)blockIdx.x, (int)gridDim.x);
}

/* keys on the even workgroups, values on the odd ones */
template <int XT, int NTERMS, bool GENERAL, bool DEEP>
__global__ __launch_bounds__(512) void pq_encode_short_pair_kernel(EncodeArgs k, EncodeArgs v)
{
    if ((blockIdx.x & 1) == 0) encode_tiles_together<XT, PQ_KEY, NTERMS, GENERAL, DEEP>(k, (int)blockIdx.x >> 1, (int)gridDim.x >> 1);
    else encode_tiles_together<XT, PQ_VALUE, NTERMS, GENERAL, DEEP>(v, (int)blockIdx.x >> 1, (int)gridDim.x >> 1);
}

template <int XT, int KIND, int NTERMS, bool GENERAL, bool DEEP>
__global__ __launch_bounds__(EncodeShape<XT>::waves * 64) void pq_encode_kernel(EncodeArgs a)
{
    encode_tiles<XT, KIND, NTERMS, GENERAL, DEEP>(a, (int)blockIdx.x, (int)gridDim.x);
}

/* Keys and values of the same tokens in one launch: workgroups [0, k_blocks) encode the key tiles, the
   rest the value tiles.  One launch instead of two, S staged once per CU, twice as many tiles per
   wavefront to spread the start-up over. */
template <int XT, int NTERMS, bool GENERAL, bool DEEP>
__global__ __launch_bounds__(EncodeShape<XT>::waves * 64) void pq_encode_pair_kernel(EncodeArgs k, EncodeArgs v, int k_blocks)
{
    if ((int)blockIdx.x < k_blocks) encode_tiles<XT, PQ_KEY, NTERMS, GENERAL, DEEP>(k, (int)blockIdx.x, k_blocks);
    else encode_tiles<XT, PQ_VALUE, NTERMS, GENERAL, DEEP>(v, (int)blockIdx.x - k_blocks, (int)gridDim.x - k_blocks);
}

template <int XT, int KIND>
__global__ __launch_bounds__(512) void pq_append_kernel(AppendArgs a, int n)
{
    append_vectors<XT, 1>(a, KIND, (int)blockIdx.x, n);
}

/* keys and values of the same tokens in one launch: workgroups [0, n) take the key vectors,
   [n, 2n) the value vectors (a decode step appends both; one launch saves a dispatch) */
template <int XT>
__global__ __launch_bounds__(512) void pq_append_pair_kernel(AppendArgs k, AppendArgs v, int n)
{
    if ((int)blockIdx.x < n) append_vectors<XT, 1>(k, PQ_KEY, (int)blockIdx.x, n);
    else append_vectors<XT, 1>(v, PQ_VALUE, (int)blockIdx.x - n, n);
}

/* Tiles per CU up to which the workgroup-per-tile kernel is the faster one (keys and values of 8 heads, us, it against the
   wavefront-per-tile kernel: bf16 4000 tokens 11.8 / 16.1, 12000 25.4 / 29.2, 16000 31.9 / 31.7, 32768 66 / 58; fp32 1000 tokens
   9.7 / 15.4, 3000 14.1 / 19.5, 6000 21.5 / 24.0, 8000 24.6 / 23.7; bf16 10000 at depth 7, where two wavefronts do the upper
   levels of a tile, 30.5 / 28.5).  The other kernel's rounds of 2048 tiles make its times steps. */
template <int XT, bool DEEP> constexpr int short_tiles_per_cu() { return XT == PQ_BF16 && !DEEP ? 12 : 6; }

template <int XT, int KIND, int NTERMS, bool GENERAL, bool DEEP>
pq_status launch_encode(const EncodeArgs &a, hipStream_t stream)
{
    static int cached_cus[PQ_MAX_DEVICES] = {0};
    int dev = 0;
    PQ_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= PQ_MAX_DEVICES) return PQ_EUNSUPPORTED;
    if (cached_cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached_cus[dev] = n;
    }
    const int cus = cached_cus[dev];
    constexpr int kWaves = EncodeShape<XT>::waves, kThreads = kWaves * 64;
    const int64_t blocks = a.n_items < cus ? a.n_items : cus; /* n_items >= 1 */
    pq_prof_before(1, stream);
    if (a.n_items <= short_tiles_per_cu<XT, DEEP>() * (int64_t)cus)
        hipLaunchKernelGGL((pq_encode_short_kernel<XT, KIND, NTERMS, GENERAL, DEEP>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((pq_encode_kernel<XT, KIND, NTERMS, GENERAL, DEEP>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, a);
    pq_prof_after(1, stream);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}

template <int XT, int NTERMS, bool GENERAL, bool DEEP>
pq_status launch_encode_pair(const EncodeArgs &k, const EncodeArgs &v, hipStream_t stream)
{
    int dev = 0, cus = 0;
    PQ_HIP_TRY(hipGetDevice(&dev));
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    constexpr int kWaves = EncodeShape<XT>::waves, kThreads = kWaves * 64;
    /* both streams have the same number of items: half of the CUs each, at least one workgroup */
    int64_t per_kind = k.n_items < cus / 2 ? k.n_items : cus / 2;
    if (per_kind < 1) per_kind = 1;
    pq_prof_before(1, stream);
    if (2 * k.n_items <= short_tiles_per_cu<XT, DEEP>() * (int64_t)cus)
        hipLaunchKernelGGL((pq_encode_short_pair_kernel<XT, NTERMS, GENERAL, DEEP>), dim3((unsigned)(2 * per_kind)), dim3(kThreads), 0,
                           stream, k, v);
    else
        hipLaunchKernelGGL((pq_encode_pair_kernel<XT, NTERMS, GENERAL, DEEP>), dim3((unsigned)(2 * per_kind)), dim3(kThreads), 0,
                           stream, k, v, (int)per_kind);
    pq_prof_after(1, stream);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}

/* bf16 terms of S for bf16 input, binary16 ones for fp32 input where S allows them (see Operands) */
int s_terms(const pq_ctx *ctx, pq_dtype xt) { return ctx->unit_entries ? 1 : (xt == PQ_F32 && ctx->mixing ? 2 : 3); }

/* launch(input type, terms of S, caller-set codebooks, full depth), each an integral_constant */
template <typename F>
pq_status dispatch_variant(const pq_ctx *ctx, pq_dtype xt, F launch)
{
    auto with_depth = [&](auto x, auto terms, auto general) {
        return ctx->depth == 7 ? launch(x, terms, general, std::true_type{}) : launch(x, terms, general, std::false_type{});
    };
    auto with_books = [&](auto x, auto terms) {
        return ctx->general_codebooks ? with_depth(x, terms, std::true_type{}) : with_depth(x, terms, std::false_type{});
    };
    constexpr std::integral_constant<int, PQ_BF16> bf16{};
    constexpr std::integral_constant<int, PQ_F32> f32{};
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 3> three{};
    const int terms = s_terms(ctx, xt);
    if (xt == PQ_BF16) return terms == 1 ? with_books(bf16, one) : with_books(bf16, three);
    return terms == 1 ? with_books(f32, one) : (terms == 2 ? with_books(f32, two) : with_books(f32, three));
}

} // namespace

extern "C" const char *pq_kernel_name_encode(void) { return "pq_encode_kernel"; }

namespace {

/* argument checks and launch geometry shared by pq_encode_kv and pq_encode_kv_pair */
pq_status make_encode_args(const void *x, pq_dtype xt, int64_t n_tokens, int n_heads, int64_t ld_token, int64_t ld_head,
                           uint8_t *codes, uint16_t *radii, int64_t pool_tokens, int64_t dst_token0, EncodeArgs &a)
{
    if (!x || !codes || !radii) return PQ_EINVAL;
    if (n_tokens < 0 || n_heads <= 0 || pool_tokens <= 0 || (pool_tokens & 63) || dst_token0 < 0) return PQ_EINVAL;
    if (n_tokens > pool_tokens || dst_token0 > pool_tokens - n_tokens) return PQ_EINVAL;
    if (ld_token < 0 || ld_head < 0) return PQ_EINVAL;
    const int64_t elems16 = xt == PQ_BF16 ? 8 : 4;
    if (!pq_aligned16(x) || !pq_aligned16(codes) || !pq_aligned16(radii)) return PQ_EALIGN;
    if ((ld_token % elems16) || (ld_head % elems16)) return PQ_EALIGN;
    a = EncodeArgs{};
    a.x = x; a.ld_token = ld_token; a.ld_head = ld_head;
    a.codes = codes; a.radii = radii; a.pool_tiles = pool_tokens / 64; a.pool_tokens = pool_tokens;
    a.dst0 = dst_token0; a.n_tokens = n_tokens;
    a.first_tile = dst_token0 / 64;
    a.n_tiles = (dst_token0 + n_tokens + 63) / 64 - a.first_tile;
    a.n_heads = n_heads;
    a.n_items = a.n_tiles * n_heads;
    return PQ_OK;
}

void set_device_tables(EncodeArgs &a, const PqDeviceState *ds)
{
    a.S_bf16x3 = reinterpret_cast<const uint4 *>(ds->S_bf16x3);
    a.consts = ds->consts;
}

} // namespace

extern "C" pq_status pq_encode_kv(const pq_ctx *ctx, const void *x, pq_dtype xt, pq_kind kind,
                                  int64_t n_tokens, int n_heads, int64_t ld_token, int64_t ld_head,
                                  uint8_t *codes, uint16_t *radii, int64_t pool_tokens,
                                  int64_t dst_token0, void *hip_stream)
{
    if (!ctx) return PQ_EINVAL;
    if (n_tokens == 0) return PQ_OK;
    if (xt != PQ_F32 && xt != PQ_BF16) return PQ_EINVAL;
    if (kind != PQ_KEY && kind != PQ_VALUE) return PQ_EINVAL;
    EncodeArgs a;
    pq_status st = make_encode_args(x, xt, n_tokens, n_heads, ld_token, ld_head, codes, radii, pool_tokens, dst_token0, a);
    if (st != PQ_OK) return st;
    const PqDeviceState *ds = nullptr;
    st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    set_device_tables(a, ds);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    return dispatch_variant(ctx, xt, [&](auto x, auto terms, auto general, auto deep) {
        constexpr int X = decltype(x)::value, T = decltype(terms)::value;
        constexpr bool G = decltype(general)::value, D = decltype(deep)::value;
        return kind == PQ_KEY ? launch_encode<X, PQ_KEY, T, G, D>(a, stream) : launch_encode<X, PQ_VALUE, T, G, D>(a, stream);
    });
}

extern "C" pq_status pq_encode_kv_pair(const pq_ctx *ctx, const void *xk, const void *xv, pq_dtype xt,
                                       int64_t n_tokens, int n_heads, int64_t ld_token, int64_t ld_head,
                                       uint8_t *k_codes, uint16_t *k_radii, uint8_t *v_codes, uint16_t *v_radii,
                                       int64_t pool_tokens, int64_t dst_token0, void *hip_stream)
{
    if (!ctx) return PQ_EINVAL;
    if (n_tokens == 0) return PQ_OK;
    if (xt != PQ_F32 && xt != PQ_BF16) return PQ_EINVAL;
    EncodeArgs ak, av;
    pq_status st = make_encode_args(xk, xt, n_tokens, n_heads, ld_token, ld_head, k_codes, k_radii, pool_tokens, dst_token0, ak);
    if (st != PQ_OK) return st;
    st = make_encode_args(xv, xt, n_tokens, n_heads, ld_token, ld_head, v_codes, v_radii, pool_tokens, dst_token0, av);
    if (st != PQ_OK) return st;
    const PqDeviceState *ds = nullptr;
    st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    set_device_tables(ak, ds);
    set_device_tables(av, ds);
    return dispatch_variant(ctx, xt, [&](auto x, auto terms, auto general, auto deep) {
        return launch_encode_pair<decltype(x)::value, decltype(terms)::value, decltype(general)::value, decltype(deep)::value>(
            ak, av, static_cast<hipStream_t>(hip_stream));
    });
}

extern "C" pq_status pq_append_kv(const pq_ctx *ctx, const void *x, pq_dtype xt, pq_kind kind,
                                  int n_seq, int n_heads, uint8_t *codes, uint16_t *radii,
                                  int64_t pool_tokens, const int64_t *dst_token, void *hip_stream)
{
    if (!ctx) return PQ_EINVAL;
    if (n_seq == 0) return PQ_OK;
    if (!x || !codes || !radii || !dst_token) return PQ_EINVAL;
    if (xt != PQ_F32 && xt != PQ_BF16) return PQ_EINVAL;
    if (kind != PQ_KEY && kind != PQ_VALUE) return PQ_EINVAL;
    if (n_seq < 0 || n_heads <= 0 || pool_tokens <= 0 || (pool_tokens & 63)) return PQ_EINVAL;
    if ((int64_t)n_seq * n_heads > 0x7FFFFFFF) return PQ_EINVAL;
    if (!pq_aligned16(x) || !pq_aligned16(codes) || !pq_aligned16(radii)) return PQ_EALIGN;
    const PqDeviceState *ds = nullptr;
    pq_status st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    AppendArgs a{x, codes, radii, pool_tokens / 64, pool_tokens, dst_token, n_heads, ds->S_f32, ds->consts, ctx->hadamard};
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    dim3 grid((unsigned)(n_seq * n_heads)), block(512);
    if (xt == PQ_BF16) {
        if (kind == PQ_KEY) hipLaunchKernelGGL((pq_append_kernel<PQ_BF16, PQ_KEY>), grid, block, 0, s, a, n_seq * n_heads);
        else hipLaunchKernelGGL((pq_append_kernel<PQ_BF16, PQ_VALUE>), grid, block, 0, s, a, n_seq * n_heads);
    } else {
        if (kind == PQ_KEY) hipLaunchKernelGGL((pq_append_kernel<PQ_F32, PQ_KEY>), grid, block, 0, s, a, n_seq * n_heads);
        else hipLaunchKernelGGL((pq_append_kernel<PQ_F32, PQ_VALUE>), grid, block, 0, s, a, n_seq * n_heads);
    }
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}

extern "C" pq_status pq_append_kv_pair(const pq_ctx *ctx, const void *xk, const void *xv, pq_dtype xt,
                                       int n_seq, int n_heads, uint8_t *k_codes, uint16_t *k_radii,
                                       uint8_t *v_codes, uint16_t *v_radii, int64_t pool_tokens,
                                       const int64_t *dst_token, void *hip_stream)
{
    if (!ctx) return PQ_EINVAL;
    if (n_seq == 0) return PQ_OK;
    if (!xk || !xv || !k_codes || !k_radii || !v_codes || !v_radii || !dst_token) return PQ_EINVAL;
    if (xt != PQ_F32 && xt != PQ_BF16) return PQ_EINVAL;
    if (n_seq < 0 || n_heads <= 0 || pool_tokens <= 0 || (pool_tokens & 63)) return PQ_EINVAL;
    if (2 * (int64_t)n_seq * n_heads > 0x7FFFFFFF) return PQ_EINVAL;
    if (!pq_aligned16(xk) || !pq_aligned16(xv) || !pq_aligned16(k_codes) || !pq_aligned16(k_radii) ||
        !pq_aligned16(v_codes) || !pq_aligned16(v_radii)) return PQ_EALIGN;
    const PqDeviceState *ds = nullptr;
    pq_status st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    AppendArgs ak{xk, k_codes, k_radii, pool_tokens / 64, pool_tokens, dst_token, n_heads, ds->S_f32, ds->consts, ctx->hadamard};
    AppendArgs av{xv, v_codes, v_radii, pool_tokens / 64, pool_tokens, dst_token, n_heads, ds->S_f32, ds->consts, ctx->hadamard};
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int n = n_seq * n_heads;
    dim3 grid((unsigned)(2 * n)), block(512);
    if (xt == PQ_BF16) hipLaunchKernelGGL((pq_append_pair_kernel<PQ_BF16>), grid, block, 0, s, ak, av, n);
    else hipLaunchKernelGGL((pq_append_pair_kernel<PQ_F32>), grid, block, 0, s, ak, av, n);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}
