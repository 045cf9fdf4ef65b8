/*
 * pq_decode.hip -- pq_decode_kv (Algorithm 1, procedure DeQuant) and
 * pq_export_canonical (tile layout -> canonical records: 62 bytes, or 50 at
 * full recursion depth, where the block radii are themselves rebuilt from the
 * vector's radius and the codes of levels 7, 6, 5).
 *
 * DeQuant rebuilds each block top-down from its stored radius: at level l the
 * radius of node j splits into (r cos theta, r sin theta) with theta the
 * centroid selected by the node's code; after level 1 the 16 coordinates of
 * the block are known.  The optional trailing product with S^T is a 128x128
 * mat-vec per vector, on the matrix cores.  Without it, and in the export
 * kernel, the tile is read through the generic field accessors.
 */
#include <type_traits>

#include "pq_common.h"

namespace {

typedef _Float16 dq_h2 __attribute__((ext_vector_type(2)));
typedef _Float16 dq_h4 __attribute__((ext_vector_type(4)));
typedef _Float16 dq_h8 __attribute__((ext_vector_type(8)));
typedef float dq_f2 __attribute__((ext_vector_type(2)));
typedef float dq_f16 __attribute__((ext_vector_type(16)));

constexpr int kDecodeWaves = 16, kDecodeThreads = kDecodeWaves * 64;
constexpr int kTileDwords = (PQL_CODE_BYTES + 2 * PQL_RADII) / 4; /* 992 */

struct DecodeArgs {
    const uint8_t *codes;
    const uint16_t *radii;
    int64_t pool_tiles;
    int64_t token0, n_tokens;
    int64_t first_tile, n_tiles, n_items; /* tiles that the range touches; halves of them over all heads */
    void *out;
    int64_t ld_token, ld_head;
    const PqDeviceConsts *consts;
    const float *S;      /* S[i*128 + j] */
    int paired;          /* both strides even: two neighbouring coordinates of the output can be written at once */
    int deep;            /* recursion depth 7: the radius plane holds one word per token */
};

/* What a lane needs of its token: the indices of blocks 4 H .. 4 H + 3 and their radii (fp32). */
struct TokenHalf {
    uint32_t q[4][4], bi[4];
    float r[4];
    uint32_t top; /* largest stored radius of the token, binary16 bits */
};

/* Between a wavefront's own writes to LDS and its reads: LDS instructions of a wavefront are carried out in order, so the
   compiler's order is all that is asked for, and neither loads nor stores in flight are waited for. */
__device__ __forceinline__ void dq_own_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

/* The lane, as a value that the compiler takes for a new one at each call: what is derived from it is computed where it is
   used and not kept in registers over the whole loop. */
__device__ __forceinline__ int dq_lane()
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

/* A tile to LDS as it is (codes, then the radius plane of `radii_bytes`), by loads that write there and take no registers. */
__device__ __forceinline__ void dq_request_tile(uint32_t *img, const uint8_t *tc, const uint16_t *tr, int radii_bytes, int lane)
{
    typedef const __attribute__((address_space(1))) void *Global;
    typedef __attribute__((address_space(3))) void *Lds;
    __builtin_amdgcn_global_load_lds((Global)(tc + 16 * lane), (Lds)img, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((Global)(tc + 1024 + 16 * lane), (Lds)(img + 256), 16, 0, 0);
    if (lane < (PQL_CODE_BYTES - 2048) / 16) __builtin_amdgcn_global_load_lds((Global)(tc + 2048 + 16 * lane), (Lds)(img + 512), 16, 0, 0);
    if (16 * lane < radii_bytes)
        __builtin_amdgcn_global_load_lds((Global)(reinterpret_cast<const uint8_t *>(tr) + 16 * lane), (Lds)(img + PQL_CODE_BYTES / 4), 16, 0, 0);
}

/* `width` bits at bit BIT of a string of dwords */
template <int BIT, int WIDTH>
__device__ __forceinline__ uint32_t dq_field(const uint32_t *w)
{
    constexpr int d = BIT >> 5, s = BIT & 31;
    if constexpr (s + WIDTH <= 32) return (w[d] >> s) & ((1u << WIDTH) - 1u);
    else return __builtin_amdgcn_alignbit(w[d + 1], w[d], s) & ((1u << WIDTH) - 1u);
}

template <int B>
__device__ __forceinline__ void dq_key_block(TokenHalf &t, const uint32_t *w)
{
    t.q[B][0] = dq_field<PQL_BLOCK_BITS * B, 10>(w);
    t.q[B][1] = dq_field<PQL_BLOCK_BITS * B + 10, 10>(w);
    t.q[B][2] = dq_field<PQL_BLOCK_BITS * B + 20, 10>(w);
    t.q[B][3] = dq_field<PQL_BLOCK_BITS * B + 30, 10>(w);
    t.bi[B] = dq_field<PQL_BLOCK_BITS * B + 40, 6>(w);
}

/* Key tile: the token's 368-bit string and its eight radii straight from memory; blocks 4 H .. are its half
   [184 H, 184 H + 184), brought to bit 0 so that every field sits at a fixed position. */
__device__ __forceinline__ void dq_read_key(TokenHalf &t, const uint8_t *tc, const uint16_t *tr, int tau, int H, bool deep)
{
    const uint4 a = *reinterpret_cast<const uint4 *>(tc + PQL_OFF_P0 + 16 * tau);
    const uint4 b = *reinterpret_cast<const uint4 *>(tc + PQL_OFF_P1 + 16 * tau);
    const uint32_t *p2 = reinterpret_cast<const uint32_t *>(tc + PQL_OFF_P2 + 12 * tau);
    const uint32_t w[12] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, p2[0], p2[1], p2[2],
                            *reinterpret_cast<const uint16_t *>(tc + PQL_OFF_KP3 + 2 * tau)};
    uint32_t s[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] = H ? __builtin_amdgcn_alignbit(w[6 + k > 11 ? 11 : 6 + k], w[5 + k], 24) : w[k];
    dq_key_block<0>(t, s); dq_key_block<1>(t, s); dq_key_block<2>(t, s); dq_key_block<3>(t, s);
    if (!deep) {
        const uint4 r = *reinterpret_cast<const uint4 *>(tr + 8 * tau);
        const uint32_t lo = H ? r.z : r.x, hi = H ? r.w : r.y;
        t.r[0] = pq_half_bits_to_float(lo & 0xFFFFu); t.r[1] = pq_half_bits_to_float(lo >> 16);
        t.r[2] = pq_half_bits_to_float(hi & 0xFFFFu); t.r[3] = pq_half_bits_to_float(hi >> 16);
        const uint32_t h[4] = {r.x, r.y, r.z, r.w};
        t.top = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) t.top = max(t.top, max(h[k] & 0x7FFFu, (h[k] >> 16) & 0x7FFFu));
    }
}

/* Value tile: staged in the wavefront's LDS image (codes, then radii); a token's slots are spread over the strings of
   the 16 half-blocks at one bit position. */
__device__ __forceinline__ void dq_read_value(TokenHalf &t, const uint32_t *img, int tau, int H, bool deep)
{
    const uint32_t g = ((uint32_t)tau >> 2) & 3u, s = 4u * ((uint32_t)tau >> 4) + ((uint32_t)tau & 3u);
    auto base = [](uint32_t d) { return d < 4u ? d : d < 8u ? PQL_OFF_P1 / 4 + d - 4u : PQL_OFF_P2 / 4 + d - 8u; };
    const uint32_t d0 = (PQL_SLOT_BITS * s) >> 5, d1 = min(d0 + 1u, 9u), sh = (PQL_SLOT_BITS * s) & 31u;
    const uint32_t m0 = d0 < 8u ? 4u : 2u, m1 = d1 < 8u ? 4u : 2u, lam = 16u * g + 8u * (uint32_t)H;
    const uint32_t *p0 = img + base(d0) + lam * m0, *p1 = img + base(d1) + lam * m1;
    const uint32_t owner = 8u * g + 4u * (uint32_t)H;
    const uint32_t *pb = img + PQL_OFF_VB / 4 + 3u * owner + ((6u * s) >> 5);
    const uint16_t *pr = reinterpret_cast<const uint16_t *>(img) + PQL_CODE_BYTES / 2 + 16u * owner + s;
    t.top = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t v = __builtin_amdgcn_alignbit(p1[(2 * b + h) * m1], p0[(2 * b + h) * m0], sh);
            t.q[b][2 * h] = v & 1023u;
            t.q[b][2 * h + 1] = (v >> 10) & 1023u;
        }
        /* the dword after a string's last one is the next string's, or the first radii: its bits are masked off */
        t.bi[b] = __builtin_amdgcn_alignbit(pb[3 * b + 1], pb[3 * b], (6u * s) & 31u) & 63u;
        if (!deep) {
            const uint32_t r = pr[16 * b];
            t.r[b] = pq_half_bits_to_float(r);
            t.top = max(t.top, r & 0x7FFFu);
        }
    }
    if (!deep) t.top = max(t.top, (uint32_t)__shfl_xor((int)t.top, 32));
}

__device__ __forceinline__ uint32_t dq_bf16(float f) /* round to nearest even, in the upper half */
{
    const uint32_t u = __float_as_uint(f);
    return u + 0x7FFFu + ((u >> 16) & 1u);
}

/* output coordinates c and c + 1 of one token (`at`: element offset of the first) */
template <int OT>
__device__ __forceinline__ void dq_store_pair(void *out, int64_t at, float a, float b, bool paired)
{
    if (OT == PQ_F32) {
        float *p = static_cast<float *>(out) + at;
        if (paired) *reinterpret_cast<float2 *>(p) = make_float2(a, b);
        else { p[0] = a; p[1] = b; }
    } else {
        uint16_t *p = static_cast<uint16_t *>(out) + at;
        const uint32_t ua = dq_bf16(a), ub = dq_bf16(b);
        if (paired) *reinterpret_cast<uint32_t *>(p) = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
        else { p[0] = (uint16_t)(ua >> 16); p[1] = (uint16_t)(ub >> 16); }
    }
}

/* DeQuant, one wavefront per half tile (32 tokens of one head plane; four wavefronts per SIMD); lane (H, j) rebuilds blocks
 * 4 H .. 4 H + 3 of token j in fp32 from products of centroid cosines and sines (tables in LDS).
 *
 * The trailing S^T runs on the matrix cores: out = y S^T with y and S each as two binary16 terms of 22
 * significant bits (a power of two taken out of every token, so that its largest radius sits at 2^14, and out of S) and
 * the three products above 2^-22.  UNIT: all entries of S are +-1/sqrt(128); +-1 is one exact term and two products.
 * Against 64 bits the result is as exact as the fp32 sums in index order that this replaces (1.5e-7 of the vector's norm,
 * 1.1e-7 for UNIT, against 2.2e-7).
 * v_mfma_f32_32x32x16_f16 multiplies 32 tokens by 32 output coordinates.  Tokens are the rows of the product, so that a
 * store writes whole lines: the columns of a pair of products are the even and the odd coordinates of 64, a lane
 * holds two neighbouring ones and 32 lanes 128 or 256 consecutive bytes of a token.  (With tokens as columns a lane
 * held 16 coordinates of one token and every store touched 64 lines: 52 us for the case below, 106 to fp32.)
 *
 * Bound by the vector and matrix instructions (about 600 and 96 per half tile); the bytes alone would take 18 us of a
 * copy.  262144 vectors to bf16: 242 us with the generic bit reader and fp32 sums on 16 tokens per workgroup -> 33 us
 * for keys, 35 for values; to fp32 243 -> 48 and 51.  Every register counts: with what follows from the lane number kept
 * over the loop, up to 11 spilled registers cost values 39.5 us (fp32 57; Hadamard 34 against 28 now), and requesting the
 * next half tile ahead of the products in registers spills more than it hides (45).  AHEAD: it is requested to LDS, which takes none; it
 * travels under the rebuild and the products of this half tile.  (Values spill one register to bf16 and three with AHEAD, keys
 * one with AHEAD; measured as they are.)  Whole tiles on eight wavefronts of 256 registers (S fetched half as often)
 * spill 100 registers; value slots are read from an image in LDS because a token's 16 slots are spread over 16 strings. */
template <int KIND, int OT, bool UNIT, bool AHEAD>
__global__ __launch_bounds__(kDecodeThreads, 1) void pq_decode_kernel(DecodeArgs a)
{
    constexpr int kChunks = 4 * 8 * 64; /* of eight halves: (64-coordinate group, parity), k-step, lane */
    __shared__ uint4 sS[(UNIT ? 1 : 2) * kChunks];
    __shared__ __attribute__((aligned(16))) float tq[2][64][2], tb[64][4];
    __shared__ float2 tup[24];
    __shared__ __attribute__((aligned(16))) float sUn[kDecodeWaves][32];
    __shared__ __attribute__((aligned(16))) uint32_t img[AHEAD || KIND == PQ_VALUE ? kDecodeWaves : 1][AHEAD || KIND == PQ_VALUE ? kTileDwords : 4];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PqDeviceConsts &K = *a.consts;
    /* consecutive half tiles go to different workgroups: a short range occupies every CU */
    const int64_t stride = (int64_t)kDecodeWaves * gridDim.x;
    const int radii_halves = a.deep ? PQ_DEEP_RADII_HALVES : PQL_RADII;
    auto request = [&](int64_t item, int lane) {
        const int64_t full_tile = item >> 1, head = full_tile / a.n_tiles, tile = a.first_tile + (full_tile - head * a.n_tiles);
        const int64_t at = head * a.pool_tiles + tile;
        dq_request_tile(img[wave], a.codes + at * PQL_CODE_BYTES, a.radii + at * radii_halves, 2 * radii_halves, lane);
    };
    int64_t item = (int64_t)wave * gridDim.x + blockIdx.x;
    /* The wavefront's first tile is under way to LDS while S is staged (without, values to bf16: 12000 tokens of 8 heads 17.6
       instead of 17.2 us, 3000 of 8 9.8 instead of 9.6; 32768 of 8 within the spread, 35.2 and 35.4). */
    bool requested = KIND == PQ_VALUE || AHEAD;
    if (requested && item < a.n_items) request(item, dq_lane());
    {
        /* chunk (grp, par, ks, lane): S[64 grp + 2 (lane & 31) + par][64 (lane >> 5) + 8 ks .. + 7], the k order of the
           tokens' operand below.  A wavefront fetches eight rows of one parity, 128 bytes each: whole lines, and 32 LDS banks
           when they are written (a chunk per lane touched 64 lines per load, each line in four loads: 10.5 us for 24000 values, now
           9.8; 96000 18.4, now 17.6; 262144 within the spread, from 35.3 on and from 34.6 on). */
        float4 s[4]; /* all requested before the first is stored */
        const int lane = tid & 63, kk = lane & 7;
        auto place = [&](int i, int &row, int &k, int &chunk) {
            const int w = 4 * wave + i, rg = w >> 2, cg = w & 3, par = rg & 1, grp = (rg >> 1) & 1, l31 = 8 * (rg >> 2) + (lane >> 3);
            row = 64 * grp + 2 * l31 + par;
            k = 32 * cg + 4 * kk;
            chunk = ((2 * grp + par) * 8 + 4 * (cg & 1) + (kk >> 1)) * 64 + 32 * (cg >> 1) + l31;
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int row, k, chunk;
            place(i, row, k, chunk);
            s[i] = *reinterpret_cast<const float4 *>(a.S + row * PQ_D + k);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int row, k, chunk;
            place(i, row, k, chunk);
            const float f[4] = {s[i].x, s[i].y, s[i].z, s[i].w};
            dq_h4 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = UNIT ? (f[e] < 0.f ? -1.f : 1.f) : f[e] * 32768.f; /* entries are at most 1 */
                hi[e] = (_Float16)v;
                lo[e] = (_Float16)(v - (float)hi[e]);
            }
            uint2 *to = reinterpret_cast<uint2 *>(sS + chunk) + (kk & 1);
            *to = __builtin_bit_cast(uint2, hi);
            if (!UNIT) to[2 * kChunks] = __builtin_bit_cast(uint2, lo);
        }
        static_assert(kDecodeWaves == 16, "sixteen groups of eight rows, four loads each");
    }
    if (tid < 256) {
        (&tq[0][0][0])[tid] = (&K.dq_quarter[0][0][0])[tid];
        (&tb[0][0])[tid] = __uint_as_float(K.attn_tab[PQ_TAB_TBF + tid]);
    }
    if (tid < 48) reinterpret_cast<float *>(tup)[tid] = (&K.up_cs[0][0][0])[tid];
    const int b5 = K.up_bits[0], b6 = K.up_bits[1], b7 = K.up_bits[2];
    __syncthreads();

    for (; item < a.n_items; item += stride) {
        const int lane = dq_lane(), j = lane & 31, H = lane >> 5;
        const int64_t full_tile = item >> 1, head = full_tile / a.n_tiles, tile = a.first_tile + (full_tile - head * a.n_tiles);
        const int half = (int)(item & 1), tau = 32 * half + j;
        const int64_t row0 = tile * 64 + 32 * half - a.token0; /* output row of the half tile's first slot */
        if (!AHEAD && (row0 + 32 <= 0 || row0 >= a.n_tokens)) {
            if (requested) asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); /* nothing writes to LDS behind the wavefront's back */
            requested = false;
            continue;
        }
        TokenHalf t;
        const uint8_t *tc = a.codes + (head * a.pool_tiles + tile) * PQL_CODE_BYTES;
        const uint16_t *tr = a.radii + (head * a.pool_tiles + tile) * radii_halves;
        if constexpr (AHEAD) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); /* the tile is in LDS */
            tc = reinterpret_cast<const uint8_t *>(img[wave]);
            tr = reinterpret_cast<const uint16_t *>(tc + PQL_CODE_BYTES);
        } else if constexpr (KIND == PQ_VALUE) {
            if (!requested) {
                uint4 *im = reinterpret_cast<uint4 *>(img[wave]);
                for (int c = lane; c < PQL_CODE_BYTES / 16; c += 64) im[c] = reinterpret_cast<const uint4 *>(tc)[c];
                if (!a.deep) im[PQL_CODE_BYTES / 16 + lane] = reinterpret_cast<const uint4 *>(tr)[lane];
                dq_own_order();
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); /* a requested tile is in LDS (and the stores of the half tile before are out) */
            requested = false;
        }
        if (KIND == PQ_KEY) dq_read_key(t, tc, tr, tau, H, a.deep != 0);
        else dq_read_value(t, img[wave], tau, H, a.deep != 0);
        if (a.deep) {
            const uint32_t word = reinterpret_cast<const uint32_t *>(tr)[tau];
#pragma unroll
            for (int b = 0; b < 4; ++b) t.r[b] = pq_deep_block_radius(word, b5, b6, b7, tup, 4 * H + b);
            t.top = (word >> 16) & 0x7FFFu;
        }
        if constexpr (AHEAD) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); /* and has been read: the next one may follow */
            if (item + stride < a.n_items) request(item + stride, lane);
            if (row0 + 32 <= 0 || row0 >= a.n_tokens) continue;
        }
        /* the token's largest radius goes to [2^14, 2^15) */
        const uint32_t exponent = max(t.top >> 10, 1u);
        const float scale = __uint_as_float((127u + 29u - exponent) << 23);
        if (H == 0)
            sUn[wave][j] = UNIT ? __uint_as_float((127u - 29u + exponent) << 23) * PQ_INV_SQRT_D : __uint_as_float((127u - 44u + exponent) << 23);
        dq_h8 yh[8], yl[8]; /* k-step ks: coordinates 64 H + 8 ks .. + 7 */
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const float4 f = *reinterpret_cast<const float4 *>(tb[t.bi[b]]);
            const float rs = t.r[b] * scale;
            const float rq[4] = {rs * f.x, rs * f.y, rs * f.z, rs * f.w};
            float y[16];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float2 pa = *reinterpret_cast<const float2 *>(tq[0][t.q[b][k] & 63u]);
                const float2 pb = *reinterpret_cast<const float2 *>(tq[1][t.q[b][k] >> 4]);
                y[4 * k] = rq[k] * pa.x; y[4 * k + 1] = rq[k] * pa.y;
                y[4 * k + 2] = rq[k] * pb.x; y[4 * k + 3] = rq[k] * pb.y;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                /* the two terms must come from one and the same rounded product (the compiler would otherwise
                   round the exact product to binary16 for the one and the fp32 product for the other) */
                asm("" : "+v"(y[e]));
                const _Float16 hi = (_Float16)y[e];
                yh[2 * b + (e >> 3)][e & 7] = hi;
                yl[2 * b + (e >> 3)][e & 7] = (_Float16)(y[e] - (float)hi);
            }
            __builtin_amdgcn_sched_barrier(0); /* gathers of all four blocks at once would not fit the registers */
        }
        dq_own_order(); /* the image is read before the next one replaces it; the scales are written */
        {
            const bool whole = a.paired && row0 >= 0 && row0 + 32 <= a.n_tokens; /* every store of the half tile is a pair */
            /* element offset of this lane's first token, column pair 0; the rows of a register differ by scalar multiples */
            __builtin_amdgcn_sched_barrier(0);
            const int lane = dq_lane(), j = lane & 31, H = lane >> 5;
            const int64_t row_h = row0 + 4 * H;
            int64_t at0 = row_h * a.ld_token + head * a.ld_head + 2 * j;
#pragma unroll 1
            for (int grp = 0; grp < 2; ++grp, at0 += 64) {
                asm volatile("" : "+v"(at0)); /* 16 row addresses kept over both groups would spill */
                dq_f16 acc[2]; /* even and odd coordinates of the group */
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[p][e] = 0.f;
                const uint4 *sg = sS + 2 * grp * 8 * 64 + lane;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const dq_h8 s_hi = __builtin_bit_cast(dq_h8, sg[(p * 8 + ks) * 64]);
                        if (!UNIT) {
                            const dq_h8 s_lo = __builtin_bit_cast(dq_h8, sg[(UNIT ? 0 : kChunks) + (p * 8 + ks) * 64]);
                            acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(yh[ks], s_lo, acc[p], 0, 0, 0);
                        }
                        acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(yl[ks], s_hi, acc[p], 0, 0, 0);
                        acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(yh[ks], s_hi, acc[p], 0, 0, 0);
                    }
                /* register r of lane (H, j): token 8 (r >> 2) + 4 H + (r & 3) of the half, coordinates 64 grp + 2 j, + 1 */
                auto store = [&](auto whole_c) {
                    constexpr bool WHOLE = decltype(whole_c)::value;
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const float4 un4 = *reinterpret_cast<const float4 *>(&sUn[wave][8 * r4 + 4 * H]);
                        const float un[4] = {un4.x, un4.y, un4.z, un4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int64_t row = row_h + 8 * r4 + e;
                            if (WHOLE || (row >= 0 && row < a.n_tokens))
                                dq_store_pair<OT>(a.out, at0 + (8 * r4 + e) * a.ld_token, acc[0][4 * r4 + e] * un[e],
                                                  acc[1][4 * r4 + e] * un[e], WHOLE || a.paired != 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                if (whole) store(std::true_type{});
                else store(std::false_type{});
            }
            dq_own_order(); /* the scales are read before the next ones replace them */
        }
    }
}

/* DeQuant without the trailing S^T: sixteen tokens per workgroup, a thread per (token, block) rebuilds its sixteen
 * coordinates, and every row is then written by the 128 threads as whole lines; any strides.  Bound by the generic reader's
 * loads and the stores: 262144 vectors to bf16 36 us for keys, 38 for values, to fp32 62 and 64.  (Stored by the kernel above
 * from the lanes that rebuild them, a pair of coordinates and a line of its own per lane, they took 78 to 82 and 171 to 175.) */
constexpr int kRotatedTokens = 16;

template <int KIND, int OT>
__global__ __launch_bounds__(128) void pq_decode_rotated_kernel(DecodeArgs a)
{
    __shared__ float sy[kRotatedTokens][PQ_D];
    const int head = blockIdx.y, tid = threadIdx.x;
    const int64_t t_base = (int64_t)blockIdx.x * kRotatedTokens;
    const PqDeviceConsts &K = *a.consts;
    const int64_t t = t_base + (tid >> 3);
    if (t < a.n_tokens) {
        const int b = tid & 7, tau = (int)((a.token0 + t) & 63);
        const int64_t tile = head * a.pool_tiles + ((a.token0 + t) >> 6);
        const uint8_t *tc = a.codes + tile * PQL_CODE_BYTES;
        const uint16_t *tr = a.radii + tile * (a.deep ? PQ_DEEP_RADII_HALVES : PQL_RADII);
        const PqBlockFields f = pql_read_block(KIND, tc, a.deep ? nullptr : tr, tau, b);
        float r4;
        if (a.deep)
            r4 = pq_deep_block_radius(reinterpret_cast<const uint32_t *>(tr)[tau], K.up_bits[0], K.up_bits[1], K.up_bits[2],
                                      reinterpret_cast<const float2 *>(&K.up_cs[0][0][0]), b);
        else
            r4 = (float)__builtin_bit_cast(_Float16, f.radius);
        const float r3[2] = {r4 * K.cs234[2][f.c4][0], r4 * K.cs234[2][f.c4][1]};
        float *y = &sy[tid >> 3][16 * b];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t g6 = f.g6[h], c2a = g6 >> 4, c3 = (g6 >> 2) & 3, c2b = g6 & 3;
            const float r2a = r3[h] * K.cs234[1][c3][0], r2b = r3[h] * K.cs234[1][c3][1];
            const float r1[4] = {r2a * K.cs234[0][c2a][0], r2a * K.cs234[0][c2a][1], r2b * K.cs234[0][c2b][0], r2b * K.cs234[0][c2b][1]};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t c1 = (f.l1 >> (4 * (4 * h + q))) & 15;
                y[8 * h + 2 * q] = r1[q] * K.cs1[c1][0];
                y[8 * h + 2 * q + 1] = r1[q] * K.cs1[c1][1];
            }
        }
    }
    __syncthreads();
    const int n = (int)min((int64_t)kRotatedTokens, a.n_tokens - t_base);
#pragma unroll
    for (int k = 0; k < kRotatedTokens; ++k) {
        if (k >= n) break;
        const int64_t at = (t_base + k) * a.ld_token + head * a.ld_head + tid;
        if (OT == PQ_F32) static_cast<float *>(a.out)[at] = sy[k][tid];
        else static_cast<uint16_t *>(a.out)[at] = (uint16_t)(dq_bf16(sy[k][tid]) >> 16);
    }
}

template <int KIND, int OT>
void launch_decode(const DecodeArgs &a, bool unit, int rotated, int n_heads, hipStream_t s)
{
    if (rotated) {
        const dim3 grid((unsigned)((a.n_tokens + kRotatedTokens - 1) / kRotatedTokens), (unsigned)n_heads);
        hipLaunchKernelGGL((pq_decode_rotated_kernel<KIND, OT>), grid, dim3(128), 0, s, a);
        return;
    }
    const dim3 grid((unsigned)(a.n_items < 256 ? a.n_items : 256)); /* one workgroup per CU */
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kDecodeThreads), 0, s, a); };
    /* The next tile ahead of this one's rebuild: for fp32 output, once a wavefront has more than one (32768 tokens of 8 heads, us with
       and without: values 44.8 / 50.3, keys with a +-1 S 38.0 / 44.5; to bf16 36.4 / 35.2, whose stores leave less to wait for than the
       LDS pass costs; 3001 fp32 keys 11.1 / 10.6). */
    const bool ahead = OT == PQ_F32 && a.n_items > 256 * kDecodeWaves;
    if constexpr (OT == PQ_F32)
        if (ahead) return unit ? launch(pq_decode_kernel<KIND, OT, true, true>) : launch(pq_decode_kernel<KIND, OT, false, true>);
    if (unit) launch(pq_decode_kernel<KIND, OT, true, false>);
    else launch(pq_decode_kernel<KIND, OT, false, false>);
}

struct ExportArgs {
    const uint8_t *codes;
    const uint16_t *radii;
    int64_t pool_tiles;
    int64_t token0, n_tokens;
    uint8_t *rec;
    int deep;
};

/* one thread per (token, block): writes the block's share of the canonical record */
template <int KIND>
__global__ __launch_bounds__(256) void pq_export_kernel(ExportArgs a)
{
    const int head = blockIdx.y;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t t = idx >> 3;
    const int b = (int)(idx & 7);
    if (t >= a.n_tokens) return;
    const int64_t slot = a.token0 + t;
    const int64_t tile = slot >> 6;
    const int tau = (int)(slot & 63);
    const uint8_t *tc = a.codes + ((int64_t)head * a.pool_tiles + tile) * PQL_CODE_BYTES;
    const uint16_t *tr = a.radii + ((int64_t)head * a.pool_tiles + tile) * (a.deep ? PQ_DEEP_RADII_HALVES : PQL_RADII);
    PqBlockFields f = pql_read_block(KIND, tc, a.deep ? nullptr : tr, tau, b);
    uint8_t *rec = a.rec + ((int64_t)head * a.n_tokens + t) * (a.deep ? PQ_DEEP_RECORD_BYTES : PQ_RECORD_BYTES);
    /* level 1: pairs 8b..8b+7 -> bytes 4b..4b+3, earlier code in the high nibble */
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t c_even = (f.l1 >> (8 * k)) & 15, c_odd = (f.l1 >> (8 * k + 4)) & 15;
        rec[4 * b + k] = (uint8_t)((c_even << 4) | c_odd);
    }
    /* level 2: nodes 4b..4b+3 -> byte 32 + b, earlier code in the higher bits */
    uint32_t c2_0 = f.g6[0] >> 4, c2_1 = f.g6[0] & 3, c2_2 = f.g6[1] >> 4, c2_3 = f.g6[1] & 3;
    rec[32 + b] = (uint8_t)((c2_0 << 6) | (c2_1 << 4) | (c2_2 << 2) | c2_3);
    uint32_t c3_0 = (f.g6[0] >> 2) & 3, c3_1 = (f.g6[1] >> 2) & 3;
    /* level 3 (2 codes) and level 4 (1 code) share bytes with the neighbouring
       blocks: gather them across the 8 lanes that hold one token's blocks */
    uint32_t nib3 = (c3_0 << 2) | c3_1; /* 4 bits of byte 40 + b/2 */
    uint32_t other3 = __shfl_xor(nib3, 1);
    if ((b & 1) == 0) rec[40 + (b >> 1)] = (uint8_t)((nib3 << 4) | other3);
    uint32_t acc4 = f.c4 << (6 - 2 * (b & 3)); /* 2 bits of byte 44 + b/4 */
    acc4 |= __shfl_xor(acc4, 1);
    acc4 |= __shfl_xor(acc4, 2);
    if ((b & 3) == 0) rec[44 + (b >> 2)] = (uint8_t)acc4;
    if (a.deep) {
        if (b == 0) { /* code word of levels 5..7, then the vector's radius, both little endian */
            const uint32_t word = reinterpret_cast<const uint32_t *>(tr)[tau];
            rec[46] = (uint8_t)(word & 0xFF);
            rec[47] = (uint8_t)((word >> 8) & 0xFF);
            rec[48] = (uint8_t)((word >> 16) & 0xFF);
            rec[49] = (uint8_t)(word >> 24);
        }
    } else {
        rec[46 + 2 * b] = (uint8_t)(f.radius & 0xFF);
        rec[47 + 2 * b] = (uint8_t)(f.radius >> 8);
    }
}

} // namespace

extern "C" pq_status pq_decode_kv(const pq_ctx *ctx, pq_kind kind, const uint8_t *codes, const uint16_t *radii,
                                  int64_t pool_tokens, int64_t token0, int64_t n_tokens, int n_heads,
                                  void *out, pq_dtype ot, int64_t ld_token, int64_t ld_head,
                                  int rotated, void *hip_stream)
{
    if (!ctx || !codes || !radii || !out) return PQ_EINVAL;
    if (kind != PQ_KEY && kind != PQ_VALUE) return PQ_EINVAL;
    if (ot != PQ_F32 && ot != PQ_BF16) return PQ_EINVAL;
    if (n_tokens < 0 || n_heads <= 0 || n_heads > 65535 || pool_tokens <= 0 || (pool_tokens & 63) || token0 < 0) return PQ_EINVAL;
    if (n_tokens > pool_tokens || token0 > pool_tokens - n_tokens || ld_token < 0 || ld_head < 0) return PQ_EINVAL;
    if (!pq_aligned16(codes) || !pq_aligned16(radii) || !pq_aligned16(out)) return PQ_EALIGN;
    if (n_tokens == 0) return PQ_OK;
    const PqDeviceState *ds = nullptr;
    pq_status st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    DecodeArgs a{};
    a.codes = codes; a.radii = radii; a.pool_tiles = pool_tokens / 64;
    a.token0 = token0; a.n_tokens = n_tokens;
    a.first_tile = token0 / 64;
    a.n_tiles = (token0 + n_tokens + 63) / 64 - a.first_tile;
    a.n_items = 2 * a.n_tiles * n_heads;
    a.out = out; a.ld_token = ld_token; a.ld_head = ld_head;
    a.consts = ds->consts; a.S = ds->S_f32;
    a.paired = ld_token % 2 == 0 && ld_head % 2 == 0; /* out itself is 16-byte aligned */
    a.deep = ctx->depth == 7 ? 1 : 0;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (kind == PQ_KEY) {
        if (ot == PQ_F32) launch_decode<PQ_KEY, PQ_F32>(a, ctx->unit_entries, rotated, n_heads, s);
        else launch_decode<PQ_KEY, PQ_BF16>(a, ctx->unit_entries, rotated, n_heads, s);
    } else {
        if (ot == PQ_F32) launch_decode<PQ_VALUE, PQ_F32>(a, ctx->unit_entries, rotated, n_heads, s);
        else launch_decode<PQ_VALUE, PQ_BF16>(a, ctx->unit_entries, rotated, n_heads, s);
    }
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}

extern "C" pq_status pq_export_canonical(const pq_ctx *ctx, pq_kind kind, const uint8_t *codes,
                                         const uint16_t *radii, int64_t pool_tokens, int64_t token0,
                                         int64_t n_tokens, int n_heads, uint8_t *rec, void *hip_stream)
{
    if (!ctx || !codes || !radii || !rec) return PQ_EINVAL;
    if (kind != PQ_KEY && kind != PQ_VALUE) return PQ_EINVAL;
    if (n_tokens < 0 || n_heads <= 0 || n_heads > 65535 || pool_tokens <= 0 || (pool_tokens & 63) || token0 < 0) return PQ_EINVAL;
    if (n_tokens > pool_tokens || token0 > pool_tokens - n_tokens) return PQ_EINVAL;
    if (!pq_aligned16(codes) || !pq_aligned16(radii)) return PQ_EALIGN;
    if (n_tokens == 0) return PQ_OK;
    ExportArgs a{codes, radii, pool_tokens / 64, token0, n_tokens, rec, ctx->depth == 7 ? 1 : 0};
    dim3 grid((unsigned)((n_tokens * 8 + 255) / 256), (unsigned)n_heads), block(256);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (kind == PQ_KEY) hipLaunchKernelGGL((pq_export_kernel<PQ_KEY>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((pq_export_kernel<PQ_VALUE>), grid, block, 0, s, a);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}
