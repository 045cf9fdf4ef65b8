/*
 * pq_general.hip -- the general PolarQuant format: any recursion depth from 4 to 7
 * and other bit widths than Section 4.1's (Definition 1 recurses to log2 d; the
 * remark after Theorem 1 leaves the codebook size of each level free).
 *
 * This is the plain path next to the tuned one: records are kept one after
 * another in the canonical general layout (all codes of level 1, then level 2,
 * ..., in one little-endian bit stream padded to a byte, then the 128 >> depth
 * binary16 radii), every field goes through a generic bit reader, and the
 * kernels are fp32 code:
 *   encode     y = x S (fp32 matrix instructions, sums in index order), procedure Polar
 *              level by level between lanes, procedure Quant as a count of the cell
 *              boundaries (midpoints of neighbouring centroids) below the angle
 *   decode     procedure DeQuant: centroid cos/sin products from the top level
 *              down, then the trailing S^T; one wavefront per vector
 *   attention  Eq. 5 in the rotated domain: q' = q S once, every cached token
 *              dequantised without its S^T, one token per lane, softmax
 *              weights, one S^T at the end; one workgroup per row, or, with a
 *              workspace, several per sequence
 * Section 4.1's own configuration (depth 4, bits 4/2/2/2) and its depth-7
 * extension have the tuned kernels of pq_encode.hip / pq_attn.hip; this file
 * accepts them too (same numbers, other layout), which is how it is tested
 * against them.
 */
#include <atomic>
#include <chrono>
#include <type_traits>

#include "pq_common.h"

#include <cmath>
#include <cstring>

namespace {

constexpr int kGenMaxCells = 16, kGenUpperCells = 8; /* of level 1, of the levels above */
constexpr int kGenMaxRecord = 96; /* bytes: depth 4 with bits 4/3/3/3 needs 53 + 16 */

/* Kernel arguments are copied for every launch: a kernel gets the format and, of the codebooks, the boundaries or the centroids'
   cosines and sines, whichever it looks at (1.3 KB with both: the attention call took the host 13.1 us, now 11.9, an encode 7.2, now 6.6). */
struct GenFormat {
    int depth;
    int bits[7];
    int bit_off[7];    /* first bit of level l in the record's bit stream */
    int code_bytes, rec_bytes, n_radii;
    int rec_dwords, rec_inv; /* dwords of a record (the last may be partial); 65536 / rec_dwords, rounded up */
};

struct GenBounds { /* inner cell boundaries, +inf beyond the level's last one */
    float first[kGenMaxCells - 1], upper[6][kGenUpperCells - 1];
};

struct GenCentroids { /* (cos, sin): 16 of level 1, then eight each of the levels above */
    float2 cs[kGenMaxCells + 6 * kGenUpperCells];
};

bool general_format_ok(const pq_general_format *f)
{
    if (!f || f->depth < 4 || f->depth > 7) return false;
    if (f->bits[0] != 3 && f->bits[0] != 4) return false;
    for (int l = 1; l < 4; ++l)
        if (f->bits[l] != 2 && f->bits[l] != 3) return false;
    for (int l = 4; l < f->depth; ++l)
        if (f->bits[l] < 1 || f->bits[l] > 3) return false;
    return true;
}

int general_code_bits(const pq_general_format *f)
{
    int n = 0;
    for (int l = 0; l < f->depth; ++l) n += (PQ_D >> (l + 1)) * f->bits[l];
    return n;
}

pq_status make_format(const pq_general_format *f, const double *cbg, GenFormat *g)
{
    if (!general_format_ok(f) || !cbg) return PQ_EINVAL;
    memset(g, 0, sizeof(*g));
    g->depth = f->depth;
    int cboff = 0;
    const double half_pi = 1.57079632679489661923, two_pi = 6.28318530717958647692;
    for (int l = 0; l < f->depth; ++l) {
        const int K = 1 << f->bits[l];
        g->bits[l] = f->bits[l];
        g->bit_off[l] = l == 0 ? 0 : g->bit_off[l - 1] + (PQ_D >> l) * f->bits[l - 1];
        for (int k = 0; k < K; ++k) {
            const double c = cbg[cboff + k];
            if (!std::isfinite(c) || c < 0.0 || c > (l == 0 ? two_pi : half_pi)) return PQ_EINVAL;
            if (k > 0 && !(c > cbg[cboff + k - 1])) return PQ_EINVAL;
        }
        cboff += K;
    }
    g->code_bytes = (general_code_bits(f) + 7) / 8;
    g->n_radii = PQ_D >> f->depth;
    g->rec_bytes = g->code_bytes + 2 * g->n_radii;
    g->rec_dwords = (g->rec_bytes + 3) / 4;
    g->rec_inv = (65536 + g->rec_dwords - 1) / g->rec_dwords;
    return PQ_OK;
}

/* of a format and codebooks that make_format has accepted */
GenBounds make_bounds(const GenFormat &g, const double *cbg)
{
    GenBounds b;
    for (int l = 0; l < 7; ++l) {
        const int K = l < g.depth ? 1 << g.bits[l] : 1, most = l == 0 ? kGenMaxCells : kGenUpperCells;
        float *to = l == 0 ? b.first : b.upper[l - 1];
        for (int k = 1; k < most; ++k) to[k - 1] = k < K ? (float)(0.5 * (cbg[k] + cbg[k - 1])) : INFINITY;
        if (l < g.depth) cbg += K;
    }
    return b;
}

GenCentroids make_centroids(const GenFormat &g, const double *cbg)
{
    GenCentroids c{};
    for (int l = 0; l < g.depth; ++l) {
        float2 *to = l == 0 ? c.cs : c.cs + kGenMaxCells + (l - 1) * kGenUpperCells;
        for (int k = 0; k < 1 << g.bits[l]; ++k, ++cbg) to[k] = make_float2((float)cos(*cbg), (float)sin(*cbg));
    }
    return c;
}

__device__ __forceinline__ uint32_t gen_get_bits(const uint8_t *stream, int pos, int width)
{
    uint32_t v = stream[pos >> 3] | ((uint32_t)stream[(pos >> 3) + 1] << 8); /* width <= 4: two bytes suffice */
    return (v >> (pos & 7)) & ((1u << width) - 1u);
}

__device__ __forceinline__ uint16_t gen_radius_bits(float r)
{
    return __builtin_bit_cast(uint16_t, (_Float16)fminf(r, 65504.f)); /* saturates at the largest finite binary16 */
}

/* ---- encode: sixteen vectors per workgroup of 512 threads ----
 * Wavefront w forms columns 16 w .. 16 w + 15 of the sixteen products on v_mfma_f32_16x16x4_f32 (fp32 products and sums, y_c =
 * sum_i x_i S[i][c], i ascending); S comes straight from memory, each element once per workgroup.  Then thread (vector, quarter)
 * takes four coordinates through levels 1 and 2, and the levels above join neighbouring lanes: a level's inputs never leave
 * the wavefront.  The codes are OR-ed into an image of the sixteen records, which lie one after another.
 * Bound by the launch and the chain of loads and levels up to some 4096 vectors, by vector instructions (the arctangents)
 * beyond.  bf16, depth 5: 4096 vectors 10.1 -> 7.2 us, 65536 62 -> 50 (products on the vector ALU with the vectors broadcast from LDS,
 * 1024 reads of sixteen bytes per workgroup, and a barrier per level -> this).  Same sums in the same order: the records are the
 * same, bit for bit, infinities, subnormal vectors and NaN included. */
constexpr int kGenEncVecs = 16, kGenEncThreads = 512;
constexpr int kGenRow = PQ_D + 4; /* floats from vector to vector in LDS: lanes of neighbouring vectors read neighbouring banks */

typedef float gen_f4 __attribute__((ext_vector_type(4)));

/* number of the first N boundaries below the angle: nearest centroid, ties to the lower cell (boundaries that a level does not
   have are +inf; reading them all at once is a third of the time of a loop over those it has) */
template <int N>
__device__ __forceinline__ uint32_t gen_cell(const float (&bound)[N], float ang)
{
    uint32_t code = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) code += ang > bound[k] ? 1u : 0u;
    return code;
}

__device__ __forceinline__ void gen_emit(uint32_t *image, int pos, uint32_t v, int width)
{
    atomicOr(&image[pos >> 5], v << (pos & 31));
    if ((pos & 31) + width > 32) atomicOr(&image[(pos >> 5) + 1], v >> (32 - (pos & 31)));
}

template <int XT>
__global__ __launch_bounds__(kGenEncThreads) void pq_general_encode_kernel(GenFormat f, GenBounds bounds, const void *x, int64_t ld_vector, int64_t n,
                                                                           const float *S, uint8_t *rec)
{
    __shared__ __attribute__((aligned(16))) float buf[kGenEncVecs][kGenRow], sy[kGenEncVecs][kGenRow];
    __shared__ uint32_t srec[kGenEncVecs * kGenMaxRecord / 4 + 1];
    const int64_t v0 = (int64_t)blockIdx.x * kGenEncVecs;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nv = (int)(n - v0 < kGenEncVecs ? n - v0 : kGenEncVecs);
    float val[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = 4 * i + (tid >> 7), c = tid & 127;
        val[i] = 0.f; /* vectors beyond the last one: computed along, not written */
        if (v < nv) {
            const int64_t at = (v0 + v) * ld_vector + c;
            val[i] = XT == PQ_BF16 ? __uint_as_float((uint32_t)static_cast<const uint16_t *>(x)[at] << 16)
                                   : static_cast<const float *>(x)[at];
        }
    }
    float s[PQ_D / 4]; /* all of the lane's elements of S in flight */
#pragma unroll
    for (int k = 0; k < PQ_D / 4; ++k) s[k] = S[(4 * k + (lane >> 4)) * PQ_D + 16 * wave + (lane & 15)];
#pragma unroll
    for (int i = 0; i < 4; ++i) buf[4 * i + (tid >> 7)][tid & 127] = val[i];
    for (int c = tid; c < kGenEncVecs * kGenMaxRecord / 4 + 1; c += kGenEncThreads) srec[c] = 0u;
    __syncthreads();
    {
        gen_f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < PQ_D / 4; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(buf[lane & 15][4 * k + (lane >> 4)], s[k], acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) sy[4 * (lane >> 4) + i][16 * wave + (lane & 15)] = acc[i];
    }
    __syncthreads();
    {
        const int v = tid >> 5, q = tid & 31, base = 8 * f.rec_bytes * v;
        const float4 y = *reinterpret_cast<const float4 *>(&sy[v][4 * q]);
        auto angle1 = [](float a, float b) {
            const float ang = atan2f(b, a);
            return ang < 0.f ? ang + 6.28318530717958647692f : ang;
        };
        /* level 1: two angles, next to each other in the stream */
        const uint32_t c0 = gen_cell(bounds.first, angle1(y.x, y.y));
        const uint32_t c1 = gen_cell(bounds.first, angle1(y.z, y.w));
        gen_emit(srec, base + 2 * q * f.bits[0], c0 | c1 << f.bits[0], 2 * f.bits[0]);
        float a = sqrtf(y.x * y.x + y.y * y.y), b = sqrtf(y.z * y.z + y.w * y.w);
        gen_emit(srec, base + f.bit_off[1] + q * f.bits[1], gen_cell(bounds.upper[0], atan2f(b, a)), f.bits[1]);
        float r = sqrtf(a * a + b * b);
#pragma unroll
        for (int l = 2; l < 7; ++l) { /* the 2^(l-1) lanes of a node all know its radius, the first of them has the code to write */
            if (l < f.depth) {
                const float other = __shfl_xor(r, 1 << (l - 2));
                const bool up = (q >> (l - 2)) & 1;
                a = up ? other : r;
                b = up ? r : other;
                const uint32_t code = gen_cell(bounds.upper[l - 1], atan2f(b, a));
                if ((q & ((1 << (l - 1)) - 1)) == 0) gen_emit(srec, base + f.bit_off[l] + (q >> (l - 1)) * f.bits[l], code, f.bits[l]);
                r = sqrtf(a * a + b * b);
            }
        }
        const int per = f.depth - 2; /* 2^per quarters to a radius */
        if ((q & ((1 << per) - 1)) == 0) gen_emit(srec, base + 8 * f.code_bytes + 16 * (q >> per), gen_radius_bits(r), 16);
    }
    __syncthreads();
    const uint8_t *img = reinterpret_cast<const uint8_t *>(srec);
    uint8_t *out = rec + v0 * f.rec_bytes;
    const int n_bytes = nv * f.rec_bytes;
    int done = 0;
    if ((reinterpret_cast<uintptr_t>(out) & 3) == 0) { /* sixteen records are a whole number of dwords */
        for (int c = tid; c < n_bytes / 4; c += kGenEncThreads) reinterpret_cast<uint32_t *>(out)[c] = srec[c];
        done = n_bytes & ~3;
    }
    for (int c = done + tid; c < n_bytes; c += kGenEncThreads) out[c] = img[c];
}

/* orders the LDS accesses of the lanes of one wavefront (the buffers below belong to a single wavefront) */
__device__ __forceinline__ void gen_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

/* DeQuant's loops for one record by one wavefront (lane = 0..63): r^(0) (rotated domain) into
   buf[returned index][0..127]; buf is the wavefront's own */
__device__ __forceinline__ int gen_dequant_rotated(const GenFormat &f, const GenCentroids &centroids, const uint8_t *rec, float (&buf)[2][PQ_D], int lane)
{
    int cur = 0;
    if (lane < f.n_radii) {
        const uint16_t h = (uint16_t)(rec[f.code_bytes + 2 * lane] | (rec[f.code_bytes + 2 * lane + 1] << 8));
        buf[0][lane] = (float)__builtin_bit_cast(_Float16, h);
    }
    gen_wave_sync();
    for (int l = f.depth - 1; l >= 0; --l) {
        const int n_ang = PQ_D >> (l + 1);
        if (lane < n_ang) {
            const uint32_t code = gen_get_bits(rec, f.bit_off[l] + lane * f.bits[l], f.bits[l]);
            const float r = buf[cur][lane];
            const float2 t = centroids.cs[(l == 0 ? 0 : kGenMaxCells + (l - 1) * kGenUpperCells) + code];
            buf[cur ^ 1][2 * lane] = r * t.x;
            buf[cur ^ 1][2 * lane + 1] = r * t.y;
        }
        cur ^= 1;
        gen_wave_sync();
    }
    return cur;
}

/* ---- decode: one wavefront per record; out[i] = sum_j y_j S[i][j] with St[j][i] = S[i][j] ---- */
__global__ __launch_bounds__(64) void pq_general_decode_kernel(GenFormat f, GenCentroids centroids, const uint8_t *rec, int64_t n, const float *St,
                                                               int rotated, float *out)
{
    __shared__ float buf[2][PQ_D];
    const int64_t v = blockIdx.x;
    const int tid = threadIdx.x;
    if (v >= n) return;
    const int cur = gen_dequant_rotated(f, centroids, rec + v * f.rec_bytes, buf, tid);
    float a0 = 0.f, a1 = 0.f;
    if (rotated) {
        a0 = buf[cur][2 * tid];
        a1 = buf[cur][2 * tid + 1];
    } else {
        for (int j = 0; j < PQ_D; ++j) {
            const float2 s2 = *reinterpret_cast<const float2 *>(St + j * PQ_D + 2 * tid);
            a0 = fmaf(buf[cur][j], s2.x, a0);
            a1 = fmaf(buf[cur][j], s2.y, a1);
        }
    }
    out[v * PQ_D + 2 * tid] = a0;
    out[v * PQ_D + 2 * tid + 1] = a1;
}

/* x of the lane that the DPP control names, inside rows of sixteen lanes */
template <int CTRL>
__device__ __forceinline__ float gen_dpp(float x)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}

/* sum of lanes i, i ^ 16, i ^ 32, i ^ 48 */
__device__ __forceinline__ float gen_rows_sum(float x)
{
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

__device__ __forceinline__ float gen_wave_sum(float x)
{
    x += gen_dpp<0xB1>(x);
    x += gen_dpp<0x4E>(x);
    x += gen_dpp<0x141>(x);
    x += gen_dpp<0x140>(x);
    return gen_rows_sum(x);
}

__device__ __forceinline__ float gen_wave_max(float x)
{
    x = fmaxf(x, gen_dpp<0xB1>(x));
    x = fmaxf(x, gen_dpp<0x4E>(x));
    x = fmaxf(x, gen_dpp<0x141>(x));
    x = fmaxf(x, gen_dpp<0x140>(x));
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}

/* Of 2 HALF values a lane keeps the half that bit HALF of its lane number names, summed with those of the lane that CTRL pairs
   it with, which keeps the other half. */
template <int HALF, int CTRL>
__device__ __forceinline__ void gen_halve(float (&a)[16], int lane)
{
    const bool up = (lane & HALF) != 0;
#pragma unroll
    for (int c = 0; c < HALF; ++c) {
        const float keep = up ? a[c + HALF] : a[c], give = up ? a[c] : a[c + HALF];
        a[c] = keep + gen_dpp<CTRL>(give);
    }
}

/* ---- attention: one workgroup of eight or sixteen wavefronts per (sequence, HEADS query heads of one kv head) ----
 * Without a workspace a sequence is not split over workgroups (pq_general_piece_kernel does that); inside one, wavefront (tg, b) takes block
 * b (sixteen coordinates) of 64 tokens at a time, one token per lane:
 *   - the records of 64 or 128 tokens are copied to LDS, every record on a dword boundary, while those before are worked on;
 *   - a lane rebuilds its block from the codes on the path from the top radius down (the same fp32 products in the same
 *     order as DeQuant; fields are read with wave-uniform positions, centroids gathered from a 16-entry table), and leaves
 *     its part of the scores in LDS; the eight parts of a token are summed by every wavefront of its group;
 *   - softmax weights against an exponent reference per lane that moves only when a score exceeds it by more than kGenSlack;
 *   - the weighted values stay in the lane (sixteen sums per head); lanes, token groups and S^T come at the end.
 * Bound by LDS reads (36 centroid gathers and 16 field reads per wavefront and 64 tokens), then by vector instructions
 * (some 330).  4 sequences of 2048 tokens, 8 query heads: 646 us with one token per wavefront at a time -> 46 us.
 * Rebuilding the values ahead of the weights measured the same here and 4 to 9 % slower on 512 rows and more.
 * Sixteen wavefronts leave a lane 128 registers: enough for one head (124); two heads spilled 29 of them and four 66, which made
 * a workgroup of two or four heads take 20 to 30 us however short its sequence.  Eight wavefronts (163 and 195 registers) spill
 * nothing: 1024 rows of 10 tokens in fours 30.5 -> 14.6 us, of 600 tokens 63.9 -> 43.8. */
constexpr int kGenMaxDwords = (69 + 3) / 4 + 1; /* dwords of a record in LDS (an odd number: token strides spread over the banks) */
constexpr float kGenSlack = 16.f;

/* 32 bits at bit `pos` (the same in all lanes) of a lane's record */
__device__ __forceinline__ uint32_t gen_bits_at(const uint32_t *rec, int pos)
{
    return __builtin_amdgcn_alignbit(rec[(pos >> 5) + 1], rec[pos >> 5], pos & 31);
}

/* The sixteen coordinates of block `blk` (the same in all lanes) of a lane's record. */
__device__ __forceinline__ void gen_block(const GenFormat &f, const uint32_t *rec, const float2 (&cs)[7][kGenMaxCells], int blk,
                                          float (&v)[16])
{
    float r = (float)__builtin_bit_cast(_Float16, (uint16_t)gen_bits_at(rec, 8 * f.code_bytes + 16 * (blk >> (f.depth - 4))));
#pragma unroll
    for (int l = 6; l >= 4; --l) { /* levels above 4: the branch that leads to the block */
        if (l >= f.depth) continue;
        const uint32_t code = gen_bits_at(rec, f.bit_off[l] + (blk >> (l - 3)) * f.bits[l]) & ((1u << f.bits[l]) - 1u);
        const float2 t = cs[l][code];
        r *= ((blk >> (l - 4)) & 1) ? t.y : t.x;
    }
    const int b1 = f.bits[0], b2 = f.bits[1], b3 = f.bits[2], b4 = f.bits[3];
    const uint32_t g4 = gen_bits_at(rec, f.bit_off[3] + blk * b4), g3 = gen_bits_at(rec, f.bit_off[2] + 2 * blk * b3);
    const uint32_t g2 = gen_bits_at(rec, f.bit_off[1] + 4 * blk * b2), g1 = gen_bits_at(rec, f.bit_off[0] + 8 * blk * b1);
    const float2 t4 = cs[3][g4 & ((1u << b4) - 1u)];
    const float r3[2] = {r * t4.x, r * t4.y};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float2 t3 = cs[2][__builtin_amdgcn_ubfe(g3, h * b3, b3)];
        const float r2[2] = {r3[h] * t3.x, r3[h] * t3.y};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float2 t2 = cs[1][__builtin_amdgcn_ubfe(g2, (2 * h + q) * b2, b2)];
            const float r1[2] = {r2[q] * t2.x, r2[q] * t2.y};
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int k = 4 * h + 2 * q + p;
                const float2 t1 = cs[0][__builtin_amdgcn_ubfe(g1, k * b1, b1)];
                v[2 * k] = r1[p] * t1.x;
                v[2 * k + 1] = r1[p] * t1.y;
            }
        }
    }
}

/* Dword k of a record in memory (no alignment); a last, partial one is read with the record's last four bytes and has to be
   shifted right by gen_dword_shift bits, which is left to where the value is used: the loads then all go out together. */
__device__ __forceinline__ uint32_t gen_load_dword(const uint8_t *rec, int k, int rec_bytes)
{
    uint32_t w;
    __builtin_memcpy(&w, rec + min(4 * k, rec_bytes - 4), 4);
    return w;
}

__device__ __forceinline__ int gen_dword_shift(int k, int rec_bytes) { return 8 * max(4 * k + 4 - rec_bytes, 0); }

/* tokens of a sequence that take part: one outside the pool is treated as empty */
__device__ __forceinline__ int gen_tokens(int64_t n, int64_t t0, int64_t pool_tokens)
{
    return n < 0 || t0 < 0 || n > pool_tokens || t0 > pool_tokens - n ? 0 : (int)n; /* t0 + n could overflow */
}

/* ---- the same over several workgroups per sequence, for callers with a workspace ----
 * The chunks of kGenChunk tokens of all sequences are dealt out in pieces of `share` chunks (the last of a sequence may be
 * smaller), so that there are at most `slots` pieces and one more per sequence, numbered along the sequences.  Every wavefront
 * forms that by itself from the lengths, which the host does not know: lane b looks after sequence b.  `share` follows from the
 * lengths of all sequences and, by way of the slots, from B and Hq, so a row's pieces and the rounding of its sums do too. */
constexpr int kGenChunk = 64, kGenSplitBatch = 64; /* tokens; sequences of a split call */
constexpr int kGenWhole = 2; /* nothing is split in a call whose sequences all have at most so many chunks */

__device__ __forceinline__ int gen_wave_scan(int x) /* inclusive sum over the lanes */
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
    return x;
}

struct GenPlan {
    int len; /* as loaded */
    int64_t t0;
    int tokens, upto, share; /* of the lane's sequence; pieces of the sequences up to it; chunks per piece */

    __device__ __forceinline__ void load(const int64_t *seq_start, const int32_t *ctx_len, int B)
    {
        const int b = min((int)(threadIdx.x & 63), B - 1);
        len = ctx_len[b];
        t0 = seq_start[b];
    }
    __device__ __forceinline__ void form(int B, int64_t pool_tokens, int slots)
    {
        tokens = (int)(threadIdx.x & 63) < B ? gen_tokens(len, t0, pool_tokens) : 0;
        const int chunks = (tokens + kGenChunk - 1) / kGenChunk;
        const int sum = __builtin_amdgcn_readlane(gen_wave_scan(chunks), 63);
        share = __ballot(chunks > kGenWhole) == 0ull ? kGenWhole : max((sum + slots - 1) / slots, 1);
        upto = gen_wave_scan((chunks + share - 1) / share);
    }
    __device__ __forceinline__ int first(int b) const { return b > 0 ? __builtin_amdgcn_readlane(upto, b - 1) : 0; }
    __device__ __forceinline__ int pieces(int b) const { return __builtin_amdgcn_readlane(upto, b) - first(b); }
    __device__ __forceinline__ int tokens_of(int b) const { return __builtin_amdgcn_readlane(tokens, b); }
    __device__ __forceinline__ int64_t start_of(int b) const
    {
        return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(t0 >> 32), b) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)t0, b));
    }
};

struct GenSplit {
    int B, slots, pieces; /* pieces: the most there can be */
    float *o, *ml;        /* [piece][query head][128], [piece][query head][2]: weighted values, reference and sum of the weights */
    unsigned long long *arrived, call; /* [sequence][group of heads][kGenWordStride]: see gen_begin_count */
};

constexpr int kGenWordStride = 16; /* a line for each word: eight of them on one, 256 arrivals, took 4 us */
constexpr int kGenMostPieces = 256; /* of a sequence: GenPlan's share leaves no more than the slots, and general_split gives no more than that */

/* What a workgroup leaves for another one of the same launch, which may be on another XCD, behind another L2: written and read at the
   scope of the device, eight bytes at a time.  (Fences that write back an L2 for it took 3 us and more per piece.) */
__device__ __forceinline__ void gen_put(float *to, float x, float y)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(to), (unsigned long long)__float_as_uint(y) << 32 | __float_as_uint(x),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float2 gen_get(const float *from)
{
    const unsigned long long x = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(from), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)x), __uint_as_float((uint32_t)(x >> 32)));
}

/* Arrivals are counted at a word of the workspace, whose contents are anything at first.  Its upper 48 bits name the call.  Every
   workgroup, before it arrives, begins the count if it finds another name there; where its exchange fails, somebody else has.
   Nobody waits for anybody. */
__device__ __forceinline__ void gen_begin_count(unsigned long long *word, unsigned long long call)
{
    unsigned long long seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((seen >> 16) != call)
        __hip_atomic_compare_exchange_strong(word, &seen, call << 16, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* True for the last of `all`, which leaves a word that names no call: the same launch may follow on the same workspace (a graph
   that is replayed). */
__device__ __forceinline__ bool gen_arrive(unsigned long long *word, uint32_t all)
{
    const unsigned long long before = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = (uint32_t)(before & 0xFFFFull) == all - 1;
    if (last) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last;
}

template <int HEADS, int WAVES>
__global__ __launch_bounds__(WAVES * 64, HEADS == 1 ? 4 : 2) void pq_general_attn_kernel(
    GenFormat f, GenCentroids centroids, const uint16_t *q, float *out, const uint8_t *k_rec, const uint8_t *v_rec, const int64_t *seq_start,
    const int32_t *ctx_len, int Hq, int Hkv, int64_t pool_tokens, float scale, const float *S, const float *St)
{
    constexpr int kThreads = WAVES * 64, kTokens = kThreads / 8; /* eight blocks of a token, one per wavefront */
    constexpr int kGroups = kTokens / 64;
    __shared__ uint32_t srec[2][2][kTokens * kGenMaxDwords + 1]; /* [buffer][keys, values] */
    __shared__ float2 cs[7][kGenMaxCells];
    __shared__ float spart[HEADS][8][PQ_D];  /* a block's part of the scores; at the ends partial products with S */
    __shared__ __attribute__((aligned(16))) float sq[HEADS][PQ_D];
    __shared__ float so[HEADS][PQ_D]; /* sq: q, then its rotation; so: the weighted values */
    __shared__ float part_o[HEADS][kGroups][PQ_D], part_m[HEADS][kGroups], part_l[HEADS][kGroups];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tg = wave >> 3, blk = wave & 7;
    /* products with a matrix: thread (part, c) sums kTerms terms of column c; its slice is requested ahead */
    constexpr int kParts = kThreads / PQ_D, kTerms = PQ_D / kParts;
    const int my_part = tid >> 7, my_col = tid & 127;
    float slice[kTerms];
    auto load_slice = [&](const float *M) {
#pragma unroll
        for (int k = 0; k < kTerms; ++k) slice[k] = M[(kTerms * my_part + k) * PQ_D + my_col];
    };
    load_slice(S);
    const int groups = Hq / HEADS, b = blockIdx.x / groups, head0 = (blockIdx.x % groups) * HEADS, hk = head0 / (Hq / Hkv);
    const int64_t t0 = seq_start[b];
    const int64_t n = gen_tokens(ctx_len[b], t0, pool_tokens);
    const int64_t row0 = (int64_t)b * Hq + head0;

    /* records of tokens [first, first + kTokens) of the sequence: dword (stream, token, k) -> registers -> LDS */
    const int per_stream = kTokens * f.rec_dwords;
    constexpr int kMaxStage = (2 * kTokens * (kGenMaxDwords - 1) + kThreads - 1) / kThreads;
    uint32_t stage[kMaxStage];
    const int64_t slot0 = (int64_t)hk * pool_tokens + t0;
    struct Place { int stream, t, k; };
    auto place = [&](int at) { /* threads beyond the last dword repeat it */
        at = min(at, 2 * per_stream - 1);
        Place p;
        p.stream = at >= per_stream ? 1 : 0;
        const int in = at - p.stream * per_stream; /* below 2304: the multiplication by the inverse is exact */
        p.t = (int)(((uint32_t)in * (uint32_t)f.rec_inv) >> 16);
        p.k = in - p.t * f.rec_dwords;
        return p;
    };
    auto fetch = [&](int64_t first) {
#pragma unroll
        for (int i = 0; i < kMaxStage; ++i) {
            const Place p = place(tid + i * kThreads);
            const int64_t t = first + p.t < n ? first + p.t : n - 1; /* tokens beyond the sequence repeat its last one */
            stage[i] = gen_load_dword((p.stream ? v_rec : k_rec) + (slot0 + t) * f.rec_bytes, p.k, f.rec_bytes);
        }
    };
    auto store = [&](int buffer) {
#pragma unroll
        for (int i = 0; i < kMaxStage; ++i) {
            const Place p = place(tid + i * kThreads);
            srec[buffer][p.stream][p.t * kGenMaxDwords + p.k] = stage[i] >> gen_dword_shift(p.k, f.rec_bytes);
        }
    };
    if (n > 0) fetch(0);
    if (tid < kGenMaxCells + 6 * kGenUpperCells) (tid < kGenMaxCells ? cs[0][tid] : cs[(tid >> 3) - 1][tid & 7]) = centroids.cs[tid];
    for (int t = tid; t < HEADS * PQ_D; t += kThreads) sq[t >> 7][t & 127] = __uint_as_float((uint32_t)q[row0 * PQ_D + t] << 16);
    __syncthreads();
    auto times_slice = [&](const float (&in)[HEADS][PQ_D]) {
        float acc[HEADS];
#pragma unroll
        for (int h = 0; h < HEADS; ++h) acc[h] = 0.f;
#pragma unroll
        for (int k = 0; k < kTerms; ++k)
#pragma unroll
            for (int h = 0; h < HEADS; ++h) acc[h] = fmaf(in[h][kTerms * my_part + k], slice[k], acc[h]);
#pragma unroll
        for (int h = 0; h < HEADS; ++h) spart[h][my_part][my_col] = acc[h];
        __syncthreads();
    };
    auto product = [&](int h, int c) {
        float a[kParts];
#pragma unroll
        for (int k = 0; k < kParts; ++k) a[k] = spart[h][k][c];
#pragma unroll
        for (int d = kParts / 2; d >= 1; d >>= 1)
#pragma unroll
            for (int k = 0; k < d; ++k) a[k] = a[2 * k] + a[2 * k + 1];
        return a[0];
    };
    times_slice(sq); /* q' = q S */
    for (int t = tid; t < HEADS * PQ_D; t += kThreads) sq[t >> 7][t & 127] = product(t >> 7, t & 127);
    if (n > 0) store(0);
    __syncthreads();
    /* q' of the wavefront's block: the same in all lanes, in scalar registers */
    float qv[HEADS][16];
#pragma unroll
    for (int h = 0; h < HEADS; ++h)
#pragma unroll
        for (int c = 0; c < 16; ++c)
            qv[h][c] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(sq[h][16 * blk + c])));

    float m[HEADS], l[HEADS], acc[HEADS][16];
#pragma unroll
    for (int h = 0; h < HEADS; ++h) {
        m[h] = -INFINITY;
        l[h] = 0.f;
#pragma unroll
        for (int c = 0; c < 16; ++c) acc[h][c] = 0.f;
    }
    const int tok = 64 * tg + lane;
    int cur = 0;
    for (int64_t first = 0; first < n; first += kTokens, cur ^= 1) { /* n is the same in all threads */
        const bool more = first + kTokens < n;
        if (more) fetch(first + kTokens);
        {
            float v[16];
            gen_block(f, srec[cur][0] + tok * kGenMaxDwords, cs, blk, v);
#pragma unroll
            for (int h = 0; h < HEADS; ++h) {
                float d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < 16; ++c) d[c & 3] = fmaf(qv[h][c], v[c], d[c & 3]);
                spart[h][blk][tok] = (d[0] + d[1]) + (d[2] + d[3]);
            }
        }
        __syncthreads(); /* the parts are written, and everyone is through with the other buffer */
        if (more) store(cur ^ 1);
        const bool valid = first + tok < n;
        float p[HEADS];
#pragma unroll
        for (int h = 0; h < HEADS; ++h) {
            /* The parts are summed, scaled and compared with the reference in 64 bits: a score of 20 rounded to fp32
               would put 1e-6 on its token's weight, the largest error of the whole result. */
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) sum += (double)spart[h][k][tok];
            const double s = sum * (double)scale;
            float over = (float)(s - (double)m[h]); /* +inf at a lane's first token */
            const bool move = valid && over > kGenSlack;
            if (__ballot(move) != 0ull) {
                const float alpha = move ? expf(-over) : 1.f; /* exp(-inf) = 0 */
                if (move) {
                    m[h] = (float)s;
                    over = (float)(s - (double)m[h]);
                }
                l[h] *= alpha;
#pragma unroll
                for (int c = 0; c < 16; ++c) acc[h][c] *= alpha;
            }
            p[h] = valid ? expf(over) : 0.f;
            l[h] += p[h];
        }
        {
            float v[16];
            gen_block(f, srec[cur][1] + tok * kGenMaxDwords, cs, blk, v);
#pragma unroll
            for (int c = 0; c < 16; ++c)
#pragma unroll
                for (int h = 0; h < HEADS; ++h) acc[h][c] = fmaf(p[h], v[c], acc[h][c]);
        }
        __syncthreads(); /* the next records are in place, and the parts have been read */
    }
    load_slice(St);
    /* the lanes of a wavefront: everything to one reference, then sums; after four halving steps inside the rows of sixteen
       lanes a lane holds the coordinate that its lower four lane bits name */
#pragma unroll
    for (int h = 0; h < HEADS; ++h) {
        const float mw = gen_wave_max(m[h]);
        const float w = m[h] == -INFINITY ? 0.f : expf(m[h] - mw);
        const float lw = gen_wave_sum(l[h] * w);
        float a[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) a[c] = acc[h][c] * w;
        gen_halve<8, 0x140>(a, lane); /* with lane 15 - i of the row */
        gen_halve<4, 0x141>(a, lane); /* 7 - i of the half row */
        gen_halve<2, 0x1B>(a, lane);  /* 3 - i of the quad */
        gen_halve<1, 0xB1>(a, lane);  /* i ^ 1 */
        const float o = gen_rows_sum(a[0]);
        if (lane < 16) part_o[h][tg][16 * blk + lane] = o;
        if (blk == 0 && lane == 0) {
            part_m[h][tg] = mw;
            part_l[h][tg] = lw;
        }
    }
    __syncthreads();
    for (int t = tid; t < HEADS * PQ_D; t += kThreads) {
        const int h = t >> 7, c = t & 127;
        const float mm = fmaxf(part_m[h][0], part_m[h][kGroups - 1]);
        float lt = 0.f, a = 0.f;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const float w = part_m[h][g] == -INFINITY ? 0.f : expf(part_m[h][g] - mm); /* a group without a token */
            lt = fmaf(part_l[h][g], w, lt);
            a = fmaf(part_o[h][g][c], w, a);
        }
        so[h][c] = lt > 0.f ? a / lt : 0.f;
    }
    __syncthreads();
    times_slice(so);
    for (int t = tid; t < HEADS * PQ_D; t += kThreads) out[row0 * PQ_D + t] = product(t >> 7, t & 127);
}

/* A piece and HEADS query heads of its kv head: sixteen wavefronts, chunks of 64 tokens, one token per lane.  Wavefront b < 8
 * rebuilds block b of the keys and forms its part of the scores, wavefront 8 + b rebuilds block b of the values meanwhile; one
 * wavefront per head turns the parts into weights, and the value wavefronts multiply them with their values on
 * v_mfma_f32_16x16x4_f32 (fp32 products and sums; the values change places by way of LDS) while the others are at the next keys.
 * A sequence that is one piece is finished by its workgroup, of any other the workgroup that arrives last joins the pieces, in their order.
 * Bound by the chain of a piece: lengths 1 us, records and S 1.4, q S 1.2, a chunk 2.4, the end 1, joining 3.  4 sequences of 2000 tokens, 8
 * query heads: 45.2 us on 32 workgroups -> 12.7; one sequence of 8000 tokens 155 -> 16.9.  A second launch that joined the pieces took 13.9 and 17.2,
 * and sequences of up to 64 tokens, which have nothing to join, waited for it: 11.9 us, 10.2 on 32 workgroups, now 9.6; of up to 128
 * tokens 12.9, 10.4, 11.3.  Against 64 bits 3.1e-7 to 4.5e-7, one workgroup per row 3.2e-7 to 5.4e-7.  Weights against a reference per lane, sums
 * in the lanes and eight wavefronts for keys and values one after the other: 15.8 us for this launch alone, now 10.7. */
constexpr int kGenSplitThreads = 1024;

template <int HEADS>
__global__ __launch_bounds__(kGenSplitThreads, 4) void pq_general_piece_kernel(
    GenFormat f, GenCentroids centroids, const uint16_t *q, float *out, const uint8_t *k_rec, const uint8_t *v_rec, const int64_t *seq_start,
    const int32_t *ctx_len, int Hq, int Hkv, int64_t pool_tokens, float scale, const float *S, const float *St, GenSplit split)
{
    constexpr int kThreads = kGenSplitThreads, kParts = kThreads / PQ_D, kTerms = PQ_D / kParts;
    __shared__ uint32_t srec[2][2][kGenChunk * kGenMaxDwords + 1]; /* [buffer][keys, values] */
    __shared__ float2 cs[7][kGenMaxCells];
    __shared__ float spart[HEADS][kParts][PQ_D]; /* partial products with S; a block's part of the scores in its first 64 */
    __shared__ __attribute__((aligned(16))) float sq[HEADS][PQ_D]; /* q, then its rotation; at the end the weighted values */
    /* values of a wavefront's block, sixteen floats per token, and as many to spare after sixteen tokens: four tokens sixteen apart
       are read at a time, each from its own sixteen banks */
    __shared__ __attribute__((aligned(16))) float sv[8][(kGenChunk + 4) * 16];
    __shared__ __attribute__((aligned(16))) float sw[HEADS][kGenChunk], salpha[4]; /* weights of the chunk; factors on what was summed before */
    __shared__ float sm[HEADS], sl[HEADS];
    __shared__ bool last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), blk = wave & 7;
    const int my_part = tid >> 7, my_col = tid & 127;
    GenPlan plan;
    plan.load(seq_start, ctx_len, split.B); /* ahead of the loads below: they come back in order */
    float slice[kTerms];
    auto load_slice = [&](const float *M) {
#pragma unroll
        for (int k = 0; k < kTerms; ++k) slice[k] = M[(kTerms * my_part + k) * PQ_D + my_col];
    };
    load_slice(S);
    if (tid < kGenMaxCells + 6 * kGenUpperCells) (tid < kGenMaxCells ? cs[0][tid] : cs[(tid >> 3) - 1][tid & 7]) = centroids.cs[tid];
    const int groups = Hq / HEADS, item = blockIdx.x / groups, head0 = (blockIdx.x % groups) * HEADS, hk = head0 / (Hq / Hkv);
    plan.form(split.B, pool_tokens, split.slots);
    const int b = __popcll(__ballot(plan.upto <= item));
    if (b >= split.B) { /* fewer pieces than there could be, by at least one for every sequence without tokens: its row is zeros */
        uint64_t empty = __ballot(lane < split.B && plan.tokens == 0);
        for (int k = item - __builtin_amdgcn_readlane(plan.upto, 63); k > 0 && empty != 0; --k) empty &= empty - 1;
        if (empty != 0 && tid < HEADS * PQ_D) out[((int64_t)(__ffsll((unsigned long long)empty) - 1) * Hq + head0) * PQ_D + tid] = 0.f;
        return;
    }
    const bool whole = plan.pieces(b) == 1;
    unsigned long long *word = &split.arrived[(int64_t)(b * groups + (int)(blockIdx.x % groups)) * kGenWordStride];
    const int begin = (item - plan.first(b)) * plan.share * kGenChunk;
    const int n = (int)min((int64_t)plan.tokens_of(b), (int64_t)begin + (int64_t)plan.share * kGenChunk); /* begin < n */
    const int64_t row0 = (int64_t)b * Hq + head0, slot0 = (int64_t)hk * pool_tokens + plan.start_of(b);

    /* records of tokens [first, first + 64): dword (stream, token, k) -> registers -> LDS */
    const int per_stream = kGenChunk * f.rec_dwords;
    constexpr int kMaxStage = (2 * kGenChunk * (kGenMaxDwords - 1) + kThreads - 1) / kThreads;
    uint32_t stage[kMaxStage];
    struct Place { int stream, t, k; };
    auto place = [&](int at) { /* threads beyond the last dword repeat it */
        at = min(at, 2 * per_stream - 1);
        Place p;
        p.stream = at >= per_stream ? 1 : 0;
        const int in = at - p.stream * per_stream; /* below 1152: the multiplication by the inverse is exact */
        p.t = (int)(((uint32_t)in * (uint32_t)f.rec_inv) >> 16);
        p.k = in - p.t * f.rec_dwords;
        return p;
    };
    auto fetch = [&](int first) {
#pragma unroll
        for (int i = 0; i < kMaxStage; ++i) {
            const Place p = place(tid + i * kThreads);
            const int t = min(first + p.t, n - 1); /* tokens beyond the piece repeat its last one */
            stage[i] = gen_load_dword((p.stream ? v_rec : k_rec) + (slot0 + t) * f.rec_bytes, p.k, f.rec_bytes);
        }
    };
    auto store = [&](int buffer) {
#pragma unroll
        for (int i = 0; i < kMaxStage; ++i) {
            const Place p = place(tid + i * kThreads);
            srec[buffer][p.stream][p.t * kGenMaxDwords + p.k] = stage[i] >> gen_dword_shift(p.k, f.rec_bytes);
        }
    };
    fetch(begin);
    for (int t = tid; t < HEADS * PQ_D; t += kThreads) sq[t >> 7][t & 127] = __uint_as_float((uint32_t)q[row0 * PQ_D + t] << 16);
    __syncthreads();
    auto times_slice = [&](const float (&in)[HEADS][PQ_D]) {
#pragma unroll
        for (int h = 0; h < HEADS; ++h) {
            float acc = 0.f;
#pragma unroll
            for (int k = 0; k < kTerms; k += 4) {
                const float4 x = *reinterpret_cast<const float4 *>(&in[h][kTerms * my_part + k]);
                acc = fmaf(x.x, slice[k], acc);
                acc = fmaf(x.y, slice[k + 1], acc);
                acc = fmaf(x.z, slice[k + 2], acc);
                acc = fmaf(x.w, slice[k + 3], acc);
            }
            spart[h][my_part][my_col] = acc;
        }
        __syncthreads();
    };
    auto product = [&](int h, int c) {
        float a[kParts];
#pragma unroll
        for (int k = 0; k < kParts; ++k) a[k] = spart[h][k][c];
        return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    };
    times_slice(sq); /* q' = q S */
    for (int t = tid; t < HEADS * PQ_D; t += kThreads) sq[t >> 7][t & 127] = product(t >> 7, t & 127);
    store(0);
    __syncthreads();
    if (whole) load_slice(St);
    else if (tid == kThreads - 1) gen_begin_count(word, split.call);

    float m = -INFINITY, l = 0.f; /* wavefront h < HEADS: reference and sum of the weights of head h, for the lane's tokens */
    gen_f4 acc = {0.f, 0.f, 0.f, 0.f}; /* wavefront 8 + b, lane j < 16: coordinate 16 b + j for head 0, 1, ... */
    int cur = 0;
    for (int first = begin; first < n; first += kGenChunk, cur ^= 1) { /* n is the same in all threads */
        const bool more = first + kGenChunk < n;
        if (more) fetch(first + kGenChunk);
        float v[16];
        gen_block(f, srec[cur][wave >> 3] + lane * kGenMaxDwords, cs, blk, v);
        if (wave < 8) {
#pragma unroll
            for (int h = 0; h < HEADS; ++h) {
                float d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < 16; c += 4) {
                    const float4 qc = *reinterpret_cast<const float4 *>(&sq[h][16 * blk + c]);
                    d[0] = fmaf(qc.x, v[c], d[0]);
                    d[1] = fmaf(qc.y, v[c + 1], d[1]);
                    d[2] = fmaf(qc.z, v[c + 2], d[2]);
                    d[3] = fmaf(qc.w, v[c + 3], d[3]);
                }
                spart[h][blk][lane] = (d[0] + d[1]) + (d[2] + d[3]);
            }
        } else {
            float4 *to = reinterpret_cast<float4 *>(&sv[blk][16 * (lane + (lane >> 4))]);
#pragma unroll
            for (int c = 0; c < 16; c += 4) to[c / 4] = make_float4(v[c], v[c + 1], v[c + 2], v[c + 3]);
        }
        __syncthreads(); /* the parts are written, and everyone is through with the other buffer */
        if (more) store(cur ^ 1);
        if (wave < HEADS) {
            const bool valid = first + lane < n;
            /* The parts are summed, scaled and compared with the reference in 64 bits: a score of 20 rounded to fp32
               would put 1e-6 on its token's weight, the largest error of the whole result. */
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) sum += (double)spart[wave][k][lane];
            const double s = sum * (double)scale;
            const float top = gen_wave_max(valid ? (float)s : -INFINITY);
            float alpha = 1.f;
            if (top > m + kGenSlack || m == -INFINITY) { /* the same in all lanes */
                alpha = m == -INFINITY ? 0.f : expf(m - top);
                m = top;
            }
            const float p = valid ? expf((float)(s - (double)m)) : 0.f;
            l = l * alpha + p;
            sw[wave][lane] = p;
            if (lane == 0) salpha[wave] = alpha;
        }
        __syncthreads(); /* the next records are in place, the parts have been read, the weights are written */
        if (wave >= 8) { /* contraction: step k takes tokens k, 16 + k, 32 + k and 48 + k */
            const int g = lane >> 4, j = lane & 15;
            gen_f4 o = {0.f, 0.f, 0.f, 0.f};
            const float4 *w4 = reinterpret_cast<const float4 *>(&sw[min(j, HEADS - 1)][16 * g]);
            const float *from = &sv[blk][16 * 17 * g + j];
#pragma unroll
            for (int k = 0; k < 16; k += 4) {
                float4 w = w4[k / 4];
                if (j >= HEADS) w = make_float4(0.f, 0.f, 0.f, 0.f);
                o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, from[16 * k], o, 0, 0, 0);
                o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, from[16 * k + 16], o, 0, 0, 0);
                o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, from[16 * k + 32], o, 0, 0, 0);
                o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, from[16 * k + 48], o, 0, 0, 0);
            }
#pragma unroll
            for (int h = 0; h < HEADS; ++h) acc[h] = fmaf(acc[h], salpha[h], o[h]);
        }
    }
    if (wave < HEADS) {
        l = gen_wave_sum(l);
        if (lane == 0) {
            sm[wave] = m;
            sl[wave] = l;
        }
    }
    __syncthreads();
    if (wave >= 8 && lane < 16) {
#pragma unroll
        for (int h = 0; h < HEADS; ++h) sq[h][16 * blk + lane] = whole ? acc[h] / sl[h] : acc[h]; /* a piece has a token: sl > 0 */
    }
    __syncthreads();
    if (!whole) {
        /* The piece's sums go to the workspace; the workgroup that arrives last joins the pieces of its row.  Other XCDs have other
           L2s: the sums are written and read at the scope of the device, and every wavefront waits until its own have arrived there. */
        constexpr int kPairs = HEADS * PQ_D / 2, kSums = kThreads / kPairs, kBatch = 16;
        const int64_t at = (int64_t)item * Hq + head0;
        if (tid < kPairs) gen_put(&split.o[at * PQ_D + 2 * tid], (&sq[0][0])[2 * tid], (&sq[0][0])[2 * tid + 1]);
        if (tid < HEADS) gen_put(&split.ml[(at + tid) * 2], sm[tid], sl[tid]);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const int first_piece = plan.first(b), used = plan.pieces(b);
        if (tid == 0) last = gen_arrive(word, (uint32_t)used);
        __syncthreads();
        if (!last) return;
        /* thread (share, pair): pieces share, share + kSums, ... of two neighbouring columns, kBatch of them requested at once */
        const int pair = tid % kPairs, share = tid / kPairs, h = pair >> 6;
        const float *ml = split.ml + ((int64_t)first_piece * Hq + head0 + min(wave, HEADS - 1)) * 2;
        const float *po = split.o + ((int64_t)first_piece * Hq + head0) * PQ_D + 2 * pair;
        float2 v[kGenMostPieces / 64], batch[kBatch];
        if (wave < HEADS)
#pragma unroll
            for (int i = 0; i < kGenMostPieces / 64; ++i) {
                v[i] = make_float2(-INFINITY, 0.f);
                if (lane + 64 * i < used) v[i] = gen_get(ml + (int64_t)(lane + 64 * i) * Hq * 2);
            }
        auto request = [&](int p) {
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                batch[i] = make_float2(0.f, 0.f);
                if (p + i * kSums < used) batch[i] = gen_get(po + (int64_t)(p + i * kSums) * Hq * PQ_D);
            }
        };
        request(share);
        load_slice(St);
        float *weight = reinterpret_cast<float *>(&srec[0][0][0]); /* [HEADS][kGenMostPieces], on one reference */
        static_assert(sizeof(srec) >= sizeof(float) * HEADS * kGenMostPieces, "the records' buffers hold the weights");
        if (wave < HEADS) {
            float top = -INFINITY, sum = 0.f;
#pragma unroll
            for (int i = 0; i < kGenMostPieces / 64; ++i) top = fmaxf(top, v[i].x);
            top = gen_wave_max(top);
#pragma unroll
            for (int i = 0; i < kGenMostPieces / 64; ++i) {
                const float w = expf(v[i].x - top); /* a piece has a token, and a reference; one that is not there has weight 0 */
                weight[wave * kGenMostPieces + lane + 64 * i] = w;
                sum = fmaf(v[i].y, w, sum);
            }
            sum = gen_wave_sum(sum);
            if (lane == 0) sl[wave] = sum;
        }
        __syncthreads();
        float2 o = make_float2(0.f, 0.f);
        for (int p = share; p < used; p += kBatch * kSums) {
            if (p != share) request(p);
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                if (p + i * kSums < used) {
                    const float w = weight[h * kGenMostPieces + p + i * kSums];
                    o.x = fmaf(batch[i].x, w, o.x);
                    o.y = fmaf(batch[i].y, w, o.y);
                }
        }
        float2 *sums = reinterpret_cast<float2 *>(&sv[0][0]);
        sums[tid] = o;
        __syncthreads();
        if (tid < kPairs) {
            float2 a = sums[tid];
#pragma unroll
            for (int k = 1; k < kSums; ++k) {
                a.x += sums[k * kPairs + tid].x;
                a.y += sums[k * kPairs + tid].y;
            }
            (&sq[0][0])[2 * tid] = a.x / sl[h];
            (&sq[0][0])[2 * tid + 1] = a.y / sl[h];
        }
        __syncthreads();
    }
    times_slice(sq);
    for (int t = tid; t < HEADS * PQ_D; t += kThreads) out[row0 * PQ_D + t] = product(t >> 7, t & 127);
}

/* heads of a kv head that a workgroup of a split call takes together */
int gen_split_heads(int G) { return G % 4 == 0 ? 4 : (G % 2 == 0 ? 2 : 1); }

/* How a call is split: not at all (slots 0) where the heads alone occupy half of the CUs, or where the pool holds no more than
   eight chunks per sequence (three sequences, 8 heads, us for the call, split and not: 2000 tokens 12.8 / 45.2, 500 12.3 / 17.0, 300 12.0 /
   14.7, 200 12.0 / 12.3; the lengths are on the device, so the pool stands for them).  Nor in a pool of more than kGenSplitTokens: the
   split kernel counts tokens in 32 bits, and up to there a token plus a chunk, and the chunks of kGenSplitBatch sequences that
   overlap (2^30 of them), stay below 2^31.  The row kernel counts in 64. */
constexpr int64_t kGenSplitTokens = (int64_t)1 << 30;

GenSplit general_split(int B, int Hq, int Hkv, int64_t pool_tokens)
{
    GenSplit p{};
    p.B = B;
    const int64_t rows = (int64_t)B * Hq, chunks = (pool_tokens + kGenChunk - 1) / kGenChunk;
    if (rows > 128 || B > kGenSplitBatch || chunks <= 8 * (int64_t)B || pool_tokens > kGenSplitTokens) return p;
    const int groups = Hq / gen_split_heads(Hq / Hkv);
    p.slots = groups < 256 ? 256 / groups : 1;
    p.pieces = p.slots + B;
    return p;
}

/* the sums of the pieces, then the arrivals: a word per query head is more than there are groups */
size_t general_split_bytes(const GenSplit &p, int Hq)
{
    return p.slots ? (size_t)p.pieces * Hq * (PQ_D + 2) * sizeof(float) + (size_t)p.B * Hq * kGenWordStride * sizeof(unsigned long long) : 0;
}

/* Names a call in 48 bits, never 0, beginning anywhere: a workspace that happens to hold the name of this call before it
   (1 in 2^48) is what is left to chance. */
unsigned long long next_call()
{
    static std::atomic<uint64_t> calls{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ULL >> 16};
    unsigned long long c;
    do c = calls.fetch_add(1, std::memory_order_relaxed) & 0xFFFFFFFFFFFFull;
    while (c == 0);
    return c;
}

} // namespace

extern "C" size_t pq_general_record_bytes(const pq_general_format *f)
{
    if (!general_format_ok(f)) return 0;
    return (size_t)((general_code_bits(f) + 7) / 8 + 2 * (PQ_D >> f->depth));
}

extern "C" int pq_general_codebook_entries(const pq_general_format *f)
{
    if (!general_format_ok(f)) return 0;
    int n = 0;
    for (int l = 0; l < f->depth; ++l) n += 1 << f->bits[l];
    return n;
}

extern "C" pq_status pq_general_codebooks(const pq_general_format *f, double *cbg)
{
    if (!general_format_ok(f) || !cbg) return PQ_EINVAL;
    const double two_pi = 6.28318530717958647692;
    int off = 0;
    for (int l = 0; l < f->depth; ++l) {
        const int K = 1 << f->bits[l];
        if (l == 0) {
            for (int k = 0; k < K; ++k) cbg[off + k] = two_pi * (k + 0.5) / K; /* uniform on [0, 2 pi): equal cells */
        } else {
            double bnd[kGenMaxCells + 1];
            pq_lloyd_max(l + 1, K, cbg + off, bnd);
        }
        off += K;
    }
    return PQ_OK;
}

extern "C" pq_status pq_general_encode(const pq_ctx *ctx, const pq_general_format *f, const double *cbg, const void *x,
                                       pq_dtype xt, int64_t n_vectors, int64_t ld_vector, uint8_t *records,
                                       void *hip_stream)
{
    if (!ctx || !x || !records || n_vectors < 0 || ld_vector < PQ_D) return PQ_EINVAL;
    if (xt != PQ_F32 && xt != PQ_BF16) return PQ_EINVAL;
    if (n_vectors > 0x7FFFFFFF) return PQ_EUNSUPPORTED;
    GenFormat g;
    pq_status st = make_format(f, cbg, &g);
    if (st != PQ_OK) return st;
    if (n_vectors == 0) return PQ_OK;
    const PqDeviceState *ds = nullptr;
    st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const GenBounds bounds = make_bounds(g, cbg);
    if (xt == PQ_BF16)
        hipLaunchKernelGGL(pq_general_encode_kernel<PQ_BF16>, dim3((unsigned)((n_vectors + kGenEncVecs - 1) / kGenEncVecs)), dim3(kGenEncThreads), 0, s, g, bounds, x, ld_vector, n_vectors, ds->S_f32, records);
    else
        hipLaunchKernelGGL(pq_general_encode_kernel<PQ_F32>, dim3((unsigned)((n_vectors + kGenEncVecs - 1) / kGenEncVecs)), dim3(kGenEncThreads), 0, s, g, bounds, x, ld_vector, n_vectors, ds->S_f32, records);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}

extern "C" pq_status pq_general_decode(const pq_ctx *ctx, const pq_general_format *f, const double *cbg,
                                       const uint8_t *records, int64_t n_vectors, int rotated, float *out, void *hip_stream)
{
    if (!ctx || !records || !out || n_vectors < 0) return PQ_EINVAL;
    if (n_vectors > 0x7FFFFFFF) return PQ_EUNSUPPORTED;
    GenFormat g;
    pq_status st = make_format(f, cbg, &g);
    if (st != PQ_OK) return st;
    if (n_vectors == 0) return PQ_OK;
    const PqDeviceState *ds = nullptr;
    st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    hipLaunchKernelGGL(pq_general_decode_kernel, dim3((unsigned)n_vectors), dim3(64), 0, static_cast<hipStream_t>(hip_stream),
                       g, make_centroids(g, cbg), records, n_vectors, ds->St_f32, rotated, out);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}

extern "C" size_t pq_general_attn_workspace_bytes(int B, int Hq, int Hkv, int64_t pool_tokens)
{
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || Hq % Hkv || pool_tokens <= 0) return 0;
    return general_split_bytes(general_split(B, Hq, Hkv, pool_tokens), Hq);
}

extern "C" pq_status pq_general_attn_decode(const pq_ctx *ctx, const pq_general_format *f, const double *cbg, const void *q,
                                            float *out, const uint8_t *k_records, const uint8_t *v_records,
                                            const int64_t *seq_start, const int32_t *ctx_len, int B, int Hq, int Hkv,
                                            int64_t pool_tokens, float softmax_scale, void *hip_stream)
{
    return pq_general_attn_decode_ws(ctx, f, cbg, q, out, k_records, v_records, seq_start, ctx_len, B, Hq, Hkv, pool_tokens,
                                     softmax_scale, nullptr, 0, hip_stream);
}

extern "C" pq_status pq_general_attn_decode_ws(const pq_ctx *ctx, const pq_general_format *f, const double *cbg, const void *q,
                                               float *out, const uint8_t *k_records, const uint8_t *v_records,
                                               const int64_t *seq_start, const int32_t *ctx_len, int B, int Hq, int Hkv,
                                               int64_t pool_tokens, float softmax_scale, void *workspace, size_t workspace_bytes,
                                               void *hip_stream)
{
    if (!ctx || !q || !out || !k_records || !v_records || !seq_start || !ctx_len) return PQ_EINVAL;
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || Hq % Hkv || pool_tokens <= 0) return PQ_EINVAL;
    if ((int64_t)B * Hq > 0x7FFFFFFF) return PQ_EUNSUPPORTED;
    GenFormat g;
    pq_status st = make_format(f, cbg, &g);
    if (st != PQ_OK) return st;
    const PqDeviceState *ds = nullptr;
    st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    /* Heads of a kv head in one workgroup rebuild its tokens once for all of them: as soon as that leaves a workgroup for
       every CU (2048 rows of 600 tokens: 85.5 us with four heads, 100.6 with two, 107.5 with one; 1024 rows of 10 tokens: 14.5, 18.0
       and 18.3; 512 rows of 2000 tokens: 67 with two, 82 with one).  Below, a workgroup per head has more of the chip at work: sixteen
       wavefronts while every one finds a CU, else eight, two workgroups to a CU (300 rows of 4 tokens: 11.3 us against
       18.5 in two rounds of sixteen, of 600 tokens 30 against 38). */
    const int64_t rows = (int64_t)B * Hq;
    const int G = Hq / Hkv;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const GenCentroids centroids = make_centroids(g, cbg);
    GenSplit split = workspace ? general_split(B, Hq, Hkv, pool_tokens) : GenSplit{};
    if (split.slots && workspace_bytes < general_split_bytes(split, Hq)) split = GenSplit{};
    if (split.slots && !pq_aligned16(workspace)) return PQ_EALIGN;
    if (split.slots) {
        split.o = static_cast<float *>(workspace);
        split.ml = split.o + (size_t)split.pieces * Hq * PQ_D;
        split.arrived = reinterpret_cast<unsigned long long *>(split.ml + (size_t)split.pieces * Hq * 2);
        split.call = next_call();
        const int heads = gen_split_heads(G);
        const dim3 grid((unsigned)((int64_t)split.pieces * (Hq / heads))), blk(kGenSplitThreads);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, blk, 0, stream, g, centroids, static_cast<const uint16_t *>(q), out, k_records, v_records, seq_start,
                               ctx_len, Hq, Hkv, pool_tokens, softmax_scale, ds->S_f32, ds->St_f32, split);
        };
        if (heads == 4) launch(pq_general_piece_kernel<4>);
        else if (heads == 2) launch(pq_general_piece_kernel<2>);
        else launch(pq_general_piece_kernel<1>);
        PQ_HIP_TRY(hipGetLastError());
        return PQ_OK;
    }
    auto launch = [&](auto heads, auto waves) {
        constexpr int H = decltype(heads)::value, W = decltype(waves)::value;
        hipLaunchKernelGGL((pq_general_attn_kernel<H, W>), dim3((unsigned)(rows / H)), dim3(W * 64), 0, stream, g, centroids,
                           static_cast<const uint16_t *>(q), out, k_records, v_records, seq_start, ctx_len, Hq, Hkv, pool_tokens,
                           softmax_scale, ds->S_f32, ds->St_f32);
    };
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 4> four{};
    constexpr std::integral_constant<int, 8> eight{};
    constexpr std::integral_constant<int, 16> sixteen{};
    if (G % 4 == 0 && rows >= 4 * 256) launch(four, eight);
    else if (G % 2 == 0 && rows >= 2 * 256) launch(two, eight);
    else if (rows > 256) launch(one, eight);
    else launch(one, sixteen);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}
