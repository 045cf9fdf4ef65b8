/*
 * pq_fit.hip -- pq_fit_codebooks: online codebook construction (Section 4.1,
 * line 3 of Algorithm 1 in its online variant: 1-D k-means on the angles of the
 * polar-transformed inputs), for gfx950.
 *
 * The heavy part runs on the GPU: every input vector is rotated (y = x S), its
 * 120 angles are formed (procedure Polar) and counted into fine histograms,
 * one per level (8192 bins over [0, 2 pi) for level 1, 2048 over [0, pi/2] for
 * levels 2-4; for a full-depth context 2048 more for each of levels 5-7, see
 * pq_fit_codebooks_deep).  A second kernel forms the running sums of the counts and
 * leaves both in host memory, and the k-means rounds then look up what they need there,
 * in fp64 on the host, where the result is wanted (pq_set_codebooks takes host centroids).
 *
 * Kernel: one wavefront per tile of 64 vectors, sixteen wavefronts per
 * workgroup, S and the histograms in LDS.
 *   Rotation on the matrix cores as in the encode kernel (same operand image of
 *   S, same register layout of the result: a lane ends up with complete blocks
 *   of 16 rotated coordinates of one vector), with the two leading bf16 terms
 *   of S (16 significant bits; bf16 inputs are exact operands, fp32 inputs are
 *   split into two terms and the three products above 2^-16 are used): the
 *   angle error of 1e-5 rad is a hundredth of a bin.
 *   Bins are uniform in the pseudo-angle t = v / (u + v) of a node's two inputs
 *   (level 1: quadrant + t, with |y| or |x| on top so that it grows with the
 *   angle), which is monotone in the angle and costs a reciprocal instead of
 *   an arctangent: bin edge k / 2048 is the angle atan2(k, 2048 - k).  The
 *   host part knows the edges and treats the angles of a bin as spread evenly
 *   between them.
 * Counts are integers: the result does not depend on scheduling.
 * Bound by the vector instructions of a tile and, for short inputs, by the
 * launch, its latencies and the workgroups' additions to the call's counters (some
 * 6 us for 256 workgroups).  The square roots are correctly rounded (the hardware's
 * own would move nodes next to a bin edge, and count every upper angle of a vector
 * below 1e-19 as 0), in five instructions where the squares are in a middle range;
 * with sqrtf's fourteen, one half of a tile fetched after the other, a wavefront per
 * tile and a workgroup per tile up to 256, the clear included: 8000 bf16 vectors
 * 21.8 -> 13.4 us, 32000 29.7 -> 19.5, 262144 50.7 -> 43.4; fp32 23.7 -> 18.9,
 * 32.8 -> 23.9, 59.5 -> 54.5.
 */
#include "pq_common.h"
#include "pq_root.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

namespace {

constexpr int kBins1 = 8192, kBinsU = 2048;
constexpr int kHistSize = kBins1 + 3 * kBinsU; /* 14336 counters */
constexpr int kHistUpper = 3 * kBinsU;         /* levels 5..7 (full-depth recursion): 6144 more */
constexpr int kFitWaves = 16, kFitThreads = kFitWaves * 64;
constexpr int kTileVecs = 64;
constexpr int kFitTerms = 2;                   /* bf16 terms of S that take part */

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct FitArgs {
    const void *x;
    int64_t ld_token, ld_head, n_tokens;
    int n_heads;
    int64_t tiles_per_head, n_items;
    const uint4 *S_bf16x3; /* the encode kernel's operand image of S, term-major */
    uint32_t *hist;        /* [kHistSize], zeroed before the launch */
    uint32_t *hist_up;     /* [kHistUpper] or NULL: angles of levels 5..7 */
};

union FitOperand {
    bf16x8 v;
    uint4 q;
    uint32_t w[4];
};

__device__ __forceinline__ uint32_t fit_bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

/* (u^2 + v^2)^(1/2), correctly rounded; MID: see fit_root */
template <bool MID = false>
__device__ __forceinline__ float fit_radius(float u, float v) { return fit_root<MID>(__builtin_fmaf(u, u, v * v)); }

/* byte offset of the counter of t = part / sum among `bins` equal ones; atan2(0, 0) counts as 0 */
template <int BINS>
__device__ __forceinline__ uint32_t bin_offset(float part, float sum)
{
    const float t = part * __builtin_amdgcn_rcpf(fmaxf(sum, 1e-37f));
    return min((uint32_t)(t * (float)BINS), (uint32_t)BINS - 1u) << 2;
}

__device__ __forceinline__ void count_at(uint32_t *hist, uint32_t byte_offset)
{
    atomicAdd(reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(hist) + byte_offset), 1u);
}

/* Counts the angle of (u, v), both >= 0, in a histogram of kBinsU bins uniform in t = v / (u + v). */
__device__ __forceinline__ void count_upper(uint32_t *hist, float u, float v) { count_at(hist, bin_offset<kBinsU>(v, u + v)); }

/* Angles of one block of 16 rotated coordinates, with the squared radii q of its pairs, into the LDS histograms; returns the
   block's radius. */
template <bool MID>
__device__ __forceinline__ float count_block_angles(const f32x16 &y, const float (&q)[8], uint32_t *sh)
{
    float r[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const float a = y[2 * p], b = y[2 * p + 1];
        /* quadrants of [0, 2 pi): (+,+), (-,+), (-,-), (+,-); the sign bits go straight to their places in the offset */
        const uint32_t ub = __float_as_uint(b), x = __float_as_uint(a) ^ ub; /* sign of x: an odd quadrant */
        const uint32_t quadrant = ((ub >> 17) & 0x4000u) | ((x >> 18) & 0x2000u);
        const uint32_t in = bin_offset<kBins1 / 4>((int32_t)x < 0 ? fabsf(a) : fabsf(b), fabsf(a) + fabsf(b));
        count_at(sh, quadrant | in);
        r[p] = fit_root<MID>(q[p]);
    }
    static_assert(kBins1 == 8192, "0x2000 bytes are a quadrant's 2048 counters");
    int base = kBins1;
#pragma unroll
    for (int n = 4; n >= 1; n >>= 1) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (p < n) {
                const float u = r[2 * p], v = r[2 * p + 1];
                count_upper(sh + base, u, v);
                r[p] = fit_radius<MID>(u, v);
            }
        }
        base += kBinsU;
    }
    return r[0];
}

/* The short roots where all squares of a wavefront's blocks are in their range (an upper one is at most eight times the
   largest of them); sqrtf for vectors of zeros, below 2^-50, above 2^48, infinite or not a number. */
__device__ __forceinline__ float count_block(const f32x16 &y, uint32_t *sh)
{
    float q[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) q[p] = __builtin_fmaf(y[2 * p], y[2 * p], y[2 * p + 1] * y[2 * p + 1]);
    bool mid = true;
#pragma unroll
    for (int p = 0; p < 8; ++p) mid = mid && q[p] >= 0x1p-100f && q[p] <= 0x1p96f;
    return __ballot(!mid) == 0ull ? count_block_angles<true>(y, q, sh) : count_block_angles<false>(y, q, sh);
}

/* Adds a workgroup's counters to the call's, two at a time: no total reaches 2^32, so nothing carries from one into the
   other.  The workgroups end together; each begins elsewhere, so that they don't all add to the same lines (262144 bf16 vectors
   44.4 -> 42.0 us). */
__device__ __forceinline__ void add_counts(uint32_t *total, const uint32_t *sh, int n)
{
    const uint2 *pairs = reinterpret_cast<const uint2 *>(sh);
    unsigned long long *out = reinterpret_cast<unsigned long long *>(total);
    const int n2 = n / 2, begin = (int)((uint32_t)blockIdx.x * (uint32_t)n2 / gridDim.x) & ~15; /* whole lines of 128 bytes */
    for (int c = threadIdx.x; c < n2; c += kFitThreads) {
        const int at = c + begin < n2 ? c + begin : c + begin - n2;
        const uint2 v = pairs[at];
        if (v.x | v.y) atomicAdd(&out[at], ((unsigned long long)v.y << 32) | v.x);
    }
}

/* bf16 terms of fp32 input; bf16 input is one exact term */
template <int XT> constexpr int fit_terms() { return XT == PQ_BF16 ? 1 : 2; }

/* B operands of a vector's lane: its 8-coordinate slices (coordinates 64 H + 8 ks .. + 7) from element offset `at` */
template <int XT>
__device__ __forceinline__ void load_vector(const FitArgs &a, int64_t at, int H, FitOperand (&xb)[fit_terms<XT>()][8])
{
    if constexpr (XT == PQ_BF16) {
        const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(a.x) + at);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) xb[0][ks].q = xr[8 * H + ks];
    } else {
        const float4 *xr = reinterpret_cast<const float4 *>(static_cast<const float *>(a.x) + at);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const float4 p0 = xr[16 * H + 2 * ks], p1 = xr[16 * H + 2 * ks + 1];
            const float f[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                uint32_t hi[2], lo[2];
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    hi[z] = fit_bf16_rne(f[e + z]);
                    lo[z] = fit_bf16_rne(f[e + z] - __uint_as_float(hi[z] << 16));
                }
                xb[0][ks].w[e / 2] = hi[0] | (hi[1] << 16);
                xb[1][ks].w[e / 2] = lo[0] | (lo[1] << 16);
            }
        }
    }
}

/* D[i][j] = sum_k S[k][col(rt, i)] x[j][k]: lane (H, j) receives rotated coordinates 16 (4 H + rt) .. + 15 of vector j */
template <int XT>
__device__ __forceinline__ f32x16 rotate_block(const uint4 *sS, int rt, const FitOperand (&xb)[fit_terms<XT>()][8], int lane)
{
    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int term = kFitTerms - 1; term >= 0; --term)
#pragma unroll
            for (int xt = 0; xt < fit_terms<XT>(); ++xt) {
                if (term + xt > 1) continue; /* below 2^-16 of the leading product */
                FitOperand sa;
                sa.q = sS[((term * 4 + rt) * 8 + ks) * 64 + lane];
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa.v, xb[xt][ks].v, acc, 0, 0, 0);
            }
    return acc;
}

/* SPLIT, for short inputs of four levels: eight wavefronts share a tile, wavefront (half, row tile) counts the 32 x 2 blocks of its
   part (a tile is a chain of 128 matrix and some 3000 vector instructions: see the launch for what it takes alone). */
template <int XT, bool SPLIT>
__global__ __launch_bounds__(kFitThreads, 1) void pq_angle_histogram_kernel(FitArgs a)
{
    __shared__ uint4 sS[kFitTerms * 4 * 8 * 64];    /* 64 KB */
    __shared__ __attribute__((aligned(16))) uint32_t sh[kHistSize + kHistUpper]; /* 80 KB */
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 31, H = lane >> 5; /* vector within a 32-vector half, lane half */
    /* element offset of vector 32 v + j of an item; a lane without a vector reads the tile's first one again and counts nothing */
    auto vector_at = [&](int64_t item, int v, bool &valid) {
        const int64_t t0 = (item % a.tiles_per_head) * kTileVecs, tok = t0 + 32 * v + j;
        valid = tok < a.n_tokens;
        return (valid ? tok : t0) * a.ld_token + (item / a.tiles_per_head) * a.ld_head;
    };
    /* consecutive tiles go to different workgroups: a short input occupies every CU */
    constexpr int kShare = SPLIT ? 8 : 1; /* wavefronts of a tile */
    const int64_t stride = (int64_t)gridDim.x * (kFitWaves / kShare);
    int64_t item = (int64_t)(wave / kShare) * gridDim.x + blockIdx.x;
    const int my_v = (wave >> 2) & 1, my_rt = wave & 3; /* SPLIT */
    FitOperand xb[2][fit_terms<XT>()][8];
    bool valid[2] = {false, false};
    /* of bf16 input both halves' rows are requested at once: the second's arrive under the first's work */
    auto load_item = [&](int64_t it) {
        if (SPLIT) {
            load_vector<XT>(a, vector_at(it, my_v, valid[0]), H, xb[0]);
        } else if (XT == PQ_BF16) {
#pragma unroll
            for (int v = 0; v < 2; ++v) load_vector<XT>(a, vector_at(it, v, valid[v]), H, xb[v]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (SPLIT && item < a.n_items) load_item(item); /* under way while S is staged (whole tiles would hold S up: 46.6 against 42.6 us) */
    {
        uint4 stage[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) stage[i] = a.S_bf16x3[tid + i * kFitThreads];
#pragma unroll
        for (int i = 0; i < 4; ++i) sS[tid + i * kFitThreads] = stage[i];
    }
    for (int c = tid; c < kHistSize + kHistUpper; c += kFitThreads) sh[c] = 0u;
    __syncthreads();

    while (item < a.n_items) {
        if constexpr (SPLIT) {
            const f32x16 acc = rotate_block<XT>(sS, my_rt, xb[0], lane);
            if (valid[0]) count_block(acc, sh);
        } else {
            load_item(item);
            float rb[2][4]; /* radii of blocks 4H .. 4H+3 of this lane's two vectors */
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                if (XT != PQ_BF16) load_vector<XT>(a, vector_at(item, v, valid[v]), H, xb[0]);
#pragma unroll
                for (int rt = 0; rt < 4; ++rt) {
                    const f32x16 acc = rotate_block<XT>(sS, rt, xb[XT == PQ_BF16 ? v : 0], lane);
                    rb[v][rt] = valid[v] ? count_block(acc, sh) : 0.f;
                }
            }
            if (a.hist_up) {
                /* levels 5 and 6 inside the lane (blocks 4H .. 4H+3), level 7 joins the two lane halves */
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const float r50 = fit_radius(rb[v][0], rb[v][1]), r51 = fit_radius(rb[v][2], rb[v][3]);
                    const float r6 = fit_radius(r50, r51);
                    const float other = __shfl_xor(r6, 32);
                    if (valid[v]) {
                        uint32_t *up = sh + kHistSize;
                        count_upper(up, rb[v][0], rb[v][1]);
                        count_upper(up, rb[v][2], rb[v][3]);
                        count_upper(up + kBinsU, r50, r51);
                        if (H == 0) count_upper(up + 2 * kBinsU, r6, other);
                    }
                }
            }
        }
        item += stride;
        if (SPLIT && item < a.n_items) load_item(item);
    }
    __syncthreads();
    add_counts(a.hist, sh, kHistSize);
    if (a.hist_up) add_counts(a.hist_up, sh + kHistSize, kHistUpper);
}

/* angle of the lower edge of bin b of a level's histogram (b = bins gives the upper end of the range) */
double bin_edge(int b, int bins, bool level1)
{
    const double half_pi = 1.57079632679489661923132169163975144;
    const int per = level1 ? bins / 4 : bins; /* bins per quarter turn */
    const int q = b / per, k = b % per;
    return q * half_pi + atan2((double)k, (double)(per - k));
}

/* the bins of a level: their edges, ascending, and the middle of each in units of 2^-60 rad; formed once per process */
struct Bins {
    std::vector<double> edge;
    std::vector<uint64_t> middle;
};

const Bins &bins_of(bool level1)
{
    auto make = [](int bins, bool first) {
        Bins e;
        for (int b = 0; b <= bins; ++b) e.edge.push_back(bin_edge(b, bins, first));
        for (int b = 0; b < bins; ++b) e.middle.push_back((uint64_t)ldexp(0.5 * (e.edge[b] + e.edge[b + 1]), 60));
        return e;
    };
    static const Bins first = make(kBins1, true), upper = make(kBinsU, false);
    return level1 ? first : upper;
}

/* k-means rounds on one level's histogram.  The angles of a bin are taken as spread evenly over
   it: a bin that a cell boundary (midpoint of two centroids) cuts gives each side its share of
   the count, centred on its part of the bin; an uncut bin stands for its centre.  Nearest
   centroid by linear distance (procedure Quant); a centroid whose cell is empty stays.
   A cell is its part of its first bin, the whole bins behind it and its part of its last bin.  The parts are formed by
   themselves; the whole bins come from running sums of counts and of counts times middles, which are integers (below 2^45 and
   2^108), so that their differences are exact: a cell of a sliver of one bin keeps its centroid next to any count elsewhere.
   (Running sums make a round a few lookups; walking over all bins in every round, and forming the edges in every call,
   took 430 us for ten rounds on the four histograms of 262144 vectors; pq_fit_codebooks as a whole 565 -> 115 us.  A round takes
   some 0.4 us.) */
constexpr int kRunBins = 8;

struct BinSum { /* of the bins below kRunBins r of a level */
    uint64_t lo;
    uint32_t hi, count; /* moment, 2^64 hi + lo: below 2^96, and a level's angles fit 32 bits, where the device counted */
};

typedef unsigned __int128 wide;

struct Sum {
    uint64_t count;
    wide moment;
};

/* run(r): the sum below bin kRunBins r */
template <class Run>
void lloyd_rounds(const uint32_t *hist, int bins, bool level1, int K, int iterations, double *c, const Run &run)
{
    const std::vector<double> &edge = bins_of(level1).edge;
    const std::vector<uint64_t> &middle = bins_of(level1).middle;
    auto below = [&](int b) {
        Sum s = run(b / kRunBins);
        for (int i = b / kRunBins * kRunBins; i < b; ++i) {
            s.count += hist[i];
            s.moment += (wide)middle[i] * hist[i];
        }
        return s;
    };
    auto bin_at = [&](double x) { return (int)(std::upper_bound(edge.begin(), edge.end(), x) - edge.begin()) - 1; };
    for (int it = 0; it < iterations; ++it) {
        double next[16], from = edge[0];
        int first = 0; /* the bin that `from` lies in */
        for (int k = 0; k < K; ++k) {
            const double cut = k + 1 < K ? 0.5 * (c[k] + c[k + 1]) : edge[bins];
            const double to = cut < edge[bins] ? cut : edge[bins];
            next[k] = c[k];
            if (!(to > from)) continue; /* the cell lies outside the range */
            const int last = bin_at(to);
            double mass = 0.0, sum = 0.0;
            auto add = [&](int b, double lo, double hi) {
                const double m = (double)hist[b] * ((hi - lo) / (edge[b + 1] - edge[b]));
                mass += m;
                sum += m * (0.5 * (lo + hi));
            };
            if (first == last) {
                add(first, from, to);
            } else {
                add(first, from, edge[first + 1]);
                const Sum hi = below(last), lo = below(first + 1);
                mass += (double)(hi.count - lo.count);
                sum += (double)(hi.moment - lo.moment) * 0x1p-60;
                if (last < bins) add(last, edge[last], to);
            }
            if (mass > 0.0) next[k] = std::min(std::max(sum / mass, from), to);
            from = to;
            first = last;
        }
        for (int k = 0; k < K; ++k) c[k] = next[k];
    }
}

/* the running sums of a histogram in host memory, and the rounds */
void lloyd_on_histogram(const uint32_t *hist, int bins, bool level1, int K, int iterations, double *c)
{
    const std::vector<uint64_t> &middle = bins_of(level1).middle;
    std::vector<Sum> sums((size_t)bins / kRunBins + 1);
    Sum all{0, 0};
    for (int b = 0; b < bins; ++b) {
        if (b % kRunBins == 0) sums[b / kRunBins] = all;
        all.count += hist[b];
        all.moment += (wide)middle[b] * hist[b];
    }
    sums[bins / kRunBins] = all;
    lloyd_rounds(hist, bins, level1, K, iterations, c, [&](int r) { return sums[r]; });
}

} // namespace

extern "C" size_t pq_fit_workspace_bytes(void) { return (size_t)(kHistSize + kHistUpper) * sizeof(uint32_t); }

namespace {

/* clears the histograms with a kernel of the library's own: a memset node would not survive graph capture */
__global__ __launch_bounds__(256) void pq_fit_clear_kernel(uint32_t *hist, int n)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) hist[i] = 0u;
}

/* Tiles up to which eight wavefronts share one (bf16, us with and without: 8000 vectors 13.4 / 20.0, 64000 26.5 / 28.5, 96000 28.7 /
   31.6, 131072 34.1 / 32.1; fp32 rows, split by every wavefront of a tile, leave no gain from 32000 vectors on: 33.8 / 29.6). */
constexpr int64_t kSplitItems = 1536;
pq_status check_start(const pq_ctx *ctx, const double *cb_init, const double *cbt_init, bool upper, double (&c)[28],
                      double (&ct)[3][8])
{
    if (cb_init) {
        memcpy(c, cb_init, sizeof(c));
    } else {
        for (int k = 0; k < 16; ++k) c[k] = ctx->centroids[0][k];
        for (int l = 1; l < 4; ++l)
            for (int k = 0; k < 4; ++k) c[16 + 4 * (l - 1) + k] = ctx->centroids[l][k];
    }
    const int off[4] = {0, 16, 20, 24}, K[4] = {16, 4, 4, 4};
    for (int l = 0; l < 4; ++l)
        for (int k = 0; k < K[l]; ++k) {
            if (!std::isfinite(c[off[l] + k])) return PQ_EINVAL;
            if (k > 0 && !(c[off[l] + k] > c[off[l] + k - 1])) return PQ_EINVAL;
        }
    if (upper) {
        for (int l = 0; l < 3; ++l) {
            const int Kl = 1 << ctx->upper_bits[l];
            for (int k = 0; k < 8; ++k) ct[l][k] = cbt_init ? cbt_init[8 * l + k] : (k < Kl ? ctx->upper_centroids[l][k] : 0.0);
            for (int k = 0; k < Kl; ++k) {
                if (!std::isfinite(ct[l][k])) return PQ_EINVAL;
                if (k > 0 && !(ct[l][k] > ct[l][k - 1])) return PQ_EINVAL;
            }
        }
    }
    return PQ_OK;
}

pq_status check_count(const pq_ctx *ctx, const void *x, pq_dtype xt, int64_t n_tokens, int n_heads, int64_t ld_token, int64_t ld_head,
                      const void *workspace, size_t workspace_bytes)
{
    if (!ctx || !x || !workspace) return PQ_EINVAL;
    if (xt != PQ_F32 && xt != PQ_BF16) return PQ_EINVAL;
    if (n_tokens <= 0 || n_heads <= 0 || ld_token < 0 || ld_head < 0) return PQ_EINVAL;
    if (workspace_bytes < pq_fit_workspace_bytes()) return PQ_ENOMEM;
    const int64_t elems16 = xt == PQ_BF16 ? 8 : 4;
    if (!pq_aligned16(workspace) || !pq_aligned16(x) || (ld_token % elems16) || (ld_head % elems16)) return PQ_EALIGN;
    /* every bin counter must hold the angles of a level: 64 per vector at level 1 */
    if ((double)n_tokens * n_heads * 64.0 >= 4294967295.0) return PQ_EUNSUPPORTED;
    return PQ_OK;
}

} // namespace

extern "C" pq_status pq_fit_count_angles(const pq_ctx *ctx, const void *x, pq_dtype xt, int64_t n_tokens, int n_heads,
                                         int64_t ld_token, int64_t ld_head, void *workspace, size_t workspace_bytes,
                                         void *hip_stream)
{
    const pq_status args = check_count(ctx, x, xt, n_tokens, n_heads, ld_token, ld_head, workspace, workspace_bytes);
    if (args != PQ_OK) return args;
    const bool upper = ctx->depth == 7;
    const PqDeviceState *ds = nullptr;
    pq_status st = pq_device_state(ctx, &ds);
    if (st != PQ_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    uint32_t *hist = static_cast<uint32_t *>(workspace);
    hipLaunchKernelGGL(pq_fit_clear_kernel, dim3(16), dim3(256), 0, s, hist, kHistSize + kHistUpper);
    FitArgs a{};
    a.x = x; a.ld_token = ld_token; a.ld_head = ld_head; a.n_tokens = n_tokens; a.n_heads = n_heads;
    a.tiles_per_head = (n_tokens + kTileVecs - 1) / kTileVecs;
    a.n_items = a.tiles_per_head * n_heads;
    a.S_bf16x3 = reinterpret_cast<const uint4 *>(ds->S_bf16x3);
    a.hist = hist;
    a.hist_up = upper ? hist + kHistSize : nullptr;
    const bool split = !upper && xt == PQ_BF16 && a.n_items <= kSplitItems;
    /* every workgroup adds its counters to the call's: no more of them than keep each SIMD of the used CUs at work (16000 bf16
       vectors 21.2 us with a workgroup per tile, 17.0 per two; 32000 24.3 on 256 CUs, 19.5 on 128; 16000 fp32 vectors 29.4 with a
       workgroup per tile, 20.5 per four) */
    int64_t blocks = split ? (a.n_items + 1) / 2 : (a.n_items + 3) / 4;
    const int64_t most = split && a.n_items <= 512 ? 128 : 256;
    if (blocks > most) blocks = most;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kFitThreads), 0, s, a); };
    if (xt == PQ_BF16) split ? launch(pq_angle_histogram_kernel<PQ_BF16, true>) : launch(pq_angle_histogram_kernel<PQ_BF16, false>);
    else launch(pq_angle_histogram_kernel<PQ_F32, false>);
    PQ_HIP_TRY(hipGetLastError());
    return PQ_OK;
}

extern "C" pq_status pq_fit_cluster(const pq_ctx *ctx, const uint32_t *hist, const double *cb_init, const double *cbt_init,
                                    int iterations, double *cb_out, double *cbt_out)
{
    if (!ctx || !hist || !cb_out || iterations < 0) return PQ_EINVAL;
    const bool upper = ctx->depth == 7;
    if (upper && !cbt_out) return PQ_EINVAL;
    double c[28], ct[3][8] = {};
    const pq_status st = check_start(ctx, cb_init, cbt_init, upper, c, ct);
    if (st != PQ_OK) return st;
    const int off[4] = {0, 16, 20, 24};
    lloyd_on_histogram(hist, kBins1, true, 16, iterations, c);
    for (int l = 1; l < 4; ++l)
        lloyd_on_histogram(hist + kBins1 + (l - 1) * kBinsU, kBinsU, false, 4, iterations, c + off[l]);
    memcpy(cb_out, c, sizeof(c));
    if (upper) {
        for (int l = 0; l < 3; ++l)
            lloyd_on_histogram(hist + kHistSize + l * kBinsU, kBinsU, false, 1 << ctx->upper_bits[l], iterations, ct[l]);
        memcpy(cbt_out, ct, sizeof(ct));
    }
    return PQ_OK;
}

namespace {

/* ---- what the rounds look at, brought to the host by a kernel: the counts and their running sums ----
 * One workgroup per level: a thread takes eight bins, a scan over the workgroup gives the sums below them, and both go
 * straight to host memory that the device writes to: 5.5 us, where a copy of the counts to pageable memory took 12 us beyond
 * the wait and forming the sums on the host some 7.  262144 bf16 vectors, ten rounds: 81.5 -> 73.6 us for the call, 8000 vectors
 * 56 -> 48.  (The rounds themselves are a chain of divisions and lookups for 28 numbers: 22 us as a kernel for ten of them, some 4 on
 * the host.) */
constexpr int kLevels = 7, kSumThreads = 1024;

struct FitResult { /* in host memory */
    uint32_t hist[kHistSize + kHistUpper]; /* as in the workspace */
    BinSum run1[kBins1 / kRunBins + 1], run_upper[kLevels - 1][kBinsU / kRunBins + 1];
};

__device__ __forceinline__ void bin_add(BinSum &s, const BinSum &t)
{
    s.count += t.count;
    s.lo += t.lo;
    s.hi += t.hi + (s.lo < t.lo ? 1u : 0u);
}

__global__ __launch_bounds__(kSumThreads) void pq_fit_sums_kernel(const uint32_t *hist, const uint64_t *middles, FitResult *out)
{
    static_assert(kBins1 == kRunBins * kSumThreads && kRunBins == 8, "a thread takes one run of bins, two 16-byte loads");
    __shared__ BinSum wave_sum[kSumThreads / 64];
    const int level = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int runs = (level == 0 ? kBins1 : kBinsU) / kRunBins, first = level == 0 ? 0 : kBins1 + (level - 1) * kBinsU;
    BinSum mine{0, 0, 0};
    if (tid < runs) {
        const uint64_t *m = middles + (level == 0 ? 0 : kBins1) + kRunBins * tid;
        const uint4 a = *reinterpret_cast<const uint4 *>(hist + first + kRunBins * tid);
        const uint4 b = *reinterpret_cast<const uint4 *>(hist + first + kRunBins * tid + 4);
        const uint32_t n[kRunBins] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < kRunBins; ++i) bin_add(mine, BinSum{m[i] * n[i], (uint32_t)__umul64hi(m[i], n[i]), n[i]});
        *reinterpret_cast<uint4 *>(out->hist + first + kRunBins * tid) = a;
        *reinterpret_cast<uint4 *>(out->hist + first + kRunBins * tid + 4) = b;
    }
    BinSum upto = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        BinSum t;
        t.lo = __shfl_up((unsigned long long)upto.lo, d);
        t.hi = __shfl_up(upto.hi, d);
        t.count = __shfl_up(upto.count, d);
        if (lane >= d) bin_add(upto, t);
    }
    if (lane == 63) wave_sum[wave] = upto;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSumThreads / 64 - 1; ++w) {
        const BinSum t = wave_sum[w];
        if (w < wave) bin_add(upto, t);
    }
    BinSum *run = level == 0 ? out->run1 : out->run_upper[level - 1];
    if (tid < runs) run[tid + 1] = upto; /* up to and with this thread: below the next one's bins */
    if (tid == 0) run[0] = BinSum{0, 0, 0};
}

/* the middles of the bins on every device, level 1 and then the others, uploaded by the first call there */
__device__ uint64_t g_middles[kBins1 + kBinsU];

pq_status device_middles(const uint64_t **out)
{
    static std::mutex mu;
    static bool ready[PQ_MAX_DEVICES];
    int dev = -1;
    PQ_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= PQ_MAX_DEVICES) return PQ_EUNSUPPORTED;
    void *at = nullptr;
    PQ_HIP_TRY(hipGetSymbolAddress(&at, HIP_SYMBOL(g_middles)));
    std::lock_guard<std::mutex> lock(mu);
    if (!ready[dev]) {
        const std::vector<uint64_t> &first = bins_of(true).middle, &upper = bins_of(false).middle;
        PQ_HIP_TRY(hipMemcpy(at, first.data(), first.size() * sizeof(uint64_t), hipMemcpyHostToDevice));
        PQ_HIP_TRY(hipMemcpy(static_cast<uint64_t *>(at) + kBins1, upper.data(), upper.size() * sizeof(uint64_t), hipMemcpyHostToDevice));
        ready[dev] = true;
    }
    *out = static_cast<const uint64_t *>(at);
    return PQ_OK;
}

/* Host memory for a FitResult: one block per call under way, kept for the next call (four of 130 KB at most; more callers at a
   time allocate and free their own). */
class ResultBlock {
  public:
    ResultBlock()
    {
        {
            std::lock_guard<std::mutex> lock(pool().mu);
            if (pool().n > 0) p_ = pool().kept[--pool().n];
        }
        if (!p_ && hipHostMalloc(reinterpret_cast<void **>(&p_), sizeof(FitResult), hipHostMallocPortable) != hipSuccess) p_ = nullptr;
    }
    ~ResultBlock()
    {
        if (!p_) return;
        {
            std::lock_guard<std::mutex> lock(pool().mu);
            if (pool().n < kKept) {
                pool().kept[pool().n++] = p_;
                return;
            }
        }
        (void)hipHostFree(p_);
    }
    ResultBlock(const ResultBlock &) = delete;
    ResultBlock &operator=(const ResultBlock &) = delete;
    FitResult *get() const { return p_; }

  private:
    static constexpr int kKept = 4;
    struct Pool { /* what is kept goes with the process */
        std::mutex mu;
        FitResult *kept[kKept];
        int n = 0;
    };
    static Pool &pool()
    {
        static Pool p;
        return p;
    }
    FitResult *p_ = nullptr;
};

/* counting, sums, a wait for the stream, the rounds */
pq_status fit_codebooks(const pq_ctx *ctx, const void *x, pq_dtype xt, int64_t n_tokens, int n_heads,
                        int64_t ld_token, int64_t ld_head, const double *cb_init, const double *cbt_init, bool upper,
                        int iterations, double *cb_out, double *cbt_out, void *workspace, size_t workspace_bytes,
                        void *hip_stream)
{
    if (!ctx || !cb_out || (upper && !cbt_out) || iterations < 0) return PQ_EINVAL;
    if (upper && ctx->depth != 7) return PQ_EINVAL;
    double c[28], ct[3][8] = {};
    pq_status st = check_start(ctx, cb_init, cbt_init, upper, c, ct);
    if (st != PQ_OK) return st;
    st = check_count(ctx, x, xt, n_tokens, n_heads, ld_token, ld_head, workspace, workspace_bytes);
    if (st != PQ_OK) return st;
    /* Everything that can be refused is, before the first launch: a capturing stream, which has no results to wait for, would
       otherwise keep the launches in its graph, and every replay would write to the workspace. */
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) == hipSuccess && capture != hipStreamCaptureStatusNone) return PQ_EHIP;
    const uint64_t *middles = nullptr;
    st = device_middles(&middles);
    if (st != PQ_OK) return st;
    ResultBlock result;
    FitResult *r = result.get();
    if (!r) return PQ_ENOMEM;
    st = pq_fit_count_angles(ctx, x, xt, n_tokens, n_heads, ld_token, ld_head, workspace, workspace_bytes, hip_stream);
    if (st != PQ_OK) return st;
    hipLaunchKernelGGL(pq_fit_sums_kernel, dim3(upper ? kLevels : 4), dim3(kSumThreads), 0, s, static_cast<const uint32_t *>(workspace),
                       middles, r);
    PQ_HIP_TRY(hipGetLastError());
    PQ_HIP_TRY(hipStreamSynchronize(s));
    auto rounds = [&](int level, int K, double *centroids) {
        const BinSum *run = level == 0 ? r->run1 : r->run_upper[level - 1];
        lloyd_rounds(r->hist + (level == 0 ? 0 : kBins1 + (level - 1) * kBinsU), level == 0 ? kBins1 : kBinsU, level == 0, K, iterations,
                     centroids, [&](int i) { return Sum{run[i].count, (wide)run[i].hi << 64 | run[i].lo}; });
    };
    rounds(0, 16, c);
    for (int l = 1; l < 4; ++l) rounds(l, 4, c + 12 + 4 * l);
    memcpy(cb_out, c, sizeof(c));
    if (upper) {
        for (int l = 0; l < 3; ++l) rounds(4 + l, 1 << ctx->upper_bits[l], ct[l]);
        memcpy(cbt_out, ct, sizeof(ct));
    }
    return PQ_OK;
}

} // namespace

extern "C" pq_status pq_fit_codebooks(const pq_ctx *ctx, const void *x, pq_dtype xt, int64_t n_tokens, int n_heads,
                                      int64_t ld_token, int64_t ld_head, const double *cb_init, int iterations,
                                      double *cb_out, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return fit_codebooks(ctx, x, xt, n_tokens, n_heads, ld_token, ld_head, cb_init, nullptr, false, iterations, cb_out,
                         nullptr, workspace, workspace_bytes, hip_stream);
}

extern "C" pq_status pq_fit_codebooks_deep(const pq_ctx *ctx, const void *x, pq_dtype xt, int64_t n_tokens, int n_heads,
                                           int64_t ld_token, int64_t ld_head, const double *cb_init,
                                           const double *cbt_init, int iterations, double *cb_out, double *cbt_out,
                                           void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return fit_codebooks(ctx, x, xt, n_tokens, n_heads, ld_token, ld_head, cb_init, cbt_init, true, iterations, cb_out,
                         cbt_out, workspace, workspace_bytes, hip_stream);
}
