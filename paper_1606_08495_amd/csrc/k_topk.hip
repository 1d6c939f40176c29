// Retrieval by cosine similarity (Section 2; Section 7.3: K = 30, threshold tau): for every query
// vector the K most similar candidate vectors.
//
// Candidates are taken in rounds, in index order.  A round's scores are screened: every (query,
// candidate) pair that may beat the query's current K-th best is put on the query's pending list, and
// topk_fold_kernel gives each listed pair its similarity in fp32, folds those that do beat the K-th
// best into the sorted best list and raises the threshold.  The similarity of a pair is
// fl(fl(dot * 1/|q|) * 1/|c|) with dot one fused-multiply-add chain over the columns in order -- whoever
// forms it, so results depend neither on the round length nor on which screen listed the pair.
//
// The screen need not be exact, only never miss: two of the three work in 16 bits on the matrix cores,
// sixteen times the rate of fp32 there, with a margin that covers their error for certain (below):
//   wide    (many queries): a round's candidates are normalised and rounded to fp16 once, in the order in
//           which the matrix cores take them, and multiplied tile by tile.
//   stream  (few): bound by reading the candidates; a wavefront reads 32 of them once, rounds them
//           to bf16 in registers (no scale is known yet; bf16 has fp32's range), and forms norms,
//           rounding errors and products with all queries on the way.
//   fp32    exact scores from the fp32 matrix cores: where the workspace is too small for the rounded
//           queries, in the first rounds of a wide search, and in blocks whose similarities are crowded.
//
// Margin.  Let a = q/|q|, b = c/|c| in fp32 and a', b' their rounded forms.  |a.b - a'.b'| <=
// |a - a'| |b| + |a'| |b - b'|, and the norms of the two rounding errors are computed per row
// (about 2e-4 for fp16, 9e-4 for bf16: a tenth of the distance to the K-th best that a crowded list
// has).  What fp32 arithmetic adds on either side (products summed in any order, norms, the two
// scalings) is at most a few d 2^-24; topk_rounding(d) below holds twice that.  Rows whose squared length
// is too small to be precise are always listed.
#include "common.h"

#include <algorithm>
#include <math.h>
#include <type_traits>

namespace w2v {

static inline unsigned blocks_for(uint64_t items, unsigned per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));

constexpr int TK_BQ = 128;          // fp32 screen: queries per block tile (2 x 2 wavefronts x 2 x 2 tiles of 32)
constexpr int TK_BC = 128;          // candidates per block tile; granularity of a round
constexpr int TK_BK = 16;           // columns per panel; two panels are held in LDS
constexpr int TK_LD = TK_BK + 1;    // LDS row pitch (odd: conflict-free column reads)
constexpr int TK_THREADS = 256;     // four wavefronts
constexpr int TK_LIST = 64;         // slots of a query's best list (K <= 64)
constexpr uint32_t TK_NONE = 0xFFFFFFFFu;
constexpr uint32_t TK_STREAM_Q = 128;     // queries of the stream screen's tile, at most
constexpr int TK_KS = 16;                 // columns of one 16-bit matrix-core step
constexpr float TK_F16_SCALE = 256.f;     // fp16 rows are stored times this: components below 2.4e-7 of the
                                          // row's length (fp16 subnormals) are taken as zero
constexpr float TK_TINY = 1e-30f;         // squared lengths below this are not precise
// Crowded similarities.  Where more candidates lie within the margin than a round lists in earnest, listing
// them (a row read each in the fold) costs far more than forming all similarities in fp32 at once.  So a block
// that finds more hits than twice what the thresholds let pass plus TK_DENSE_* drops them and does that
// (exact_block) -- all but the first TK_SPARE, for one block alone takes longer that way; and once half of
// the blocks so far have, the rounds that follow do not screen.
// Vectors around one direction, noise 0.03 of the components, K = 30; us, in brackets with every pair in fp32:
// 4096 queries over 200 000 x 300 4760 [4550], 300 1070 [880], 100 530 [700], 7 480 [485]; with hits of a
// tile of 32 x 32 above 128 re-formed by its own wavefront, as it was, 13 200, 1970, 14 600, 390.  Rows of 100 columns,
// whose next round is rounded beside the products: 4096 queries 2055, 1000 739, 300 504; where a round that does not
// screen is left out of the count, so that the next one screens again, 2175, 790, 549.  What the
// count costs where nothing is crowded: a barrier per block, 2 % at most (300 queries over 200 000 x 16).
// (TK_DENSE_WIDE 256, 1024, 2048 on the first at noise 0.1: 3.90, 3.91, 5.05 ms against 3.74.
// TK_DENSE_STREAM 8, 16: 10 queries over 100 000 x 300, noise 0.3, 303 and 483 us against 302.
// TK_SPARE 0, 16, 32: 1 query over 200 000 x 100, no crowd, 140, 126, 127 us, noise 0.03 187, 208, 259.)
constexpr uint32_t TK_DENSE_WIDE = 512;           // of 256 queries x 128 candidates
constexpr uint32_t TK_DENSE_STREAM = 4;           // per query (64 at most), of 128 candidates
constexpr uint32_t TK_SPARE = 8;
constexpr double TK_EXACT_ROUND = 100000;         // pairs
// Queries of one launch of the fold, query tiles of one launch of the stream screen, candidates of one
// launch: a grid holds less than 2^32 threads in x (past that the runtime wraps it without an error) and
// 2^16 blocks in y, so very long lists are served in slices.
constexpr uint32_t TK_FOLD_SLICE = 1u << 21;
constexpr uint32_t TK_STREAM_SLICE = 1u << 15;
constexpr uint32_t TK_CAND_SLICE = 1u << 30;

__host__ __device__ inline uint32_t topk_steps(uint32_t d) { return 2 * ((d + 2 * TK_KS - 1) / (2 * TK_KS)); }   // even
__device__ __forceinline__ float topk_rounding(uint32_t d) { return (float)(d + 64) * 0x1p-22f; }

template <bool VEC4>
__device__ __forceinline__ float4 load_cols(const float* __restrict__ row, bool row_ok, uint32_t k,
                                            uint32_t d) {
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!row_ok) return r;
    if (VEC4) {
        if (k < d) r = *(const float4*)(row + k);            // d % 4 == 0: all four inside
    } else {
        if (k + 0 < d) r.x = row[k + 0];
        if (k + 1 < d) r.y = row[k + 1];
        if (k + 2 < d) r.z = row[k + 2];
        if (k + 3 < d) r.w = row[k + 3];
    }
    return r;
}

// The same from a row that may be read, and without a branch: what lies past the last column is read elsewhere in the
// row.  (Loads behind branches cannot be counted, so that each wait is for all of them.)
template <bool VEC4>
__device__ __forceinline__ float4 load_cols_flat(const float* __restrict__ row, uint32_t k, uint32_t d) {
    float4 r;
    if (VEC4) {
        r = *(const float4*)(row + (k < d ? k : 0u));
    } else {
        r.x = row[k + 0 < d ? k + 0 : 0u]; r.y = row[k + 1 < d ? k + 1 : 0u];
        r.z = row[k + 2 < d ? k + 2 : 0u]; r.w = row[k + 3 < d ? k + 3 : 0u];
    }
    return r;
}
template <bool VEC4>
__device__ __forceinline__ float4 cols_inside(float4 r, uint32_t k, uint32_t d) {
    if (k + 0 >= d) r.x = 0.f;
    if (k + (VEC4 ? 0 : 1) >= d) r.y = 0.f;
    if (k + (VEC4 ? 0 : 2) >= d) r.z = 0.f;
    if (k + (VEC4 ? 0 : 3) >= d) r.w = 0.f;
    return r;
}

// Squared length of a row: sixteen chains by column number mod 16, then a fixed tree -- the same bits
// from one lane that walks the whole row and from two lanes that take alternate groups of eight.
__device__ __forceinline__ void square8(const float4& a, const float4& b, float (&s)[8]) {
    s[0] = fmaf(a.x, a.x, s[0]); s[1] = fmaf(a.y, a.y, s[1]); s[2] = fmaf(a.z, a.z, s[2]); s[3] = fmaf(a.w, a.w, s[3]);
    s[4] = fmaf(b.x, b.x, s[4]); s[5] = fmaf(b.y, b.y, s[5]); s[6] = fmaf(b.z, b.z, s[6]); s[7] = fmaf(b.w, b.w, s[7]);
}
__device__ __forceinline__ float tree8(const float (&s)[8]) {
    return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}
__device__ __forceinline__ float inv_length(float square) { return square > 0.f ? 1.0f / sqrtf(square) : 0.f; }

// The same of row `row` by a lane pair (l, l ^ 32): the half fk takes columns 16 i + 8 fk + 0..7.
template <bool VEC4>
__device__ __forceinline__ float pair_square(const float* __restrict__ row, bool ok, uint32_t d, int fk) {
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (uint32_t k = 8 * fk; k < d + 8 * fk; k += TK_KS)
        square8(load_cols<VEC4>(row, ok, k, d), load_cols<VEC4>(row, ok, k + 4, d), s);
    const float own = tree8(s);
    return own + __shfl_xor(own, 32, 64);
}

struct TopkArgs {
    const float* Qm; const float* Cm; uint32_t Q, N, d;
    uint32_t c_begin, c_end;            // candidates of this round
    uint32_t nq_tiles, nc_tiles;
    uint32_t q_first;                   // first query (fold) or query tile (stream) of this launch
    const float* invq; const float* invc; const float* theta;
    uint32_t* cnt; uint32_t* pend; uint32_t cap;
    uint32_t* bits; uint32_t pitch;              // stream: a bit per candidate of the round, `pitch` words per query
    uint64_t* parts;                             // fold: best lists of the blocks that share a query
    uint32_t* err;
    // 16-bit screens
    const void* qfrag; const float* qmargin;     // rounded queries, and what to lower their thresholds by
    const void* cfrag; const float* cmargin;     // wide: the round's rounded candidates and their margins
    // a block with more hits than dense_limit (TK_NONE: none has) is counted in *dense and, past the first
    // TK_SPARE, forms its similarities in fp32.  A block that finds dense_skip (TK_NONE: never) or more
    // counted does not screen; the first of a round's `blocks` then counts them all, so that they stay so
    uint32_t dense_limit, dense_skip, blocks;
    uint32_t* dense;
};

// A row's normalised form, rounded, in matrix-core order: tile of 32 rows, step of 16 columns, lane
// (row, half) its eight columns; and the norm of what rounding took away.  One wavefront per tile.
// HOLD > 0: rows of up to HOLD steps stay in registers, every load in flight at once, between the norm
// and the rounding; else they are read twice.
// Held against read twice, whole search in us: 300 queries over 200 000 x 320 504, 549, x 300 491, 540, x 128
// 317, 329, x 64 279, 279, x 16 229, 221 (twenty steps whatever the row holds): rows of 65 to 320 columns.
constexpr int TK_HOLD = 20, TK_HOLD_LEAST = 5;                // steps
// Candidates are rounded beside the products of the round before, in the registers that leaves, hence read twice, except
// where rows are long and could be held.  Rounding apart and beside, whole search in us: 150 queries over 40 000 x 100
// 172, 152, 500 over 300 000 x 31 332, 300, 1000 over 400 000 x 100 568, 534, 700 over 3000 x 200 141, 136, 2000 over
// 500 000 x 512 2338, 2267; but 300 over 100 000 x 300 342, 344, 4096 over 2^20 x 300 4531, 4602.
constexpr uint32_t TK_BESIDE = 14;                            // steps, or more than TK_HOLD
template <bool F16>
__device__ __forceinline__ void round_step(const float4& x, const float4& y, float inv, bool on, void* __restrict__ frag,
                                           uint64_t at, float& e2) {
    const float scale = F16 ? TK_F16_SCALE : 1.f;
    const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    v8h h; v8b g;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float t = on ? (v[e] * inv) * scale : 0.f;      // (times a power of two: exact)
        float back;
        if (F16) { h[e] = (_Float16)(fabsf(t) < 6.2e-5f ? 0.f : t); back = (float)h[e]; }
        else { g[e] = (__bf16)t; back = (float)g[e]; }
        e2 = fmaf(t - back, t - back, e2);
    }
    if (F16) ((v8h*)frag)[at] = h; else ((v8b*)frag)[at] = g;
}

template <bool F16, bool VEC4, int HOLD>
__device__ __forceinline__ void round_rows(const float* __restrict__ M, uint32_t row, bool ok, uint32_t d,
                                           uint32_t steps, void* __restrict__ frag, uint32_t tile, int lane,
                                           float& square, float& inv, float& lost) {
    const int fk = lane >> 5;
    const float* p = M + (uint64_t)(ok ? row : 0u) * d;
    const uint64_t at = (uint64_t)tile * steps * 64 + lane;
    float e2 = 0.f;
    if constexpr (HOLD > 0) {
        float4 x[HOLD], y[HOLD];
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < HOLD; ++i) {
            x[i] = load_cols<VEC4>(p, ok, i * TK_KS + 8 * fk, d);
            y[i] = load_cols<VEC4>(p, ok, i * TK_KS + 8 * fk + 4, d);
        }
#pragma unroll
        for (int i = 0; i < HOLD; ++i) square8(x[i], y[i], s);       // (zeros past d leave the sums alone)
        const float own = tree8(s);
        square = own + __shfl_xor(own, 32, 64);
        inv = inv_length(square);
        const bool on = square >= TK_TINY && inv > 0.f;       // else the rounded row is zero
#pragma unroll
        for (int i = 0; i < HOLD; ++i)
            if ((uint32_t)i < steps) round_step<F16>(x[i], y[i], inv, on, frag, at + (uint64_t)i * 64, e2);
    } else {
        square = pair_square<VEC4>(p, ok, d, fk);
        inv = inv_length(square);
        const bool on = square >= TK_TINY && inv > 0.f;
#pragma unroll 4
        for (uint32_t i = 0; i < steps; ++i) {               // (of a panel of four the loads are in flight together)
            const uint32_t k = i * TK_KS + 8 * fk;
            round_step<F16>(load_cols<VEC4>(p, ok, k, d), load_cols<VEC4>(p, ok, k + 4, d), inv, on, frag,
                            at + (uint64_t)i * 64, e2);
        }
    }
    e2 += __shfl_xor(e2, 32, 64);
    lost = sqrtf(e2) / (F16 ? TK_F16_SCALE : 1.f) * 1.004f;
    if (square > 0.f && square < TK_TINY) lost = INFINITY;     // always listed
}

// Queries: 1/|q|, rounded rows, margins; the state of an empty search.  Margin < 0: a query without
// length (every similarity is 0).
template <bool F16, bool VEC4>
__global__ __launch_bounds__(64) void topk_queries_kernel(const float* __restrict__ Qm, uint32_t Q, uint32_t d,
                                                          float theta0, float* __restrict__ invq,
                                                          float* __restrict__ theta, uint32_t* __restrict__ cnt,
                                                          uint32_t* __restrict__ best_cnt, void* __restrict__ frag,
                                                          float* __restrict__ margin, uint32_t* __restrict__ err) {
    const int lane = threadIdx.x;
    const uint32_t q = blockIdx.x * 32u + (lane & 31);
    float square, inv, lost;
    if (frag) {
        round_rows<F16, VEC4, 0>(Qm, q, q < Q, d, topk_steps(d), frag, blockIdx.x, lane, square, inv, lost);
        if (lane < 32) margin[q] = inv > 0.f ? lost + topk_rounding(d) : -1.f;
    } else {
        square = pair_square<VEC4>(Qm + (uint64_t)(q < Q ? q : 0u) * d, q < Q, d, lane >> 5);
        inv = inv_length(square);
    }
    if (lane < 32 && q < Q) { invq[q] = inv; theta[q] = theta0; cnt[q] = 0u; best_cnt[q] = 0u; }
    if (blockIdx.x == 0 && lane < 2) err[lane] = 0u;           // (err[1]: TopkArgs::dense)
}

// The wide screen's candidates of one round (rows c_end .. the end of the last tile are zero and have
// a margin that no threshold meets).  Bound by memory: 4 d bytes read (a second time, for the rounding,
// out of the caches) and 2 d written per row.
struct RoundArgs { const float* Cm; uint32_t c_begin, c_end, d, tiles; float* invc; void* frag; float* margin; };
template <bool VEC4, int HOLD>
__device__ __forceinline__ void round_tile(const RoundArgs& r, uint32_t tile, int lane) {
    const uint32_t c = r.c_begin + tile * 32 + (lane & 31);
    float square, inv, lost;
    round_rows<true, VEC4, HOLD>(r.Cm, c, c < r.c_end, r.d, topk_steps(r.d), r.frag, tile, lane, square, inv, lost);
    if (lane < 32) {
        r.margin[tile * 32 + lane] = c < r.c_end ? lost * (TK_F16_SCALE * TK_F16_SCALE) : -INFINITY;
        if (c < r.c_end) r.invc[c] = inv;
    }
}
template <bool VEC4, int HOLD>
__global__ __launch_bounds__(64) void topk_round_kernel(RoundArgs r) {
    round_tile<VEC4, HOLD>(r, blockIdx.x, threadIdx.x);
}

// 1 / |row| alone, for the fp32 screen: one wavefront per 32 rows.
template <bool VEC4>
__global__ __launch_bounds__(256) void inv_length_kernel(const float* __restrict__ M, uint32_t rows, uint32_t d,
                                                         float* __restrict__ inv) {
    const uint32_t r = (blockIdx.x * 4 + threadIdx.x / 64) * 32u + (threadIdx.x & 31);
    const float s = pair_square<VEC4>(M + (uint64_t)(r < rows ? r : 0u) * d, r < rows, d, (threadIdx.x & 63) >> 5);
    if ((threadIdx.x & 32) == 0 && r < rows) inv[r] = inv_length(s);
}

// Whether a block goes without the screen: thread 0 asks (early: loads come back in order) and tells the
// others by way of *s_dense before a barrier.  (An ordinary read, which may be served by a cache: what
// matters is what earlier rounds have counted.)
__device__ __forceinline__ uint32_t dense_so_far(const TopkArgs& a) {
    return threadIdx.x == 0 && a.dense_skip != TK_NONE ? *a.dense : 0u;
}
__device__ __forceinline__ void tell_dense(const TopkArgs& a, uint32_t counted, bool first, uint32_t* s_hits, uint32_t* s_dense) {
    if (threadIdx.x) return;
    const bool skip = counted >= a.dense_skip;               // (TK_NONE: never reached)
    if (skip && first) atomicAdd(a.dense, a.blocks);
    *s_hits = 0; *s_dense = skip;
}

// Whether a block with that many hits is to drop them and form its similarities in fp32 (all threads; `hits`
// of a wavefront, the same in its lanes; s_hits is zero before).
__device__ __forceinline__ bool dense_block(const TopkArgs& a, int hits, uint32_t* s_hits, uint32_t* s_dense) {
    if (a.dense_limit == TK_NONE) return false;
    if (hits && threadIdx.x % 64 == 0) atomicAdd(s_hits, (uint32_t)hits);
    __syncthreads();
    if (*s_hits <= a.dense_limit) return false;
    if (threadIdx.x == 0) *s_dense = atomicAdd(a.dense, 1u) >= TK_SPARE;
    __syncthreads();
    return *s_dense != 0;
}

// What a 16-bit product must reach before the candidate's own margin: the query's threshold less its
// margin, in units of the product.
__device__ __forceinline__ float screen_level(float theta, float margin, float unit) {
    if (margin < 0.f) return theta < 0.f ? -INFINITY : INFINITY;          // every similarity is 0
    const float t = (theta - margin) * unit;
    return fabsf(t) < INFINITY ? t - fabsf(t) * 0x1p-20f : t;
}

// A slot on its query's pending list for every set bit: bit v of lane (fr, fk) is the pair of query
// q0 + 8 (v / 4) + 4 fk + v % 4 and the lane's candidate.  Lane (v, fk) reserves the slots of that
// query for the tile: one atomic instruction, one round trip for all 32 lists.  SCORED: the list holds
// (similarity, candidate), score(v) tells it.
template <bool SCORED, typename Score>
__device__ __forceinline__ void append_tile(const TopkArgs& a, uint32_t bits, uint32_t q0, uint32_t c, int lane, Score score) {
    const int fr = lane & 31, fk = lane >> 5;
    if (__ballot(bits != 0) == 0) return;                     // uniform per wavefront
    uint32_t mine = 0, base = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const uint64_t both = __ballot((bits >> v) & 1u);
        if (fr == v) mine = (uint32_t)__popc(fk ? (uint32_t)(both >> 32) : (uint32_t)both);
    }
    if (mine) base = atomicAdd(&a.cnt[q0 + 8 * (fr / 4) + 4 * fk + fr % 4], mine);   // (fr < 16)
    bool lost = false;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const bool pass = (bits >> v) & 1u;
        const uint64_t both = __ballot(pass);
        if (both == 0) continue;
        const uint32_t half = fk ? (uint32_t)(both >> 32) : (uint32_t)both;
        const uint32_t slot = __shfl(base, v + 32 * fk, 64) + (uint32_t)__popc(half & ((1u << fr) - 1u));
        const uint32_t q = q0 + 8 * (v / 4) + 4 * fk + v % 4;
        if (pass && slot < a.cap) {
            if (SCORED) ((uint2*)a.pend)[(uint64_t)q * a.cap + slot] = make_uint2(__float_as_uint(score(v)), c);
            else a.pend[(uint64_t)q * a.cap + slot] = c;
        }
        lost |= pass && slot >= a.cap;                        // (a list holds a whole round: cannot happen)
    }
    if (lost) atomicOr(a.err, 1u);
}

// The same bits, as one word per query: lane (v, fk), v < 16, holds that of query 8 (v / 4) + 4 fk + v % 4.
__device__ __forceinline__ uint32_t tile_words(uint32_t bits, int lane) {
    const int fr = lane & 31, fk = lane >> 5;
    uint32_t mine = 0;
    if (__ballot(bits != 0) == 0) return 0;                   // uniform per wavefront
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const uint64_t both = __ballot((bits >> v) & 1u);
        if (fr == v) mine = fk ? (uint32_t)(both >> 32) : (uint32_t)both;
    }
    return mine;
}

// A tile's 16-bit products against the thresholds: the bits of append_tile, and how many (added to `hits`,
// the same in every lane).  Most tiles hold none once the thresholds have risen: two instructions per
// element tell.  level: LDS, the 32 levels of the tile's queries (+inf past Q: no bits); `unit_c` scales
// this lane's products (its candidate) into the levels' units; `own` is the candidate's margin there, -inf
// for a lane without a candidate.
__device__ __forceinline__ uint32_t screen_tile(const v16f& acc, float unit_c, float own, const float* level, int lane,
                                                int& hits) {
    const int fk = lane >> 5;
    float lv[16];
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
        const float4 t = *reinterpret_cast<const float4*>(level + 4 * fk + 8 * v4);
        lv[4 * v4 + 0] = t.x; lv[4 * v4 + 1] = t.y; lv[4 * v4 + 2] = t.z; lv[4 * v4 + 3] = t.w;
    }
    float over = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) over = fmaxf(over, fmaf(acc[v], unit_c, -lv[v]));
    if (__ballot(over + own >= 0.f) == 0) return 0;           // uniform per wavefront
    const bool c_ok = own > -INFINITY;
    uint32_t bits = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const bool p = c_ok && fmaf(acc[v], unit_c, -lv[v]) + own >= 0.f;
        bits |= p ? 1u << v : 0u;
        hits += __popcll(__ballot(p));
    }
    return bits;
}

// ---------------------------------------------------------------------------------------------
// Similarities of a block of 64 WM queries x 64 WN candidates in fp32 on the matrix cores, and the pairs
// above the threshold listed.  WM x WN wavefronts, each 2 x 2 tiles of 32 x 32.
// v_mfma_f32_32x32x2_f32: lane l feeds A[i = l % 32][k = l / 32] and B[k = l / 32][j = l % 32];
// accumulator register v of lane l is D[8 (v / 4) + 4 (l / 32) + v % 4][l % 32], and each element is
// the fused-multiply-add chain over its columns in order.
// 2 x 2 tiles per wavefront at four wavefronts per SIMD (128 registers, accumulators included) measured
// best: 2 x 4 and 4 x 2 tiles (two wavefronts per SIMD) ran 9 % slower, 4 x 4 (one) 2.3 times slower --
// this lives on having other wavefronts to switch to at its barriers.
// STREAM: the pairs are left as bits, and the candidates' inverse lengths are formed here, else they are in a.invc.
// ---------------------------------------------------------------------------------------------
template <int WM, int WN> struct ExactLds {
    struct Panels { float A[2][64 * WM][TK_LD], B[2][64 * WN][TK_LD]; };
    struct Tables { float level[64 * WM], invq[64 * WM], theta[64 * WM], invc[64 * WN]; };
    union { alignas(16) Panels p; Tables t; };               // (the tables once the products are done)
    __device__ ExactLds() {}
};

template <int WM, int WN, bool VEC4, bool SCORED, bool STREAM>
__device__ __forceinline__ void exact_block(const TopkArgs& a, uint32_t q0, uint32_t c0, ExactLds<WM, WN>& s) {
    constexpr int TM = 2, TN = 2, BQ = 64 * WM, BC = 64 * WN, THREADS = 64 * WM * WN;
    constexpr int RPM = THREADS / (TK_BK / 4);               // rows covered by one move of the block
    constexpr int MOVES_A = BQ / RPM, MOVES_B = BC / RPM;
    static_assert(BQ % RPM == 0 && BC % RPM == 0, "whole moves");
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int wm = wave / WN, wn = wave % WN;
    static_assert(THREADS >= BQ && (!STREAM || 32 * WM * WN == BC), "a query per thread, 32 candidates per wavefront");
    const bool q_ok = tid < BQ && q0 + tid < a.Q;
    const float iq = q_ok ? a.invq[q0 + tid] : 0.f, th = q_ok ? a.theta[q0 + tid] : INFINITY;
    // Staging through two LDS buffers of TK_BK columns: while a panel is multiplied, the next one
    // is written to the other buffer (from registers loaded during the panel before) and the one
    // after is requested from memory; one barrier per panel.  Thread t moves float4 number t,
    // t + THREADS, ... of a panel, i.e. the same four columns of rows srow0, srow0 + RPM, ...
    // (One buffer of 32 columns with a barrier on either side of its refill measured 1 % slower.)
    const int srow0 = tid / (TK_BK / 4), scol = (tid % (TK_BK / 4)) * 4;
    const float* arow0 = a.Qm + (uint64_t)(q0 + srow0) * a.d;      // not dereferenced past Q / c_end
    const float* brow0 = a.Cm + (uint64_t)(c0 + srow0) * a.d;
    const uint64_t row_step = (uint64_t)RPM * a.d;
    float4 ra[MOVES_A], rb[MOVES_B];
    auto fetch = [&](uint32_t col0) {
#pragma unroll
        for (int i = 0; i < MOVES_A; ++i)
            ra[i] = load_cols<VEC4>(arow0 + i * row_step, q0 + srow0 + i * RPM < a.Q, col0 + scol, a.d);
#pragma unroll
        for (int i = 0; i < MOVES_B; ++i)
            rb[i] = load_cols<VEC4>(brow0 + i * row_step, c0 + srow0 + i * RPM < a.c_end, col0 + scol, a.d);
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < MOVES_A; ++i) {
            float* pa = &s.p.A[buf][srow0 + i * RPM][scol];
            pa[0] = ra[i].x; pa[1] = ra[i].y; pa[2] = ra[i].z; pa[3] = ra[i].w;
        }
#pragma unroll
        for (int i = 0; i < MOVES_B; ++i) {
            float* pb = &s.p.B[buf][srow0 + i * RPM][scol];
            pb[0] = rb[i].x; pb[1] = rb[i].y; pb[2] = rb[i].z; pb[3] = rb[i].w;
        }
    };
    float inv = 0.f;
    if (STREAM) {
        const uint32_t c = c0 + wave * 32 + (lane & 31);
        inv = inv_length(pair_square<VEC4>(a.Cm + (uint64_t)(c < a.c_end ? c : 0u) * a.d, c < a.c_end, a.d, lane >> 5));
    }
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    const int fr = lane & 31, fk = lane >> 5;
    fetch(0);
    stash(0);
    if (TK_BK < a.d) fetch(TK_BK);
    __syncthreads();
    int cur = 0;
    for (uint32_t kb = 0; kb < a.d; kb += TK_BK, cur ^= 1) {
        if (kb + TK_BK < a.d) {
            stash(cur ^ 1);
            if (kb + 2 * TK_BK < a.d) fetch(kb + 2 * TK_BK);
        }
        // (columns beyond d hold zeros: skipped; so are a wavefront's queries past the last)
        const int kmax = q0 + wm * 32 * TM < a.Q ? (int)min((uint32_t)TK_BK, a.d - kb) : 0;
        // one step of two columns per trip (longer straight runs, which would let the compiler
        // issue LDS reads under earlier products, measured the same; 16-byte LDS accesses on a
        // column order that gives each lane four adjacent floats per four steps measured slower)
#pragma unroll 1
        for (int kk = 0; kk < kmax; kk += 2) {
            float av[TM], bv[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) av[i] = s.p.A[cur][wm * 32 * TM + i * 32 + fr][kk + fk];
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[j] = s.p.B[cur][wn * 32 * TN + j * 32 + fr][kk + fk];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

    if (tid < BQ) {
        s.t.invq[tid] = iq;
        s.t.theta[tid] = th;
        // The same threshold for the raw product dot x (1/|c|), lowered by 2^-20 of itself so that
        // no score the exact test below accepts is missed (the two roundings of the score and the
        // ones made here stay under 2^-22 relative); -inf sends every element to the exact test.
        float t;
        if (iq == 0.f) {
            t = th <= 0.f ? -INFINITY : INFINITY;         // every score of a zero query is 0
        } else {
            const float r = th / iq;
            t = fabsf(r) < INFINITY ? r - fabsf(r) * 0x1p-20f : (r > 0.f && th == INFINITY ? INFINITY : -INFINITY);
        }
        s.t.level[tid] = t;
    }
    if (STREAM && lane < 32) s.t.invc[wave * 32 + lane] = inv;
    __syncthreads();

    // filter: a score above the query's threshold joins the query's pending list.  Most tiles hold no
    // such score once the thresholds have risen, so each 32 x 32 tile is first screened with two
    // instructions per element (raw product against the lowered threshold); only a tile with a hit
    // goes through the exact test.
#pragma unroll
    for (int ti = 0; ti < TM; ++ti) {
        const int qbase = wm * 32 * TM + ti * 32 + 4 * fk;   // this lane's queries: qbase + 8 (v/4) + v%4
        float tq[16];
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            const float4 t4 = *reinterpret_cast<const float4*>(&s.t.level[qbase + 8 * v4]);
            tq[4 * v4 + 0] = t4.x; tq[4 * v4 + 1] = t4.y; tq[4 * v4 + 2] = t4.z; tq[4 * v4 + 3] = t4.w;
        }
#pragma unroll
        for (int tj = 0; tj < TN; ++tj) {
            const uint32_t c = c0 + wn * 32 * TN + tj * 32 + fr;
            const bool c_ok = c < a.c_end;
            const float ic = STREAM ? s.t.invc[c - c0] : (c_ok ? a.invc[c] : 0.f);
            float over = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) over = fmaxf(over, fmaf(acc[ti][tj][v], ic, -tq[v]));
            if (!STREAM && __ballot(over >= 0.f) == 0) continue;       // uniform per wavefront
            uint32_t bits = 0;
            auto score = [&](int v) { return acc[ti][tj][v] * s.t.invq[qbase + 8 * (v / 4) + v % 4] * ic; };
#pragma unroll
            for (int v = 0; v < 16; ++v)                     // (padded queries carry +inf: never)
                bits |= c_ok && score(v) > s.t.theta[qbase + 8 * (v / 4) + v % 4] ? 1u << v : 0u;
            if constexpr (STREAM) {
                const uint32_t word = tile_words(bits, lane), q = q0 + wm * 32 * TM + ti * 32 + 8 * (fr / 4) + 4 * fk + fr % 4;
                if (fr < 16 && q < a.Q) a.bits[(uint64_t)q * a.pitch + (c - a.c_begin) / 32] = word;   // (c - fr: of this tile)
            } else {
                append_tile<SCORED>(a, bits, q0 + wm * 32 * TM + ti * 32, c, lane, score);
            }
        }
    }
}
// ---------------------------------------------------------------------------------------------
// Wide screen: WM x WN wavefronts, each TM x TN matrix-core tiles of 32 x 32.  Operands come in
// matrix-core order, so staging is a straight copy and LDS reads are 16 adjacent bytes per lane.
// Panels of two steps (32 columns) go through two LDS buffers: while one is multiplied, the next is
// written from registers and the one after is on its way from memory; one barrier per panel.
// Block b is mapped so that the blocks an XCD receives (b mod 8) walk through the query tiles of one
// candidate tile after the other: that tile and the queries stay in its L2.
// After = RoundArgs: the launch's first blocks (a multiple of eight) round the candidates of the round after this one:
// that is bound by memory and this by the matrix cores (TK_BESIDE).
// ---------------------------------------------------------------------------------------------
struct NoRound {};
template <int TM, int TN, int WM, int WN, int WPE, bool VEC4, class After>
__global__ __launch_bounds__(64 * WM * WN, WPE) void topk_wide_kernel(TopkArgs a, After after) {
    constexpr int THREADS = 64 * WM * WN, QT = TM * WM, CT = TN * WN, KC = 2;
    constexpr int PANEL = (QT + CT) * KC * 64;               // 16-byte units
    constexpr int MOVES = PANEL / THREADS;
    static_assert(PANEL % THREADS == 0, "whole moves");
    union Lds { v8h panel[2][PANEL]; ExactLds<WM, WN> exact; __device__ Lds() {} };
    __shared__ Lds lds;
    auto& s_panel = lds.panel;
    __shared__ __align__(16) float s_level[QT * 32];
    __shared__ uint32_t s_hits, s_dense;
    static_assert(QT == 2 * WM && CT == 2 * WN, "the tile of exact_block");
    const uint32_t total = a.nq_tiles * a.nc_tiles;
    const uint32_t per_xcd = (total + 7u) / 8u;
    uint32_t block = blockIdx.x;
    if constexpr (std::is_same<After, RoundArgs>::value) {
        const uint32_t round_blocks = ((after.tiles + WM * WN - 1) / (WM * WN) + 7) / 8 * 8;
        if (block < round_blocks) {                          // uniform per block
            const uint32_t tile = block * (WM * WN) + threadIdx.x / 64;
            if (tile < after.tiles) round_tile<VEC4, 0>(after, tile, threadIdx.x % 64);
            return;
        }
        block -= round_blocks;
    }
    const uint32_t logical = (block % 8u) * per_xcd + block / 8u;
    if (logical >= total) return;                            // uniform per block, before any barrier
    const uint32_t qt0 = (logical % a.nq_tiles) * QT, ct0 = (logical / a.nq_tiles) * CT;
    const uint32_t counted = dense_so_far(a);
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int wm = wave / WN, wn = wave % WN;
    const uint32_t steps = topk_steps(a.d), panels = steps / KC;
    for (int i = tid; i < QT * 32; i += THREADS) {
        const uint32_t q = qt0 * 32 + i;
        s_level[i] = q < a.Q ? screen_level(a.theta[q], a.qmargin[q], TK_F16_SCALE * TK_F16_SCALE) : INFINITY;
    }
    // unit u of a panel: tile u / (KC 64) -- queries first -- then step and lane
    const v8h* from[MOVES];
#pragma unroll
    for (int i = 0; i < MOVES; ++i) {
        const uint32_t u = tid + i * THREADS, t = u / (KC * 64), w = u % (KC * 64);
        from[i] = t < (uint32_t)QT ? (const v8h*)a.qfrag + (uint64_t)(qt0 + t) * steps * 64 + w
                                   : (const v8h*)a.cfrag + (uint64_t)(ct0 + t - QT) * steps * 64 + w;
    }
    v8h r[MOVES];
    auto fetch = [&](uint32_t p) {
#pragma unroll
        for (int i = 0; i < MOVES; ++i) r[i] = from[i][(uint64_t)p * (KC * 64)];
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < MOVES; ++i) s_panel[buf][tid + i * THREADS] = r[i];
    };
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    fetch(0);
    stash(0);
    tell_dense(a, counted, block == 0, &s_hits, &s_dense);       // (the first that screens)
    if (panels > 1) fetch(1);
    __syncthreads();
    bool dense = s_dense != 0;                               // uniform per block
    for (uint32_t p = dense ? panels : 0; p < panels; ++p) {
        const int cur = p & 1;
        if (p + 1 < panels) {
            stash(cur ^ 1);
            if (p + 2 < panels) fetch(p + 2);
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            v8h av[TM], bv[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) av[i] = s_panel[cur][((wm * TM + i) * KC + k) * 64 + lane];
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[j] = s_panel[cur][((QT + wn * TN + j) * KC + k) * 64 + lane];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }
    if (!dense) {
        uint32_t bits[TM][TN];
        int hits = 0;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const float own = a.cmargin[(ct0 + wn * TN + j) * 32 + (lane & 31)];
#pragma unroll
            for (int i = 0; i < TM; ++i) bits[i][j] = screen_tile(acc[i][j], 1.f, own, s_level + (wm * TM + i) * 32, lane, hits);
        }
        dense = dense_block(a, hits, &s_hits, &s_dense);
        if (!dense && hits) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    append_tile<false>(a, bits[i][j], (qt0 + wm * TM + i) * 32, a.c_begin + (ct0 + wn * TN + j) * 32 + (lane & 31), lane,
                                       [](int) { return 0.f; });
        }
    }
    if (dense) exact_block<WM, WN, VEC4, false, false>(a, qt0 * 32, a.c_begin + ct0 * 32, lds.exact);
}

// ---------------------------------------------------------------------------------------------
// Stream screen: a wavefront takes 32 candidates and TQ tiles of 32 queries (q_first + blockIdx.y: which).  The
// lane pair (l, l ^ 32) walks candidate l % 32, eight columns at a time each; the rounded columns are
// a matrix-core operand as they stand.  Four steps of candidate columns are in flight ahead of the
// four in work.  The queries' operands go through two LDS buffers of as many steps, asked for one panel ahead of the
// columns: read from memory where they are multiplied, every one of them waited for all columns on their way as well
// (whole search, us, that way and this: 200 queries over 200 001 x 512 555, 469; 32 over 500 000 x 300 476, 436; 100 over
// 200 003 x 100 129, 122; 250 over 100 001 x 31 155, 155).  Held to three wavefronts per SIMD at 128 queries, it spills:
// 522 and 130.
// The pairs to look at are left as a bit each: a block
// writes sixteen bytes per query, needs no counters, and a round may be as long as there is room for bits.
// (With lists of four bytes a pair a search of 100 queries over 200 003 x 100 took five rounds, 193 us; with three, 123.)
// ---------------------------------------------------------------------------------------------
constexpr int TK_AHEAD = 4;
template <int TQ, bool VEC4>
__global__ __launch_bounds__(256, TQ == 1 ? 4 : (TQ == 2 ? 3 : 2)) void topk_stream_kernel(TopkArgs a) {
    __shared__ __align__(16) float s_level[TQ * 32];
    constexpr int PANEL = TQ * TK_AHEAD * 64;                // 16-byte units, TQ of them a thread
    static_assert(PANEL == TQ * 256, "a step of a tile per wavefront and move");
    union Lds { v8b panel[2][PANEL]; ExactLds<2, 2> exact; __device__ Lds() {} };
    __shared__ Lds lds;
    __shared__ uint32_t s_hits, s_dense;
    __shared__ __align__(16) uint32_t s_words[TQ * 32][4];
    const int tid = threadIdx.x, lane = tid % 64, fk = lane >> 5;
    const uint32_t qt0 = (a.q_first + blockIdx.y) * TQ;
    const uint32_t c0 = a.c_begin + blockIdx.x * 128u;
    const uint32_t c = c0 + (tid / 64) * 32 + (lane & 31);
    const bool c_ok = c < a.c_end;
    const float* row = a.Cm + (uint64_t)(c_ok ? c : 0u) * a.d;
    float4 x[TK_AHEAD][2], nx[TK_AHEAD][2];
    auto fetch = [&](float4 (&r)[TK_AHEAD][2], uint32_t ks) {
#pragma unroll
        for (int i = 0; i < TK_AHEAD; ++i) {
            const uint32_t k = (ks + i) * TK_KS + 8 * fk;
            r[i][0] = load_cols_flat<VEC4>(row, k, a.d);
            r[i][1] = load_cols_flat<VEC4>(row, k + 4, a.d);
        }
    };
    const uint32_t steps = topk_steps(a.d);
    const v8b* qf = (const v8b*)a.qfrag + (uint64_t)qt0 * steps * 64 + lane;
    v8b qr[TQ];
    auto fetch_queries = [&](uint32_t ks) {                  // this thread's part of the panel of steps ks ..
        const uint32_t step = min(ks + tid / 64, steps - 1);
#pragma unroll
        for (int t = 0; t < TQ; ++t) qr[t] = qf[((uint64_t)t * steps + step) * 64];
    };
    const uint32_t counted = dense_so_far(a);
    fetch_queries(0);
    fetch(x, 0);
    for (int i = tid; i < TQ * 32; i += 256) {
        const uint32_t q = qt0 * 32 + i;
        s_level[i] = q < a.Q ? screen_level(a.theta[q], a.qmargin[q], 1.f) : INFINITY;
    }
    tell_dense(a, counted, a.q_first + blockIdx.y + blockIdx.x == 0, &s_hits, &s_dense);
    __syncthreads();
    bool dense = s_dense != 0;                               // uniform per block
    if (!dense) {
        v16f acc[TQ];
#pragma unroll
        for (int t = 0; t < TQ; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
        float sq[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, e2 = 0.f;
        int buf = 0;
        for (uint32_t ks0 = 0; ks0 < steps; ks0 += TK_AHEAD, buf ^= 1) {
#pragma unroll
            for (int t = 0; t < TQ; ++t) lds.panel[buf][t * 256 + tid] = qr[t];
            if (ks0 + TK_AHEAD < steps) {
                fetch_queries(ks0 + TK_AHEAD);
                fetch(nx, ks0 + TK_AHEAD);
            }
            __syncthreads();                                 // (a buffer is written again a barrier after its last read)
#pragma unroll
            for (int i = 0; i < TK_AHEAD; ++i) {
                const uint32_t ks = ks0 + i, k = ks * TK_KS + 8 * fk;
                if (ks < steps) {
                    const float4 xa = c_ok ? cols_inside<VEC4>(x[i][0], k, a.d) : make_float4(0.f, 0.f, 0.f, 0.f);
                    const float4 xb = c_ok ? cols_inside<VEC4>(x[i][1], k + 4, a.d) : make_float4(0.f, 0.f, 0.f, 0.f);
                    const float v[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
                    v8b g;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        g[e] = (__bf16)v[e];
                        const float lost = v[e] - (float)g[e];
                        e2 = fmaf(lost, lost, e2);
                    }
                    square8(xa, xb, sq);
#pragma unroll
                    for (int t = 0; t < TQ; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds.panel[buf][t * 256 + i * 64 + lane], g, acc[t], 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < TK_AHEAD; ++i) { x[i][0] = nx[i][0]; x[i][1] = nx[i][1]; }
        }
        const float half = tree8(sq);
        const float square = half + __shfl_xor(half, 32, 64);
        const float ic = inv_length(square);
        e2 += __shfl_xor(e2, 32, 64);
        float own = sqrtf(e2) * ic * 1.004f;
        if (square > 0.f && (square < TK_TINY || ic == 0.f)) own = INFINITY;   // imprecise, or too long to square
        if (!(own >= 0.f)) own = INFINITY;
        if (!c_ok) own = -INFINITY;
        int hits = 0;
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
            if (own == INFINITY || ic == 0.f)                    // products that may not be finite: the margin decides
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
            const uint32_t word = tile_words(screen_tile(acc[t], ic, own, s_level + t * 32, lane, hits), lane);
            const int fr = lane & 31;
            if (fr < 16) s_words[t * 32 + 8 * (fr / 4) + 4 * fk + fr % 4][tid / 64] = word;
        }
        dense = dense_block(a, hits, &s_hits, &s_dense);
        if (!dense) {
            __syncthreads();
            const uint32_t q = qt0 * 32 + tid;
            if (tid < TQ * 32 && q < a.Q)                        // (the pitch is a multiple of four words)
                *(uint4*)(a.bits + (uint64_t)q * a.pitch + blockIdx.x * 4) = *(const uint4*)s_words[tid];
        }
    }
    if (dense) exact_block<2, 2, VEC4, false, true>(a, qt0 * 32, c0, lds.exact);
}

// The fp32 screen: nothing but such blocks, mapped to XCDs as above.
template <bool VEC4>
__global__ __launch_bounds__(TK_THREADS, 4) void topk_scores_kernel(TopkArgs a) {
    __shared__ ExactLds<2, 2> lds;
    const uint32_t total = a.nq_tiles * a.nc_tiles;
    const uint32_t per_xcd = (total + 7u) / 8u;
    const uint32_t logical = (blockIdx.x % 8u) * per_xcd + blockIdx.x / 8u;
    if (logical >= total) return;                            // uniform per block, before any barrier
    exact_block<2, 2, VEC4, true, false>(a, (logical % a.nq_tiles) * TK_BQ, a.c_begin + (logical / a.nq_tiles) * TK_BC, lds);
}

// ---------------------------------------------------------------------------------------------
// Fold: one block per query gives the pairs listed (or left as bits) their similarities -- a lane per candidate, its
// row read by lanes side by side (wave_scores) or by itself (exact_score); the fp32 screen has them listed already -- and merges those above
// the threshold into the sorted best list (higher score first, equal scores by lower index), then raises
// the threshold to the K-th best and empties the list.  Rounds come in index order, so a later candidate that only equals the K-th best
// never enters.  Each wavefront keeps its own 64 best, sorted across its lanes; the lists are merged
// through LDS at the end.  `out_idx` (last round): the results are written as well.
// Bits may name any share of a long round: where similarities rise with the index, nearly all of it passes thresholds as
// old as the round before.  Past FOLD_PICK candidates gridDim.y blocks share the query (fold_parts; with fewer all but
// the first have only counted), and the last one done merges their lists.  Rising order, K = 30, us, with rounds as short
// as lists of four bytes a pair allow, with the long ones and one block a query, and shared: 1 query over 200 000 x 100
// 1760, 2570, 295, over 10^6 3250, 9900, 865; 100 queries 1820, 1545, 795 and 3520, 6250, 2950; 200 over 200 000
// 1720, 2240, 1480.
// ---------------------------------------------------------------------------------------------
// (score, index) as one number that grows with the rank: order-preserving bits of the score, then ~index
__device__ __forceinline__ uint64_t rank_key(float s, uint32_t c) {
    const uint32_t b = __float_as_uint(s + 0.f);             // (-0 and 0 are equal scores)
    return ((uint64_t)((b & 0x80000000u) ? ~b : b | 0x80000000u) << 32) | (uint32_t)~c;
}
__device__ __forceinline__ float key_score(uint64_t k) {
    const uint32_t b = (uint32_t)(k >> 32);
    return __uint_as_float((b & 0x80000000u) ? b & 0x7FFFFFFFu : ~b);
}
__device__ __forceinline__ uint64_t lane_xor(uint64_t k, int m) {
    return ((uint64_t)(uint32_t)__shfl_xor((int)(k >> 32), m, 64) << 32) | (uint32_t)__shfl_xor((int)(uint32_t)k, m, 64);
}
__device__ __forceinline__ uint64_t sort64(uint64_t k, int lane) {             // descending over the lanes
    for (int size = 2; size <= 64; size <<= 1)
        for (int j = size >> 1; j > 0; j >>= 1) {
            const uint64_t o = lane_xor(k, j);
            const bool keep_max = ((lane & j) == 0) == ((lane & size) == 0 || size == 64);
            k = (k > o) == keep_max ? k : o;
        }
    return k;
}
// the 64 largest of a sorted list and `rev`, a sorted list read backwards
__device__ __forceinline__ uint64_t merge64(uint64_t list, uint64_t rev, int lane) {
    uint64_t k = list > rev ? list : rev;
    for (int j = 32; j > 0; j >>= 1) {
        const uint64_t o = lane_xor(k, j);
        k = (k > o) == ((lane & j) == 0) ? k : o;
    }
    return k;
}

// The similarities of a wavefront's candidates, lane r the one of candidate c of lane r (lanes 0 .. nr - 1, nr at least 1).
// Rows are read 32 columns at a time by lanes side by side and go through LDS, from where each lane walks its own: a
// lane that reads its row from memory takes a line of its own for every access, 64 to an instruction, and the fold was bound by
// those (a round, us, that way and this: 4096 queries over 2^20 x 300 in the median 27, 15, on average, with the two early ones
// that list hundreds of candidates a query, 36, 24; 100 over 200 003 x 100 29, 22; one over 500 000 x 300 67, 33).
constexpr int FS_COLS = 32, FS_PITCH = FS_COLS + 4;      // (16-byte aligned, eight rows a pass over the banks)
struct FoldRows { float x[65][FS_PITCH]; uint32_t c[64]; };      // row 64: the query
template <bool VEC4, int AHEAD>
__device__ __forceinline__ float wave_scores(const float* __restrict__ q, const float* __restrict__ Cm, uint32_t c, uint32_t nr,
                                             uint32_t d, float iq, FoldRows& lds) {
    constexpr int PER_ROW = VEC4 ? 8 : 32;               // lanes to a row
    constexpr int ROWS = 64 / PER_ROW, STEPS = 64 / ROWS;
    const uint32_t lane = threadIdx.x % 64, in_row = lane / PER_ROW, col = (lane % PER_ROW) * (VEC4 ? 4 : 1);
    lds.c[lane] = c;
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    fence();
    typedef typename std::conditional<VEC4, float4, float>::type word;
    struct Part { word x[STEPS], y; } part[AHEAD];       // columns asked for
    auto none = [](uint32_t k, uint32_t d_) { return k >= d_; };
    auto fetch = [&](uint32_t k0, Part& p) {                      // (past the last column: elsewhere in the row, zero when stored)
        const uint32_t k = none(k0 + col, d) ? 0u : k0 + col;
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            if ((uint32_t)(i * ROWS) >= nr) break;       // uniform
            const uint32_t row = lds.c[min(i * ROWS + in_row, nr - 1)];
            p.x[i] = *reinterpret_cast<const word*>(Cm + (uint64_t)row * d + k);
        }
        p.y = *reinterpret_cast<const word*>(q + k);
    };
    auto put = [&](uint32_t k0, const Part& p) {
        const bool past = none(k0 + col, d);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            if ((uint32_t)(i * ROWS) >= nr) break;
            *reinterpret_cast<word*>(&lds.x[i * ROWS + in_row][col]) = past ? word{} : p.x[i];
        }
        if (lane < (uint32_t)PER_ROW) *reinterpret_cast<word*>(&lds.x[64][col]) = past ? word{} : p.y;
    };
    float dot = 0.f, lo[8], hi[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { lo[e] = 0.f; hi[e] = 0.f; }
#pragma unroll
    for (int t = 0; t < AHEAD; ++t)
        if ((uint32_t)(t * FS_COLS) < d) fetch(t * FS_COLS, part[t]);
    const uint32_t own = min(lane, nr - 1);
#pragma unroll 1
    for (uint32_t k1 = 0; k1 < d; k1 += AHEAD * FS_COLS) {
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) {
            const uint32_t k0 = k1 + t * FS_COLS;
            if (k0 >= d) break;                          // uniform
            put(k0, part[t]);
            fence();
            if (k0 + AHEAD * FS_COLS < d) fetch(k0 + AHEAD * FS_COLS, part[t]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {                // eight columns
                const float4 u = *reinterpret_cast<const float4*>(&lds.x[own][8 * i]), v = *reinterpret_cast<const float4*>(&lds.x[own][8 * i + 4]);
                const float4 f = *reinterpret_cast<const float4*>(&lds.x[64][8 * i]), g = *reinterpret_cast<const float4*>(&lds.x[64][8 * i + 4]);
                dot = fmaf(f.x, u.x, dot); dot = fmaf(f.y, u.y, dot); dot = fmaf(f.z, u.z, dot); dot = fmaf(f.w, u.w, dot);
                dot = fmaf(g.x, v.x, dot); dot = fmaf(g.y, v.y, dot); dot = fmaf(g.z, v.z, dot); dot = fmaf(g.w, v.w, dot);
                square8(u, v, i % 2 ? hi : lo);
            }
            fence();
        }
    }
    return dot * iq * inv_length(tree8(lo) + tree8(hi));
}

// The same by one lane from memory: rows of a line or two (fold_by_lane), and long ones, no multiple of four columns, of which few
// are asked for (fold_few).
template <bool VEC4>
__device__ __forceinline__ float exact_score(const float* __restrict__ q, const float* __restrict__ c, uint32_t d,
                                             float iq) {
    float dot = 0.f, lo[8], hi[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { lo[e] = 0.f; hi[e] = 0.f; }
    float4 x[8], nx[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = load_cols<VEC4>(c, true, 4 * i, d);
    for (uint32_t k0 = 0; k0 < d; k0 += 32) {
#pragma unroll
        for (int i = 0; i < 8; ++i) nx[i] = load_cols<VEC4>(c, true, k0 + 32 + 4 * i, d);   // (zero past the row's end)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float4 y = load_cols<VEC4>(q, true, k0 + 4 * i, d);
            dot = fmaf(y.x, x[i].x, dot); dot = fmaf(y.y, x[i].y, dot);
            dot = fmaf(y.z, x[i].z, dot); dot = fmaf(y.w, x[i].w, dot);
        }
        square8(x[0], x[1], lo); square8(x[2], x[3], hi);
        square8(x[4], x[5], lo); square8(x[6], x[7], hi);
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = nx[i];
    }
    return dot * iq * inv_length(tree8(lo) + tree8(hi));
}

// Rows that lanes read on their own: of bits by sixteen wavefronts up to TK_STREAM_Q queries, eight past that, of a list by four.
// Searches of 200 000 rows, us, this way and through LDS, by columns: 100 queries 7: 86, 95, 13: 96, 97, 17: 102, 98; 16: 78, 84,
// 40: 91, 91, 52: 100, 92; 129 queries 21: 127, 117; 56, crowded, 646, 543; 200 queries 7: 116, 127; 40: 114, 122.  600 queries 7: 233, 249,
// 27: 255, 259; 16: 266, 267, 56: 268, 264.  Where similarities rise with the index the lines would lie higher: 100 of 17 315, 420;
// 300 of 60 1210, 1310.
static bool fold_by_lane(bool bits, uint32_t d, bool vec4) {
    return d <= (bits ? (vec4 ? 40u : 16u) : (vec4 ? 48u : 24u));
}
// Whether so few candidates are expected that lanes read rows on their own, sixteen wavefronts to a query: as long as their lines
// fit the L1 that is faster than four bytes at a time through LDS.  `passing`: candidates of the round times the
// share that the thresholds let through.  The first round has only tau to go by.  Searches, us, this way throughout, by this rule and through LDS
// throughout: 1 query over 18 030 x 511, K = 1, tau = 0.3: 168, 168, 202; 19 over 5000 x 495, K = 10, tau = 0.65 138, 138, 169; 100 over
// 100 000 x 301, K = 30, no tau 1190, 330, 330; limit 20, 50, 100, 200, 400 on K = 10 over 5000 to 400 000 x 511, geometric mean against this way
// throughout 1.19, 1.24, 1.24, 1.00, 1.00; 1 over 100 000 x 65, K = 1, 69, 69, 64, x 99 81, 81, 84.
static bool fold_few(uint32_t Q, uint32_t d, bool vec4, bool first, double passing, float tau) {
    return !vec4 && d > 96 && Q <= TK_STREAM_Q && (first ? tau > 0.f : passing <= 100.);
}
constexpr uint32_t FOLD_PICK = 2048;             // candidates named by bits that a block lists before it scores them
constexpr uint32_t FOLD_CHUNK = 16;              // words: where they are more
// candidates of a round for every block of a query (a block more costs what it takes to count: 100 queries over 200 003 x
// 100, not crowded, 116.6 us, in five blocks each 116.9, and two in the round before 117.2)
static uint32_t fold_share(uint32_t Q) { return Q <= 32 ? 1u << 13 : 1u << 15; }
constexpr uint32_t FOLD_WORDS = 8;           // of a thread, in flight
// Queries from which two wavefronts fold a list, and one: most lists fill one, and what LDS a block asks for says how many
// are on the chip; long lists want the chip filled.  Searches, us, by one, two and four wavefronts: 4096 over 2^20 x 300 4497, 4552,
// 4720; over 200 000 rows 2500 x 99 652, 682, - (x 60, crowded, 1042, 1020, -); 2000 x 60 432, 430, 438 (crowded 886, 859, 860); 1024 x 99 457, 432,
// 449, x 300 620, 594, 579; 600 x 300 571, -, 508.  Where similarities rise with the index, and last by four without LDS: 1024 x 100
// 6817, 4208, 3463, 4837; 2000 x 100 8778, 6686, 6559, 11 170; 3000 x 255 33.1 ms, 44.8, 44.7, 170.
constexpr uint32_t FOLD_PAIR_Q = 1024, FOLD_ALONE_Q = 2048;
enum FoldFrom { FOLD_LIST, FOLD_SCORED, FOLD_BITS };
template <int WAVES, bool VEC4, FoldFrom FROM, bool BY_LANE = false>
__global__ __launch_bounds__(64 * WAVES) void topk_fold_kernel(TopkArgs a, uint32_t K, float tau,
                                                               uint64_t* __restrict__ best,
                                                               uint32_t* __restrict__ best_cnt,
                                                               float* __restrict__ theta,
                                                               uint32_t* __restrict__ out_idx,
                                                               float* __restrict__ out_score,
                                                               uint32_t* __restrict__ out_count) {
    __shared__ uint64_t s_list[WAVES][64];
    union Picked {
        uint32_t pick[FROM == FOLD_BITS ? FOLD_PICK : 1];
        uint32_t queue[FROM == FOLD_BITS ? WAVES : 1][64 + 32 * FOLD_CHUNK];
    };
    __shared__ Picked lds;
    __shared__ uint32_t s_picked;
    __shared__ __align__(16) FoldRows s_rows[FROM == FOLD_SCORED || BY_LANE ? 1 : WAVES];
    const uint32_t q = a.q_first + blockIdx.x;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const uint32_t part = FROM == FOLD_BITS ? blockIdx.y : 0u, n_parts = FROM == FOLD_BITS ? gridDim.y : 1u;
    const uint32_t bc = best_cnt[q];
    const float th = theta[q], iq = a.invq[q];
    // (key 0 is below that of every score: an empty place)
    uint64_t list = part == 0 && wave == 0 && (uint32_t)lane < bc ? best[(uint64_t)q * TK_LIST + lane] : 0ull;
    uint32_t n_new;
    const uint32_t words = (a.c_end - a.c_begin + 31) / 32;
    const uint32_t* bits = a.bits + (uint64_t)q * a.pitch;
    if constexpr (FROM == FOLD_BITS) {
        // the candidates whose bits are set, in any order: ranks decide
        if (threadIdx.x == 0) s_picked = 0;
        __syncthreads();
        for (uint32_t i0 = threadIdx.x; i0 < words; i0 += FOLD_WORDS * 64 * WAVES) {
            uint32_t word[FOLD_WORDS];                       // (asked for together, then looked at)
#pragma unroll
            for (uint32_t e = 0; e < FOLD_WORDS; ++e) word[e] = bits[min(i0 + e * 64 * WAVES, words - 1)];
#pragma unroll
            for (uint32_t e = 0; e < FOLD_WORDS; ++e) {
                const uint32_t i = i0 + e * 64 * WAVES;
                if (i >= words || word[e] == 0) continue;
                uint32_t at = atomicAdd(&s_picked, (uint32_t)__popc(word[e]));
                for (uint32_t left = word[e]; left; left &= left - 1, ++at)
                    if (at < FOLD_PICK) lds.pick[at] = a.c_begin + i * 32 + __builtin_ctz(left);
            }
        }
        __syncthreads();
        n_new = s_picked;
        if (part && n_new <= FOLD_PICK) return;              // uniform per block; all blocks of a query count the same
    } else {
        n_new = min(a.cnt[q], a.cap);
    }
    if (n_new == 0 && !out_idx) return;                      // uniform per block
    const bool spilled = FROM == FOLD_BITS && n_new > FOLD_PICK;        // each wavefront looks through words of its own
    const int waves = spilled ? WAVES : min(WAVES, (int)((n_new + 63) / 64));      // that have any
    if (wave && wave >= waves) return;
    // spilled: sixteen words at a time are turned into candidates in order, until there is one for every lane
    uint32_t words_at = (part * WAVES + wave) * FOLD_CHUNK, queued = 0, taken = 0;
    for (uint32_t base = wave * 64u; spilled || base < n_new; base += 64u * WAVES) {
        bool on = base + lane < n_new;
        uint32_t c = 0;
        float s = 0.f;
        if constexpr (FROM == FOLD_BITS) {
            if (spilled) {
                uint32_t* queue = lds.queue[wave];
                const uint32_t left = queued - taken, keep = taken + lane < queued ? queue[taken + lane] : 0u;
                if (left < 64) {                             // (uniform per wavefront, as all of these)
                    queue[lane] = keep;
                    queued = left; taken = 0;
                }
                while (queued - taken < 64 && words_at < words) {
                    uint32_t word = lane < (int)FOLD_CHUNK && words_at + lane < words ? bits[words_at + lane] : 0u;
                    const uint32_t n = (uint32_t)__popc(word);
                    uint32_t incl = n;
#pragma unroll
                    for (int d = 1; d < (int)FOLD_CHUNK; d <<= 1) {
                        const uint32_t y = __shfl_up(incl, d, 64);
                        if (lane >= d) incl += y;
                    }
                    for (uint32_t at = queued + incl - n; word; word &= word - 1, ++at)
                        queue[at] = a.c_begin + (words_at + lane) * 32 + __builtin_ctz(word);
                    queued += (uint32_t)__builtin_amdgcn_readlane((int)incl, FOLD_CHUNK - 1);
                    words_at += FOLD_CHUNK * WAVES * n_parts;
                }
                if (queued == taken) break;
                on = taken + lane < queued;
                if (on) c = queue[taken + lane];
                taken = min(taken + 64, queued);
            } else if (on) {
                c = lds.pick[base + lane];
            }
        } else if (on && FROM == FOLD_LIST) {
            c = a.pend[(uint64_t)q * a.cap + base + lane];
        } else if (on) {
            const uint2 e = ((const uint2*)a.pend)[(uint64_t)q * a.cap + base + lane];
            s = __uint_as_float(e.x); c = e.y;
        }
        if constexpr (BY_LANE) {
            if (on) s = exact_score<VEC4>(a.Qm + (uint64_t)q * a.d, a.Cm + (uint64_t)c * a.d, a.d, iq);
        } else if constexpr (FROM != FOLD_SCORED) {          // (those that are on come first, and are some)
            s = wave_scores<VEC4, (WAVES == 8 ? 2 : 1)>(a.Qm + (uint64_t)q * a.d, a.Cm, c, (uint32_t)__popcll(__ballot(on)), a.d, iq, s_rows[wave]);
        }
        const uint64_t k = on && s > th ? rank_key(s, c) : 0ull;       // (a similarity that is no number never passes)
        if (__ballot(k != 0)) list = merge64(list, __shfl((unsigned long long)sort64(k, lane), 63 - lane, 64), lane);
    }
    int half = 1;                                            // half of the wavefronts, rounded up to a power of two
    while (2 * half < waves) half *= 2;
    for (int w = waves > 1 ? half : 0; w >= 1; w >>= 1) {
        __syncthreads();
        if (wave >= w && wave < 2 * w) s_list[wave][63 - lane] = list;
        __syncthreads();
        if (wave < w && wave + w < waves) list = merge64(list, s_list[wave + w][lane], lane);
    }
    if (wave) return;
    if (FROM == FOLD_BITS && spilled && n_parts > 1) {       // (a.cnt is zero: the lists it counts are not used here)
        uint64_t* lists = a.parts + (uint64_t)q * n_parts * TK_LIST;
        __hip_atomic_store(lists + part * TK_LIST + lane, list, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
        uint32_t done = 0;
        if (lane == 0) done = __hip_atomic_fetch_add(&a.cnt[q], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)done) + 1 < n_parts) return;
        __threadfence();
        for (uint32_t p = 0; p < n_parts; ++p)
            if (p != part)
                list = merge64(list, __hip_atomic_load(lists + p * TK_LIST + (63 - lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), lane);
    }
    const uint32_t have = min(K, (uint32_t)__popcll(__ballot(list != 0)));
    if ((uint32_t)lane >= have) list = 0;
    best[(uint64_t)q * TK_LIST + lane] = list;
    const float s = key_score(list);
    if (lane == 0) { best_cnt[q] = have; a.cnt[q] = 0u; }
    if (have == K && (uint32_t)lane == K - 1) theta[q] = s;
    if (out_idx) {
        const bool ok = list != 0 && s > tau;
        if ((uint32_t)lane < K) {
            out_idx[(uint64_t)q * K + lane] = ok ? (uint32_t)~(uint32_t)list : TK_NONE;
            out_score[(uint64_t)q * K + lane] = ok ? s : 0.f;
        }
        const uint64_t mask = __ballot(ok);
        if (lane == 0 && out_count) out_count[q] = (uint32_t)__popcll(mask);
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
struct TopkLayout {
    size_t invq, invc, theta, cnt, best_cnt, err, best, pend, fixed_bytes;
};

static TopkLayout topk_layout(uint32_t Q, uint32_t N) {
    TopkLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = (off + bytes + 255) & ~(size_t)255; return o; };
    L.invq = take(sizeof(float) * Q);
    L.invc = take(sizeof(float) * N);
    L.theta = take(sizeof(float) * Q);
    L.cnt = take(sizeof(uint32_t) * Q);
    L.best_cnt = take(sizeof(uint32_t) * Q);
    L.err = take(256);
    L.best = take(sizeof(uint64_t) * (size_t)Q * TK_LIST);
    L.pend = off;
    L.fixed_bytes = off;
    return L;
}

// (sized for eight bytes per query and candidate of a round; what the pending lists do not take -- four
// bytes each -- holds the rounded rows)
size_t topk_workspace_bytes(uint32_t Q, uint32_t N, uint32_t round_candidates) {
    uint32_t cap = ((round_candidates + TK_BC - 1) / TK_BC) * TK_BC;
    return topk_layout(Q, N).fixed_bytes + 8 * (size_t)Q * cap;
}

bool topk_workspace_fits(uint32_t Q, uint32_t N, size_t workspace_bytes) {
    return workspace_bytes >= topk_workspace_bytes(Q, N, TK_BC);
}

// The wide screen's tile: 256 queries x 128 candidates by eight wavefronts of 64 x 64, four to a SIMD.
// (Measured on 4096 x 2^20 x 300, whole search: 4.75 ms; 128 x 128 by four wavefronts 4.87, 256 x 256 by
// sixteen 4.84; wavefronts of 128 x 64, two to a SIMD, 5.05 - 5.5; of 128 x 128 alone on a SIMD 33.)
constexpr int TK_WTM = 2, TK_WTN = 2, TK_WWM = 4, TK_WWN = 2, TK_WWPE = 4;
constexpr uint32_t WIDE_Q = 32 * TK_WTM * TK_WWM, WIDE_C = 32 * TK_WTN * TK_WWN;

// How a search is served: by which screen, in rounds of how many candidates, and with how many rounded
// queries (a whole number of the screen's tiles: 32, 64 or 128 for the stream screen, 256 for the wide one).
// `list`: room of a query's list, pairs of four bytes.  The stream screen needs a bit per pair, so its rounds may be
// longer, as the same memory holds.
// `ahead`: there is room for the rounded candidates of two rounds.  `parts`: blocks that may share a query's fold.
struct TopkPlan { TopkScreen screen; uint64_t cap, q_up, list; bool ahead; uint32_t parts; };
// Up to sixteen where there are few queries, in a sixteenth of the room that the bits have at most.  A block of eight wavefronts with
// rows in LDS has a compute unit to itself, so these numbers fill the chip two times over, eight past TK_STREAM_Q queries.  Where every
// query has as much to fold, once would do (rising order, 200 000 x 300, us, filled once and as it is: 64 queries 1243, 1647; 128 1987, 2325;
// 256 3600, 3852; 100 1942, 1748); where one of many has, its list is folded by that many compute units (129 queries over 100 000 x 301,
// crowded: 5688, 3577).
static uint32_t fold_parts(uint32_t Q, uint64_t room) {
    const uint32_t parts = Q > 2 * TK_STREAM_Q ? 1u : std::min(16u, (Q > TK_STREAM_Q ? 2048u : 512u) / Q);
    return (uint64_t)Q * parts * TK_LIST * 8 <= room / 16 ? parts : 1u;
}
static uint32_t stream_tiles(uint32_t Q) { return Q <= 32 ? 1 : (Q <= 64 ? 2 : 4); }    // of 32 queries, per wavefront

static TopkPlan topk_plan(uint32_t Q, uint32_t N, uint32_t d, size_t workspace_bytes) {
    const uint64_t row_bytes = (uint64_t)topk_steps(d) * TK_KS * 2;
    const uint64_t n_up = ((uint64_t)N + 255) / 256 * 256;
    const uint64_t free_bytes = workspace_bytes - topk_layout(Q, N).fixed_bytes;          // (fits 128 candidates of eight bytes)
    // Up to one tile of queries the stream screen reads every candidate once; with more it reads and rounds
    // them again for each tile, which from some 256 queries on costs more than rounding them once into the
    // workspace -- unless that leaves short rounds (us, wide and stream: 4096 over 200 000 x 300 with room for
    // 900, 3800 candidates 4750, 5670 and 2990, 4230; 1000 with room for 3400 2230, 2150; 300 over 200 000
    // x 60 280, 264).  With 129 to 256 the wide screen is ahead only over few candidates, whose rows it need
    // not read twice (129 over 20 000 x 300 187, 206; over 200 000 x 60 246, 224; x 512 840, 600; x 1000
    // 2030, 1130).  (`cap` of the stream screen, here: what its lists would hold, close to twice what the fp32 screen's
    // do; where the rounded queries take much of that, the fp32 screen is taken: 4096 over 20 000 x 800 with room
    // for 512 candidates 3870, stream with lists 4590.)
    TopkPlan p{TOPK_FP32, free_bytes / (8ull * Q) / TK_BC * TK_BC, 0, 0, false, 1};
    const uint64_t cap_fp32 = p.cap;
    // (`per_round`: of the candidates' bytes, those that are better held twice, for this round and the next)
    auto room = [&](uint64_t tile, uint64_t per_candidate, uint64_t per_round, uint64_t granule, uint64_t least, TopkScreen screen) {
        const uint64_t q_up = (Q + tile - 1) / tile * tile, q_bytes = q_up * (row_bytes + 4) + 512;
        if (free_bytes <= q_bytes) return false;
        const uint64_t cap = (free_bytes - q_bytes) / per_candidate / granule * granule;
        if (cap < n_up && cap < least) return false;
        const uint64_t twice = (free_bytes - q_bytes) / (per_candidate + per_round) / granule * granule;
        const uint32_t steps = topk_steps(d);
        const bool ahead = per_round && (steps <= TK_BESIDE || steps > (uint32_t)TK_HOLD) && (twice >= n_up || twice >= least);
        uint64_t held = ahead ? twice : cap, longest = held;
        uint32_t parts = 1;
        if (screen == TOPK_STREAM) {
            uint64_t bytes = free_bytes - q_bytes;
            parts = fold_parts(Q, bytes);
            if (parts > 1) bytes -= (uint64_t)Q * parts * TK_LIST * 8 + 256;
            held = std::min(held, bytes / per_candidate / granule * granule);
            longest = bytes / Q * 8 / TK_BC * TK_BC;
        }
        p = TopkPlan{screen, longest, q_up, std::min<uint64_t>({held, n_up, TK_CAND_SLICE}), ahead, parts};
        return true;
    };
    const bool wide = Q > 2 * TK_STREAM_Q || (Q > TK_STREAM_Q && N <= (1u << 16) && topk_steps(d) <= TK_HOLD);
    const uint64_t least_wide = std::min<uint64_t>(8192, std::max<uint64_t>(1024, (1u << 22) / Q));
    const uint64_t least_stream = Q > TK_STREAM_Q ? std::max<uint64_t>(2 * TK_BC, cap_fp32 + cap_fp32 / 2) : 2 * TK_BC;
    if (!wide || !room(WIDE_Q, 4ull * Q + row_bytes + 4, row_bytes + 4, 256, least_wide, TOPK_WIDE))
        room(32 * stream_tiles(Q), 4ull * Q, 0, TK_BC, least_stream, TOPK_STREAM);
    p.cap = std::min<uint64_t>({p.cap, n_up, TK_CAND_SLICE});
    return p;
}

uint32_t topk_screen(uint32_t Q, uint32_t N, uint32_t d, size_t workspace_bytes) {
    return topk_plan(Q, N, d, workspace_bytes).screen;
}

uint32_t* launch_topk_cosine(const float* Qm, uint32_t Q, const float* Cm, uint32_t N, uint32_t d,
                             uint32_t K, float tau, uint32_t* out_idx, float* out_score,
                             uint32_t* out_count, void* workspace, size_t workspace_bytes, hipStream_t st) {
    const TopkLayout L = topk_layout(Q, N);
    char* ws = (char*)workspace;
    float* theta = (float*)(ws + L.theta);
    uint32_t* best_cnt = (uint32_t*)(ws + L.best_cnt);
    uint64_t* best = (uint64_t*)(ws + L.best);
    TopkArgs a{};
    a.Qm = Qm; a.Cm = Cm; a.Q = Q; a.N = N; a.d = d;
    a.invq = (float*)(ws + L.invq); a.invc = (float*)(ws + L.invc); a.theta = theta;
    a.cnt = (uint32_t*)(ws + L.cnt); a.err = (uint32_t*)(ws + L.err); a.dense = a.err + 1;
    const bool vec4 = d % 4 == 0 && ((uintptr_t)Qm % 16 == 0) && ((uintptr_t)Cm % 16 == 0);

    const uint64_t row_bytes = (uint64_t)topk_steps(d) * TK_KS * 2;
    const TopkPlan plan = topk_plan(Q, N, d, workspace_bytes);
    const TopkScreen screen = plan.screen;
    const uint64_t cap = plan.cap, q_up = plan.q_up;
    char* at = ws + L.pend;
    a.pend = (uint32_t*)at;
    a.cap = (uint32_t)cap;
    a.bits = a.pend;
    a.pitch = (uint32_t)(cap / 32);
    at += (std::max(screen == TOPK_STREAM ? cap * Q / 8 : cap * Q * 4, plan.list * Q * 4) + 255) / 256 * 256;
    if (plan.parts > 1) { a.parts = (uint64_t*)at; at += (uint64_t)Q * plan.parts * TK_LIST * 8; }
    void* qfrag = nullptr; float* qmargin = nullptr; void* cfrag[2] = {nullptr, nullptr}; float* cmargin[2] = {nullptr, nullptr};
    if (screen != TOPK_FP32) {
        qfrag = at; at += q_up * row_bytes;
        qmargin = (float*)at; at += q_up * 4;
        for (int b = 0; screen == TOPK_WIDE && b < (plan.ahead ? 2 : 1); ++b) {
            cfrag[b] = at; at += cap * row_bytes;
            cmargin[b] = (float*)at; at += cap * 4;
        }
    }
    a.qfrag = qfrag; a.qmargin = qmargin;

    // nothing below the threshold is ever wanted; without one, every cosine passes (-2 < -1)
    const float theta0 = tau > -2.0f ? tau : -2.0f;
    {
        const dim3 grid(blocks_for(qfrag ? q_up : Q, 32)), block(64);
#define W2V_QUERIES(F16, VEC4)                                                                             \
    hipLaunchKernelGGL((topk_queries_kernel<F16, VEC4>), grid, block, 0, st, Qm, Q, d, theta0, (float*)a.invq, \
                       theta, a.cnt, best_cnt, qfrag, qmargin, a.err)
        if (screen == TOPK_WIDE) { if (vec4) W2V_QUERIES(true, true); else W2V_QUERIES(true, false); }
        else { if (vec4) W2V_QUERIES(false, true); else W2V_QUERIES(false, false); }
#undef W2V_QUERIES
    }
    auto inverse_lengths = [&](uint64_t begin, uint64_t count) {
        for (uint64_t first = begin; first < begin + count; first += TK_CAND_SLICE) {
            const uint32_t rows = (uint32_t)std::min<uint64_t>(TK_CAND_SLICE, begin + count - first);
            const dim3 grid(blocks_for(rows, 128)), block(256);
            const float* at = Cm + first * d;
            float* inv = (float*)a.invc + first;
            if (vec4) hipLaunchKernelGGL(inv_length_kernel<true>, grid, block, 0, st, at, rows, d, inv);
            else hipLaunchKernelGGL(inv_length_kernel<false>, grid, block, 0, st, at, rows, d, inv);
        }
    };
    if (screen == TOPK_FP32) inverse_lengths(0, N);
    // Short rounds first: with a threshold from the first few hundred candidates only a small share of a
    // full round's scores reaches the pending lists.  Many queries: rounds grow fourfold from 256 (every
    // pair listed costs a row read).  Few: sixteenfold from 1024 -- there launches cost more than pairs.
    const bool many = Q > 2 * TK_STREAM_Q || screen == TOPK_WIDE;
    const uint64_t growth = many || screen == TOPK_FP32 ? 4 : 16;
    uint64_t blocks_seen = 0;                  // that screened or might have
    uint64_t len = screen == TOPK_FP32 ? TK_BC : (many ? 256 : 1024);
    auto longer = [&](uint64_t x) { return x * growth < cap ? x * growth : cap; };
    // With many queries an early round that would list many pairs goes through the fp32 screen, whose fold
    // reads no rows: listing 4096 x 256 pairs of 300 columns and folding them takes 237 us, this way 85
    // (4096 x 20 000, K = 64: 1047 -> 614 us in all; 4096 x 200 000, K = 30: 1540 -> 1360).  Below some 10^5
    // pairs the fp32 product is not faster: 300 x 100 000 328 us, 334 with TK_EXACT_ROUND 50 000.
    // (Where tau prunes from the start, nothing is known of how many pairs pass: screened.)
    auto in_fp32 = [&](uint64_t begin, uint64_t len) {
        const uint64_t m = std::min(len, N - begin);
        const double share = begin ? std::min(1.0, (double)K / (double)begin) : 1.0;
        return screen == TOPK_FP32 || (many && tau <= 0.f && 2 * m <= plan.list && share > 0.01 &&
                                       share * (double)m * Q > TK_EXACT_ROUND);
    };
    int buffer = 0;                            // of the wide screen's rounded candidates: this round's
    bool ready = false;                        // it holds them: rounded beside the round before
    if (len > cap) len = cap;
    for (uint64_t begin = 0; begin < N; begin += len, len = longer(len)) {
        a.c_begin = (uint32_t)begin;
        a.c_end = (uint32_t)(begin + len < N ? begin + len : N);
        const uint32_t m = a.c_end - a.c_begin;
        // The thresholds are those of `begin` candidates: about m K / begin of this round pass.
        const double share = begin ? std::min(1.0, (double)K / (double)begin) : 1.0;
        const uint32_t tile_q = std::min(Q, screen == TOPK_WIDE ? WIDE_Q : TK_STREAM_Q);
        a.dense_limit = a.dense_skip = TK_NONE;
        if (begin > 0) {
            a.dense_limit = (uint32_t)(2.0 * share * 128.0 * tile_q) +
                            (screen == TOPK_WIDE ? TK_DENSE_WIDE : TK_DENSE_STREAM * std::min(tile_q, 64u));
            if (blocks_seen) a.dense_skip = (uint32_t)std::min<uint64_t>(TK_NONE - 1, TK_SPARE + (blocks_seen + 1) / 2);
        }
        a.blocks = 0;
        const bool exact_round = in_fp32(begin, len);
        a.cap = (uint32_t)(screen == TOPK_FP32 ? cap : exact_round ? plan.list / 2 : plan.list);   // (eight bytes a pair or four)
        if (screen == TOPK_WIDE && !exact_round) {
            a.nq_tiles = (Q + WIDE_Q - 1) / WIDE_Q;
            a.nc_tiles = (m + WIDE_C - 1) / WIDE_C;
            const uint32_t total = a.nq_tiles * a.nc_tiles;
            if (begin > 0) blocks_seen += a.blocks = total;
            auto rounded = [&](uint64_t first, uint64_t count, int buf) {
                const uint32_t end = (uint32_t)std::min<uint64_t>(first + count, N);
                return RoundArgs{Cm, (uint32_t)first, end, d, blocks_for(end - (uint32_t)first, WIDE_C) * (WIDE_C / 32),
                                 (float*)a.invc, cfrag[buf], cmargin[buf]};
            };
            if (!ready) {
                const RoundArgs now = rounded(begin, len, buffer);
#define W2V_ROUND(VEC4, HOLD) hipLaunchKernelGGL((topk_round_kernel<VEC4, HOLD>), dim3(now.tiles), dim3(64), 0, st, now)
                if (vec4 && topk_steps(d) >= TK_HOLD_LEAST && topk_steps(d) <= TK_HOLD) W2V_ROUND(true, TK_HOLD);
                else if (vec4) W2V_ROUND(true, 0);
                else W2V_ROUND(false, 0);
#undef W2V_ROUND
            }
            a.cfrag = cfrag[buffer]; a.cmargin = cmargin[buffer];
            buffer ^= plan.ahead ? 1 : 0;
            RoundArgs after{};
            const uint64_t next = begin + len;
            ready = plan.ahead && next < N && !in_fp32(next, longer(len));
            if (ready) after = rounded(next, longer(len), buffer);
            const uint32_t round_blocks = (blocks_for(after.tiles, TK_WWM * TK_WWN) + 7) / 8 * 8;
            const dim3 grid(((total + 7u) / 8u) * 8u + round_blocks), block(64 * TK_WWM * TK_WWN);
#define W2V_WIDE(VEC4, AFTER)                                                                              \
    hipLaunchKernelGGL((topk_wide_kernel<TK_WTM, TK_WTN, TK_WWM, TK_WWN, TK_WWPE, VEC4, std::decay_t<decltype(AFTER)>>), grid, \
                       block, 0, st, a, AFTER)
            if (ready) { if (vec4) W2V_WIDE(true, after); else W2V_WIDE(false, after); }
            else { if (vec4) W2V_WIDE(true, NoRound{}); else W2V_WIDE(false, NoRound{}); }
#undef W2V_WIDE
        } else if (screen == TOPK_STREAM && !exact_round) {
            const uint32_t tq = stream_tiles(Q);
            const uint32_t q_tiles = blocks_for(Q, 32 * tq);
            if (begin > 0) blocks_seen += a.blocks = q_tiles * blocks_for(m, 128);
#define W2V_STREAM(TQ)                                                                                     \
    do {                                                                                                   \
        if (vec4) hipLaunchKernelGGL((topk_stream_kernel<TQ, true>), grid, block, 0, st, a);               \
        else hipLaunchKernelGGL((topk_stream_kernel<TQ, false>), grid, block, 0, st, a);                   \
    } while (0)
            for (a.q_first = 0; a.q_first < q_tiles; a.q_first += TK_STREAM_SLICE) {
                const dim3 grid(blocks_for(m, 128), std::min(TK_STREAM_SLICE, q_tiles - a.q_first)), block(256);
                if (tq == 1) W2V_STREAM(1); else if (tq == 2) W2V_STREAM(2); else W2V_STREAM(4);
            }
#undef W2V_STREAM
        } else {
            if (screen != TOPK_FP32) inverse_lengths(a.c_begin, m);
            a.nq_tiles = (Q + TK_BQ - 1) / TK_BQ;
            a.nc_tiles = (m + TK_BC - 1) / TK_BC;
            const uint32_t total = a.nq_tiles * a.nc_tiles;
            const dim3 grid(((total + 7u) / 8u) * 8u), block(TK_THREADS);
            if (vec4) hipLaunchKernelGGL((topk_scores_kernel<true>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((topk_scores_kernel<false>), grid, block, 0, st, a);
        }
        const bool last = begin + len >= N;
        uint32_t* oi = last ? out_idx : nullptr;
        const bool bits = screen == TOPK_STREAM && !exact_round;
        const uint32_t parts = bits ? std::max(1u, std::min(plan.parts, m / fold_share(Q))) : 1u;
#define W2V_FOLD(WAVES, VEC4, ...)                                                                         \
    hipLaunchKernelGGL((topk_fold_kernel<WAVES, VEC4, __VA_ARGS__>), dim3(std::min(TK_FOLD_SLICE, Q - a.q_first), parts), \
                       dim3(64 * WAVES), 0, st, a, K, tau, best, best_cnt, theta, oi, out_score, out_count)
        for (a.q_first = 0; a.q_first < Q; a.q_first += TK_FOLD_SLICE) {
            if (exact_round) W2V_FOLD(4, false, FOLD_SCORED);
            else if (!bits && fold_by_lane(bits, d, vec4)) { if (vec4) W2V_FOLD(4, true, FOLD_LIST, true); else W2V_FOLD(4, false, FOLD_LIST, true); }
            else if (!bits && Q >= FOLD_ALONE_Q) { if (vec4) W2V_FOLD(1, true, FOLD_LIST); else W2V_FOLD(1, false, FOLD_LIST); }
            else if (!bits && Q >= FOLD_PAIR_Q) { if (vec4) W2V_FOLD(2, true, FOLD_LIST); else W2V_FOLD(2, false, FOLD_LIST); }
            else if (!bits) { if (vec4) W2V_FOLD(4, true, FOLD_LIST); else W2V_FOLD(4, false, FOLD_LIST); }
            else if (fold_by_lane(bits, d, vec4)) {
                if (Q > TK_STREAM_Q) { if (vec4) W2V_FOLD(8, true, FOLD_BITS, true); else W2V_FOLD(8, false, FOLD_BITS, true); }
                else { if (vec4) W2V_FOLD(16, true, FOLD_BITS, true); else W2V_FOLD(16, false, FOLD_BITS, true); }
            }
            else if (fold_few(Q, d, vec4, begin == 0, share * m, tau)) W2V_FOLD(16, false, FOLD_BITS, true);
            else { if (vec4) W2V_FOLD(8, true, FOLD_BITS); else W2V_FOLD(8, false, FOLD_BITS); }
        }
#undef W2V_FOLD
    }
    return a.err;
}

}  // namespace w2v
