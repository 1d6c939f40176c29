// Initial values, row get/set, negative sampling (destination keys), gather dot products and the
// client's coefficient step.  gfx950, wave64.
#include <algorithm>

#include "rows.h"
#include "loss.h"

namespace w2v {

static inline unsigned blocks_for(uint64_t items, unsigned per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

// ---------------------------------------------------------------------------------------------
// Initial vectors: component (word w, global column c) of matrix m is
//   ((R >> 8) * 2^-24 - 0.5) / d_total,  R = word (c mod 4) of Philox(counter = (w, c/4, m, INIT)).
// One thread per float4 of a row; columns past d_slice inside the stride stay zero.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void init_kernel(float4* __restrict__ M, uint32_t V, RowGeom g,
                                                   uint32_t d_slice, float d_total,
                                                   uint32_t col_begin, uint32_t k0, uint32_t k1,
                                                   uint32_t matrix, int zero) {
    uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    uint64_t total = (uint64_t)V * g.stride4;
    if (i >= total) return;
    uint32_t w = (uint32_t)(i / g.stride4);
    uint32_t q = (uint32_t)(i % g.stride4);
    float vals[4] = {0.f, 0.f, 0.f, 0.f};
    if (!zero) {
        uint32_t have_block = 0xFFFFFFFFu;
        U4 r{0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t local = q * 4 + e;
            if (local < d_slice) {
                uint32_t c = col_begin + local;
                if ((c >> 2) != have_block) {
                    have_block = c >> 2;
                    r = philox4x32_10(w, have_block, matrix, DOM_INIT, k0, k1);
                }
                uint32_t lane = c & 3u;
                uint32_t bits = lane == 0 ? r.x : lane == 1 ? r.y : lane == 2 ? r.z : r.w;
                float x = (float)(bits >> 8) * (1.0f / 16777216.0f) - 0.5f;
                vals[e] = x / d_total;
            }
        }
    }
    M[i] = make_float4(vals[0], vals[1], vals[2], vals[3]);
}

void launch_init(float* M, uint32_t V, RowGeom g, uint32_t d_slice, uint32_t d_total,
                 uint32_t col_begin, uint64_t seed, uint32_t matrix, bool zero, hipStream_t st) {
    uint64_t total = (uint64_t)V * g.stride4;
    hipLaunchKernelGGL(init_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, st, (float4*)M, V,
                       g, d_slice, (float)d_total, col_begin, (uint32_t)seed,
                       (uint32_t)(seed >> 32), matrix, zero ? 1 : 0);
}

// ---------------------------------------------------------------------------------------------
// Listed rows between a matrix and the caller's row array (get, set, and the column slices of an
// export).  Bound by memory: a block moves a whole number of rows, MOVE_ITEMS accesses per thread, each
// as wide as the widths, the pitch and the caller's pointer allow (16 bytes when the row length is a
// multiple of four floats), four of them in flight; the words are read and range-checked once per row.
// (One 4-byte access per thread, a division and a word load each, before: reading back 0.5 M + 2.7 M
// rows of 1200 bytes took 3.11 ms, now 1.56 ms, 4.9 TB/s read and written.)
// ---------------------------------------------------------------------------------------------
constexpr int MOVE_ITEMS = 8;
constexpr int MOVE_ROWS_MAX = 1024;               // rows of a block, at most (their words sit in LDS)
constexpr uint32_t MOVE_GROUPS = 1u << 18;        // blocks of rows of several parts in x, at most (32 parts of them are less than 2^32 threads)
enum MoveDir { MOVE_OUT, MOVE_IN };

struct MovePart {                                 // one matrix and its columns on the caller's side
    float* M; uint32_t stride;                    // stride in floats (a multiple of 4)
    uint32_t col, width;                          // row r starts at ext + r * pitch + col
    uint32_t magic;                               // ceil(2^32 / (width / VEC)): exact below 2^22 items a block
    uint32_t* err;
};
template <int PARTS> struct MoveRows {
    float* ext; uint32_t pitch, m, V, rows_per_block, parts, in_x;
    bool together;                                // parts of the same rows are blocks that follow each other
    const uint32_t* rows;
    MovePart part[PARTS];
};

template <int VEC> struct MoveWord;
template <> struct MoveWord<1> { typedef float type; };
template <> struct MoveWord<2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct MoveWord<4> { typedef v4f type; };

template <int VEC, MoveDir DIR, int PARTS>
__global__ __launch_bounds__(256) void move_rows_kernel(MoveRows<PARTS> a) {
    typedef typename MoveWord<VEC>::type word;
    __shared__ uint32_t s_row[MOVE_ROWS_MAX];
    // Where one part's columns end inside a line of the caller's rows, the parts of some rows are blocks that follow each
    // other on one die (blocks go to the eight in turn): the line is still in that die's L2 when the next part's are written.
    // (130 000 rows of five parts of 60 columns one part after the other 94 us, this way 71; where parts end with their
    // lines, 200 000 rows of four of 32, 39 and 41.  For which widths: launch_move_rows.)
    const uint32_t which = PARTS > 1 ? (a.together ? blockIdx.x / 8 % a.parts : blockIdx.x / a.in_x) : 0u;
    const uint32_t group_x = a.together ? blockIdx.x / (8 * a.parts) * 8 + blockIdx.x % 8 : blockIdx.x % a.in_x;
    const uint64_t group = PARTS > 1 ? (uint64_t)blockIdx.y * MOVE_GROUPS + group_x : blockIdx.x;
    const MovePart& part = a.part[which];
    const uint64_t r0_64 = group * a.rows_per_block;
    if (r0_64 >= a.m) return;                                    // (of several parts the grid is rounded up)
    const uint32_t r0 = (uint32_t)r0_64;
    const uint32_t nr = min(a.rows_per_block, a.m - r0);
    for (uint32_t i = threadIdx.x; i < nr; i += 256) {
        uint32_t w = a.rows[r0 + i];
        if (w >= a.V) { atomicOr(part.err, 1u); w = DIR == MOVE_OUT ? 0u : KEY_NONE; }
        s_row[i] = w;
    }
    __syncthreads();
    const uint32_t dv = part.width / VEC, count = nr * dv;
    for (uint32_t i0 = threadIdx.x; i0 < count; i0 += 4 * 256) {
        word x[4];                       // (vectors of the compiler's own: an array of structs lands in LDS)
        word* to[4];
        bool on[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t i = min(i0 + e * 256, count - 1);     // (past the end: a load that is not stored)
            const uint32_t r = dv == 1 ? i : __umulhi(i, part.magic), c = i - r * dv;
            const uint32_t w = s_row[r];
            word* ext = (word*)(a.ext + (uint64_t)(r0 + r) * a.pitch + part.col) + c;
            word* mat = (word*)(part.M + (uint64_t)(w == KEY_NONE ? 0u : w) * part.stride) + c;
            const word* from = DIR == MOVE_OUT ? mat : ext;
            x[e] = *from;
            to[e] = DIR == MOVE_OUT ? ext : mat;
            on[e] = i0 + e * 256 < count && w != KEY_NONE;       // (a word outside is not written)
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (on[e]) *to[e] = x[e];
    }
}

// (PARTS = 1 keeps the kernel's arguments short for a plain get or set)
template <MoveDir DIR, int PARTS>
static void launch_move_rows(const RowPart* parts, uint32_t S, float* ext, uint32_t pitch,
                             const uint32_t* rows, uint32_t m, uint32_t V, hipStream_t st) {
    if (m == 0) return;
    MoveRows<PARTS> a{};
    a.ext = ext; a.pitch = pitch; a.m = m; a.V = V; a.rows = rows;
    uint32_t mix = pitch | (uint32_t)((uintptr_t)ext / 4), width = 0;
    uint64_t widths = 0;
    bool lines_shared = false;
    for (uint32_t s = 0; s < S; ++s) {
        mix |= parts[s].width | parts[s].col;
        lines_shared |= (parts[s].col | pitch | (uint32_t)((uintptr_t)ext / 4)) % 32 != 0;
        width = std::max(width, parts[s].width);
        widths += parts[s].width;
    }
    // Blocks of narrow parts hold the places of others with little to do, so parts are moved together where they are nearly
    // equal, and somewhat unequal ones where the caches would not keep the shared lines anyway.  One part after the other and
    // together, us, 100 000 and 600 000 rows: 150 + 150 columns 52, 46 and 407, 292; 200 + 100 51, 56 and 402, 359; 60 + 100 + 140 55, 51 and
    // 428, 341; 100 + 28 21.5, 22.2 and 150, 172; 280 + 20 49, 62 and 363, 374.
    const bool large = (uint64_t)m * pitch * 4 >= 200000000u;
    a.together = lines_shared && 10 * widths >= (large ? 7 : 9) * (uint64_t)S * width;
    const uint32_t vec = (uintptr_t)ext % 4 ? 1 : (mix % 4 == 0 ? 4 : (mix % 2 == 0 ? 2 : 1));
    for (uint32_t s = 0; s < S; ++s) {
        const uint32_t dv = parts[s].width / vec;                 // (dv = 1: the magic is not used)
        a.part[s] = MovePart{parts[s].M, parts[s].stride4 * 4, parts[s].col, parts[s].width,
                             (uint32_t)(((1ull << 32) + dv - 1) / dv), parts[s].err};
    }
    // as many rows as give every thread MOVE_ITEMS accesses, fewer (down to one access per thread) while
    // that leaves the chip short of blocks
    const uint32_t dv_max = width / vec;
    const uint32_t most = std::min((uint32_t)MOVE_ROWS_MAX, std::max(1u, 256u * MOVE_ITEMS / dv_max));
    const uint32_t least = std::min(most, std::max(1u, 256u / dv_max));
    const uint32_t rb = std::min(most, std::max(least, (uint32_t)((uint64_t)m * S / 2048u)));
    a.rows_per_block = rb; a.parts = S;
    const uint32_t groups = blocks_for(m, rb), in_x = std::min(a.together ? (groups + 7) / 8 * 8 : groups, MOVE_GROUPS);
    a.in_x = in_x;
    const dim3 grid(PARTS > 1 ? in_x * S : groups, PARTS > 1 ? blocks_for(groups, in_x) : 1u), block(256);
    if (vec == 4) hipLaunchKernelGGL((move_rows_kernel<4, DIR, PARTS>), grid, block, 0, st, a);
    else if (vec == 2) hipLaunchKernelGGL((move_rows_kernel<2, DIR, PARTS>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((move_rows_kernel<1, DIR, PARTS>), grid, block, 0, st, a);
}

void launch_get_rows(const RowPart* parts, uint32_t S, float* dst, uint32_t pitch, const uint32_t* rows,
                     uint32_t m, uint32_t V, hipStream_t st) {
    if (S == 1) launch_move_rows<MOVE_OUT, 1>(parts, S, dst, pitch, rows, m, V, st);
    else launch_move_rows<MOVE_OUT, ROW_PARTS_MAX>(parts, S, dst, pitch, rows, m, V, st);
}

void launch_set_rows(const RowPart& part, const float* src, const uint32_t* rows, uint32_t m, uint32_t V,
                     hipStream_t st) {
    launch_move_rows<MOVE_IN, 1>(&part, 1, const_cast<float*>(src), part.width, rows, m, V, st);
}

// ---------------------------------------------------------------------------------------------
// Destination keys: slot 0 of pair p is its positive output word, slot j >= 1 its j-th negative.
// A negative is the first alias-table candidate (attempt t = 0..15, Philox counter (p, j, t, NEG))
// that differs from the positive word; after 16 rejections it is the next word index, cyclically.
// One thread per slot, so the generator runs with all 64 lanes busy.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void dest_key_item(const uint2* __restrict__ bins, uint32_t V,
                                              const uint32_t* __restrict__ out_idx, uint32_t n,
                                              uint32_t T, uint32_t k0, uint32_t k1,
                                              uint32_t* __restrict__ keys, uint32_t* err, uint32_t i) {
    if (i >= n * T) return;
    uint32_t p = i / T, j = i - p * T;
    uint32_t wo = out_idx[p];
    if (wo >= V) { wo = 0; if (j == 0) atomicOr(err, 1u); }
    uint32_t key;
    if (j == 0) {
        key = wo;
    } else {
        key = wo + 1 == V ? 0u : wo + 1;           // the fallback
        for (uint32_t t = 0; t < 16; ++t) {
            U4 r = philox4x32_10(p, j, t, DOM_NEG, k0, k1);
            uint64_t r64 = ((uint64_t)r.y << 32) | (uint64_t)r.x;
            uint32_t bin = (uint32_t)__umul64hi(r64, (uint64_t)V);
            uint2 b = bins[bin];
            uint32_t cand = (r.z < b.x) ? bin : b.y;
            if (cand != wo) { key = cand; break; }
        }
    }
    keys[i] = key;
}

__global__ __launch_bounds__(256) void dest_keys_kernel(const uint2* __restrict__ bins, uint32_t V,
                                                        const uint32_t* __restrict__ out_idx,
                                                        uint32_t n, uint32_t T, uint32_t k0,
                                                        uint32_t k1, uint32_t* __restrict__ keys,
                                                        uint32_t* err) {
    dest_key_item(bins, V, out_idx, n, T, k0, k1, keys, err, blockIdx.x * 256 + threadIdx.x);
}

// After the sort of the destination keys: an entry whose two neighbours carry other keys is the
// only slot of the minibatch that names its row.  Such slots get KEY_ALONE set in the slot-ordered
// key array (each slot is written by at most one thread), so that the input-side kernel, which
// holds everything the row's update needs, can write it, and the output side can leave it out.
__global__ __launch_bounds__(256) void mark_alone_kernel(const uint32_t* __restrict__ skey,
                                                         const uint32_t* __restrict__ sidx,
                                                         uint32_t M, uint32_t* __restrict__ keys) {
    uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= M) return;
    const uint32_t k = skey[i], before = skey[max(i, 1u) - 1], after = skey[min(i + 1, M - 1)], slot = sidx[i];
    const bool left = i > 0 && before == k;
    const bool right = i + 1 < M && after == k;
    if (!left && !right) keys[slot] = k | KEY_ALONE;
}

void launch_dest_keys(NoiseTable nt, const uint32_t* out_idx, uint32_t n, uint32_t k, uint64_t seed,
                      uint32_t* keys, uint32_t* err, hipStream_t st) {
    if (n == 0) return;
    uint32_t T = k + 1;
    hipLaunchKernelGGL(dest_keys_kernel, dim3(blocks_for((uint64_t)n * T, 256)), dim3(256), 0, st,
                       nt.bins, nt.V, out_idx, n, T, (uint32_t)seed, (uint32_t)(seed >> 32), keys,
                       err);
}

void launch_mark_alone(const uint32_t* skey, const uint32_t* sidx, uint32_t M, uint32_t* keys,
                       hipStream_t st) {
    if (M == 0) return;
    hipLaunchKernelGGL(mark_alone_kernel, dim3(blocks_for(M, 256)), dim3(256), 0, st, skey, sidx, M,
                       keys);
}

// Range-checked copy of the input words: an index >= V raises *err and is replaced by word 0, so no
// later kernel can be sent outside the matrices.
__device__ __forceinline__ void check_input_item(const uint32_t* __restrict__ in_idx, uint32_t n,
                                                 uint32_t V, uint32_t* __restrict__ in_safe,
                                                 uint32_t* err, uint32_t p) {
    if (p >= n) return;
    uint32_t wi = in_idx[p];
    if (wi >= V) { atomicOr(err, 1u); wi = 0; }
    in_safe[p] = wi;
}

__global__ __launch_bounds__(256) void check_inputs_kernel(const uint32_t* __restrict__ in_idx,
                                                           uint32_t n, uint32_t V,
                                                           uint32_t* __restrict__ in_safe,
                                                           uint32_t* err) {
    check_input_item(in_idx, n, V, in_safe, err, blockIdx.x * 256 + threadIdx.x);
}

void launch_check_inputs(const uint32_t* in_idx, uint32_t n, uint32_t V, uint32_t* in_safe,
                         uint32_t* err, hipStream_t st) {
    if (n == 0) return;
    hipLaunchKernelGGL(check_inputs_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, in_idx, n, V,
                       in_safe, err);
}

// The index work that depends on nothing but the call's arguments, in ONE launch: destination
// keys, checked input words and up to two plain fills (the sort's counters, the output side's
// border slots).  Each block does one part, told by its number.  A step of a few thousand pairs is
// a chain of dependent launches of a few microseconds each, and these were four of them.
__global__ __launch_bounds__(256) void index_prologue_kernel(IndexPrologue a) {
    const uint32_t b = blockIdx.x;
    if (b < a.b_check) {
        dest_key_item(a.nt.bins, a.nt.V, a.out_idx, a.n, a.T, a.seed_lo, a.seed_hi, a.keys, a.err,
                      b * 256 + threadIdx.x);
    } else if (b < a.b_fill[0]) {
        check_input_item(a.in_idx, a.n, a.nt.V, a.in_safe, a.err, (b - a.b_check) * 256 + threadIdx.x);
    } else {
        const int f = b < a.b_fill[1] ? 0 : 1;
        const uint32_t i = (b - a.b_fill[f]) * 256 + threadIdx.x;
        if (i < a.fill[f].count) a.fill[f].p[i] = a.fill[f].value;
    }
}

void launch_index_prologue(IndexPrologue a, hipStream_t st) {
    if (a.n == 0) { a.fill[0].count = 0; a.fill[1].count = 0; }   // (no pairs: nothing follows)
    a.b_check = blocks_for((uint64_t)a.n * a.T, 256);
    a.b_fill[0] = a.b_check + blocks_for(a.n, 256);
    a.b_fill[1] = a.b_fill[0] + blocks_for(a.fill[0].count, 256);
    const uint32_t blocks = a.b_fill[1] + blocks_for(a.fill[1].count, 256);
    if (blocks == 0) return;
    hipLaunchKernelGGL(index_prologue_kernel, dim3(blocks), dim3(256), 0, st, a);
}

__global__ __launch_bounds__(256) void copy_negatives_kernel(const uint32_t* __restrict__ keys,
                                                             uint32_t n, uint32_t k,
                                                             uint32_t* __restrict__ neg) {
    uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n * k) return;
    uint32_t p = i / k, j = i - p * k;
    neg[i] = keys[p * (k + 1) + 1 + j];
}

void launch_copy_negatives(const uint32_t* keys, uint32_t n, uint32_t k, uint32_t* neg,
                           hipStream_t st) {
    if (n == 0 || k == 0) return;
    hipLaunchKernelGGL(copy_negatives_kernel, dim3(blocks_for((uint64_t)n * k, 256)), dim3(256), 0,
                       st, keys, n, k, neg);
}

// ---------------------------------------------------------------------------------------------
// Gather dot products: one lane group per pair.  The group loads u once, then the T output rows in
// batches of TB with every load of a batch issued before the first multiply.
// ---------------------------------------------------------------------------------------------
constexpr int DOT_THREADS = 128;     // (256: the kernel 40 % slower beside other work, 64: the same)
template <int G, int NV, int TB, bool FULL>
__global__ __launch_bounds__(DOT_THREADS) void dots_kernel(const float4* __restrict__ Um, const float4* __restrict__ Wm, RowGeom g,
                                                   const uint32_t* __restrict__ in_idx,
                                                   const uint32_t* __restrict__ keys, uint32_t n,
                                                   uint32_t T, float* __restrict__ dots) {
    const int l = threadIdx.x % G;
    const uint32_t grp = group_value<G>((blockIdx.x * (uint32_t)DOT_THREADS + threadIdx.x) / G);
    const bool live = grp < n;
    const uint32_t p = live ? grp : n - 1;
    const Rows<G, NV, OneMatrix, 0> U(OneMatrix{}, Um, g, l);
    const Rows<G, NV, OneMatrix, 1> W(OneMatrix{}, Wm, g, l);
    const uint32_t in[1] = {group_value<G>(in_idx[p])};      // already range-checked (launch_check_inputs)
    float4 u[1][NV], w[TB][NV];
    for (uint32_t jb = 0; jb < T; jb += TB) {
        const uint32_t slots = FULL ? TB : min((uint32_t)TB, T - jb);      // (FULL: T is a multiple of TB)
        uint32_t row[TB];                                    // (a prepared set's keys may carry the mark)
#pragma unroll
        for (int t = 0; t < TB; ++t) row[t] = group_value<G>(keys[p * T + min(jb + t, T - 1)]);
        if (jb == 0) U.template load_all<false>(in, 1u, u);
        W.template load_all<false>(row, slots, w);
        float s[TB];
#pragma unroll
        for (int t = 0; t < TB; ++t) s[t] = dot_part_of<NV>(W, u[0], w[t]);
#pragma unroll
        for (int t = 0; t < TB; ++t) s[t] = group_sum<G>(s[t]);
#pragma unroll
        for (int t = 0; t < TB; ++t)
            if (l == t && live && (uint32_t)t < slots) dots[p * T + jb + t] = s[t];
    }
}

void launch_dots(const float* U, const float* W, RowGeom g, const uint32_t* in_idx,
                 const uint32_t* keys, uint32_t n, uint32_t T, float* dots, hipStream_t st) {
    if (n == 0) return;
#define CALL_BATCH(G, NV, TB, FULL)                                                               \
    hipLaunchKernelGGL((dots_kernel<G, NV, TB, FULL>),                                            \
                       dim3(blocks_for((uint64_t)n * G, DOT_THREADS)), dim3(DOT_THREADS), 0, st, (const float4*)U, \
                       (const float4*)W, g, in_idx, keys, n, T, dots)
#define CALL(G, NV)                                                                               \
    do {                                                                                          \
        constexpr int TB = NV <= 2 ? 6 : 4;                                                       \
        if (T % TB) CALL_BATCH(G, NV, TB, false); else CALL_BATCH(G, NV, TB, true);               \
    } while (0)
    W2V_DISPATCH_GEOM(g.d4, CALL);
#undef CALL
#undef CALL_BATCH
}

// ---------------------------------------------------------------------------------------------
// Client step between the two calls: f = sum over shards of the partial dots (shard order), then
// the coefficient label - sigma(f), written as sigma(-f) for the positive slot so that it keeps
// its relative accuracy when f is large.  Loss terms are softplus(-f) / softplus(f), summed in double
// in a fixed order, per block and then over the blocks.
// Bound by what it issues: two exponentials, a logarithm and a division a slot, once for both kinds of slot (each
// evaluated for all lanes, with a remainder by T a slot, 6.3 M slots took 52 us; now 33; reading and writing them
// takes 11).
// ---------------------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void coeffs_kernel(PartialPtrs parts, uint32_t S, uint32_t total,
                                                     uint32_t T, float* __restrict__ coeffs,
                                                     double* __restrict__ block_loss) {
    __shared__ double red[4];
    const uint32_t terms = loss_terms_of(total), lo = blockIdx.x * terms, hi = min(total - lo, terms) + lo;
    double sum = 0.0;
    SlotInPair slot(lo + threadIdx.x, T, 256);
    for (uint32_t i0 = lo + threadIdx.x; i0 < hi; i0 += 4 * 256) {
        float f[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t i = i0 + e * 256;
            f[e] = 0.f;
            for (uint32_t s = 0; s < S; ++s) f[e] += i < hi ? parts.p[s][i] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t i = i0 + e * 256;
            const bool positive = slot.first();
            const float x = positive ? f[e] : -f[e], g = 1.0f / (1.0f + expf(x));
            if (i < hi) {
                coeffs[i] = positive ? g : -g;
                if (block_loss) sum += (double)softplus(-x);
            }
            slot.next();
        }
    }
    if (block_loss) {
        const double s = block_tree_sum<256>(sum, red);
        if (threadIdx.x == 0) block_loss[blockIdx.x] = s;
    }
}

__global__ __launch_bounds__(256) void sum_doubles_kernel(const double* __restrict__ x, uint32_t n,
                                                          double* __restrict__ out) {
    __shared__ double red[4];
    sum_doubles_block<256>(x, n, out, red);
}

static void launch_sum_doubles(const double* x, uint32_t n, double* out, hipStream_t st) {
    hipLaunchKernelGGL(sum_doubles_kernel, dim3(1), dim3(256), 0, st, x, n, out);
}

// doubles of scratch for the loss: one per block of terms (most blocks: at the end of the short ones)
size_t coeffs_loss_scratch_doubles(uint32_t n, uint32_t T) {
    const uint32_t total = n * T, short_total = std::min(total, LOSS_SHORT_TERMS);
    return std::max(blocks_for(total, loss_terms_of(total)), blocks_for(short_total, loss_terms_of(short_total))) + 8;
}

void launch_coeffs(PartialPtrs parts, uint32_t S, uint32_t n, uint32_t T, float* coeffs,
                   double* block_loss, double* loss_out, hipStream_t st) {
    uint32_t total = n * T;
    if (total == 0) {
        if (loss_out) launch_sum_doubles(nullptr, 0, loss_out, st);
        return;
    }
    unsigned nb = blocks_for(total, loss_terms_of(total));
    hipLaunchKernelGGL(coeffs_kernel, dim3(nb), dim3(256), 0, st, parts, S, total, T, coeffs,
                       loss_out ? block_loss : (double*)nullptr);
    if (loss_out) launch_sum_doubles(block_loss, nb, loss_out, st);
}

// Minibatch loss of the fused step, from the dots the input-side kernel leaves behind: the same
// softplus terms as coeffs_kernel, so that the fused and the unfused form of a step report the
// same loss, finite however far sigma saturates.
__global__ __launch_bounds__(256) void loss_from_dots_kernel(const float* __restrict__ dots,
                                                             uint32_t total, uint32_t T,
                                                             double* __restrict__ block_loss) {
    __shared__ double red[4];
    loss_terms_block<256>(dots, total, T, block_loss, blockIdx.x, red);
}

void launch_loss_from_dots(const float* dots, uint32_t n, uint32_t T, double* tmp, double* loss_out,
                           hipStream_t st) {
    uint32_t total = n * T;
    if (total == 0) { launch_sum_doubles(nullptr, 0, loss_out, st); return; }
    unsigned nb = blocks_for(total, loss_terms_of(total));
    hipLaunchKernelGGL(loss_from_dots_kernel, dim3(nb), dim3(256), 0, st, dots, total, T, tmp);
    launch_sum_doubles(tmp, nb, loss_out, st);
}

}  // namespace w2v
