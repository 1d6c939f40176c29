// Client-side pair formation on the device (Eq.1's index sets): subsample each token, then pair
// every surviving center with the surviving tokens at most b positions away inside its sentence,
// b uniform on 1..B per center.  Three passes:
//   draws   : per token, keep flag and b from Philox(counter = (position lo, position hi, epoch,
//             TOKEN)): word 0 < keep threshold keeps the token; b = 1 + ((word 1 * B) >> 32).  The flags of
//             64 tokens are one word, with the survivors before it in its tile; a scan of the tiles' survivors
//             is all that stands between this and the number of any survivor (survivors_before)
//   compact : surviving tokens get consecutive numbers; each learns the range
//             of surviving neighbours it pairs with and how many pairs that is; pairs are counted
//             per PAIR_BLOCK survivors on the way
//   emit    : a block takes PAIR_BLOCK centers, adds up the counts of the blocks before it (of long texts
//             these are scanned first), scans its own pair counts in LDS and writes its stretch of the output
//             one pair per thread
// A block of two million tokens is a chain of four launches bound by their latencies and, in emit, by
// the 8 bytes a pair has to be written.  (One center per thread with a serial loop over its pairs, full
// scans around it: ten launches, 265 us for 2^21 tokens; six launches, with a scan of the flags and one of the pair
// counts, 118; now 81.)
#include "common.h"

namespace w2v {

static inline unsigned blocks_for(uint64_t items, unsigned per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

constexpr uint32_t PAIR_BLOCK = 256;             // centers per block of the emission
// Up to as many such blocks each adds up the counts before it, past that they are scanned, a launch more.  (Every token
// surviving, added up and scanned, us: 2^21 tokens 89, 94; 2^22 147, 152; 2^23 329, 297.)
constexpr uint32_t PAIR_SUM_BLOCKS = 16384;
constexpr uint32_t DRAW_TILE = 2048;             // tokens of a block of the draws
constexpr uint32_t DRAW_WORDS = DRAW_TILE / 64;
constexpr uint32_t COMPACT_TOKENS = 1024;        // tokens of a block of the compaction
constexpr uint32_t COMPACT_SENTS = 256;          // sentences of such a block that are held in LDS

// Which tokens survive.  (words and tiles cover position n_tokens too: survivors_before(n_tokens) is their number.)
struct Survivors {
    const uint64_t* flags;           // bit t % 64 of word t / 64
    const uint32_t* in_tile;         // survivors of the word's tile before the word
    const uint32_t* before_tile;     // survivors before each tile (scanned sums)
};
__device__ __forceinline__ uint32_t survivors_before(const Survivors& s, uint32_t t) {
    const uint32_t w = t / 64;
    return s.before_tile[t / DRAW_TILE] + s.in_tile[w] + (uint32_t)__popcll(s.flags[w] & ((1ull << (t % 64)) - 1ull));
}

// Pairs and examples per PAIR_BLOCK survivors.
struct PairSums { uint32_t *pairs, *ex; };

// (one random 8-byte read per token, eight of them in flight)
__global__ __launch_bounds__(256) void token_draws_kernel(const uint32_t* __restrict__ tokens,
                                                          uint32_t n_tokens, uint64_t token_base,
                                                          uint32_t epoch, uint32_t k0, uint32_t k1,
                                                          uint32_t B,
                                                          const uint64_t* __restrict__ keep,
                                                          uint32_t V, uint32_t* __restrict__ fw,
                                                          uint64_t* __restrict__ flags,
                                                          uint32_t* __restrict__ in_tile,
                                                          uint32_t* __restrict__ sums,
                                                          uint32_t* __restrict__ clear, uint32_t n_clear,
                                                          uint32_t* err) {
    constexpr int ITEMS = DRAW_TILE / 256;
    __shared__ uint32_t s_kept[DRAW_WORDS];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    const uint64_t t0 = (uint64_t)blockIdx.x * DRAW_TILE + threadIdx.x;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n_clear; i += gridDim.x * 256) clear[i] = 0;
    uint32_t w[ITEMS], x[ITEMS];
    uint64_t th[ITEMS];
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) w[e] = t0 + e * 256 < n_tokens ? tokens[t0 + e * 256] : 0u;
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        if (w[e] >= V) { atomicOr(err, 1u); w[e] = 0; }
        th[e] = keep ? keep[w[e]] : ~0ull;
    }
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        const uint64_t gpos = token_base + t0 + e * 256;
        const U4 r = philox4x32_10((uint32_t)gpos, (uint32_t)(gpos >> 32), epoch, DOM_TOKEN, k0, k1);
        x[e] = r.x;
        if (t0 + e * 256 < n_tokens) fw[t0 + e * 256] = 1u + (uint32_t)(((uint64_t)r.y * (uint64_t)B) >> 32);
    }
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        const uint64_t kept = __ballot(t0 + e * 256 < n_tokens && (uint64_t)x[e] < th[e]);
        if (lane == 0) {
            flags[(uint64_t)blockIdx.x * DRAW_WORDS + e * 4 + wave] = kept;
            s_kept[e * 4 + wave] = (uint32_t)__popcll(kept);
        }
    }
    __syncthreads();
    if (threadIdx.x < DRAW_WORDS) {
        uint32_t before = 0;
#pragma unroll
        for (uint32_t i = 0; i < DRAW_WORDS; ++i) before += i < threadIdx.x ? s_kept[i] : 0u;
        in_tile[(uint64_t)blockIdx.x * DRAW_WORDS + threadIdx.x] = before;
        if (threadIdx.x == DRAW_WORDS - 1) sums[blockIdx.x] = before + s_kept[threadIdx.x];
    }
}

// The last s in 0 .. n_sent - 1 with sent_off[s] <= t (0 if there is none): one wavefront, 64 probes a step.
__device__ __forceinline__ uint32_t wave_sentence(const uint64_t* __restrict__ sent_off, uint32_t n_sent,
                                                  uint64_t t) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t lo = 0, hi = n_sent;                 // invariant: sent_off[lo] <= t < sent_off[hi]
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + 63) / 64;
        const uint64_t at = (uint64_t)lo + (uint64_t)(lane + 1) * step;
        const uint32_t below = (uint32_t)__popcll(__ballot(at < hi && sent_off[at < hi ? at : lo] <= t));
        const uint64_t next = (uint64_t)lo + (uint64_t)below * step;
        lo = (uint32_t)next;
        hi = next + step < hi ? (uint32_t)(next + step) : hi;
    }
    return lo;
}

__device__ __forceinline__ uint32_t wave_add(uint32_t x) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) x += __shfl_xor(x, s, 64);
    return x;
}

// Bound by latency: the search for the block's first and last sentence, its sentences' offsets, the survivors
// before them, then everything else out of LDS.  (A block of 256 tokens that bisected the offsets in memory, a
// chain of some fourteen reads, 22 us for 2^21 tokens; this way 19.)
__global__ __launch_bounds__(256) void compact_kernel(const uint32_t* __restrict__ tokens,
                                                      uint32_t n_tokens,
                                                      const uint64_t* __restrict__ sent_off,
                                                      uint32_t n_sent,
                                                      const uint32_t* __restrict__ fw, Survivors sv,
                                                      uint32_t V, uint32_t* __restrict__ kword,
                                                      uint32_t* __restrict__ klo,
                                                      uint32_t* __restrict__ kcnt,
                                                      uint32_t* __restrict__ kj, PairSums out) {
    constexpr int ITEMS = COMPACT_TOKENS / 256;
    constexpr uint32_t PARTS = COMPACT_TOKENS / PAIR_BLOCK + 1;   // stretches of PAIR_BLOCK survivors it reaches into
    __shared__ uint32_t s_sent[2], s_sum[PARTS], s_ex[PARTS], s_off[COMPACT_SENTS + 1], s_num[COMPACT_SENTS + 1];
    const uint32_t t0 = blockIdx.x * COMPACT_TOKENS, lane = threadIdx.x & 63;
    // (asked for ahead of the search)
    uint32_t word[ITEMS], width[ITEMS], q[ITEMS];
    bool kept[ITEMS];
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        const uint32_t t = t0 + e * 256 + threadIdx.x;       // (below 2^32: 2 B n_tokens is)
        const bool in = t < n_tokens;
        word[e] = in ? tokens[t] : 0u;
        width[e] = in ? fw[t] : 0u;
        kept[e] = in && ((sv.flags[t / 64] >> (t % 64)) & 1ull);
        q[e] = in ? survivors_before(sv, t) : 0u;
    }
    const uint32_t first = survivors_before(sv, t0) / PAIR_BLOCK;
    if (threadIdx.x < 128) {                      // sentences of the block's first and last token
        const uint32_t which = threadIdx.x / 64;
        const uint32_t s = wave_sentence(sent_off, n_sent, which ? min(t0 + COMPACT_TOKENS - 1, n_tokens - 1) : t0);
        if (lane == 0) s_sent[which] = s;
    }
    if (threadIdx.x < PARTS) { s_sum[threadIdx.x] = 0; s_ex[threadIdx.x] = 0; }
    __syncthreads();
    const uint32_t s0 = s_sent[0], count = s_sent[1] >= s0 ? s_sent[1] - s0 + 1 : 1u;      // (at most n_sent - s0)
    const bool held = count <= COMPACT_SENTS;
    auto clamped = [&](uint64_t off) { return off < n_tokens ? (uint32_t)off : n_tokens; };  // never past the flags
    if (held) {
        for (uint32_t i = threadIdx.x; i <= count; i += 256) {
            const uint32_t off = clamped(sent_off[s0 + i]);
            s_off[i] = off;
            s_num[i] = survivors_before(sv, off);
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        const uint32_t t = t0 + e * 256 + threadIdx.x;
        uint32_t pairs = 0, part = 0;
        if (kept[e]) {
            uint32_t begin, end, lo = 0, hi = count;
            if (held) {
                while (hi > lo + 1) {
                    const uint32_t mid = lo + (hi - lo) / 2;
                    if (s_off[mid] <= t) lo = mid; else hi = mid;
                }
                begin = s_num[lo]; end = s_num[lo + 1];
            } else {
                while (hi > lo + 1) {
                    const uint32_t mid = lo + (hi - lo) / 2;
                    if (sent_off[s0 + mid] <= (uint64_t)t) lo = mid; else hi = mid;
                }
                begin = survivors_before(sv, clamped(sent_off[s0 + lo]));
                end = survivors_before(sv, clamped(sent_off[s0 + lo + 1]));
            }
            const uint32_t j = q[e] - begin, m = end - begin, b = width[e];
            const uint32_t left = j < b ? j : b, right = (m - 1 - j) < b ? (m - 1 - j) : b;
            kword[q[e]] = word[e] < V ? word[e] : 0u;
            klo[q[e]] = q[e] - left;
            kcnt[q[e]] = left + right;
            if (kj) kj[q[e]] = j;                 // position among the sentence's survivors
            pairs = left + right;
            part = min(q[e] / PAIR_BLOCK - first, PARTS - 1);
        }
        // a wavefront's 64 tokens reach into two stretches at most
        const uint64_t some = __ballot(kept[e]);
        if (some == 0) continue;
        const uint32_t p0 = (uint32_t)__builtin_amdgcn_readlane((int)part, __builtin_ctzll(some));
        const uint64_t next = __ballot(kept[e] && part != p0), with = __ballot(pairs > 0);
        const uint32_t all = wave_add(pairs), later = next ? wave_add(part != p0 ? pairs : 0u) : 0u;
        if (lane == 0) {
            atomicAdd(&s_sum[p0], all - later);
            atomicAdd(&s_ex[p0], (uint32_t)__popcll(with & ~next));
            if (next) {
                atomicAdd(&s_sum[min(p0 + 1, PARTS - 1)], later);
                atomicAdd(&s_ex[min(p0 + 1, PARTS - 1)], (uint32_t)__popcll(with & next));
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < PARTS && s_sum[threadIdx.x]) {
        if (out.pairs) atomicAdd(&out.pairs[first + threadIdx.x], s_sum[threadIdx.x]);
        if (out.ex) atomicAdd(&out.ex[first + threadIdx.x], s_ex[threadIdx.x]);
    }
}

__global__ __launch_bounds__(256) void set_u32_kernel(uint32_t* __restrict__ x, uint32_t n,
                                                      uint32_t value) {
    uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) x[i] = value;
}

// Interleaved order: pairs per PAIR_BLOCK survivors taken in the order perm[0], perm[1], ...
__global__ __launch_bounds__(256) void permuted_sums_kernel(const uint32_t* __restrict__ kcnt,
                                                            const uint32_t* __restrict__ perm,
                                                            const uint32_t* __restrict__ n_kept,
                                                            uint32_t* __restrict__ pair_sums) {
    __shared__ uint32_t s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    const uint32_t r = blockIdx.x * PAIR_BLOCK + threadIdx.x;
    if (r < *n_kept) atomicAdd(&s_sum, kcnt[perm[r]]);
    __syncthreads();
    if (threadIdx.x == 0) pair_sums[blockIdx.x] = s_sum;
}

// Bag-of-words examples on top of the pair stream: a center with pairs is an example, its pairs' output
// words are its context.  (ctx_off null: pairs only)
struct ExampleOut { uint32_t* ctx_off; uint32_t* centers; uint64_t capacity; };

// The sum of the first b counts.  Every thread calls it; s_part holds one word per wavefront.
__device__ __forceinline__ uint32_t sum_before(const uint32_t* __restrict__ counts, uint32_t b, uint32_t* s_part) {
    uint32_t x = 0;
#pragma unroll 8
    for (uint32_t i = threadIdx.x; i < b; i += 256) x += counts[i];
    x = wave_add(x);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x / 64] = x;
    __syncthreads();
    return s_part[0] + s_part[1] + s_part[2] + s_part[3];
}

// totals[0], totals[1]: all pairs and examples, for the host.  `scanned`: the sums are those of the blocks before
// each, and the totals stand behind them.
constexpr uint32_t EMIT_OWNERS = 6144;           // pairs of a block whose centers are looked up, not searched for
__global__ __launch_bounds__(256) void emit_pairs_kernel(const uint32_t* __restrict__ kword,
                                                         const uint32_t* __restrict__ klo,
                                                         const uint32_t* __restrict__ kcnt,
                                                         PairSums sums, uint32_t n_blocks, bool scanned,
                                                         const uint32_t* __restrict__ n_kept,
                                                         const uint32_t* __restrict__ perm,
                                                         uint32_t* __restrict__ in_idx,
                                                         uint32_t* __restrict__ out_idx,
                                                         uint64_t capacity, ExampleOut ex, uint32_t* totals) {
    static_assert(PAIR_BLOCK == 256, "a center per thread");
    __shared__ uint32_t s_off[PAIR_BLOCK + 1], s_q[PAIR_BLOCK], s_lo[PAIR_BLOCK], s_w[PAIR_BLOCK], s_wave[4], s_exw[4];
    __shared__ uint32_t s_before[2][4], s_all[2][4];
    __shared__ uint8_t s_owner[EMIT_OWNERS];
    const uint32_t kept = *n_kept, r = blockIdx.x * PAIR_BLOCK + threadIdx.x;   // place in the order of emission
    if (blockIdx.x == 0) {                                   // (uniform per block)
        uint32_t pairs, examples = 0;
        if (scanned) {
            pairs = sums.pairs[n_blocks];
            if (ex.ctx_off) examples = sums.ex[n_blocks];
        } else {
            pairs = sum_before(sums.pairs, n_blocks, s_all[0]);
            if (ex.ctx_off) examples = sum_before(sums.ex, n_blocks, s_all[1]);
        }
        if (threadIdx.x == 0) {
            totals[0] = pairs; totals[1] = examples;
            if (ex.ctx_off) ex.ctx_off[0] = 0;
        }
    }
    if (blockIdx.x * PAIR_BLOCK >= kept) return;             // uniform per block
    uint32_t cnt = 0;
    if (r < kept) {
        const uint32_t q = perm ? perm[r] : r;               // which survivor is the center
        cnt = kcnt[q];
        s_q[threadIdx.x] = q; s_lo[threadIdx.x] = klo[q]; s_w[threadIdx.x] = kword[q];
    }
    const uint64_t start = scanned ? sums.pairs[blockIdx.x] : sum_before(sums.pairs, blockIdx.x, s_before[0]);
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    uint32_t incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d, 64);
        if (lane >= (uint32_t)d) incl += y;
    }
    const uint64_t some = __ballot(cnt > 0);
    if (lane == 63) { s_wave[wave] = incl; s_exw[wave] = (uint32_t)__popcll(some); }
    __syncthreads();
    uint32_t before = 0, examples = 0;
    for (uint32_t w = 0; w < wave; ++w) { before += s_wave[w]; examples += s_exw[w]; }
    const uint32_t total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3], off = before + incl - cnt;
    const bool listed = total <= EMIT_OWNERS;
    s_off[threadIdx.x] = off;
    if (threadIdx.x == 255) s_off[PAIR_BLOCK] = before + incl;
    if (listed)
        for (uint32_t o = off; o < off + cnt; ++o) s_owner[o] = (uint8_t)threadIdx.x;
    if (ex.ctx_off) {
        examples += scanned ? sums.ex[blockIdx.x] : sum_before(sums.ex, blockIdx.x, s_before[1]);
        const uint64_t x = (uint64_t)examples + (uint32_t)__popcll(some & ((1ull << lane) - 1ull));
        if (cnt > 0 && x < ex.capacity) {                    // this center's example
            ex.centers[x] = s_w[threadIdx.x];
            ex.ctx_off[x + 1] = (uint32_t)start + before + incl;
        }
    }
    __syncthreads();
    for (uint32_t o = threadIdx.x; o < total; o += 256) {
        uint32_t i = 0;                                      // the last center whose pairs begin at or before o
        if (listed) {
            i = s_owner[o];
        } else {
#pragma unroll
            for (uint32_t step = PAIR_BLOCK / 2; step; step >>= 1)
                if (s_off[i + step] <= o) i += step;
        }
        uint32_t c = s_lo[i] + (o - s_off[i]);               // its neighbours, itself left out
        if (c >= s_q[i]) ++c;
        const uint64_t at = start + o;
        if (at < capacity && c < kept) {                     // (c < kept holds for well-formed sentences)
            if (in_idx) in_idx[at] = s_w[i];
            out_idx[at] = kword[c];
        }
    }
}

// The scratch of one formation, in a fixed order; every part grows with the number of tokens.
struct PairPlan {
    uint32_t tiles, n_blocks;
    uint64_t* flags; uint32_t *in_tile, *tile_sums, *n_kept, *fw;
    PairSums sums; uint32_t n_sums;                  // cleared by the draws, from sums.pairs on
    uint32_t *kword, *klo, *kcnt;
    uint32_t *kj, *sort_tmp; uint2 *b0, *b1;         // interleaved order
    size_t u32;
};
static PairPlan make_pair_plan(uint32_t* base, uint32_t n, bool interleave) {
    PairPlan p{};
    size_t at = 0;
    auto take = [&](size_t count) {                  // (8-byte aligned)
        uint32_t* r = base ? base + at : nullptr;
        at += (count + 1) & ~(size_t)1;
        return r;
    };
    p.tiles = blocks_for((uint64_t)n + 1, DRAW_TILE);
    p.n_blocks = blocks_for(n, PAIR_BLOCK);
    p.flags = (uint64_t*)take((size_t)p.tiles * DRAW_WORDS * 2);
    p.in_tile = take((size_t)p.tiles * DRAW_WORDS);
    p.tile_sums = take(p.tiles);
    p.n_kept = take(1);
    const size_t first = at;
    p.sums.pairs = take((size_t)p.n_blocks + 1);     // (and their total)
    p.sums.ex = take((size_t)p.n_blocks + 1);
    p.n_sums = (uint32_t)(at - first);
    p.fw = take(n);
    p.kword = take(n); p.klo = take(n); p.kcnt = take(n);
    if (interleave) {
        p.kj = take(n);
        p.b0 = (uint2*)take(2 * (size_t)n); p.b1 = (uint2*)take(2 * (size_t)n);
        p.sort_tmp = take(sort_scratch_u32(n));
    }
    p.u32 = at;
    return p;
}

size_t pairs_scratch_u32(uint32_t n_tokens, bool interleave) { return make_pair_plan(nullptr, n_tokens, interleave).u32; }

// (at least one token)
void launch_make_pairs(const PairArgs& a, hipStream_t st) {
    const uint32_t n = a.n_tokens;
    const PairPlan p = make_pair_plan(a.scratch, n, a.interleave);
    hipLaunchKernelGGL(token_draws_kernel, dim3(p.tiles), dim3(256), 0, st,
                       a.tokens, n, a.token_base, a.epoch, (uint32_t)a.seed,
                       (uint32_t)(a.seed >> 32), a.B, a.keep, a.V, p.fw, p.flags, p.in_tile, p.tile_sums,
                       p.sums.pairs, p.n_sums, a.err);
    launch_scan_sums(p.tile_sums, p.tiles, p.n_kept, st);
    const Survivors sv{p.flags, p.in_tile, p.tile_sums};
    const dim3 grid(blocks_for(n, 256)), block(256);
    if (a.interleave) hipLaunchKernelGGL(set_u32_kernel, grid, block, 0, st, p.kj, n, n);   // sorts last
    PairSums counted = p.sums;
    if (a.interleave) counted.pairs = nullptr;       // (counted in the order of emission)
    if (!a.ctx_off) counted.ex = nullptr;
    hipLaunchKernelGGL(compact_kernel, dim3(blocks_for(n, COMPACT_TOKENS)), block, 0, st, a.tokens, n, a.sent_off,
                       a.n_sent, p.fw, sv, a.V, p.kword, p.klo, p.kcnt, p.kj, counted);
    uint32_t *sk = nullptr, *perm = nullptr;
    if (a.interleave) {
        // Round-robin over the sentences: a stable sort of the survivors by their position within the
        // sentence keeps the sentences in order among equal positions.
        uint32_t bits = 1;
        while (bits < 32 && (1ull << bits) <= (uint64_t)n) ++bits;
        launch_sort_pairs(p.kj, p.b0, p.b1, n, bits, p.sort_tmp, &sk, &perm, a.err, st);
        hipLaunchKernelGGL(permuted_sums_kernel, grid, block, 0, st, p.kcnt, perm, p.n_kept, p.sums.pairs);
    }
    const bool scanned = p.n_blocks > PAIR_SUM_BLOCKS;
    if (scanned) {
        launch_scan_sums(p.sums.pairs, p.n_blocks, p.sums.pairs + p.n_blocks, st);
        if (a.ctx_off) launch_scan_sums(p.sums.ex, p.n_blocks, p.sums.ex + p.n_blocks, st);
    }
    hipLaunchKernelGGL(emit_pairs_kernel, grid, block, 0, st, p.kword, p.klo, p.kcnt, p.sums, p.n_blocks, scanned, p.n_kept,
                       (const uint32_t*)perm, a.in_idx, a.out_idx, a.capacity,
                       ExampleOut{a.ctx_off, a.centers, a.cap_examples}, a.totals);
}

}  // namespace w2v
