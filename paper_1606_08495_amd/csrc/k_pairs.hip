// Client-side pair formation on the device (Eq.1's index sets): subsample each token, then pair
// every surviving center with the surviving tokens at most b positions away inside its sentence,
// b uniform on 1..B per center.  Three passes joined by two prefix sums:
//   draws   : per token, keep flag and b from Philox(counter = (position lo, position hi, epoch,
//             TOKEN)): word 0 < keep threshold keeps the token; b = 1 + ((word 1 * B) >> 32).  Counts
//             the survivors of its scan tile on the way.
//   compact : surviving tokens get consecutive numbers (scan of the flags); each learns the range
//             of surviving neighbours it pairs with and how many pairs that is; pairs are counted
//             per PAIR_BLOCK survivors on the way
//   emit    : a block takes PAIR_BLOCK centers, scans their pair counts in LDS and writes its stretch
//             of the output one pair per thread
// A block of two million tokens is a chain of six launches bound by their latencies and, in emit, by
// the 8 bytes a pair has to be written.  (One center per thread with a serial loop over its pairs, full
// scans around it: ten launches, 265 us for 2^21 tokens, 114 of them the scattered writes; now 118 and 23.)
#include "common.h"

namespace w2v {

static inline unsigned blocks_for(uint64_t items, unsigned per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

constexpr uint32_t PAIR_BLOCK = 256;             // centers per block of the emission
constexpr uint32_t FW_KEPT = 0x80000000u;        // keep flag beside the window width (B < 2^31)

__global__ __launch_bounds__(256) void token_draws_kernel(const uint32_t* __restrict__ tokens,
                                                          uint32_t n_tokens, uint64_t token_base,
                                                          uint32_t epoch, uint32_t k0, uint32_t k1,
                                                          uint32_t B,
                                                          const uint64_t* __restrict__ keep,
                                                          uint32_t V, uint32_t tile, uint32_t* __restrict__ fw,
                                                          uint32_t* __restrict__ sums,
                                                          uint32_t* __restrict__ pair_sums,
                                                          uint32_t* __restrict__ ex_sums, uint32_t n_pair_sums,
                                                          uint32_t* err) {
    __shared__ uint32_t s_kept[4];
    uint32_t kept_here = 0;
    for (uint32_t e = threadIdx.x; e < tile; e += 256) {
        const uint64_t t = (uint64_t)blockIdx.x * tile + e;
        bool kept = false;
        if (t < n_tokens) {
            uint64_t gpos = token_base + t;
            U4 r = philox4x32_10((uint32_t)gpos, (uint32_t)(gpos >> 32), epoch, DOM_TOKEN, k0, k1);
            uint32_t w = tokens[t];
            if (w >= V) { atomicOr(err, 1u); w = 0; }
            kept = keep ? ((uint64_t)r.x < keep[w]) : true;
            fw[t] = (kept ? FW_KEPT : 0u) | (1u + (uint32_t)(((uint64_t)r.y * (uint64_t)B) >> 32));
        } else if (t == n_tokens) {
            fw[t] = 0;                            // sentinel: the scan has n_tokens + 1 entries
        }
        kept_here += (uint32_t)__popcll(__ballot(kept));     // (the same in every lane of the wavefront)
    }
    if ((threadIdx.x & 63) == 0) s_kept[threadIdx.x / 64] = kept_here;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = s_kept[0] + s_kept[1] + s_kept[2] + s_kept[3];
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;       // (tile / 8 threads per tile, one sum per 256 tokens)
    if (i < n_pair_sums) { pair_sums[i] = 0; ex_sums[i] = 0; }
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

// kpos[t] = number of surviving tokens before t (exclusive scan of the flags, n_tokens+1 entries).
__global__ __launch_bounds__(256) void compact_kernel(const uint32_t* __restrict__ tokens,
                                                      uint32_t n_tokens,
                                                      const uint64_t* __restrict__ sent_off,
                                                      uint32_t n_sent,
                                                      const uint32_t* __restrict__ fw,
                                                      const uint32_t* __restrict__ kpos,
                                                      uint32_t V, uint32_t* __restrict__ kword,
                                                      uint32_t* __restrict__ klo,
                                                      uint32_t* __restrict__ kcnt,
                                                      uint32_t* __restrict__ kj,
                                                      uint32_t* __restrict__ pair_sums,
                                                      uint32_t* __restrict__ ex_sums) {
    __shared__ uint32_t s_sent[2], s_sum[2], s_ex[2];
    const uint32_t t0 = blockIdx.x * 256, t = t0 + threadIdx.x;
    if (threadIdx.x < 128) {                      // sentences of the block's first and last token
        const uint32_t which = threadIdx.x / 64;
        const uint32_t s = wave_sentence(sent_off, n_sent, which ? min(t0 + 255, n_tokens - 1) : t0);
        if ((threadIdx.x & 63) == 0) { s_sent[which] = s; s_sum[which] = 0; s_ex[which] = 0; }
    }
    __syncthreads();
    const uint32_t first = kpos[t0] / PAIR_BLOCK;            // the block's survivors lie in two stretches at most
    const uint32_t mine = t < n_tokens ? fw[t] : 0u;
    if (mine & FW_KEPT) {
        uint32_t lo = s_sent[0], hi = s_sent[1] + 1;
        while (hi > lo + 1) {
            uint32_t mid = lo + (hi - lo) / 2;
            if (sent_off[mid] <= (uint64_t)t) lo = mid; else hi = mid;
        }
        uint64_t ob = sent_off[lo], oe = sent_off[lo + 1];        // clamped: never index past kpos
        uint32_t s_begin = kpos[ob < n_tokens ? (uint32_t)ob : n_tokens];
        uint32_t s_end = kpos[oe < n_tokens ? (uint32_t)oe : n_tokens];
        uint32_t q = kpos[t];
        uint32_t j = q - s_begin, m = s_end - s_begin, b = mine & ~FW_KEPT;
        uint32_t left = j < b ? j : b;
        uint32_t right = (m - 1 - j) < b ? (m - 1 - j) : b;
        uint32_t w = tokens[t];
        kword[q] = w < V ? w : 0u;
        klo[q] = q - left;
        kcnt[q] = left + right;
        if (kj) kj[q] = j;                        // position among the sentence's survivors
        const uint32_t part = min(q / PAIR_BLOCK - first, 1u);
        atomicAdd(&s_sum[part], left + right);
        if (left + right) atomicAdd(&s_ex[part], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 2 && s_sum[threadIdx.x]) {
        if (pair_sums) atomicAdd(&pair_sums[first + threadIdx.x], s_sum[threadIdx.x]);
        if (ex_sums) atomicAdd(&ex_sums[first + threadIdx.x], s_ex[threadIdx.x]);
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
struct ExampleOut {
    const uint32_t* start;           // examples before each PAIR_BLOCK centers
    uint32_t* ctx_off; uint32_t* centers; uint64_t capacity;
};

__global__ __launch_bounds__(256) void emit_pairs_kernel(const uint32_t* __restrict__ kword,
                                                         const uint32_t* __restrict__ klo,
                                                         const uint32_t* __restrict__ kcnt,
                                                         const uint32_t* __restrict__ pair_start,
                                                         const uint32_t* __restrict__ n_kept,
                                                         const uint32_t* __restrict__ perm,
                                                         uint32_t* __restrict__ in_idx,
                                                         uint32_t* __restrict__ out_idx,
                                                         uint64_t capacity, ExampleOut ex) {
    static_assert(PAIR_BLOCK == 256, "a center per thread");
    __shared__ uint32_t s_off[PAIR_BLOCK + 1], s_q[PAIR_BLOCK], s_lo[PAIR_BLOCK], s_w[PAIR_BLOCK], s_wave[4], s_exw[4];
    const uint32_t kept = *n_kept, r = blockIdx.x * PAIR_BLOCK + threadIdx.x;   // place in the order of emission
    if (ex.ctx_off && blockIdx.x == 0 && threadIdx.x == 0) ex.ctx_off[0] = 0;
    if (blockIdx.x * PAIR_BLOCK >= kept) return;             // uniform per block
    uint32_t cnt = 0;
    if (r < kept) {
        const uint32_t q = perm ? perm[r] : r;               // which survivor is the center
        cnt = kcnt[q];
        s_q[threadIdx.x] = q; s_lo[threadIdx.x] = klo[q]; s_w[threadIdx.x] = kword[q];
    }
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
    s_off[threadIdx.x] = before + incl - cnt;
    if (threadIdx.x == 255) s_off[PAIR_BLOCK] = before + incl;
    __syncthreads();
    const uint32_t total = s_off[PAIR_BLOCK];
    const uint64_t start = pair_start[blockIdx.x];
    if (ex.ctx_off && cnt > 0) {                             // this center's example
        const uint64_t x = (uint64_t)ex.start[blockIdx.x] + examples + (uint32_t)__popcll(some & ((1ull << lane) - 1ull));
        if (x < ex.capacity) {
            ex.centers[x] = s_w[threadIdx.x];
            ex.ctx_off[x + 1] = (uint32_t)start + before + incl;
        }
    }
    for (uint32_t o = threadIdx.x; o < total; o += 256) {
        uint32_t i = 0;                                      // the last center whose pairs begin at or before o
#pragma unroll
        for (uint32_t step = PAIR_BLOCK / 2; step; step >>= 1)
            if (s_off[i + step] <= o) i += step;
        uint32_t c = s_lo[i] + (o - s_off[i]);               // its neighbours, itself left out
        if (c >= s_q[i]) ++c;
        const uint64_t at = start + o;
        if (at < capacity && c < kept) {                     // (c < kept holds for well-formed sentences)
            if (in_idx) in_idx[at] = s_w[i];
            out_idx[at] = kword[c];
        }
    }
}

// scratch layout (uint32): fw[n+1] kpos[n+1] pair_sums[n] kword[n] klo[n] kcnt[n] ex_sums[n]
// n_kept[8] scan_tmp[...]; interleaved order adds kj[n] b0[2n] b1[2n] sort_tmp[...]
size_t pairs_scratch_u32(uint32_t n_tokens, bool interleave) {
    size_t n = n_tokens;
    size_t base = 2 * (n + 1) + 5 * n + 8 + scan_scratch_u32(n_tokens + 1);
    if (interleave) base += 5 * n + 4 + sort_scratch_u32(n_tokens);
    return base;
}

// (at least one token)
void launch_make_pairs(const PairArgs& a, hipStream_t st) {
    const uint32_t n = a.n_tokens;
    uint32_t* fw = a.scratch;
    uint32_t* kpos = fw + (n + 1);
    uint32_t* pair_sums = kpos + (n + 1);            // one per PAIR_BLOCK survivors (at most n of them)
    uint32_t* kword = pair_sums + n;
    uint32_t* klo = kword + n;
    uint32_t* kcnt = klo + n;
    uint32_t* ex_sums = kcnt + n;                    // the same for examples
    uint32_t* n_kept = ex_sums + n;
    uint32_t* scan_tmp = n_kept + 8;
    uint32_t* extra = scan_tmp + scan_scratch_u32(n + 1);
    uint32_t* kj = a.interleave ? extra : nullptr;
    // sort buffers (8-byte words) and sort scratch start on 8-byte boundaries
    uint32_t* after_kj = extra + n;
    after_kj += ((uintptr_t)after_kj & 4) ? 1 : 0;
    uint2 *b0 = (uint2*)after_kj, *b1 = b0 + n;
    uint32_t* sort_tmp = (uint32_t*)(b1 + n);
    const uint32_t tiles = blocks_for((uint64_t)n + 1, scan_tile()), n_pair_sums = blocks_for(n, PAIR_BLOCK);
    hipLaunchKernelGGL(token_draws_kernel, dim3(tiles), dim3(256), 0, st,
                       a.tokens, n, a.token_base, a.epoch, (uint32_t)a.seed,
                       (uint32_t)(a.seed >> 32), a.B, a.keep, a.V, scan_tile(), fw, scan_tmp, pair_sums,
                       ex_sums, n_pair_sums, a.err);
    launch_scan_sums(scan_tmp, tiles, n_kept, st);
    launch_scan_apply(fw, kpos, n + 1, 31, scan_tmp, st);
    const dim3 grid(blocks_for(n, 256)), block(256);
    if (a.interleave) hipLaunchKernelGGL(set_u32_kernel, grid, block, 0, st, kj, n, n);   // sorts last
    hipLaunchKernelGGL(compact_kernel, grid, block, 0, st, a.tokens, n, a.sent_off, a.n_sent, fw,
                       kpos, a.V, kword, klo, kcnt, kj, a.interleave ? (uint32_t*)nullptr : pair_sums,
                       a.ctx_off ? ex_sums : (uint32_t*)nullptr);
    uint32_t *sk = nullptr, *perm = nullptr;
    if (a.interleave) {
        // Round-robin over the sentences: a stable sort of the survivors by their position within the
        // sentence keeps the sentences in order among equal positions.
        uint32_t bits = 1;
        while (bits < 32 && (1ull << bits) <= (uint64_t)n) ++bits;
        launch_sort_pairs(kj, b0, b1, n, bits, sort_tmp, &sk, &perm, a.err, st);
        hipLaunchKernelGGL(permuted_sums_kernel, grid, block, 0, st, kcnt, perm, n_kept, pair_sums);
    }
    launch_scan_sums(pair_sums, n_pair_sums, a.total_pairs, st, a.ctx_off ? ex_sums : nullptr, a.total_examples);
    hipLaunchKernelGGL(emit_pairs_kernel, grid, block, 0, st, kword, klo, kcnt, pair_sums, n_kept,
                       (const uint32_t*)perm, a.in_idx, a.out_idx, a.capacity,
                       ExampleOut{ex_sums, a.ctx_off, a.centers, a.cap_examples});
}

}  // namespace w2v
