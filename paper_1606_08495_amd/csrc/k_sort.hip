// Exclusive scan of a list of sums and a stable least-significant-digit radix sort of (key, index)
// pairs, up to 8 bits per pass.  Used to group the contributions of adjust by destination row:
// equal keys end up adjacent and, the sort being stable, in increasing order of their original
// slot, so the order in which a row's contributions are summed is fixed by the input alone.
#include "common.h"

#include <algorithm>

namespace w2v {

static inline unsigned blocks_for(uint64_t items, unsigned per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

// ---------------------------------------------------------------------------------------------
// Scan of a list of sums by one block with a running carry.
// ---------------------------------------------------------------------------------------------
constexpr int SCAN_THREADS = 256;

// Exclusive scan of one value per thread across the first 256 threads of a block (larger blocks
// pass through with the rest of their threads, for the barriers); returns the exclusive prefix
// and leaves the total in *total_out (shared).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* wave_sums,
                                                         uint32_t* total_out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63 && wave < SCAN_THREADS / 64) wave_sums[wave] = incl;
    __syncthreads();
    uint32_t base = 0;
#pragma unroll
    for (int w = 0; w < SCAN_THREADS / 64; ++w) {
        uint32_t s = wave_sums[w];
        if (w < wave) base += s;
    }
    if (threadIdx.x == SCAN_THREADS - 1) *total_out = base + incl;
    __syncthreads();
    return base + incl - x;
}

// (sixteen sums per thread and step: a running carry over n / 256 of them is two steps for two million)
constexpr int SCAN_SUMS_ITEMS = 16;
__global__ __launch_bounds__(SCAN_THREADS) void scan_sums_kernel(uint32_t* __restrict__ sums,
                                                                 uint32_t* __restrict__ total_out, uint32_t nb) {
    __shared__ uint32_t wave_sums[4];
    __shared__ uint32_t total;
    uint32_t carry = 0;
    for (uint32_t start = 0; start < nb; start += SCAN_THREADS * SCAN_SUMS_ITEMS) {
        const uint32_t i0 = start + threadIdx.x * SCAN_SUMS_ITEMS;
        uint32_t v[SCAN_SUMS_ITEMS], x = 0;
#pragma unroll
        for (int e = 0; e < SCAN_SUMS_ITEMS; ++e) { v[e] = i0 + e < nb ? sums[i0 + e] : 0u; x += v[e]; }
        uint32_t run = carry + block_exclusive_scan(x, wave_sums, &total);
#pragma unroll
        for (int e = 0; e < SCAN_SUMS_ITEMS; ++e) {
            if (i0 + e < nb) sums[i0 + e] = run;
            run += v[e];
        }
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total_out = carry;
}

void launch_scan_sums(uint32_t* sums, uint32_t nb, uint32_t* total, hipStream_t st) {
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(SCAN_THREADS), 0, st, sums, total, nb);
}

// ---------------------------------------------------------------------------------------------
// Radix sort.  One or two independent arrays ("jobs") are sorted by the same launches:
//   fill      : clears the digit totals, the tile tickets and the first tile-state array
//   totals    : one read of the keys gives, for every pass at once, how many keys carry each digit
//               (the totals do not depend on the order the earlier passes leave behind)
//   pass x P  : ONE launch per pass.  A block takes the next tile of THREADS x ITEMS consecutive elements
//               (ticket counter), ranks its elements among the tile's elements of the same digit in
//               tile order (-> stable), and learns how many elements of each digit the tiles before
//               it hold by looking back over the tile states: a tile first publishes its own digit
//               counts ("partial"), then walks back over its predecessors, adding partial counts
//               until it meets a tile that has already published its prefix ("inclusive"), and
//               publishes its own prefix.  A tile only ever waits for tiles with smaller tickets,
//               which are running or done; the wait is bounded all the same: past the limit the
//               block raises the error flag and goes on with what it has, so every wave ends.
//               The tile is then put in sorted order in LDS and written out position by position,
//               so that neighbouring threads write neighbouring addresses inside a digit's run.
// Between passes an element travels as one 8-byte word (key, index): one coalesced load and one
// store per element and pass, runs of 16 elements filling whole 128-byte lines.  The first pass
// reads the keys alone (the index is the position), the last one writes keys and indices to
// separate arrays, which is what the kernels of adjust read.
// Two tile-state arrays alternate between passes; each block clears its own row of the array the
// next pass will use, so no pass starts on stale states and nothing is cleared between passes.
// ---------------------------------------------------------------------------------------------
constexpr int SORT_THREADS = 256;                    // of the totals kernel
constexpr uint32_t SORT_SMALL_N = 1u << 19;
constexpr int SORT_MAX_PASSES = 4;
constexpr uint32_t SORT_SPIN_LIMIT = 1u << 22;       // fruitless look-back polls before giving up (~ a second)
constexpr int LB_WINDOW = 8;                         // tiles examined per look-back round
constexpr uint64_t ST_PARTIAL = 1ull << 62, ST_INCLUSIVE = 2ull << 62, ST_VALUE = (1ull << 62) - 1;
// Tile shapes.  A pass over few tiles is a chain of latencies -- a tile's own work, then the look-back, eight tiles a
// round trip -- so the tiles are as large as still leaves the chip enough of them, and their threads many: what
// a tile does between its loads and its counts is short then.  Joint sort of 6 n + n keys of 20 bits, us, all launches:
// keys       140 000  280 000  459 000  700 000  1.05 M  1.84 M  3.67 M  7.34 M
// 256 x 4         41       52       67       88     116     181     293     507   (so up to 2^19 keys before)
// 512 x 16        55       58       60       67      74      86     122     210   (and from there on)
// 1024 x 2        35       41       48       62      77     111     183     320
// 1024 x 4        38       42       46       54      64      95     163     274
// 1024 x 8        46       49       52       57      63      77     127     226
// (1024 x 16 alone 109 and 194 at the two largest; its blocks fill a compute unit, which beside row kernels they seldom
// get to themselves: benchmark step 3.110 ms against 3.098 with 512 x 16, dotprod and adjust of 60 columns 1.097, 1.111.)
// (Look-back windows of 4 tiles the same, of 16 and 32 up to 40 % slower.)
struct SortShape { uint32_t below, threads, items; };           // for less than `below` keys in all
constexpr SortShape SORT_SHAPES[] = {{300000u, 1024, 2}, {1u << 20, 1024, 4}, {2500000u, 1024, 8}, {0xFFFFFFFFu, 512, 16}};
static inline int sort_shape_for(uint64_t n) {
    int s = 0;
    while (s < 3 && n >= SORT_SHAPES[s].below) ++s;
    return s;
}
static inline uint32_t sort_tile_of(int shape) { return SORT_SHAPES[shape].threads * SORT_SHAPES[shape].items; }

struct SortJobDev {
    const uint32_t* keys_in;     // the caller's keys (pass 0 reads them; never written)
    uint2* buf[2];               // ping-pong buffers of (key, index) words, n each
    uint32_t* out_keys;          // last pass: separate arrays (inside the buffer it does not read)
    uint32_t* out_vals;
    uint32_t n, tiles;
};
struct SortArgs {
    SortJobDev job[2];
    uint32_t njobs, tiles0;      // tiles of job 0 come first in ticket order
    uint32_t passes, shift[SORT_MAX_PASSES], width[SORT_MAX_PASSES];
    uint32_t* totals;            // [2][SORT_MAX_PASSES][256] digit totals
    uint32_t* tickets;           // [SORT_MAX_PASSES]
    uint64_t* state[2];          // [tiles0 + tiles1][256] each
    uint32_t* err;               // sticky error flag of the shard (may be null)
};

__global__ __launch_bounds__(256) void sort_fill_kernel(uint64_t* __restrict__ p, uint64_t count) {
    uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0ull;
}

// Digit totals of every pass in one read of the keys.  A block covers 256 x 16 keys of one job and
// counts in LDS, one atomic per key and pass.  Word frequencies are skewed, so many lanes of a
// wavefront hold the same digit (in the top pass, most of them): each counter is kept in
// TOT_COPIES copies, chosen by lane number, which divides the number of lanes that queue up on
// one address by that many (integer sums: the order does not matter).
constexpr int TOT_ITEMS = 16;
constexpr int TOT_COPIES = 8;
__global__ __launch_bounds__(SORT_THREADS) void sort_totals_kernel(SortArgs a, uint32_t blocks0) {
    __shared__ uint32_t h[SORT_MAX_PASSES][256 * TOT_COPIES];
    for (int i = threadIdx.x; i < SORT_MAX_PASSES * 256 * TOT_COPIES; i += SORT_THREADS) (&h[0][0])[i] = 0;
    __syncthreads();
    const uint32_t j = blockIdx.x >= blocks0 ? 1u : 0u;
    const uint32_t b = blockIdx.x - (j ? blocks0 : 0u);
    const uint32_t* __restrict__ keys = a.job[j].keys_in;
    const uint32_t n = a.job[j].n;
    const uint32_t base = b * (uint32_t)(SORT_THREADS * TOT_ITEMS) + threadIdx.x;
    const uint32_t copy = threadIdx.x & (TOT_COPIES - 1);
    uint32_t k[TOT_ITEMS];
#pragma unroll
    for (int e = 0; e < TOT_ITEMS; ++e) {
        const uint32_t i = base + (uint32_t)e * SORT_THREADS;
        k[e] = i < n ? keys[i] : 0u;
    }
    for (uint32_t p = 0; p < a.passes; ++p) {
        const uint32_t shift = a.shift[p], mask = (1u << a.width[p]) - 1u;
#pragma unroll
        for (int e = 0; e < TOT_ITEMS; ++e) {
            const uint32_t d = (k[e] >> shift) & mask;
            if (base + (uint32_t)e * SORT_THREADS < n) atomicAdd(&h[p][d * TOT_COPIES + copy], 1u);
        }
    }
    __syncthreads();
    for (uint32_t p = 0; p < a.passes; ++p) {
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < TOT_COPIES; ++q) c += h[p][threadIdx.x * TOT_COPIES + q];
        if (c) atomicAdd(&a.totals[(j * SORT_MAX_PASSES + p) * 256 + threadIdx.x], c);
    }
}

template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void sort_pass_kernel(SortArgs a, uint32_t pass) {
    constexpr int TILE = THREADS * ITEMS;
    constexpr int WAVE_SPAN = 64 * ITEMS;
    constexpr int WAVES = THREADS / 64;
    static_assert(THREADS >= 256 && THREADS % 256 == 0, "one thread per digit for the tile's bookkeeping");
    __shared__ uint32_t cnt[WAVES][256];
    __shared__ uint32_t to_global[256];
    __shared__ uint2 s_item[TILE];
    __shared__ uint32_t wave_sums[4];
    __shared__ uint32_t total_all;
    __shared__ uint32_t s_ticket;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool owner = threadIdx.x < 256;                 // thread d < 256 keeps the books of digit d
    if (threadIdx.x == 0) s_ticket = atomicAdd(&a.tickets[pass], 1u);
    for (int i = threadIdx.x; i < WAVES * 256; i += THREADS) (&cnt[0][0])[i] = 0;
    __syncthreads();
    // (< tiles0 + tiles1: one block per tile; the same in every lane, hence a scalar)
    const uint32_t ticket = __builtin_amdgcn_readfirstlane(s_ticket);
    const uint32_t j = (a.njobs > 1 && ticket >= a.tiles0) ? 1u : 0u;
    const uint32_t first_tile = j ? a.tiles0 : 0u;       // ticket of this job's first tile
    const uint32_t tile = ticket - first_tile;
    const SortJobDev& jb = a.job[j];
    const uint32_t n = jb.n;
    const uint32_t shift = a.shift[pass], width = a.width[pass], mask = (1u << width) - 1u;
    const bool first_pass = pass == 0, last_pass = pass + 1 == a.passes;
    const uint2* __restrict__ in = jb.buf[(pass + 1) & 1];       // written by the pass before
    uint64_t* __restrict__ state = a.state[pass & 1];
    // the row of this tile in the array the next pass will use must be clear by then
    if (owner) a.state[(pass + 1) & 1][(uint64_t)ticket * 256 + threadIdx.x] = 0ull;
    // where each digit's elements start in the output: exclusive scan of the job's digit totals
    const uint32_t digit_base = block_exclusive_scan(
        owner ? a.totals[(j * SORT_MAX_PASSES + pass) * 256 + threadIdx.x] : 0u, wave_sums, &total_all);

    // element e of lane l of wave w is number w * WAVE_SPAN + e * 64 + l of the tile (n < 2^31)
    const uint32_t base = tile * (uint32_t)TILE + (uint32_t)wave * WAVE_SPAN + (uint32_t)lane;
    // (what is past the end reads the last element and is left out below: with a branch around each load, they were
    // waited for one by one)
    uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
    if (first_pass) {
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) {
            const uint32_t i = base + (uint32_t)e * 64;
            key[e] = jb.keys_in[min(i, n - 1)];
            val[e] = i;
        }
    } else {
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) {
            const uint2 x = in[min(base + (uint32_t)e * 64, n - 1)];
            key[e] = x.x; val[e] = x.y;
        }
    }
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        const bool valid = base + (uint32_t)e * 64 < n;
        const uint32_t d = (key[e] >> shift) & mask;
        // lanes of this wave holding the same digit
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            if (b < (int)width) {                        // (same in every lane)
                const uint64_t bal = __ballot((d >> b) & 1u);
                same &= ((d >> b) & 1u) ? bal : ~bal;
            }
        }
        uint32_t before = 0;
        if (valid) {
            before = cnt[wave][d];
            rank[e] = before + (uint32_t)__popcll(same & below);
        } else {
            rank[e] = 0;
        }
        // The reads above are issued before the write below by every lane of the wave (one
        // instruction stream), so the leader's update cannot be seen by this step's readers.
        if (valid && (same & below) == 0) cnt[wave][d] = before + (uint32_t)__popcll(same);
    }
    __syncthreads();
    // Thread d owns digit d: the tile's count of the digit, its place in the sorted tile, and the
    // look-back over the tiles before this one.
    uint32_t c[WAVES], tile_count = 0;
    if (owner) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { c[w] = cnt[w][threadIdx.x]; tile_count += c[w]; }
    }
    uint64_t* mine = state + (uint64_t)ticket * 256 + (threadIdx.x & 255);
    if (owner)
        __hip_atomic_store(mine, (tile == 0 ? ST_INCLUSIVE : ST_PARTIAL) | (uint64_t)tile_count,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t local_start = block_exclusive_scan(tile_count, wave_sums, &total_all);
    if (owner) {
        const uint32_t d = threadIdx.x;
        uint32_t run = local_start;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { cnt[w][d] = run; run += c[w]; }
        // Look-back, a window of LB_WINDOW tiles at a time: their states are requested together
        // (one memory round trip for the window) and taken in order from the nearest tile back,
        // up to the first that has not published yet (asked for again in the next round) or that
        // carries its prefix (done).
        uint64_t before_tiles = 0;
        if (tile > 0) {
            uint32_t cur = ticket;                       // the next tile to take is cur - 1
            uint32_t polls = 0;
            bool done = false, gave_up = false;
            while (!done) {                              // (the job's first tile is always "inclusive")
                uint64_t s[LB_WINDOW];
#pragma unroll
                for (int w = 0; w < LB_WINDOW; ++w) {
                    const bool inside = cur - first_tile > (uint32_t)w;      // tile cur-1-w is of this job
                    const uint32_t t = inside ? cur - 1u - (uint32_t)w : first_tile;
                    s[w] = __hip_atomic_load(state + (uint64_t)t * 256 + d, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
                }
                uint32_t taken = 0;
#pragma unroll
                for (int w = 0; w < LB_WINDOW; ++w) {
                    const bool inside = cur - first_tile > (uint32_t)w;
                    if (!done && taken == (uint32_t)w && inside && (s[w] >> 62) != 0) {
                        before_tiles += s[w] & ST_VALUE;
                        ++taken;
                        if ((s[w] >> 62) == 2) done = true;
                    }
                }
                cur -= taken;
                if (!done && taken == 0) {               // the nearest tile has not published yet
                    if (++polls >= SORT_SPIN_LIMIT) { gave_up = true; break; }
                    __builtin_amdgcn_s_sleep(2);
                }
            }
            if (gave_up && a.err) atomicOr(a.err, 2u);
            __hip_atomic_store(mine, ST_INCLUSIVE | ((before_tiles + tile_count) & ST_VALUE),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // output position = to_global[digit] + position in the sorted tile (mod 2^32 arithmetic)
        to_global[d] = digit_base + (uint32_t)before_tiles - local_start;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        if (base + (uint32_t)e * 64 < n) {
            const uint32_t d = (key[e] >> shift) & mask;
            s_item[cnt[wave][d] + rank[e]] = make_uint2(key[e], val[e]);
        }
    }
    __syncthreads();
    const uint32_t tile_base = tile * (uint32_t)TILE;
    const uint32_t in_tile = min((uint32_t)TILE, n - tile_base);
    uint2* __restrict__ out = jb.buf[pass & 1];
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        const uint32_t lp = (uint32_t)e * THREADS + threadIdx.x;
        if (lp < in_tile) {
            const uint2 x = s_item[lp];
            const uint32_t pos = to_global[(x.x >> shift) & mask] + lp;   // < n: ranks are a permutation
            if (pos < n) {                               // (only a timed-out look-back can fail this)
                if (last_pass) { jb.out_keys[pos] = x.x; jb.out_vals[pos] = x.y; }
                else out[pos] = x;
            }
        }
    }
}

static inline uint32_t sort_tiles(uint32_t n, int shape) { return blocks_for(n, sort_tile_of(shape)); }

// Scratch of calls over arrays of up to n0 and n1 elements, together or each alone, in uint32 (the
// region must be 8-byte aligned).  Reserved by tiles of 1024 below SORT_SMALL_N in all, which is more than any shape
// has there; past it one of the arrays alone (or a smaller call later) may still be short, and arrays of up to 2^20
// keys are cut in tiles of 4096, of which there are less than that.
static_assert((1u << 20) / 4096 + 2 <= SORT_SMALL_N / 1024 + 1, "see above");
size_t sort_scratch_u32(uint32_t n0, uint32_t n1) {
    const uint64_t n = (uint64_t)n0 + n1;
    const uint32_t tile = n < SORT_SMALL_N ? 1024u : 8192u;
    uint64_t tiles = (uint64_t)blocks_for(n0, tile) + blocks_for(n1, tile);
    if (n >= SORT_SMALL_N) tiles = std::max<uint64_t>(tiles, SORT_SMALL_N / 1024 + 1);
    return 2 * SORT_MAX_PASSES * 256 + 8 + 2 * (size_t)(2 * tiles * 256) + 16;
}

// totals, tickets and the first state array: one stretch of 8-byte words at the start of tmp
static uint64_t sort_clear_words64(uint32_t tiles) {
    return (2 * SORT_MAX_PASSES * 256 + 8) / 2 + (uint64_t)tiles * 256;
}

FillJob sort_clear_job(const SortJob* jobs, int njobs, uint32_t* tmp) {
    uint64_t n_all = 0;
    for (int i = 0; i < njobs && i < 2; ++i) n_all += jobs[i].n;
    if (n_all == 0) return FillJob{tmp, 0u, 0u};
    const int shape = sort_shape_for(n_all);
    uint32_t tiles = 0;
    for (int i = 0; i < njobs && i < 2; ++i)
        if (jobs[i].n) tiles += sort_tiles(jobs[i].n, shape);
    return FillJob{tmp, (uint32_t)(2 * sort_clear_words64(tiles)), 0u};
}

void launch_sort_jobs(const SortJob* jobs, int njobs, uint32_t bits, uint32_t* tmp, uint32_t* err,
                      hipStream_t st, bool cleared) {
    if (bits == 0) bits = 1;
    if (bits > 32) bits = 32;
    SortArgs a{};
    // empty arrays need nothing; results of an empty job are its first buffer
    int live = 0;
    uint64_t n_all = 0;
    for (int i = 0; i < njobs && i < 2; ++i) {
        *jobs[i].out_keys = (uint32_t*)jobs[i].buf0;
        *jobs[i].out_vals = (uint32_t*)jobs[i].buf0;
        if (jobs[i].n) n_all += jobs[i].n;
    }
    if (n_all == 0) return;
    const int shape = sort_shape_for(n_all);
    a.passes = (bits + 7) / 8;
    for (uint32_t p = 0, lo = 0; p < a.passes; ++p) {      // digits of nearly equal width
        const uint32_t w = (bits - lo + (a.passes - p) - 1) / (a.passes - p);
        a.shift[p] = lo; a.width[p] = w; lo += w;
    }
    for (int i = 0; i < njobs && i < 2; ++i) {
        if (jobs[i].n == 0) continue;
        SortJobDev& d = a.job[live];
        d.keys_in = jobs[i].keys_in; d.n = jobs[i].n; d.tiles = sort_tiles(jobs[i].n, shape);
        d.buf[0] = jobs[i].buf0; d.buf[1] = jobs[i].buf1;
        // the last pass reads buf[passes & 1] (or the caller's keys) and writes the other buffer
        uint2* dst = d.buf[(a.passes - 1) & 1];
        d.out_keys = (uint32_t*)dst;
        d.out_vals = (uint32_t*)dst + d.n;
        *jobs[i].out_keys = d.out_keys;
        *jobs[i].out_vals = d.out_vals;
        ++live;
    }
    a.njobs = live;
    a.tiles0 = a.job[0].tiles;
    const uint32_t tiles = a.job[0].tiles + (live > 1 ? a.job[1].tiles : 0u);
    a.totals = tmp;
    a.tickets = tmp + 2 * SORT_MAX_PASSES * 256;
    a.state[0] = (uint64_t*)(tmp + 2 * SORT_MAX_PASSES * 256 + 8);
    a.state[1] = a.state[0] + (uint64_t)tiles * 256;
    a.err = err;
    if (!cleared) {
        const uint64_t clear64 = sort_clear_words64(tiles);
        hipLaunchKernelGGL(sort_fill_kernel, dim3(blocks_for(clear64, 256)), dim3(256), 0, st,
                           (uint64_t*)tmp, clear64);
    }
    const uint32_t blocks0 = blocks_for(a.job[0].n, SORT_THREADS * TOT_ITEMS);
    const uint32_t blocks1 = live > 1 ? blocks_for(a.job[1].n, SORT_THREADS * TOT_ITEMS) : 0u;
    hipLaunchKernelGGL(sort_totals_kernel, dim3(blocks0 + blocks1), dim3(SORT_THREADS), 0, st, a, blocks0);
    for (uint32_t p = 0; p < a.passes; ++p) {
#define W2V_PASS(SHAPE)                                                                                          \
    hipLaunchKernelGGL((sort_pass_kernel<SORT_SHAPES[SHAPE].threads, SORT_SHAPES[SHAPE].items>), dim3(tiles),    \
                       dim3(SORT_SHAPES[SHAPE].threads), 0, st, a, p)
        if (shape == 0) W2V_PASS(0);
        else if (shape == 1) W2V_PASS(1);
        else if (shape == 2) W2V_PASS(2);
        else W2V_PASS(3);
#undef W2V_PASS
    }
}

void launch_sort_pairs(const uint32_t* keys_in, uint2* buf0, uint2* buf1, uint32_t n, uint32_t bits,
                       uint32_t* tmp, uint32_t** out_keys, uint32_t** out_vals, uint32_t* err,
                       hipStream_t st) {
    SortJob job{keys_in, n, buf0, buf1, out_keys, out_vals};
    launch_sort_jobs(&job, 1, bits, tmp, err, st);
}

// ---------------------------------------------------------------------------------------------
// Small arrays: equal keys brought together in ONE launch.  A block owns a bucket of keys (a fold of the
// key's bits: word numbers are frequency ranks, so frequent words spread over the buckets).  It reads ALL
// keys of its array -- a few hundred kilobytes, out of the caches --, lists the slots of its own in order and
// counts the keys of lower buckets, which is where its stretch of the output begins: no block waits for
// another.  The list is then sorted by key, slots in increasing order among equal keys: up to GS_PAIRWISE
// elements by counting each one's place against all others, more digit by digit in LDS.  The output is in
// bucket order, then key order: all that the update needs is that equal keys are adjacent.
// Each wavefront lists its stretch of the keys, at most GS_SUB of them.  Where one finds more (a very frequent
// word), the key in the middle of that wavefront's list is written out by itself and the rest listed anew.  After
// GS_ALONE such keys (many different words of one bucket) the slots of the rest are listed in global memory and sorted
// there, 1024 at a time: a step of 40 000 pairs whose words all fall into one bucket, on either side, takes 0.58 ms
// (a pass over all keys for each of them, 770).
// Bound by latency: a launch, three memory round trips, the fetch of its code -- hence loops that are
// not unrolled (with the keys held in registers and everything unrolled, 8 kB of straight code, it took 18 us
// for 28 672 keys, 13.7 this way).
// ---------------------------------------------------------------------------------------------
constexpr int GS_THREADS = 1024, GS_WAVES = GS_THREADS / 64;
constexpr uint32_t GS_MOST = 1u << 16;               // keys of one array (slots fit 16 bits)
constexpr uint32_t GS_PAIRWISE = 256;
constexpr uint32_t GS_SUB = 512;                     // list entries of a wavefront
constexpr uint32_t GS_LIST = GS_WAVES * GS_SUB;
constexpr int GS_LIST_ITEMS = GS_LIST / GS_THREADS;
constexpr int GS_ALONE = 4;                          // keys written out by themselves, at most
constexpr int GS_QUADS = 2;                          // four keys of a lane each, per step
constexpr uint32_t GS_STEP = GS_QUADS * 256;         // keys of a wavefront's step

struct GroupJobDev {
    const uint32_t* keys; uint32_t n;      // 16-byte aligned, readable up to a multiple of four
    uint32_t* out;               // n keys, then n slots
    uint32_t* other;             // n marked keys (mark: the keys in slot order, KEY_ALONE on those that occur once), then n words to spare
    bool mark;
    uint32_t fold;               // log2 of the buckets
    uint32_t passes, width;      // of the bits above `fold`, digits of the same width
};
struct GroupArgs { GroupJobDev job[2]; uint32_t blocks0; };

// bucket of a key; one above 2^31 (no key: KEY_NONE) lies past every bucket
__host__ __device__ inline uint32_t group_bucket(uint32_t k, uint32_t fold) {
    return (k ^ (k >> fold) ^ (k >> (2 * fold))) & (((1u << fold) - 1u) | 0x80000000u);
}

// row_shr:D of every sixteen lanes, zero shifted in
template <int D> __device__ __forceinline__ uint32_t shifted16(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x110 + D, 0xf, 0xf, true);
}

// The block's wavefronts' values (LDS): their sum, and that of those before this one.  (Scalars, as is `wave`: with a
// comparison for each wavefront held in scalar registers throughout, the kernel spills.)
static_assert(GS_WAVES == 16, "a lane for each");
__device__ __forceinline__ void wave_sums_of(const uint32_t* s_part, int wave, uint32_t& before, uint32_t& all) {
    uint32_t x = s_part[threadIdx.x % GS_WAVES];
    x += shifted16<1>(x); x += shifted16<2>(x); x += shifted16<4>(x); x += shifted16<8>(x);
    all = (uint32_t)__builtin_amdgcn_readlane((int)x, GS_WAVES - 1);
    before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)x, wave - 1) : 0u;
}
// The largest of them, and whose it is.
__device__ __forceinline__ void wave_most_of(const uint32_t* s_part, uint32_t& most, uint32_t& most_at) {
    const uint32_t v = s_part[threadIdx.x % GS_WAVES];
    uint32_t x = v;
    x = max(x, shifted16<1>(x)); x = max(x, shifted16<2>(x)); x = max(x, shifted16<4>(x)); x = max(x, shifted16<8>(x));
    most = (uint32_t)__builtin_amdgcn_readlane((int)x, GS_WAVES - 1);
    most_at = (uint32_t)__builtin_ctzll(__ballot(v == most));
}

// (64 registers, two blocks to a compute unit)
__global__ __launch_bounds__(GS_THREADS, 8) void group_small_kernel(GroupArgs a) {
    __shared__ __align__(16) uint32_t s_key[GS_LIST];
    __shared__ uint16_t s_val[GS_LIST];
    union Tables {
        struct { uint16_t slot[GS_WAVES][GS_SUB]; } sub;      // the wavefronts' lists
        uint32_t cnt[GS_WAVES][256];                          // once they are joined: digit counts
    };
    __shared__ Tables lds;
    __shared__ uint64_t s_done[GS_MOST / 64];                 // slots written out already, a bit each
    __shared__ __align__(16) uint32_t s_part[GS_WAVES], s_low[GS_WAVES];
    __shared__ uint32_t wave_sums[4], total_all;
    auto& s_sub = lds.sub.slot; auto& cnt = lds.cnt;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool second = blockIdx.x >= a.blocks0;
    const GroupJobDev& jb = a.job[second ? 1 : 0];
    const uint32_t bucket = blockIdx.x - (second ? a.blocks0 : 0u), n = jb.n, fold = jb.fold;
    const uint32_t* __restrict__ keys = jb.keys;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t steps = (n + GS_STEP - 1) / GS_STEP;      // wavefront w takes steps w steps / 16 .. (w + 1) steps / 16
    const uint32_t first = wave * steps / GS_WAVES, last = (wave + 1) * steps / GS_WAVES;
    int alone = 0;                                            // keys written out already
    uint32_t start = 0;
    for (;;) {
        uint32_t lower = 0, mine = 0;
        uint4 x[GS_QUADS], nx[GS_QUADS];
        auto fetch = [&](uint4 (&r)[GS_QUADS], uint32_t step) {
#pragma unroll
            for (int u = 0; u < GS_QUADS; ++u) {
                const uint32_t i = step * GS_STEP + u * 256 + lane * 4;
                r[u] = make_uint4(KEY_NONE, KEY_NONE, KEY_NONE, KEY_NONE);
                if (step < last && i < n) r[u] = *reinterpret_cast<const uint4*>(keys + i);
            }
        };
        fetch(x, first);
        fetch(nx, first + 1);
#pragma unroll 1
        for (uint32_t step = first; step < last; ++step) {
            uint32_t bits = 0;                                // bit 4 u + t: this lane's key t of quad u is of the bucket
#pragma unroll
            for (int u = 0; u < GS_QUADS; ++u) {
                const uint32_t k[4] = {x[u].x, x[u].y, x[u].z, x[u].w}, i = step * GS_STEP + u * 256 + lane * 4;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t b = i + t < n ? group_bucket(k[t], fold) : KEY_NONE;
                    lower += (uint32_t)__popcll(__ballot(b < bucket));
                    bits |= b == bucket ? 1u << (4 * u + t) : 0u;
                }
                x[u] = nx[u];
            }
            fetch(nx, step + 2);
            if (__ballot(bits != 0) == 0) continue;           // uniform per wavefront
#pragma unroll 1
            for (int u = 0; u < GS_QUADS; ++u) {
                const uint32_t i = step * GS_STEP + u * 256 + lane * 4;
                uint32_t own = (bits >> (4 * u)) & 15u;
                if (alone && own) own &= ~(uint32_t)(s_done[i / 64] >> (i % 64));
                const uint32_t c = (uint32_t)__popc(own);
                const uint64_t m0 = __ballot(c & 1u), m1 = __ballot(c & 2u), m2 = __ballot(c & 4u);
                uint32_t at = mine + (uint32_t)__popcll(m0 & below) + 2 * (uint32_t)__popcll(m1 & below) + 4 * (uint32_t)__popcll(m2 & below);
                for (; own; own &= own - 1, ++at)
                    if (at < GS_SUB) s_sub[wave][at] = (uint16_t)(i + __builtin_ctz(own));
                mine += (uint32_t)__popcll(m0) + 2 * (uint32_t)__popcll(m1) + 4 * (uint32_t)__popcll(m2);
            }
        }
        if (lane == 0) { s_part[wave] = mine; s_low[wave] = lower; }
        __syncthreads();
        uint32_t before, count, lower_all, unused, most, most_at;
        wave_sums_of(s_part, wave, before, count);
        wave_sums_of(s_low, wave, unused, lower_all);
        wave_most_of(s_part, most, most_at);
        if (!alone) start = lower_all;
        if (count == 0) return;                               // (all of these are the same in every thread)
        if (most <= GS_SUB) {
            for (uint32_t i = lane; i < mine; i += 64) {
                const uint16_t slot = s_sub[wave][i];
                s_val[before + i] = slot;
                s_key[before + i] = keys[slot];
            }
            if (threadIdx.x < 4 && count + threadIdx.x < GS_LIST) s_key[count + threadIdx.x] = KEY_NONE;   // (above every key)
            __syncthreads();                                  // (the lists are read: their place is free)
            if (count <= GS_PAIRWISE) {                       // four threads an element
                const uint32_t i = threadIdx.x / 4;
                if (i >= count) return;
                const uint32_t k = s_key[i];
                uint32_t place = 0, equal = 0;
#pragma unroll 1
                for (uint32_t j = 4 * (threadIdx.x % 4); j < count; j += 16) {
                    const uint4 y = *reinterpret_cast<const uint4*>(&s_key[j]);
                    const uint32_t o[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        place += o[t] < k || (o[t] == k && j + t < i) ? 1u : 0u;
                        equal += o[t] == k ? 1u : 0u;
                    }
                }
                place += __shfl_xor(place, 1, 64); equal += __shfl_xor(equal, 1, 64);
                place += __shfl_xor(place, 2, 64); equal += __shfl_xor(equal, 2, 64);
                if (threadIdx.x % 4) return;
                const uint32_t slot = s_val[i];
                jb.out[start + place] = k; jb.out[n + start + place] = slot;
                if (jb.mark) jb.other[slot] = equal == 1 ? k | KEY_ALONE : k;
                return;
            }
            // Digit by digit (the bucket and the bits above `fold` fix the rest).  Element e of lane l of wave w is
            // number (w items + e) 64 + l of the list.
            const uint32_t items = (count + GS_THREADS - 1) / GS_THREADS;
#pragma unroll 1
            for (uint32_t p = 0; p < jb.passes; ++p) {
                const uint32_t shift = fold + p * jb.width, dmask = (1u << jb.width) - 1u;
                for (int i = threadIdx.x; i < GS_WAVES * 256; i += GS_THREADS) (&cnt[0][0])[i] = 0;
                __syncthreads();
                uint32_t k[GS_LIST_ITEMS], slot_rank[GS_LIST_ITEMS];      // slot, and 2^16 times its rank in the wavefront
#pragma unroll
                for (int e = 0; e < GS_LIST_ITEMS; ++e) {
                    if ((uint32_t)e >= items) continue;       // uniform
                    const uint32_t i = (wave * items + e) * 64 + lane;
                    const bool valid = i < count;
                    k[e] = valid ? s_key[i] : 0u;
                    const uint32_t d = (k[e] >> shift) & dmask;
                    uint64_t same = __ballot(valid);
#pragma unroll 1
                    for (uint32_t b = 0; b < jb.width; ++b) {
                        const uint64_t bal = __ballot((d >> b) & 1u);
                        same &= ((d >> b) & 1u) ? bal : ~bal;
                    }
                    slot_rank[e] = 0;
                    uint32_t seen = 0;
                    if (valid) { seen = cnt[wave][d]; slot_rank[e] = s_val[i] | (seen + (uint32_t)__popcll(same & below)) << 16; }
                    // (every lane's read above is issued before the leader's write below: one instruction stream)
                    if (valid && (same & below) == 0) cnt[wave][d] = seen + (uint32_t)__popcll(same);
                }
                __syncthreads();
                uint32_t digit_count = 0;
                if (threadIdx.x < 256) {
#pragma unroll 4
                    for (int w = 0; w < GS_WAVES; ++w) digit_count += cnt[w][threadIdx.x];
                }
                uint32_t run = block_exclusive_scan(digit_count, wave_sums, &total_all);
                if (threadIdx.x < 256) {
#pragma unroll 4
                    for (int w = 0; w < GS_WAVES; ++w) {
                        const uint32_t c = cnt[w][threadIdx.x];
                        cnt[w][threadIdx.x] = run;
                        run += c;
                    }
                }
                __syncthreads();
#pragma unroll
                for (int e = 0; e < GS_LIST_ITEMS; ++e) {
                    if ((uint32_t)e >= items) continue;
                    if ((wave * items + e) * 64 + lane < count) {
                        const uint32_t pos = cnt[wave][(k[e] >> shift) & dmask] + (slot_rank[e] >> 16);
                        s_key[pos] = k[e]; s_val[pos] = (uint16_t)slot_rank[e];
                    }
                }
                __syncthreads();
            }
            for (uint32_t i = threadIdx.x; i < count; i += GS_THREADS) {
                const uint32_t k = s_key[i], slot = s_val[i];
                jb.out[start + i] = k; jb.out[n + start + i] = slot;
                const bool lone = (i == 0 || s_key[i - 1] != k) && (i + 1 == count || s_key[i + 1] != k);
                if (jb.mark) jb.other[slot] = lone ? k | KEY_ALONE : k;
            }
            return;
        }
        const uint32_t lo = first * GS_STEP, hi = min(last * GS_STEP, n);
        if (alone == GS_ALONE) {
            // slots in order, into the array from which an even or odd number of passes ends in the output
            uint32_t *src = jb.passes % 2 ? jb.other + n + start : jb.out + n + start, *dst = jb.passes % 2 ? jb.out + n + start : jb.other + n + start;
            uint32_t at = before;
#pragma unroll 1
            for (uint32_t i0 = lo; i0 < hi; i0 += 64) {
                const uint32_t i = i0 + lane;
                const bool own = i < hi && group_bucket(keys[i], fold) == bucket && !((s_done[i / 64] >> (i % 64)) & 1ull);
                const uint64_t m = __ballot(own);
                if (own) src[at + (uint32_t)__popcll(m & below)] = i;
                at += (uint32_t)__popcll(m);
            }
            __syncthreads();
#pragma unroll 1
            for (uint32_t p = 0; p < jb.passes; ++p) {
                const uint32_t shift = fold + p * jb.width, dmask = (1u << jb.width) - 1u;
                if (threadIdx.x < 256) s_key[threadIdx.x] = 0;
                __syncthreads();
#pragma unroll 1
                for (uint32_t i = threadIdx.x; i < count; i += GS_THREADS) atomicAdd(&s_key[(keys[src[i]] >> shift) & dmask], 1u);
                __syncthreads();
                const uint32_t digit = threadIdx.x < 256 ? s_key[threadIdx.x] : 0u;
                uint32_t run = block_exclusive_scan(digit, wave_sums, &total_all);       // where the digit's next one goes
#pragma unroll 1
                for (uint32_t i0 = 0; i0 < count; i0 += GS_THREADS) {
#pragma unroll 1
                    for (int i = threadIdx.x; i < GS_WAVES * 256; i += GS_THREADS) (&cnt[0][0])[i] = 0;
                    __syncthreads();
                    const bool valid = i0 + threadIdx.x < count;
                    const uint32_t slot = valid ? src[i0 + threadIdx.x] : 0u, d = valid ? (keys[slot] >> shift) & dmask : 0u;
                    uint64_t same = __ballot(valid);
#pragma unroll 1
                    for (uint32_t b = 0; b < jb.width; ++b) {
                        const uint64_t bal = __ballot((d >> b) & 1u);
                        same &= ((d >> b) & 1u) ? bal : ~bal;
                    }
                    if (valid && (same & below) == 0) cnt[wave][d] = (uint32_t)__popcll(same);
                    __syncthreads();
                    if (threadIdx.x < 256) {
#pragma unroll 1
                        for (int w = 0; w < GS_WAVES; ++w) {
                            const uint32_t c = cnt[w][threadIdx.x];
                            cnt[w][threadIdx.x] = run;
                            run += c;
                        }
                    }
                    __syncthreads();
                    if (valid) dst[cnt[wave][d] + (uint32_t)__popcll(same & below)] = slot;
                    __syncthreads();
                }
                uint32_t* const t = src; src = dst; dst = t;
            }
#pragma unroll 1
            for (uint32_t i = threadIdx.x; i < count; i += GS_THREADS) {
                const uint32_t slot = src[i], k = keys[slot];
                jb.out[start + i] = k;
                const bool lone = (i == 0 || keys[src[i - 1]] != k) && (i + 1 == count || keys[src[i + 1]] != k);
                if (jb.mark) jb.other[slot] = lone ? k | KEY_ALONE : k;
            }
            return;
        }
        // one key by itself: lane r of a wavefront keeps the slots of its r-th 64 keys
        static_assert(GS_MOST / GS_WAVES <= 64 * 64, "a lane for every 64 keys of a wavefront");
        const uint32_t pick = keys[s_sub[most_at][GS_SUB / 2]];
        uint64_t own = 0;
#pragma unroll 8
        for (uint32_t i0 = lo; i0 < hi; i0 += 64) {
            const uint64_t m = __ballot(i0 + lane < hi && keys[min(i0 + lane, n - 1)] == pick);
            if ((uint32_t)lane == (i0 - lo) / 64) own = m;
        }
        const uint32_t c = (uint32_t)__popcll(own);
        uint32_t incl = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
        __syncthreads();                                      // (the counts and lists above are read)
        if (lane == 63) s_part[wave] = incl;
        __syncthreads();
        uint32_t all;
        wave_sums_of(s_part, wave, before, all);
        const uint32_t slot0 = lo + (uint32_t)lane * 64;
        if (slot0 < hi) s_done[slot0 / 64] = alone ? s_done[slot0 / 64] | own : own;
        for (uint32_t at = start + before + incl - c; own; own &= own - 1, ++at) {
            const uint32_t slot = slot0 + (uint32_t)__builtin_ctzll(own);
            jb.out[at] = pick; jb.out[n + at] = slot;
            if (jb.mark) jb.other[slot] = all == 1 ? pick | KEY_ALONE : pick;
        }
        start += all;
        ++alone;
        __syncthreads();                                      // (s_done is written, s_part read)
    }
}

// Up to 80 000 keys in all (a step of d = 100 in us, radix sort and marks and this way; k = 5: 500 pairs 70, 46; 4096 81, 64;
// 10 900 96, 80; k = 1, 30 000 pairs, a skewed vocabulary: 104, 102, and with d = 300 131, 139).
bool group_small(uint32_t n0, uint32_t n1) { return std::max(n0, n1) <= GS_MOST && n0 + n1 <= 80000u; }

// Buckets of an array: about a hundred keys each, a power of two, at least 2^4 (three times that many bits are folded
// into the bucket's number, which then covers any frequent word) and at most 2^8.
static uint32_t group_fold(uint32_t n) {
    uint32_t f = 4;
    while (f < 8 && (96u << f) < n) ++f;
    return f;
}

void launch_group_jobs(const SortJob* jobs, int njobs, uint32_t bits, bool mark0, hipStream_t st) {
    GroupArgs a{};
    uint32_t blocks = 0;
    for (int i = 0; i < njobs && i < 2; ++i) {
        const SortJob& j = jobs[i];
        *j.out_keys = (uint32_t*)j.buf0;
        *j.out_vals = (uint32_t*)j.buf0 + j.n;
        const uint32_t fold = group_fold(j.n), above = bits > fold ? bits - fold : 1;
        const uint32_t passes = (above + 7) / 8, width = (above + passes - 1) / passes;
        a.job[i] = GroupJobDev{j.keys_in, j.n, (uint32_t*)j.buf0, (uint32_t*)j.buf1, mark0 && i == 0, fold, passes, width};
        blocks += j.n ? 1u << fold : 0u;
        if (i == 0) a.blocks0 = blocks;
    }
    if (blocks) hipLaunchKernelGGL(group_small_kernel, dim3(blocks), dim3(GS_THREADS), 0, st, a);
}

}  // namespace w2v
