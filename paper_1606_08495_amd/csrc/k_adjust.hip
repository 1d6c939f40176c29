// adjust: segmented, fixed-order reduction of row contributions and the single write-back.
//
// After the destination keys are sorted, the contributions to one row are a run of adjacent
// entries.  The entry list is cut into chunks of a fixed number of entries; one lane group walks one
// chunk in order with the running sum in registers.  A run that lies inside a chunk is finished by
// that group (one read-modify-write of the destination row).  A run cut by a chunk border leaves
// one partial row on each side of the border ("slots" 2b and 2b+1 of border b, tagged with the
// row); the list of slots is then reduced by the same scheme, level after level, until a level
// fits one chunk.  Which entries meet in which partial sum depends only on the entry positions, so
// the result is bitwise reproducible, and a row that collects millions of contributions is spread
// over as many groups as it has chunks.
#include "rows.h"
#include "loss.h"

#include <algorithm>
#include <type_traits>

namespace w2v {

static inline unsigned blocks_for(uint64_t items, unsigned per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

// Block sizes, measured per kernel family: the input-side kernels run 6 % faster in blocks of 128
// than of 256 (and no faster in 64); the output-side kernel is 7 % slower in 128 at one wavefront
// per row and 8 % faster at sixteen lanes per row.
constexpr int USEG_THREADS = 128;                  // input-side kernels
constexpr int adj_threads(int G) { return G == 16 ? 128 : 256; }      // everything after them
// Higher levels: entries per block, which is their chunk (even, so a border's two slots fall into one),
// and the block's size.  A lane group's share of the chunk is what it reads one batch after the other, so
// a launch that holds nothing but these levels takes the largest blocks whose pieces fit LDS (shares of
// 8 entries; 65 536 pairs, d = 100: 26 us a level with shares of 32); beside the output side's walk, or where
// a large minibatch's kernels share the memory, they have those kernels' block size and find room between
// them (benchmark step: levels of 512 threads 46 us each, of 256 42; step 3.201 -> 3.194 ms).
constexpr int tail_block(int G) { return G == 64 ? 128 : 256; }
// The input side's first level beside the output side's walk: a quarter of that, eight entries to a group.  A group
// reads its share one batch after the other, and this level was what that launch waited for (4096 pairs, d = 100: 17 us,
// the walk alone 12); there are walks above it that take as many launches anyway.
constexpr int tail_block_first(int G) { return tail_block(G) / 4; }
constexpr int tail_threads(int G, int NV) { return G == 16 || NV == 2 ? 512 : (NV > 2 ? 256 : 1024); }
constexpr uint32_t NOKEY = 0xFFFFFFFFu;   // compares unequal to every masked key
constexpr uint32_t ALONE = KEY_ALONE;

uint32_t tail_entries_per_chunk(uint32_t d4, bool first) {
    return first ? (d4 <= 32 ? tail_block_first(16) : tail_block_first(64)) : (d4 <= 32 ? tail_block(16) : tail_block(64));
}
static_assert(tail_block(16) == tail_block(32) && tail_block(64) < tail_block(16), "see above, and tail_entries_least");
uint32_t tail_entries_least() { return tail_block_first(64); }
// Pairs per chunk of the input-side kernel: about useg_e(G) entries (pairs x slots), 2..useg_maxp(G)
// pairs.  Longer chunks cut fewer runs (fewer partial rows for the higher levels: -2.7 % on the
// benchmark step, -6 % with k = 25, against chunks of 48 entries); rows of up to 64 floats take shorter ones (input side
// and walk of 2^20 pairs of d = 60, us, with 48, 96 and 192 entries: k = 5 204 + 302, 202 + 295, 206 + 293; k = 10 799 + 583, 783 + 574,
// 784 + 564).
constexpr int useg_e(int G) { return G == 16 ? 96 : 192; }
constexpr int useg_maxp(int G) { return G == 16 ? 16 : 32; }            // pairs per chunk, at most
constexpr int useg_maxe(int G) {                 // entries, at most: c T < E + T, and 2 T, T <= 65
    return useg_e(G) + 66 < 136 ? 136 : useg_e(G) + 66;
}
// A lane group walks its chunk pair by pair, one memory round trip each, so a small minibatch cut
// into long chunks leaves the chip to a handful of groups (4096 pairs in chunks of 32: 128 groups,
// 109 us of row latency in a row): below USEG_MIN_CHUNKS chunks the chunks shrink, down to two pairs.
// (32768: from 2^20 pairs on the long chunks stay; 2^18 pairs run 5 % faster per step than with
// 4096, the 2^17 examples of a bag-of-words minibatch 4 %; 4096 pairs the same.)
constexpr uint32_t USEG_MIN_CHUNKS = 32768;
uint32_t useg_pairs_per_chunk(uint32_t T, uint32_t d4, uint32_t n) {
    const int G = d4 <= 16 ? 16 : (d4 <= 32 ? 32 : 64);                 // as W2V_DISPATCH_GEOM
    uint32_t c = ((uint32_t)useg_e(G) + T - 1) / T;
    if (c < 2) c = 2;
    if (c > (uint32_t)useg_maxp(G)) c = useg_maxp(G);
    const uint32_t fill = n / USEG_MIN_CHUNKS;                          // pairs per chunk that still give that many
    if (c > fill) c = fill < 2 ? 2 : fill;
    return c;
}
// (the narrowest rows have the shortest chunks; between two steps of the chunk size the number of chunks
// peaks just before a step, highest before the first one, from two pairs to three)
uint32_t useg_slots_most(uint32_t T, uint32_t n) {
    const uint32_t before_step = std::min(n, 3 * USEG_MIN_CHUNKS - 1);
    return std::max(slots_after(n, useg_pairs_per_chunk(T, 1, n)),
                    slots_after(before_step, useg_pairs_per_chunk(T, 1, before_step)));
}

// The kernels that reach into the matrices exist for one matrix and for slices.
template <class F> static void with_slices(const Slices* sl, F&& call) {
    if (sl) call(SliceArgs{*sl}); else call(OneMatrix{});
}

struct SegArgs {
    const float4* src;          // output side, level 1: U; higher levels: partial rows of the level below
    float4* dst;                // matrix updated in place
    RowGeom g;
    const uint32_t* skey;       // destination key per entry
    const uint32_t* sidx;       // level 1 only
    const SlotRecord* rec;      // level 1 only
    uint32_t entries;
    float alpha;
    float4* prows; uint32_t* pkeys;    // this level's partial slots
    uint32_t cell_log2;                // wown_kernel: cell size
    bool skip_alone;                   // wown_kernel: runs of length one are handled elsewhere
    // input side: finished sums are not added to dst but parked in the delta buffer
    float4* defer_rows; uint32_t* defer_keys;
    uint32_t level, cp;                // level of this pass (1 = first), pairs per input-side chunk
};

// ---------------------------------------------------------------------------------------------
// Higher levels: entries are partial rows src[i] (weight 1) with destination skey[i].  A block's chunk
// is tail_block(G) entries.  Most entries hold nothing: each lane group lists the ones of its part
// that do, walks that list with several rows in flight, finishes the runs that lie inside its part and
// leaves what its borders cut in LDS (two pieces per part); then every group adds up the pieces of the
// run that begins in its part, and only what the block's own borders cut goes to the slots of the next
// level.  Bound by latency, not
// bytes -- a level costs two or three memory round trips whatever it holds -- so what counts is how few
// levels there are: they shrink 64 or 128 times.  (One lane group per chunk of 16 entries, shrinking
// eightfold, before: six launches instead of three after the output side of a 2^20-pair minibatch,
// five instead of two at 2^16 pairs.)
//
// DEFER (input side): a run finished here must not touch the input matrix yet -- the output side may
// still be reading it -- so its sum goes to the delta buffer, from where apply_delta adds it with the
// same fma.  Its place there: every entry of a higher level stands at a chunk border of the level below,
// and so, level by level, at a border of the input-side kernel's chunk grid; the pair position right
// after that border lies inside the run, is not the run's first pair (the run was cut there), and so
// holds no sum of its own.  Runs are disjoint ranges of pair positions, hence no two finished runs share
// a place.
// (vb: the block's number among the blocks of this walk -- a launch that carries several walks passes
// the block's offset within its own)
// ---------------------------------------------------------------------------------------------
enum : uint32_t { TL_POS = 0xFFFFu, TL_HAS = 1u << 16, TL_COMPLETE = 1u << 17, TL_HEAD = 1u << 18 };

template <int G, int NV, int THREADS, int CB = tail_block(G)> struct TailLds {
    static constexpr int GROUPS = THREADS / G, C = CB / GROUPS;
    float4 rows[2 * GROUPS][G * NV];                      // head and tail piece of every part
    uint32_t raw[CB + 2];                                 // keys of entries base - 1 .. base + CB
    uint32_t list[GROUPS][C];
    uint32_t gkey[2 * GROUPS];
    uint32_t out_key[2];                                  // the block's own head and tail slot
};

template <int G, int NV, int THREADS, bool DEFER, int WHICH, int CB, class SL>
__device__ __forceinline__ void tail_body(const SegArgs& a, const SL& sl, uint32_t vb, TailLds<G, NV, THREADS, CB>& lds) {
    constexpr int GROUPS = THREADS / G, C = CB / GROUPS;
    constexpr int D = NV == 1 && (DEFER || C == 8) ? 8 : (NV <= 2 ? 4 : 2);
    static_assert(C % 2 == 0, "a border's two slots fall into one part");
    constexpr int ROW4 = G * NV;                          // float4 of a row held in LDS
    auto& s_raw = lds.raw; auto& s_list = lds.list; auto& s_rows = lds.rows; auto& s_gkey = lds.gkey;
    const float alpha = a.alpha;
    const int l = threadIdx.x % G, grp = (int)group_value<G>(threadIdx.x / G);
    const uint32_t base = vb * (uint32_t)CB, count = min((uint32_t)CB, a.entries - base);
    const bool more = base + CB < a.entries;              // a block follows
    const uint32_t d4 = a.g.d4;
    const uint64_t s4 = a.g.stride4;
    const Rows<G, NV, SL, WHICH> dst(sl, a.dst, a.g, l);  // (DEFER: not used)
    int any = 0;
    for (int i = threadIdx.x; i < CB + 2; i += THREADS) {
        const int64_t pos = (int64_t)base - 1 + i;
        const uint32_t raw = pos >= 0 && pos < (int64_t)a.entries ? a.skey[pos] : KEY_NONE;
        s_raw[i] = raw;
        any |= i > 0 && i <= (int)count && (raw & KEY_MASK) < KEY_MASK;
    }
    if (threadIdx.x < 2 * GROUPS) s_gkey[threadIdx.x] = KEY_NONE;
    if (threadIdx.x < 2) lds.out_key[threadIdx.x] = KEY_NONE;
    if (__syncthreads_or(any) == 0) {                     // nothing here, and no run passes through
        if (threadIdx.x == 0) {
            if (vb > 0) a.pkeys[2 * vb - 1] = KEY_NONE;
            if (more) a.pkeys[2 * vb] = KEY_NONE;
        }
        return;
    }
    auto K = [&](int i) -> uint32_t { return s_raw[i + 1] & KEY_MASK; };      // KEY_MASK itself names no row
    auto finish = [&](uint32_t key, uint32_t entry, const float4 (&acc)[NV], const float4 (&old)[NV]) {
        if (DEFER) {
            uint32_t pos = entry;
            for (uint32_t lv = a.level; lv > 1; --lv) pos = ((pos + 2) >> 1) * (uint32_t)CB;
            pos = ((pos + 2) >> 1) * a.cp;
            store_row<G, NV>(a.defer_rows + (uint64_t)pos * s4, d4, l, acc);
            if (l == 0) a.defer_keys[pos] = key;
        } else {
            float4 out[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                out[v].x = fmaf(alpha, acc[v].x, old[v].x);
                out[v].y = fmaf(alpha, acc[v].y, old[v].y);
                out[v].z = fmaf(alpha, acc[v].z, old[v].z);
                out[v].w = fmaf(alpha, acc[v].w, old[v].w);
            }
            dst.store_part(key, out);
        }
    };
    // ---- each group's part ----
    const int e0 = grp * C;
    const int n_part = min((int)count - e0, C);           // (may be zero or less)
    const uint32_t before = K(e0 - 1);
    int listed = 0;
    const int lane0 = ((int)(threadIdx.x & 63) / G) * G;
    for (int i0 = 0; i0 < C; i0 += G) {
        const int i = i0 + l;
        const bool inside = i < n_part;
        const uint32_t k = inside ? K(e0 + i) : KEY_MASK;
        const bool use = k < KEY_MASK;
        const uint64_t wave_mask = __ballot(use);
        const uint64_t mine = G == 64 ? wave_mask : ((wave_mask >> lane0) & ((1ull << (G & 63)) - 1ull));
        if (use) {
            const bool ends = K(e0 + i + 1) != k, came_in = before == k;
            s_list[grp][listed + __popcll(mine & ((1ull << l) - 1ull))] =
                (uint32_t)(e0 + i) | ((s_raw[e0 + i + 1] & KEY_ZERO) ? 0u : (uint32_t)TL_HAS) |
                (ends ? (came_in ? (uint32_t)TL_HEAD : (uint32_t)TL_COMPLETE) : 0u);
        }
        listed += __popcll(mine);
    }
    __syncthreads();
    float4 acc[NV];
    clear<NV>(acc);
    if (listed) {
        // Rows of two float4 a lane and more: all loads of a batch, then its sums (first level of a 2^20-pair
        // minibatch of 300 columns 76 -> 60 us, the second 39 -> 29).  One: most shares are a batch, asked for at once, zeros
        // where there is nothing; the other way 2^20 pairs of 60 columns 24 -> 30 us, 2^18 of 200 33 -> 36.
        if constexpr (NV >= 2) {
            for (int b = 0; b < listed; b += D) {             // (all loads of a batch, then its sums)
                float4 srcv[D][NV], dstv[D][NV];
                uint32_t f[D];
#pragma unroll
                for (int t = 0; t < D; ++t) f[t] = group_value<G>(s_list[grp][min(b + t, listed - 1)]);
#pragma unroll
                for (int t = 0; t < D; ++t)
                    if (b + t < listed && (f[t] & TL_HAS)) load_part<G, NV>(a.src + (uint64_t)(base + (f[t] & TL_POS)) * s4, d4, l, srcv[t]);
                if (!DEFER) {
#pragma unroll
                    for (int t = 0; t < D; ++t)
                        if (b + t < listed && (f[t] & TL_COMPLETE)) dst.template load_part<false>(K((int)(f[t] & TL_POS)), dstv[t]);
                }
#pragma unroll
                for (int t = 0; t < D; ++t) {
                    if (b + t < listed) {
                        const uint32_t i = f[t] & TL_POS;
                        if (f[t] & TL_HAS) axpy<NV>(1.0f, srcv[t], acc);
                        if (f[t] & TL_COMPLETE) {
                            finish(K((int)i), base + i, acc, dstv[t]);
                            clear<NV>(acc);
                        } else if (f[t] & TL_HEAD) {          // came in from the part before and ends here
                            store_row<G, NV>(&s_rows[2 * grp][0], ROW4, l, acc);
                            if (l == 0) s_gkey[2 * grp] = K((int)i);
                            clear<NV>(acc);
                        }
                    }
                }
            }
        } else {
            float4 srcv[D][NV], dstv[D][NV];
            auto fetch = [&](int idx, float4 (&sv)[NV], float4 (&dv)[NV]) {
                const uint32_t f = idx < listed ? s_list[grp][idx] : 0u;
                const bool cm = !DEFER && (f & TL_COMPLETE);
                const uint32_t i = f & TL_POS;
                load_row_if<G, NV>((f & TL_HAS) != 0, a.src + (uint64_t)(base + i) * s4, d4, l, sv);
                if (!DEFER) dst.load_if(cm, cm ? K((int)i) : 0u, dv);
            };
#pragma unroll
            for (int t = 0; t < D; ++t) fetch(t, srcv[t], dstv[t]);
            for (int b = 0; b < listed; b += D) {
#pragma unroll
                for (int t = 0; t < D; ++t) {
                    if (b + t < listed) {
                        const uint32_t f = s_list[grp][b + t], i = f & TL_POS;
                        if (f & TL_HAS) axpy<NV>(1.0f, srcv[t], acc);
                        if (f & TL_COMPLETE) {
                            finish(K((int)i), base + i, acc, dstv[t]);
                            clear<NV>(acc);
                        } else if (f & TL_HEAD) {             // came in from the part before and ends here
                            store_row<G, NV>(&s_rows[2 * grp][0], ROW4, l, acc);
                            if (l == 0) s_gkey[2 * grp] = K((int)i);
                            clear<NV>(acc);
                        }
                    }
                    if (b + D < listed) fetch(b + t + D, srcv[t], dstv[t]);
                }
            }
        }
        const uint32_t last = K(e0 + n_part - 1);
        if (last < KEY_MASK && K(e0 + n_part) == last) {  // the last run goes on past the part
            const int piece = before == last ? 2 * grp : 2 * grp + 1;
            store_row<G, NV>(&s_rows[piece][0], ROW4, l, acc);
            if (l == 0) {
                s_gkey[piece] = last;
                if (piece == 2 * grp) s_gkey[2 * grp + 1] = last | KEY_ZERO;   // it covers the whole part
            }
        }
    }
    __syncthreads();
    // ---- what the parts' borders cut: the group of the part in which a run begins (group 0 for the run
    // that comes in from before the block) walks its pieces, which are adjacent, in order ----
    const uint32_t block_before = K(-1), block_after = K((int)count);
    for (int start = grp == 0 ? 0 : 2 * grp + 1; start <= 2 * grp + 1; ++start) {
        const uint32_t raw0 = s_gkey[start], k = raw0 & KEY_MASK;
        if (k == KEY_MASK || (raw0 & KEY_ZERO)) continue; // (flagged: the run began earlier)
        const bool came_in = block_before == k;
        float4 old[NV];
        if (!DEFER && !came_in) dst.template load_part<false>(k, old);
        clear<NV>(acc);
        int i = start;
        uint32_t raw = raw0, next;
        for (;;) {
            if (!(raw & KEY_ZERO)) {
                float4 x[NV];
                load_row<G, NV>(&s_rows[i][0], ROW4, l, x);
                axpy<NV>(1.0f, x, acc);
            }
            raw = i + 1 < 2 * GROUPS ? s_gkey[i + 1] : block_after;
            next = raw & KEY_MASK;
            if (next != k || i + 1 == 2 * GROUPS) break;
            ++i;
        }
        if (next == k || came_in) {                       // goes on past the block, or came from before it
            store_row<G, NV>(a.prows + (uint64_t)(came_in ? 2 * vb - 1 : 2 * vb) * s4, d4, l, acc);
            if (l == 0) {
                if (came_in) lds.out_key[0] = k;
                if (next == k) lds.out_key[1] = came_in ? k | KEY_ZERO : k;
            }
        } else {
            finish(k, base + (uint32_t)(i / 2) * C, acc, old);       // (ends as the head piece of a later part)
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (vb > 0) a.pkeys[2 * vb - 1] = lds.out_key[0];
        if (more) a.pkeys[2 * vb] = lds.out_key[1];
    }
}

template <int G, int NV, int THREADS, class SL>
__global__ __launch_bounds__(THREADS) void tail_kernel(SegArgs a, SL sl) {
    __shared__ TailLds<G, NV, THREADS> lds;
    tail_body<G, NV, THREADS, false, 1>(a, sl, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------------------------
// Output-vector side, level 1, with run ownership.  A grid of chunks of C entries only decides WHO
// sums a run, not where it is cut:
//  * a run that starts in chunk c and ends before the end of chunk c+1 ("short", at most 2C entries)
//    is summed entirely by group c, which reads on past its chunk's end and finishes the row with
//    one read-modify-write; the group of chunk c+1 skips those entries;
//  * a run that reaches chunk c+2 ("long": a frequent word) is cut only at multiples of L entries
//    (cells).  Each piece is summed by one group -- the group of the chunk in which the run starts,
//    or of the chunk at the cell's start -- which streams on through the cell.  A piece that is the
//    whole run is finished at once; otherwise it is left in the cell's border slots (two per cell
//    border) for the higher levels.
// Short or long follows from the run's own extent on the chunk grid, so every group that meets a
// run decides alike, from the keys at six fixed positions around its chunk.  No partial row is
// written unless a word collects more than L contributions or so.
// ---------------------------------------------------------------------------------------------
constexpr int WOWN_C = 16;
// Cell size for long runs, a multiple of C: 64 (128: the output-side kernel 9 % slower, 32: more rows for
// the levels above); 32 for minibatches of up to 2^19 slots, whose time is that of the group with the most
// entries in a row.
constexpr uint32_t WOWN_SHORT_CELLS = 1u << 19;
static uint32_t wown_cell_log2(uint32_t M) { return M <= WOWN_SHORT_CELLS ? 5u : 6u; }
constexpr int WOWN_WIN = 3 * WOWN_C + 2;     // keys staged: positions base-C-1 .. base+2C
constexpr int WOWN_E = 2 * WOWN_C;           // positions summed from LDS facts: base .. base+2C-1
constexpr uint32_t RUN_ENDS = 0x80000000u;   // a listed entry with which a sum is complete
// Rows in flight of a lane group, of either matrix: few, in many wavefronts (walk of 6.3 M slots of 60 columns, us, with two,
// four and eight 313, 302, 341; 600 000 of 320 at two float4 a lane with one, two, four and eight 123, 114, 121, 216).
constexpr int wown_depth(int NV) { return NV == 1 ? 4 : 2; }

uint32_t wseg_entries_per_chunk(uint32_t M) { return 1u << wown_cell_log2(M); }
uint32_t wseg_slots_most(uint32_t M) {
    const uint32_t before_step = std::min(M, WOWN_SHORT_CELLS);
    return std::max(slots_after(M, wseg_entries_per_chunk(M)), slots_after(before_step, wseg_entries_per_chunk(before_step)));
}

template <int G, int NV, class SL>
__device__ __forceinline__ void wown_body(const SegArgs& a, const SL& sl, uint32_t vb) {
    constexpr int WOWN_THREADS = adj_threads(G);
    constexpr int GROUPS = WOWN_THREADS / G;
    constexpr int C = WOWN_C;
    constexpr int D = wown_depth(NV);                          // rows in flight, of either matrix
    const int L = 1 << a.cell_log2;                        // a multiple of C
    static_assert(C == 16 && G >= 16, "grid shapes");
    const float alpha = a.alpha;
    __shared__ uint32_t s_key[GROUPS][WOWN_WIN];
    __shared__ SlotRecord s_rec[GROUPS][WOWN_E];           // the list: source row and coefficient,
    __shared__ uint32_t s_dst[GROUPS][WOWN_E];             // destination row, with RUN_ENDS
    const int l = threadIdx.x % G, l16 = threadIdx.x % 16, grp = (int)group_value<G>(threadIdx.x / G);
    const uint32_t c = vb * (uint32_t)GROUPS + grp;
    const uint32_t nchunks = (a.entries + C - 1) / C;
    const bool active = c < nchunks;
    const int64_t base = (int64_t)c * C;
    constexpr int PER_LANE = G < WOWN_E ? WOWN_E / G : 1;
    uint32_t slot[PER_LANE];                               // (asked for before it is known which are needed)
#pragma unroll
    for (int u = 0; u < PER_LANE; ++u) {
        const int64_t pos = base + u * G + l;
        slot[u] = active && u * G + l < WOWN_E && pos < (int64_t)a.entries ? a.sidx[pos] : 0u;
    }
    for (int i = l; i < WOWN_WIN; i += G) {
        int64_t pos = base - C - 1 + i;
        s_key[grp][i] = (active && pos >= 0 && pos < (int64_t)a.entries) ? a.skey[pos] : NOKEY;
    }
    __syncthreads();
    auto K = [&](int rel) -> uint32_t { return s_key[grp][rel + C + 1]; };   // rel = position - base
    const uint32_t kbm = K(-C - 1), kb = K(-1), k0 = K(0), kC = K(C), k2C = K(2 * C), klast = K(C - 1);
    const bool head_exists = active && kb == k0;
    const bool head_long = head_exists && !(kbm != k0 && kC != k0);
    const bool own_head = head_long && (base & (L - 1)) == 0;          // a cell begins here: the piece is ours
    const bool last_in_head = head_exists && klast == k0;
    const bool ext_ok = klast != NOKEY && !last_in_head && k2C != klast;
    // does the run through the chunk's last entry go on, as a long piece that this group owns?
    const bool cont = active && klast != NOKEY && kC == klast && (last_in_head ? own_head : k2C == klast);
    // (of a long piece the positions up to the cell's end, the window's at most, are listed; a short run has no cells)
    const int left = (int)min((int64_t)(L - (int)(base & (L - 1))), (int64_t)a.entries - base);      // to the cell's end
    const int reach = cont ? min(left, WOWN_E) : WOWN_E;
    // The positions this group sums are listed densely (positions that are skipped --
    // another group's, or rows handled elsewhere -- take no place in the loads below).
    int count = 0;
    const int group_lane0 = ((int)(threadIdx.x & 63) / G) * G;
#pragma unroll
    for (int u = 0; u < PER_LANE; ++u) {
        const int i = u * G + l;
        const bool inside = i < WOWN_E;
        const uint32_t k = inside ? K(i) : NOKEY, kn = inside ? K(i + 1) : NOKEY;
        bool use = false, ends = kn != k;
        if (active && k != NOKEY && i < reach && !(a.skip_alone && ends && K(i - 1) != k)) {
            if (i < C) {
                if (head_exists && k == k0) use = own_head;    // a run that came in from the left
                else { use = true; ends = ends && k2C != k; }  // starts here: ours entirely if short, else its first piece
            } else if (ext_ok && k == klast) {                 // the rest of our last short run
                use = true;
            } else if (cont && k == klast) {                   // our long piece goes on
                use = true; ends = false;
            }
        }
        const uint64_t wave_mask = __ballot(use);
        const uint64_t mine = (G == 64) ? wave_mask : ((wave_mask >> group_lane0) & ((1ull << G) - 1ull));
        if (use) {
            const int at = count + __popcll(mine & ((1ull << l) - 1ull));
            s_rec[grp][at] = a.rec[slot[u]];
            s_dst[grp][at] = k | (ends ? RUN_ENDS : 0u);
        }
        count += __popcll(mine);
    }
    __syncthreads();
    if (!active || count == 0) return;
    const uint32_t d4 = a.g.d4;
    const uint64_t s4 = a.g.stride4;
    const Rows<G, NV, SL, 0> src(sl, a.src, a.g, l);
    const Rows<G, NV, SL, 1> dst(sl, a.dst, a.g, l);
    const uint32_t cell = (uint32_t)(base >> a.cell_log2);
    const uint32_t head_slot = 2 * cell - 1, tail_slot = 2 * cell;   // used only when they exist

    // (what the lanes past a row's end hold is never stored)
    float4 acc[NV];
    clear<NV>(acc);
    auto finish_row = [&](uint32_t row, const float4 (&old)[NV]) {
        float4 out[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            out[v].x = fmaf(alpha, acc[v].x, old[v].x);
            out[v].y = fmaf(alpha, acc[v].y, old[v].y);
            out[v].z = fmaf(alpha, acc[v].z, old[v].z);
            out[v].w = fmaf(alpha, acc[v].w, old[v].w);
        }
        dst.store_part_nt(row, out);
    };
    for (int b = 0; b < count; b += D) {
        const int at = min(b + l16, WOWN_E - 1), n = count - b;
        const SlotRecord rec = s_rec[grp][at];
        const uint32_t row_l = rec.row, coef_l = __float_as_uint(rec.coef), dst_l = s_dst[grp][at];
        {
            float4 srcv[D][NV], dstv[D][NV];
            // Destination rows are read and written once per minibatch: with the non-temporal hint they
            // do not push the source rows (a few hundred MB that are read again and again) out of the
            // caches -- measured -7 % on this kernel; the same hint on the source rows costs +25 %.
            unrolled<D>([&](auto t) {
                constexpr int J = decltype(t)::value;
                const uint32_t row = of_lane<G, J>(row_l);
                if (J < n) src.template load_part<false>(row, srcv[J]);
            });
            unrolled<D>([&](auto t) {
                constexpr int J = decltype(t)::value;
                const uint32_t k = of_lane<G, J>(dst_l);
                if (J < n && (k & RUN_ENDS)) dst.template load_part<true>(k & ~RUN_ENDS, dstv[J]);
            });
            unrolled<D>([&](auto t) {
                constexpr int J = decltype(t)::value;
                const uint32_t k = of_lane<G, J>(dst_l);
                const float g = __uint_as_float(of_lane<G, J>(coef_l));
                if (J < n) {
                    axpy<NV>(g, srcv[J], acc);
                    if (k & RUN_ENDS) {
                        if (own_head && (k & ~RUN_ENDS) == k0) {       // our piece of a long run ends in the chunk
                            store_row<G, NV>(a.prows + (uint64_t)head_slot * s4, d4, l, acc);
                            if (l == 0) a.pkeys[head_slot] = k0;
                        } else {
                            finish_row(k & ~RUN_ENDS, dstv[J]);
                        }
                        clear<NV>(acc);
                    }
                }
            });
        }
    }
    if (!cont) return;

    // ---- the long piece goes on past the window: stream through the rest of the cell ----
    const uint32_t key = group_value<G>(klast);
    const int64_t limit = base + left;
    bool ended = K(reach) != key;                          // (all of the window's positions up to there are key's, or none after)
    for (int64_t x0 = base + WOWN_E; x0 < limit && !ended; x0 += 16) {
        const int nblk = (int)min((int64_t)16, limit - x0);
        const bool same = l16 < nblk && a.skey[x0 + l16] == key;
        const uint32_t bits = (uint32_t)(__ballot(same) >> group_lane0) & 0xFFFFu;
        const int cnt = __builtin_ctz(~bits);             // entries of the run at the block's front
        SlotRecord rec{0, 0.f};
        if (l16 < cnt) rec = a.rec[a.sidx[x0 + l16]];
        const uint32_t row_l = rec.row, coef_l = __float_as_uint(rec.coef);
        constexpr int S = 2 * D;                           // (no destination rows here)
        unrolled<16 / S>([&](auto batch) {
            constexpr int B = decltype(batch)::value * S;
            const int n = cnt - B;
            if (n <= 0) return;
            float4 srcv[S][NV];
            unrolled<S>([&](auto t) {
                constexpr int J = decltype(t)::value;
                const uint32_t row = of_lane<G, B + J>(row_l);
                if (J < n) src.template load_part<false>(row, srcv[J]);
            });
            unrolled<S>([&](auto t) {
                constexpr int J = decltype(t)::value;
                const float g = __uint_as_float(of_lane<G, B + J>(coef_l));
                if (J < n) axpy<NV>(g, srcv[J], acc);
            });
        });
        ended = cnt < nblk;
    }
    if (!ended && left > WOWN_E) ended = limit >= (int64_t)a.entries || a.skey[limit] != key;
    if (!last_in_head) {
        if (ended) {                                      // the whole run lay inside the cell
            float4 old[NV];
            dst.template load_part<true>(key, old);
            finish_row(key, old);
        } else {                                          // first piece of a run that leaves the cell
            store_row<G, NV>(a.prows + (uint64_t)tail_slot * s4, d4, l, acc);
            if (l == 0) a.pkeys[tail_slot] = key;
        }
    } else {                                              // a piece that began at the cell's start
        store_row<G, NV>(a.prows + (uint64_t)head_slot * s4, d4, l, acc);
        if (l == 0) {
            a.pkeys[head_slot] = key;
            if (!ended) a.pkeys[tail_slot] = key | KEY_ZERO;   // the run fills the cell and goes on
        }
    }
}

template <int G, int NV, class SL>
__global__ __launch_bounds__(adj_threads(G)) void wown_kernel(SegArgs a, SL sl) {
    wown_body<G, NV>(a, sl, blockIdx.x);
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t* __restrict__ x, uint32_t n,
                                                       uint32_t value) {
    uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) x[i] = value;
}

FillJob wseg_fill_job(uint32_t* pkeys, uint32_t M) {
    // border slots of the cells: only pieces of long runs write them
    const uint32_t L = wseg_entries_per_chunk(M), ncells = (M + L - 1) / L;
    return FillJob{pkeys, ncells ? 2 * (ncells - 1) : 0u, KEY_NONE};
}

void launch_wseg_fill(uint32_t* pkeys, uint32_t M, hipStream_t st) {
    const FillJob f = wseg_fill_job(pkeys, M);
    if (f.count)
        hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks_for(f.count, 256)), dim3(256), 0, st, f.p,
                           f.count, f.value);
}

static SegArgs seg_args_of(const WSideArgs& w) {
    SegArgs a{};
    a.src = (const float4*)w.U; a.dst = (float4*)w.W; a.g = w.g; a.skey = w.skey; a.sidx = w.sidx;
    a.rec = w.rec; a.entries = w.M;
    a.alpha = w.alpha; a.prows = (float4*)w.prows; a.pkeys = w.pkeys;
    a.skip_alone = w.skip_alone; a.cell_log2 = wown_cell_log2(w.M);
    return a;
}

static SegArgs seg_args_of(const TailArgs& t) {
    SegArgs a{};
    a.src = (const float4*)t.src_rows; a.dst = (float4*)t.M; a.g = t.g; a.skey = t.src_keys;
    a.sidx = nullptr; a.rec = nullptr; a.entries = t.entries;
    a.skip_alone = false;
    a.alpha = t.alpha; a.prows = (float4*)t.prows; a.pkeys = t.pkeys;
    a.defer_rows = (float4*)t.defer_rows; a.defer_keys = t.defer_keys; a.level = t.level; a.cp = t.cp;
    return a;
}

void launch_wseg(const WSideArgs& w, hipStream_t st) {
    if (w.M == 0) return;
    const SegArgs a = seg_args_of(w);
    uint32_t nchunks = (w.M + WOWN_C - 1) / WOWN_C;
#define CALL(G, NV)                                                                              \
    with_slices(w.slices, [&](const auto& sl) {                                                   \
        hipLaunchKernelGGL((wown_kernel<G, NV, std::decay_t<decltype(sl)>>),  \
                           dim3(blocks_for((uint64_t)nchunks * G, adj_threads(G))),               \
                           dim3(adj_threads(G)), 0, st, a, sl);                                  \
    })
    W2V_DISPATCH_GEOM(w.g.d4, CALL);
#undef CALL
}

void launch_tail(const TailArgs& t, hipStream_t st, bool shared) {
    if (t.entries == 0) return;
    const SegArgs a = seg_args_of(t);
#define CALL_THREADS(G, NV, THREADS)                                                             \
    with_slices(t.slices, [&](const auto& sl) {                                                   \
        hipLaunchKernelGGL((tail_kernel<G, NV, THREADS, std::decay_t<decltype(sl)>>),             \
                           dim3(blocks_for(t.entries, tail_block(G))), dim3(THREADS), 0, st, a, sl); \
    })
#define CALL(G, NV)                                                                              \
    do { if (shared) CALL_THREADS(G, NV, adj_threads(G)); else CALL_THREADS(G, NV, tail_threads(G, NV)); } while (0)
    W2V_DISPATCH_GEOM(t.g.d4, CALL);
#undef CALL
#undef CALL_THREADS
}

// ---------------------------------------------------------------------------------------------
// Write-back of the input-vector changes held in the delta buffer: U[dkey[ps]] += alpha * delta[ps]
// wherever dkey[ps] names a row.  A lane group looks at APPLY_P sorted positions and takes the few
// that do, D rows in flight: four in a joint launch (64 positions one after the other, before: 8 us for
// 4096 pairs).
// ---------------------------------------------------------------------------------------------
constexpr int APPLY_P = 16;
struct ApplyArgs {
    float4* U; RowGeom g; const float4* delta; const uint32_t* dkey; uint32_t n; float alpha;
};

template <int G, int NV, int THREADS, int D, class SL>
__device__ __forceinline__ void apply_body(const ApplyArgs& a, const SL& sl, uint32_t vb) {
    const float alpha = a.alpha;
    const int l = threadIdx.x % G;
    const uint32_t base = (vb * (uint32_t)THREADS + threadIdx.x) / G * APPLY_P;
    const uint32_t mine = l < APPLY_P && base + l < a.n ? a.dkey[base + l] : KEY_NONE;
    const int lane0 = ((int)(threadIdx.x & 63) / G) * G;
    uint32_t todo = (uint32_t)(__ballot(mine != KEY_NONE) >> lane0) & ((1u << APPLY_P) - 1u);
    const Rows<G, NV, SL, 0> U(sl, a.U, a.g, l);
    while (todo) {
        float4 dv[D][NV], uv[D][NV];
        uint32_t key[D];
#pragma unroll
        for (int t = 0; t < D; ++t) {
            const bool on = todo != 0;
            const int e = on ? __builtin_ctz(todo) : 0;
            todo &= todo - 1;                              // (0 stays 0)
            key[t] = on ? (uint32_t)__shfl(mine, e, G) : KEY_NONE;
            load_row_if<G, NV>(on, a.delta + (uint64_t)(on ? base + e : 0u) * a.g.stride4, a.g.d4, l, dv[t]);
            U.load_if(on, on ? key[t] : 0u, uv[t]);
        }
#pragma unroll
        for (int t = 0; t < D; ++t) {
            if (key[t] == KEY_NONE) continue;
            axpy<NV>(alpha, dv[t], uv[t]);
            U.store_part(key[t], uv[t]);       // (joint rows: dv holds anything where U has its padding)
        }
    }
}

// On its own, beside the output side's levels on another stream.  Where it shares the memory with them and
// with announced sorts, one row in flight per group (benchmark step with four 3.177 ms, two 3.179, one 3.168).
template <int G, int NV, int D, class SL>
__global__ __launch_bounds__(adj_threads(G)) void apply_kernel(ApplyArgs a, SL sl) {
    apply_body<G, NV, adj_threads(G), D>(a, sl, blockIdx.x);
}

void launch_apply(const ApplyDelta& x, RowGeom g, bool shared, hipStream_t st) {
    if (x.n == 0) return;
    const ApplyArgs a{(float4*)x.U, g, (const float4*)x.delta, x.dkey, x.n, x.alpha};
#define CALL_ROWS(G, NV, D)                                                                               \
    with_slices(x.slices, [&](const auto& sl) {                                                            \
        hipLaunchKernelGGL((apply_kernel<G, NV, D, std::decay_t<decltype(sl)>>),                          \
                           dim3(blocks_for((uint64_t)blocks_for(x.n, APPLY_P) * G, adj_threads(G))),      \
                           dim3(adj_threads(G)), 0, st, a, sl);                                           \
    })
#define CALL(G, NV) do { if (shared) CALL_ROWS(G, NV, 1); else CALL_ROWS(G, NV, (NV <= 2 ? 4 : 2)); } while (0)
    W2V_DISPATCH_GEOM(g.d4, CALL);
#undef CALL
#undef CALL_ROWS
}

// ---------------------------------------------------------------------------------------------
// One launch for parts of the update that do not depend on each other: a walk of the output side
// (its level-1 kernel when FIRST, else one of its higher levels), one higher level of the input
// side (beside the first walk, which reads U, it parks its sums in the delta buffer, later it adds them to U),
// one step of the loss, and, once that walk is done, the write-back of the delta buffer: a row of U has one run,
// so it gets its sum from one of these alone.  (Write-back behind all of the input side's levels instead, a launch
// more wherever there are three: four announced steps of 65 536 pairs, d = 100, 701 us against 664, a plain
// one of 1999, d = 300, 62 against 60.)
// Each block does one part, told by its number.  The update is a chain of dependent launches; this
// keeps everything that can run beside the output side out of that chain, without a second stream
// (whose event waits cost about 10 us each: the step of 65 536 pairs, d = 100, spent 90 us of 220 on
// them).
// ---------------------------------------------------------------------------------------------
struct StageDev {
    SegArgs w, u;
    ApplyArgs apply;
    uint32_t w_blocks, u_blocks, apply_blocks, loss_blocks;
    uint32_t loss_step;              // 0 none, 1 terms -> block sums, 2 block sums -> loss
    const float* dots; uint32_t total, T;
    double* block_loss; uint32_t nb; double* loss_out;
};

constexpr int stage_threads(int G, int NV, bool first) { return first ? adj_threads(G) : tail_threads(G, NV); }

template <int G, int NV, bool FIRST, class SL>
__global__ __launch_bounds__(stage_threads(G, NV, FIRST)) void adjust_stage_kernel(StageDev s, SL sl) {
    constexpr int D = NV <= 2 ? 4 : 2, THREADS = stage_threads(G, NV, FIRST);
    __shared__ TailLds<G, NV, THREADS, FIRST ? tail_block_first(G) : tail_block(G)> lds;
    __shared__ double red[THREADS / 64];
    uint32_t b = blockIdx.x;                               // the input side's level first: its blocks run longest
    if (b < s.u_blocks) {
        if (FIRST) tail_body<G, NV, THREADS, true, 0>(s.u, OneMatrix{}, b, lds);
        else tail_body<G, NV, THREADS, false, 0>(s.u, sl, b, lds);
        return;
    }
    b -= s.u_blocks;
    if (b < s.loss_blocks) {
        if (s.loss_step == 1) loss_terms_block<THREADS>(s.dots, s.total, s.T, s.block_loss, b, red);
        else sum_doubles_block<THREADS>(s.block_loss, s.nb, s.loss_out, red);
        return;
    }
    b -= s.loss_blocks;
    if (b < s.w_blocks) {
        if constexpr (FIRST) wown_body<G, NV>(s.w, sl, b);
        else tail_body<G, NV, THREADS, false, 1>(s.w, sl, b, lds);
        return;
    }
    b -= s.w_blocks;
    if (!FIRST) apply_body<G, NV, THREADS, D>(s.apply, sl, b);
}

// The input side's levels alone, beside the output side's walk on another stream: blocks no larger than
// that kernel's, which fill the places its blocks leave (of 512 threads they waited for its end).
template <int G, int NV>
__global__ __launch_bounds__(adj_threads(G)) void input_tail_kernel(SegArgs a) {
    __shared__ TailLds<G, NV, adj_threads(G)> lds;
    tail_body<G, NV, adj_threads(G), true, 0>(a, OneMatrix{}, blockIdx.x, lds);
}

void launch_input_tail(const TailArgs& t, hipStream_t st) {
    if (t.entries == 0) return;
    const SegArgs a = seg_args_of(t);
#define CALL(G, NV)                                                                                  \
    hipLaunchKernelGGL((input_tail_kernel<G, NV>), dim3(blocks_for(t.entries, tail_block(G))),       \
                       dim3(adj_threads(G)), 0, st, a)
    W2V_DISPATCH_GEOM(t.g.d4, CALL);
#undef CALL
}

template <int G, int NV, class SL>
static void launch_stage_shape(StageDev s, const SL& sl, bool first, hipStream_t st) {
    if (first) s.w_blocks = blocks_for((uint64_t)((s.w.entries + WOWN_C - 1) / WOWN_C) * G, adj_threads(G));
    else s.w_blocks = blocks_for(s.w.entries, tail_block(G));
    s.u_blocks = blocks_for(s.u.entries, first ? tail_block_first(G) : tail_block(G));
    s.apply_blocks = blocks_for((uint64_t)blocks_for(s.apply.n, APPLY_P) * G, stage_threads(G, NV, first));
    const dim3 grid(s.w_blocks + s.u_blocks + s.apply_blocks + s.loss_blocks);
    if (grid.x == 0) return;
    const dim3 block(stage_threads(G, NV, first));
    if (first) hipLaunchKernelGGL((adjust_stage_kernel<G, NV, true, SL>), grid, block, 0, st, s, sl);
    else hipLaunchKernelGGL((adjust_stage_kernel<G, NV, false, SL>), grid, block, 0, st, s, sl);
}

// (Its own launch keeps its registers to itself, and the levels run beside it; against that, events between
// streams.  Step in us, own launch and joint, k = 5: d = 300, 1.05, 2.1 and 6.3 M slots 634, 660; 1099, 1165;
// 2987, 3223; d = 200 483, 472; 835, 837; 2250, 2291.  Below: 0.3 M slots d = 300 275, 262; d = 200 229, 202; at
// 0.6 M 414, 428; 327, 309.  Rows of up to 128 floats, joint as fast or faster throughout: d = 100, 0.3 to
// 6.3 M slots 201, 172; 260, 239; 343, 333; 578, 568; 1489, 1486.)
bool adjust_walk_alone(uint32_t M, RowGeom g) { return M >= (1u << 20) && g.d4 > 32; }

void launch_adjust_stage(const AdjustStage& x, hipStream_t st) {
    StageDev s{};
    const bool first = x.wfirst != nullptr;                  // (then nothing is written back: FIRST has no such part)
    if (first) s.w = seg_args_of(*x.wfirst);
    else if (x.wtail) s.w = seg_args_of(*x.wtail);
    if (x.utail) s.u = seg_args_of(*x.utail);
    if (x.apply && !first)
        s.apply = ApplyArgs{(float4*)x.apply->U, x.g, (const float4*)x.apply->delta, x.apply->dkey, x.apply->n,
                            x.apply->alpha};
    s.loss_step = x.loss_step;
    if (x.loss_step) {
        s.dots = x.dots; s.total = x.n * x.T; s.T = x.T; s.block_loss = x.loss_tmp;
        s.nb = blocks_for(s.total, loss_terms_of(s.total)); s.loss_out = x.loss_out;
        s.loss_blocks = x.loss_step == 1 ? s.nb : 1u;
    }
#define CALL(G, NV) with_slices(x.slices, [&](const auto& sl) { launch_stage_shape<G, NV>(s, sl, first, st); })
    W2V_DISPATCH_GEOM(x.g.d4, CALL);
#undef CALL
}

// ---------------------------------------------------------------------------------------------
// Input-vector side, level 1: entries are whole pairs (T source rows each) in the order of the
// sorted input words.  Runs finished inside a chunk go to the delta buffer (the input matrix must
// stay untouched until the output side has read it); cut runs go to the partial slots.
// FUSED: the group also holds u, forms the T dots of the pair, turns them into coefficients
// (written out for the output side) and uses them at once -- the output rows are read only once.
// ---------------------------------------------------------------------------------------------
// sigma(-x) = 1 / (1 + e^x): the positive slot's coefficient 1 - sigma(f) is sigma(-f), a negative
// slot's -sigma(f) is -sigma(-(-f)); written this way the coefficient keeps its relative accuracy
// when it is small.
__device__ __forceinline__ float sigmoid_of_minus(float x) { return 1.0f / (1.0f + expf(x)); }

// Coefficients of up to sixteen slots whose dots every lane holds, j0 the number of the first: lane r of every sixteen
// takes slot r, so that the exponential and the division are issued once for all of them, and the results are
// handed round.  `dot` and `g` are this lane's own slot's, for the stores.  (The row kernels are bound by what they
// issue nearly as much as by memory: evaluated slot after slot in every lane, k = 25, d = 200, two steps of 2^18
// pairs 4450 us, this way 4216; k = 10, d = 60, 2^20 pairs 4490, 4320; k = 5, d = 100, four of 65 536 715, 694.)
template <int G, int N>
__device__ __forceinline__ void coefficients(const float (&sdot)[N], uint32_t j0, float (&gco)[N], float& dot, float& g) {
    static_assert(N <= 16, "a lane per slot");
    const int r = threadIdx.x & 15;
    dot = sdot[0];
#pragma unroll
    for (int j = 1; j < N; ++j) dot = r == j ? sdot[j] : dot;
    const bool positive = j0 + r == 0;
    const float s = sigmoid_of_minus(positive ? dot : -dot);
    g = positive ? s : -s;
    if constexpr (G == 64) {                     // (the wavefront's: scalars)
#pragma unroll
        for (int j = 0; j < N; ++j) gco[j] = lane_value(g, j);
    } else {
        share16<0>(g, gco);
    }
}


// Bound by memory where the launch fills the chip.  A pair's rows are asked for TB at a time, then used: every load of a
// batch before the first is waited for, one batch to a lane group, many lane groups.  (With a branch around each load the
// compiler waits for all loads before it: the same kernel with one or two rows in flight.  Input side of a step, us, that
// way and this: 4096 pairs of d = 100 10.8, 7.0; 65 536 58, 52; 100 003 pairs over five shards of 60 columns 182, 130.)
// FULL_BATCHES: pairs are whole batches, and no load stands behind a branch of its own; ONE_BATCH: of one batch.
// REFILLED: a register set is refilled as soon as its row is used, whole batches or not.  Input side, us, batch by batch and refilled:
// at thirty-two lanes a row k = 10, 2^18 pairs of d = 100 299, 282; k = 12, d = 128 364, 326; k = 7, d = 100 234, 228; but 4096 pairs of
// d = 100, in chunks of two pairs, 13.9, 14.9.  At sixteen the same within 3 %: k = 10, 2^20 of d = 60 474, 473; k = 25, 2^18 287, 281; k = 12,
// d = 16 108, 111.  At one float4 of sixty-four batch by batch (k = 25, d = 200 538, 569).  At two float4 a lane and more where a small launch
// leaves each wavefront to hide its own latency: 4096 pairs, k = 20, d = 300 35.7, 32.9, over three slices 48.4, 41.1, d = 600 60.7, 52.9; k = 15,
// 16 384 of d = 300 76.0, 71.5, but of d = 1000 218, 228, and steps of 65 536 of d = 300, k = 8 335, 365.  (The number of slots must stay a
// variable: as a constant, the refilled rows get registers of their own, are waited for and moved at the batch's end, and three
// wavefronts fit instead of four: 2^20 of d = 60 500.)
enum Batches { ANY_BATCH, FULL_BATCHES, ONE_BATCH, REFILLED };
constexpr int VMCNT_0 = 0x0F70;                  // s_waitcnt for loads and stores alone
template <int G, int NV, int TB, Batches FORM, bool FUSED, bool OWN, class SL>
__global__ __launch_bounds__(USEG_THREADS) void useg_kernel(USideArgs a, uint32_t CP, SL sl) {
    constexpr bool NEED_U = FUSED || OWN;      // the pair's input row: for the dots, for own rows
    constexpr bool WHOLE = FORM == FULL_BATCHES || FORM == ONE_BATCH;
    const float alpha = a.alpha;
    constexpr int GROUPS = USEG_THREADS / G;
    // The chunk's indices are staged in LDS first (two dependent gathers for the whole chunk), so
    // that the row loads of the main loop depend on nothing but LDS reads.
    constexpr int MAXP = useg_maxp(G), MAXE = FORM == ONE_BATCH ? MAXP * TB : useg_maxe(G);
    __shared__ uint32_t s_key[GROUPS][MAXE];                      // output row of every entry
    __shared__ float s_cf[FUSED ? 1 : GROUPS][FUSED ? 1 : MAXE];  // given coefficients
    __shared__ uint32_t s_pair[GROUPS][MAXP];                     // pair number of every sorted pair
    __shared__ uint32_t s_skey[GROUPS][MAXP + 2];                 // input word: [0] before, [cnt+1] after
    const int l = threadIdx.x % G, grp = (int)group_value<G>(threadIdx.x / G);
    const uint32_t c = blockIdx.x * (uint32_t)GROUPS + grp;
    const uint32_t nchunks = (a.n + CP - 1) / CP;
    const bool active = c < nchunks;
    const uint32_t ps0 = active ? c * CP : 0u;
    const uint32_t cnt = active ? min(CP, a.n - ps0) : 0u;
    const uint32_t T = FORM == ONE_BATCH ? TB : a.T;
    // (the output side's border slots must be clear before its kernel: a share of them per block)
    for (uint32_t i = blockIdx.x * USEG_THREADS + threadIdx.x; i < a.clear_count; i += gridDim.x * USEG_THREADS)
        a.clear_keys[i] = KEY_NONE;
    for (uint32_t i = l; i < cnt; i += G) {
        s_pair[grp][i] = a.perm[ps0 + i];
        s_skey[grp][i + 1] = a.skey[ps0 + i];
        a.dkey[ps0 + i] = KEY_NONE;
    }
    if (active && l == 0) {
        s_skey[grp][0] = ps0 > 0 ? a.skey[ps0 - 1] : NOKEY;
        s_skey[grp][cnt + 1] = ps0 + cnt < a.n ? a.skey[ps0 + cnt] : NOKEY;
    }
    __syncthreads();
    for (uint32_t i = l; i < cnt * T; i += G) {
        uint32_t pi = i / T, j = i - pi * T;
        uint32_t q = s_pair[grp][pi] * T + j;
        s_key[grp][i] = a.keys[q];                 // may carry ALONE (fused, own rows)
        if (!FUSED) {
            const float g = a.coeffs_in[q];
            s_cf[grp][i] = g;
            a.rec_out[q] = SlotRecord{s_skey[grp][pi + 1], g};
        }
    }
    __syncthreads();
    if (!active) return;

    const uint32_t d4 = a.g.d4;
    const uint64_t s4 = a.g.stride4;
    const Rows<G, NV, SL, 0> U(sl, (const float4*)a.U, a.g, l);
    const Rows<G, NV, SL, 1> W(sl, (const float4*)a.W, a.g, l);
    float4* delta = (float4*)a.delta;
    float4* prows = (float4*)a.prows;

    uint32_t key = group_value<G>(s_skey[grp][1]);
    const bool open_head = (group_value<G>(s_skey[grp][0]) == key);
    uint32_t run_start = ps0;
    uint32_t head_key = KEY_NONE, tail_key = KEY_NONE;
    const uint32_t head_slot = 2 * c - 1, tail_slot = 2 * c;

    // (what the lanes past a row's end hold is not stored; of joint rows the padding between slices is, in the delta buffer and
    // the partial slots, and left out when a row is written back)
    float4 acc[NV];
    clear<NV>(acc);
    float4 w[TB][NV], u[1][NV], un[NV];
    uint32_t row[TB];
    if (FORM == REFILLED) {
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            row[t] = (uint32_t)t < T ? s_key[grp][t] : 0u;
            if ((uint32_t)t < T) W.template load_part<false>(row[t] & ~ALONE, w[t]);
        }
        if (NEED_U) U.template load_part<false>(key, u[0]);
    }
    for (uint32_t pi = 0; pi < cnt; ++pi) {
        const uint32_t p = s_pair[grp][pi];
        const uint32_t next = group_value<G>(s_skey[grp][pi + 2]);
        if (FORM == REFILLED && NEED_U) {                   // the next pair's input row, ahead of need
            if (pi + 1 < cnt) U.template load_part<false>(next, un);
        } else if (NEED_U) {
            const uint32_t in[1] = {key};
            U.template load_all<false>(in, 1u, u);
        }
        for (uint32_t jb = 0; jb < T; jb += TB) {
            const uint32_t slots = WHOLE ? TB : min((uint32_t)TB, T - jb);
            const bool last_batch = jb + TB >= T;
            const uint32_t npi = last_batch ? pi + 1 : pi, njb = last_batch ? 0u : jb + TB;      // the batch that follows
            if (FORM != REFILLED) {
#pragma unroll
                for (int t = 0; t < TB; ++t) row[t] = (uint32_t)t < slots ? group_value<G>(s_key[grp][pi * T + jb + t]) : 0u;
            }
            // a row that no other slot names is read here once and written once: the
            // non-temporal hint keeps it out of the caches' way (without it, step of 2^20 pairs of d = 300, this kernel
            // 1.98 ms, with it 1.73)
            if (FORM != REFILLED) W.template load_all<OWN && G == 64>(row, slots, w);
            float gco[TB];
            if (FUSED) {
                float sdot[TB], f, g;
#pragma unroll
                for (int t = 0; t < TB; ++t) sdot[t] = dot_part_of<NV>(W, u[0], w[t]);
#pragma unroll
                for (int t = 0; t < TB; ++t) sdot[t] = group_sum<G>(sdot[t]);
                coefficients<G>(sdot, jb, gco, f, g);
                if ((uint32_t)l < slots) {
                    a.rec_out[p * T + jb + l] = SlotRecord{key, g};
                    if (a.dots_out) a.dots_out[p * T + jb + l] = f;
                }
            } else {
#pragma unroll
                for (int t = 0; t < TB; ++t) gco[t] = (uint32_t)t < slots ? s_cf[grp][pi * T + jb + t] : 0.f;
                // (all of the batch, here: where only some rows are used, the compiler takes the others for loads in flight and waits
                // before each of the next batch's.  With the dots all are.  k = 20, us: 4096 pairs of d = 60 24.0, 11.3, of d = 300
                // 29.4, 23.3; 2^18 of d = 60 274, 223)
                if (!WHOLE) __builtin_amdgcn_s_waitcnt(VMCNT_0);
            }
            // An output row that no other slot names gets its whole update here, from the
            // registers, with the same two roundings as the output-side kernel
            // (fl(g u), then one fma with alpha); that kernel never sees the slot.
            auto own_row = [&](int t) {
                if (!OWN || (uint32_t)t >= slots || !(row[t] & ALONE)) return;
                float4 out[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    out[v].x = fmaf(alpha, fmaf(gco[t], u[0][v].x, 0.f), w[t][v].x);
                    out[v].y = fmaf(alpha, fmaf(gco[t], u[0][v].y, 0.f), w[t][v].y);
                    out[v].z = fmaf(alpha, fmaf(gco[t], u[0][v].z, 0.f), w[t][v].z);
                    out[v].w = fmaf(alpha, fmaf(gco[t], u[0][v].w, 0.f), w[t][v].w);
                }
                W.store_part_nt(row[t] & ~ALONE, out);
            };
            if (FORM == REFILLED) {
#pragma unroll
                for (int t = 0; t < TB; ++t) {
                    if ((uint32_t)t < slots) axpy<NV>(gco[t], w[t], acc);
                    own_row(t);
                    // this register set is free again: the matching row of the following batch
                    if (npi < cnt && njb + t < T) {
                        row[t] = s_key[grp][npi * T + njb + t];
                        W.template load_part<false>(row[t] & ~ALONE, w[t]);
                    }
                }
            } else {
#pragma unroll
                for (int t = 0; t < TB; ++t) own_row(t);
#pragma unroll
                for (int t = 0; t < TB; ++t)
                    if ((uint32_t)t < slots) axpy<NV>(gco[t], w[t], acc);
            }
        }
        if (next != key) {                       // the run of `key` ends with this pair
            if (run_start == ps0 && open_head) {
                store_row<G, NV>(prows + (uint64_t)head_slot * s4, d4, l, acc);
                head_key = key;
            } else {
                store_row<G, NV>(delta + (uint64_t)run_start * s4, d4, l, acc);
                if (l == 0) a.dkey[run_start] = key;
            }
            clear<NV>(acc);
            run_start = ps0 + pi + 1;
        }
        if (FORM == REFILLED && NEED_U) {
#pragma unroll
            for (int v = 0; v < NV; ++v) u[0][v] = un[v];
        }
        key = next;
    }
    if (run_start < ps0 + cnt) {                 // the last run goes on into the next chunk
        const uint32_t k_last = s_skey[grp][cnt];
        if (run_start == ps0 && open_head) {
            store_row<G, NV>(prows + (uint64_t)head_slot * s4, d4, l, acc);
            head_key = k_last;
            tail_key = k_last | KEY_ZERO;
        } else {
            store_row<G, NV>(prows + (uint64_t)tail_slot * s4, d4, l, acc);
            tail_key = k_last;
        }
    }
    if (l == 0) {
        if (c > 0) a.pkeys[head_slot] = head_key;
        if (c + 1 < nchunks) a.pkeys[tail_slot] = tail_key;
    }
}

template <int G, int NV, int TB, Batches FORM, class SL>
static void launch_useg_form(const USideArgs& a, const SL& sl, uint32_t CP, dim3 grid, dim3 block, hipStream_t st) {
    if (a.fused && a.own_rows) {                 // (only the fused form takes rows over, or slices)
        hipLaunchKernelGGL((useg_kernel<G, NV, TB, FORM, true, true, SL>), grid, block, 0, st, a, CP, sl);
    } else if constexpr (TB <= 9) {
        if (a.fused) hipLaunchKernelGGL((useg_kernel<G, NV, TB, FORM, true, false, SL>), grid, block, 0, st, a, CP, sl);
        else if constexpr (SL::ONE) hipLaunchKernelGGL((useg_kernel<G, NV, TB, FORM, false, false, SL>), grid, block, 0, st, a, CP, sl);
    }
}

template <int G, int NV, int TB, class SL>
static void launch_useg_batch(const USideArgs& a, const SL& sl, uint32_t CP, dim3 grid, dim3 block, hipStream_t st) {
    if constexpr (G <= 32) {
        if (G == 16 || CP > 2) return launch_useg_form<G, NV, TB, REFILLED>(a, sl, CP, grid, block, st);
    }
    if constexpr (NV >= 2) {
        if (a.n <= (NV == 2 ? 16384u : 8192u)) return launch_useg_form<G, NV, TB, REFILLED>(a, sl, CP, grid, block, st);
    }
    if constexpr (G > 16) {
        if constexpr (TB > 9) {
            if (a.T % TB == 0) return launch_useg_form<G, NV, TB, FULL_BATCHES>(a, sl, CP, grid, block, st);
        }
        launch_useg_form<G, NV, TB, ANY_BATCH>(a, sl, CP, grid, block, st);
    }
}

template <int G, int NV, class SL>
static void launch_useg_shape(const USideArgs& a, const SL& sl, hipStream_t st) {
    const uint32_t CP = useg_pairs_per_chunk(a.T, a.g.d4, a.n);
    const uint32_t nchunks = (a.n + CP - 1) / CP;
    dim3 grid(blocks_for((uint64_t)nchunks * G, USEG_THREADS)), block(USEG_THREADS);
    // (the number of slots is a constant for k = 5, the paper's and the benchmark's number of negatives)
    if constexpr (NV <= 2) {
        if (a.T == 6) return launch_useg_form<G, NV, 6, ONE_BATCH>(a, sl, CP, grid, block, st);
    }
    constexpr int TB = NV == 1 ? 9 : (NV == 2 ? 6 : 4);     // rows requested per batch
    if constexpr (NV == 1) {
        // With one float4 per lane there are registers for up to thirteen rows in
        // flight: of 9, 11 and 13 rows per batch, take the one that needs the fewest batches per
        // pair and then leaves the fewest empty places in them (k = 10: one batch of 11 instead of
        // 9 + 2, input-side kernel 3 % faster; k = 25: 13 + 13 instead of 9 + 9 + 8, 1 %).
        if (a.fused && a.own_rows) {
            int best = 9;
            uint32_t best_nb = (a.T + 8) / 9, best_waste = best_nb * 9 - a.T;
            for (int tb : {11, 13}) {
                const uint32_t nb = (a.T + tb - 1) / tb, waste = nb * tb - a.T;
                if (nb < best_nb || (nb == best_nb && waste < best_waste)) { best = tb; best_nb = nb; best_waste = waste; }
            }
            if (best == 11) return launch_useg_batch<G, NV, 11>(a, sl, CP, grid, block, st);
            if (best == 13) return launch_useg_batch<G, NV, 13>(a, sl, CP, grid, block, st);
        }
    }
    launch_useg_batch<G, NV, TB>(a, sl, CP, grid, block, st);
}

void launch_useg(const USideArgs& a, hipStream_t st) {
    if (a.n == 0) return;
#define SHAPE(G, NV) with_slices(a.slices, [&](const auto& sl) { launch_useg_shape<G, NV>(a, sl, st); })
    W2V_DISPATCH_GEOM(a.g.d4, SHAPE);
#undef SHAPE
}

}  // namespace w2v
