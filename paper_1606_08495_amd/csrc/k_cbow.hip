// Continuous-bag-of-words variant (Section 5.1, footnote): the kernels that are specific to it.
// Everything else of the step -- negatives, dots, coefficients, both segmented reductions -- runs in
// the skip-gram kernels, which take the matrix of hidden vectors in place of the input vectors.
#include "common.h"
#include "rows.h"

namespace w2v {

static inline unsigned blocks_for(uint64_t items, unsigned per_block) {
    return (unsigned)((items + per_block - 1) / per_block);
}

// ---------------------------------------------------------------------------------------------
// Per context entry e: the checked word, the example it belongs to and the weight 1/|C_p| with
// which the example's summed output rows enter the word's input vector.  The example is found by
// bisection of the offsets, so malformed offsets can at worst give wrong (never out-of-range)
// example numbers; they raise the error flag.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void cbow_entries_kernel(const uint32_t* __restrict__ ctx_off,
                                                           const uint32_t* __restrict__ ctx_idx,
                                                           uint32_t n, uint32_t m, uint32_t V,
                                                           uint32_t* __restrict__ ctx_safe,
                                                           SlotRecord* __restrict__ entry,
                                                           uint32_t* err) {
    uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= m) return;
    uint32_t w = ctx_idx[e];
    if (w >= V) { atomicOr(err, 1u); w = 0; }
    ctx_safe[e] = w;
    uint32_t lo = 0, hi = n;                    // largest p in [0, n) with ctx_off[p] <= e
    while (hi - lo > 1) {
        uint32_t mid = lo + (hi - lo) / 2;
        if (ctx_off[mid] <= e) lo = mid; else hi = mid;
    }
    const uint32_t a = ctx_off[lo], b = ctx_off[lo + 1];
    const bool inside = a <= e && e < b && b <= m;
    if (!inside) atomicOr(err, 1u);
    entry[e] = SlotRecord{lo, inside ? 1.0f / (float)(b - a) : 0.0f};
}

// Offsets must start at 0, never decrease and end at m.
__global__ __launch_bounds__(256) void cbow_check_offsets_kernel(const uint32_t* __restrict__ ctx_off,
                                                                 uint32_t n, uint32_t m,
                                                                 uint32_t* err) {
    uint32_t p = blockIdx.x * 256 + threadIdx.x;
    if (p > n) return;
    bool bad = ctx_off[p] > m;
    if (p == 0) bad = bad || ctx_off[0] != 0;
    if (p == n) bad = bad || ctx_off[n] != m;
    if (p < n) bad = bad || ctx_off[p + 1] < ctx_off[p];
    if (bad) atomicOr(err, 1u);
}

__global__ __launch_bounds__(256) void iota_kernel(uint32_t* __restrict__ x, uint32_t n) {
    uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) x[i] = i;
}

// ---------------------------------------------------------------------------------------------
// Hidden vectors: one lane group per example adds the input rows of its context words in list
// order (eight loads in flight, four or two of longer rows) and divides by their number.  An example without context gets zeros.
// ---------------------------------------------------------------------------------------------
template <int G, int NV>
__global__ __launch_bounds__(256) void cbow_hidden_kernel(const float4* __restrict__ U, RowGeom g,
                                                          const uint32_t* __restrict__ ctx_off,
                                                          const uint32_t* __restrict__ ctx_safe,
                                                          uint32_t n, uint32_t m,
                                                          float4* __restrict__ H) {
    constexpr int UB = NV == 1 ? 8 : (NV == 2 ? 4 : 2);
    const int l = threadIdx.x % G, l16 = threadIdx.x % 16;
    const uint32_t p = (blockIdx.x * 256u + threadIdx.x) / G;
    if (p >= n) return;                                   // whole groups leave together
    const Rows<G, NV, OneMatrix, 0> rows(OneMatrix{}, U, g, l);
    const uint32_t lo = min(group_value<G>(ctx_off[p]), m);
    const uint32_t hi = min(max(group_value<G>(ctx_off[p + 1]), lo), m);
    // (what the lanes past a row's end hold is never stored)
    float4 acc[NV];
    clear<NV>(acc);
    for (uint32_t e = lo; e < hi; e += 16) {              // sixteen words in one access, handed round
        const uint32_t word = ctx_safe[min(e + (uint32_t)l16, hi - 1)];
        unrolled<16 / UB>([&](auto batch) {
            constexpr int B = decltype(batch)::value * UB;
            if (e + B >= hi) return;
            const uint32_t left = hi - (e + B);
            float4 r[UB][NV];
            unrolled<UB>([&](auto t) {
                constexpr int J = decltype(t)::value;
                const uint32_t w = of_lane<G, B + J>(word);
                if ((uint32_t)J < left) rows.template load_part<false>(w, r[J]);
            });
#pragma unroll
            for (int t = 0; t < UB; ++t)
                if ((uint32_t)t < left) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        acc[v].x += r[t][v].x; acc[v].y += r[t][v].y;
                        acc[v].z += r[t][v].z; acc[v].w += r[t][v].w;
                    }
                }
        });
    }
    if (hi > lo) {
        const float cnt = (float)(hi - lo);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            acc[v].x /= cnt; acc[v].y /= cnt; acc[v].z /= cnt; acc[v].w /= cnt;
        }
    }
    store_row<G, NV>(H + (uint64_t)p * g.stride4, g.d4, l, acc);
}

void launch_cbow_entries(const uint32_t* ctx_off, const uint32_t* ctx_idx, uint32_t n, uint32_t m,
                         uint32_t V, uint32_t* ctx_safe, SlotRecord* entry, uint32_t* err, hipStream_t st) {
    hipLaunchKernelGGL(cbow_check_offsets_kernel, dim3(blocks_for((uint64_t)n + 1, 256)), dim3(256),
                       0, st, ctx_off, n, m, err);
    if (m == 0 || n == 0) return;
    hipLaunchKernelGGL(cbow_entries_kernel, dim3(blocks_for(m, 256)), dim3(256), 0, st, ctx_off,
                       ctx_idx, n, m, V, ctx_safe, entry, err);
}

void launch_iota(uint32_t* x, uint32_t n, hipStream_t st) {
    if (n == 0) return;
    hipLaunchKernelGGL(iota_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, x, n);
}

void launch_cbow_hidden(const float* U, RowGeom g, const uint32_t* ctx_off, const uint32_t* ctx_safe,
                        uint32_t n, uint32_t m, float* H, hipStream_t st) {
    if (n == 0) return;
#define CALL(G, NV)                                                                               \
    hipLaunchKernelGGL((cbow_hidden_kernel<G, NV>), dim3(blocks_for((uint64_t)n * G, 256)),       \
                       dim3(256), 0, st, (const float4*)U, g, ctx_off, ctx_safe, n, m, (float4*)H)
    W2V_DISPATCH_GEOM(g.d4, CALL);
#undef CALL
}

}  // namespace w2v
