// Device parts of the minibatch loss, shared by the kernels that form it on their own and by the
// launch that runs them beside other work of the step.  Sums are in double and in an order fixed by
// the block size.
#pragma once
#include "common.h"

namespace w2v {

// Terms per block: a few per thread, so that the block's reduction is a small part of its work (256 a
// block, one per thread and eight barriers each, took 0.35 ms beside the row kernels for the 11.5 M terms
// of a search minibatch) and there are still blocks for the whole chip (4096 a block: 36 us for 600 000
// terms over five shards against 13).  Past 2^24 terms more, for the one block that adds up the sums.
constexpr uint32_t LOSS_SHORT_TERMS = 1u << 24;
__host__ __device__ inline uint32_t loss_terms_of(uint32_t total) { return total <= LOSS_SHORT_TERMS ? 1024u : 16384u; }

// log(1 + e^x) without overflow or cancellation
__device__ __forceinline__ float softplus(float x) {
    return fmaxf(x, 0.f) + log1pf(expf(-fabsf(x)));
}

// Whether slot i, i + step, i + 2 step, ... is a pair's first: the remainder by T is taken once.
struct SlotInPair {
    uint32_t r, T, step;
    __device__ __forceinline__ SlotInPair(uint32_t i, uint32_t t, uint32_t by) : r(i % t), T(t), step(by % t) {}
    __device__ __forceinline__ bool first() const { return r == 0; }
    __device__ __forceinline__ void next() { r += step; r -= r >= T ? T : 0u; }
};

// fixed tree over the values of a block's threads; the sum arrives in thread 0
template <int THREADS>
__device__ __forceinline__ double block_tree_sum(double v, double* red) {       // red[THREADS / 64]
    for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    double sum = red[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) sum += red[w];
    return sum;
}

// Block vb of the loss terms: slot 0 of a pair contributes softplus(-f), the others softplus(f);
// the block's sum goes to block_loss[vb].
template <int THREADS>
__device__ __forceinline__ void loss_terms_block(const float* __restrict__ dots, uint32_t total,
                                                 uint32_t T, double* __restrict__ block_loss,
                                                 uint32_t vb, double* red) {
    const uint32_t terms = loss_terms_of(total), lo = vb * terms, hi = min(total - lo, terms) + lo;
    double v = 0.0;
    SlotInPair slot(lo + threadIdx.x, T, THREADS);
    for (uint32_t i = lo + threadIdx.x; i < hi; i += THREADS) {
        const float f = dots[i];
        v += (double)softplus(slot.first() ? -f : f);        // (one evaluation for both kinds of slot)
        slot.next();
    }
    const double s = block_tree_sum<THREADS>(v, red);
    if (threadIdx.x == 0) block_loss[vb] = s;
}

// *out = sum of x[n] in a fixed order, by one block: thread t adds elements t, t + THREADS, ... in order,
// then the block reduces by the fixed tree.
template <int THREADS>
__device__ __forceinline__ void sum_doubles_block(const double* __restrict__ x, uint32_t n,
                                                  double* __restrict__ out, double* red) {
    double s = 0.0;
#pragma unroll 8
    for (uint32_t i = threadIdx.x; i < n; i += THREADS) s += x[i];
    const double r = block_tree_sum<THREADS>(s, red);
    if (threadIdx.x == 0) *out = r;
}

}  // namespace w2v
