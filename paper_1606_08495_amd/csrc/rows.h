// Device helpers: a lane group of G consecutive lanes (G = 16, 32 or 64, aligned inside the
// 64-wide wavefront) owns one matrix row; lane l keeps float4 number l, l+G, ... of it.
#pragma once
#include "common.h"

#include <type_traits>
#include <utility>

namespace w2v {

__device__ __forceinline__ float4 f4zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }

template <int G, int NV>
__device__ __forceinline__ void load_row(const float4* __restrict__ row, uint32_t d4, int l,
                                         float4 (&r)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        uint32_t i = (uint32_t)l + (uint32_t)(G * v);
        r[v] = (i < d4) ? row[i] : f4zero();
    }
}

template <int G, int NV>
__device__ __forceinline__ void load_row_if(bool on, const float4* __restrict__ row, uint32_t d4,
                                            int l, float4 (&r)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        uint32_t i = (uint32_t)l + (uint32_t)(G * v);
        r[v] = (on && i < d4) ? row[i] : f4zero();
    }
}

// The same where this lane holds a part of the row; what r holds elsewhere is left as it is.
template <int G, int NV>
__device__ __forceinline__ void load_part(const float4* __restrict__ row, uint32_t d4, int l, float4 (&r)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const uint32_t i = (uint32_t)l + (uint32_t)(G * v);
        if (v + 1 < NV || i < d4) r[v] = row[i];
    }
}

typedef float v4f __attribute__((ext_vector_type(4)));

// store_row (below) with the non-temporal hint: rows that are touched once per minibatch and should not push reusable rows
// out of the caches.
template <int G, int NV>
__device__ __forceinline__ void store_row_nt(float4* __restrict__ row, uint32_t d4, int l,
                                             const float4 (&r)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        uint32_t i = (uint32_t)l + (uint32_t)(G * v);
        if (i < d4) {
            v4f x = {r[v].x, r[v].y, r[v].z, r[v].w};
            __builtin_nontemporal_store(x, (v4f*)row + i);
        }
    }
}

template <int G, int NV>
__device__ __forceinline__ void store_row(float4* __restrict__ row, uint32_t d4, int l,
                                          const float4 (&r)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        uint32_t i = (uint32_t)l + (uint32_t)(G * v);
        if (i < d4) row[i] = r[v];
    }
}

// A value that is the same in all lanes of a group: of a whole wavefront's group a scalar, so that what follows from it
// (addresses, branches) is scalar too.
template <int G> __device__ __forceinline__ uint32_t group_value(uint32_t x) {
    return G == 64 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)x) : x;
}

// f(0), f(1), ... f(N - 1), each number a constant of the type it is passed as.
template <class F, int... I> __device__ __forceinline__ void unrolled_list(F& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void unrolled(F f) { unrolled_list(f, std::make_integer_sequence<int, N>{}); }

// This lane's part of the rows of a matrix (WHICH: 0 input, 1 output vectors): of one matrix, or of the slices of
// several shards.  Of slices a lane keeps an address and a stride for each of its float4, as they may lie in
// different matrices.  store_part() writes the whole stride of a row, the pad as zeros.
struct OneMatrix { static constexpr bool ONE = true; };
struct SliceArgs : Slices { static constexpr bool ONE = false; };
template <int G, int NV, class SL, int WHICH> struct Rows;

template <int G, int NV, int WHICH> struct Rows<G, NV, OneMatrix, WHICH> {
    float4* M; uint64_t s4; uint32_t d4; int l;
    uint32_t at;                                           // bytes into a row
    __device__ __forceinline__ Rows(const OneMatrix&, const float4* m, RowGeom g, int lane)
        : M(const_cast<float4*>(m)), s4(g.stride4), d4(g.d4), l(lane), at((uint32_t)lane * 16) {
        asm("" : "+v"(at));      // (one register throughout: formed anew for a load, in that load's own, it has to wait for what else may write there)
    }
    __device__ __forceinline__ void load_if(bool on, uint32_t row, float4 (&r)[NV]) const {
        load_row_if<G, NV>(on, M + (uint64_t)row * s4, d4, l, r);
    }
    // Whether float4 number v of this lane is part of a row.
    __device__ __forceinline__ bool has(int v) const { return v + 1 < NV || (uint32_t)l + (uint32_t)(G * v) < d4; }
    // Rows 0 .. n - 1 of keys (the word in the low 31 bits), all their loads one after the other: a branch between two kinds
    // of load, or zeros where a lane has no part, would have the compiler wait for those before.  What r holds where there
    // is no part is left as it is.  NT: rows whose key has its top bit set are read with the non-temporal hint (one
    // group to a wavefront: its key is a scalar).
    template <bool NT, int N> __device__ __forceinline__ void load_all(const uint32_t (&key)[N], uint32_t n, float4 (&r)[N][NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (has(v)) {
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if ((uint32_t)j < n) load_one(key[j] & KEY_MASK, v, NT && (key[j] & KEY_ALONE), r[j][v]);
            }
        }
    }
    __device__ __forceinline__ void load_one(uint32_t row, int v, bool nt, float4& r) const {
        const float4* from = (const float4*)((const char*)(M + (uint64_t)row * s4) + at) + G * v;
        if (nt) {
            const v4f x = __builtin_nontemporal_load((const v4f*)from);
            r = make_float4(x.x, x.y, x.z, x.w);
        } else {
            r = *from;
        }
    }
    // One row, where this lane holds a part of it; what r holds elsewhere is left as it is.
    template <bool NT> __device__ __forceinline__ void load_part(uint32_t row, float4 (&r)[NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (has(v)) load_one(row, v, NT, r[v]);
    }
    // ... and back, the pad as zeros whatever r holds there.
    __device__ __forceinline__ void store_part_nt(uint32_t row, float4 (&r)[NV]) const {
        if (!has(NV - 1)) r[NV - 1] = f4zero();
        store_nt(row, r);
    }
    __device__ __forceinline__ void store_part(uint32_t row, float4 (&r)[NV]) const {
        if (!has(NV - 1)) r[NV - 1] = f4zero();
        store(row, r);
    }
    __device__ __forceinline__ void store(uint32_t row, const float4 (&r)[NV]) const {
        store_row<G, NV>(M + (uint64_t)row * s4, (uint32_t)s4, l, r);
    }
    __device__ __forceinline__ void store_nt(uint32_t row, const float4 (&r)[NV]) const {
        store_row_nt<G, NV>(M + (uint64_t)row * s4, (uint32_t)s4, l, r);
    }
};

template <int G, int NV, int WHICH> struct Rows<G, NV, SliceArgs, WHICH> {
    float4* at[NV]; uint32_t s4[NV]; bool data[NV], inside[NV];      // (data: not the pad; its loads give zero)
    __device__ __forceinline__ Rows(const SliceArgs& sl, const float4*, RowGeom g, int lane) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const uint32_t i = (uint32_t)lane + (uint32_t)(G * v);
            at[v] = nullptr; s4[v] = 0; data[v] = false; inside[v] = i < g.d4;
            for (uint32_t s = 0; s < sl.count; ++s) {
                if (i >= sl.first[s]) {
                    at[v] = (float4*)sl.M[WHICH][s] + (i - sl.first[s]);
                    s4[v] = sl.stride4[s];
                    data[v] = i - sl.first[s] < sl.d4[s];
                }
            }
        }
    }
    __device__ __forceinline__ void load_if(bool on, uint32_t row, float4 (&r)[NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v) r[v] = on && data[v] ? at[v][(uint64_t)row * s4[v]] : f4zero();
    }
    __device__ __forceinline__ bool has(int v) const { return data[v]; }
    template <bool NT, int N> __device__ __forceinline__ void load_all(const uint32_t (&key)[N], uint32_t n, float4 (&r)[N][NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (data[v]) {
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    if ((uint32_t)j >= n) continue;
                    const float4* from = at[v] + (uint64_t)(key[j] & KEY_MASK) * s4[v];
                    if (NT && (key[j] & KEY_ALONE)) {
                        const v4f x = __builtin_nontemporal_load((const v4f*)from);
                        r[j][v] = make_float4(x.x, x.y, x.z, x.w);
                    } else {
                        r[j][v] = *from;
                    }
                }
            }
        }
    }
    template <bool NT> __device__ __forceinline__ void load_part(uint32_t row, float4 (&r)[NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (!data[v]) continue;
            const float4* from = at[v] + (uint64_t)row * s4[v];
            if (NT) {
                const v4f x = __builtin_nontemporal_load((const v4f*)from);
                r[v] = make_float4(x.x, x.y, x.z, x.w);
            } else {
                r[v] = *from;
            }
        }
    }
    __device__ __forceinline__ void store_part_nt(uint32_t row, float4 (&r)[NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (!data[v]) r[v] = f4zero();
        store_nt(row, r);
    }
    __device__ __forceinline__ void store_part(uint32_t row, float4 (&r)[NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (!data[v]) r[v] = f4zero();
        store(row, r);
    }
    __device__ __forceinline__ void store(uint32_t row, const float4 (&r)[NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (inside[v]) at[v][(uint64_t)row * s4[v]] = r[v];
    }
    __device__ __forceinline__ void store_nt(uint32_t row, const float4 (&r)[NV]) const {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (inside[v]) {
                v4f x = {r[v].x, r[v].y, r[v].z, r[v].w};
                __builtin_nontemporal_store(x, (v4f*)at[v] + (uint64_t)row * s4[v]);
            }
        }
    }
};

// This lane's part of a dot product: over what it has of a row, the rest of a and b may be anything.
template <int NV, class R>
__device__ __forceinline__ float dot_part_of(const R& rows, const float4 (&a)[NV], const float4 (&b)[NV]) {
    float s = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        float t = fmaf(a[v].x, b[v].x, s);
        t = fmaf(a[v].y, b[v].y, t);
        t = fmaf(a[v].z, b[v].z, t);
        t = fmaf(a[v].w, b[v].w, t);
        s = rows.has(v) ? t : s;
    }
    return s;
}

template <int NV>
__device__ __forceinline__ void axpy(float c, const float4 (&x)[NV], float4 (&acc)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        acc[v].x = fmaf(c, x[v].x, acc[v].x);
        acc[v].y = fmaf(c, x[v].y, acc[v].y);
        acc[v].z = fmaf(c, x[v].z, acc[v].z);
        acc[v].w = fmaf(c, x[v].w, acc[v].w);
    }
}

template <int NV>
__device__ __forceinline__ void clear(float4 (&acc)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = f4zero();
}

// Sum over the G lanes of a group; every lane of the group ends with the same bits.
// Inside a 16-lane row the butterfly runs on DPP lane permutations (xor 1, xor 2, then the two
// mirror patterns, in which both partners of a step still add the same two operands).  The four
// row sums of a wavefront are then fetched with v_readlane and added in a fixed order.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

__device__ __forceinline__ float row16_sum(float x) {
    x += dpp_move<0xB1>(x);    // quad_perm [1,0,3,2]
    x += dpp_move<0x4E>(x);    // quad_perm [2,3,0,1]
    x += dpp_move<0x141>(x);   // row_half_mirror: lane i <-> 7-i within 8
    x += dpp_move<0x140>(x);   // row_mirror: lane i <-> 15-i within 16
    return x;
}

// out[j] = the value of lane j of this lane's sixteen
template <int J, int N>
__device__ __forceinline__ void share16(float x, float (&out)[N]) {
    if constexpr (J < N) {
        out[J] = dpp_move<0x150 + J>(x);      // row_newbcast:J
        share16<J + 1>(x, out);
    }
}

__device__ __forceinline__ float lane_value(float x, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}

// The value that number J of a group's first sixteen lanes holds, for all of the group (every sixteen of them hold the same).
template <int G, int J> __device__ __forceinline__ uint32_t of_lane(uint32_t x) {
    if (G == 64) return (uint32_t)__builtin_amdgcn_readlane((int)x, J);
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + J, 0xF, 0xF, true);      // row_newbcast:J
}

template <int G>
__device__ __forceinline__ float group_sum(float x) {
    x = row16_sum(x);
    if (G == 16) return x;
    const float lo = lane_value(x, 0) + lane_value(x, 16);
    const float hi = lane_value(x, 32) + lane_value(x, 48);
    if (G == 32) return (threadIdx.x & 32) ? hi : lo;
    return lo + hi;
}

// Choice of group shape for a row of d4 float4.
#define W2V_DISPATCH_GEOM(d4, CALL)                   \
    do {                                              \
        if ((d4) <= 16)       { CALL(16, 1); }        \
        else if ((d4) <= 32)  { CALL(32, 1); }        \
        else if ((d4) <= 64)  { CALL(64, 1); }        \
        else if ((d4) <= 128) { CALL(64, 2); }        \
        else if ((d4) <= 192) { CALL(64, 3); }        \
        else                  { CALL(64, 4); }        \
    } while (0)

}  // namespace w2v
