// Wave-wide (64 lanes) reductions for gfx950 through the data-parallel-primitive lane moves of
// the vector ALU instead of LDS-routed lane permutes: a dependent chain of six permutes costs
// around a thousand cycles, the same chain of DPP moves a few tens.  All results are the same in
// every lane and do not depend on timing (fixed combination order).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "../../include/moespeq.h"

namespace moespeq {
namespace wave {

// DPP controls: partner lanes inside a row of 16 lanes
constexpr int kSwap1 = 0xB1;        // quad_perm [1,0,3,2]: lane ^ 1
constexpr int kSwap2 = 0x4E;        // quad_perm [2,3,0,1]: lane ^ 2
constexpr int kHalfMirror = 0x141;  // lane i <-> 7 - i inside each 8 lanes (the other quad)
constexpr int kMirror = 0x140;      // lane i <-> 15 - i inside the row (the other half)

template <int kCtrl>
__device__ inline uint32_t move(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xF, 0xF, false);
}
template <int kCtrl>
__device__ inline float move(float v) { return __uint_as_float(move<kCtrl>(__float_as_uint(v))); }
template <int kCtrl>
__device__ inline int move(int v) { return (int)move<kCtrl>((uint32_t)v); }
template <int kCtrl>
__device__ inline double move(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = move<kCtrl>((uint32_t)b), hi = move<kCtrl>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// value of lane `kLane`, as a wave-uniform value
template <int kLane>
__device__ inline uint32_t from_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, kLane); }
template <int kLane>
__device__ inline float from_lane(float v) { return __uint_as_float(from_lane<kLane>(__float_as_uint(v))); }
template <int kLane>
__device__ inline int from_lane(int v) { return __builtin_amdgcn_readlane(v, kLane); }
template <int kLane>
__device__ inline double from_lane(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = from_lane<kLane>((uint32_t)b), hi = from_lane<kLane>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// value of lane `lane` (wave-uniform, not a compile-time constant)
__device__ inline double from_lane(double v, int lane) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Reduction over each row of 16 lanes with a commutative `op`; every lane of the row gets the
// row's result.  After the two quad steps a quad's lanes agree, so the mirror moves pair
// disjoint, already reduced groups.
template <typename T, typename Op>
__device__ inline T row_all(T v, Op op) {
    v = op(v, move<kSwap1>(v));
    v = op(v, move<kSwap2>(v));
    v = op(v, move<kHalfMirror>(v));
    v = op(v, move<kMirror>(v));
    return v;
}

// Reduction over the wave: rows first, then the four row results in row order.
template <typename T, typename Op>
__device__ inline T all(T v, Op op) {
    v = row_all(v, op);
    return op(op(op(from_lane<0>(v), from_lane<16>(v)), from_lane<32>(v)), from_lane<48>(v));
}

__device__ inline float sum(float v) { return all(v, [](float a, float b) { return a + b; }); }
__device__ inline double sum(double v) { return all(v, [](double a, double b) { return a + b; }); }
__device__ inline double max(double v) { return all(v, [](double a, double b) { return fmax(a, b); }); }
__device__ inline int max(int v) { return all(v, [](int a, int b) { return a > b ? a : b; }); }
__device__ inline float row_sum(float v) { return row_all(v, [](float a, float b) { return a + b; }); }

// Sum of the values of this lane and of the lanes below it: shifts inside the rows of 16 lanes, then the row totals
__device__ inline int prefix_sum(int v, int lane) {
    v += move<0x111>(v);                // row_shr 1, 2, 4, 8: lanes that have no partner get 0
    v += move<0x112>(v);
    v += move<0x114>(v);
    v += move<0x118>(v);
    const int r0 = from_lane<15>(v), r1 = r0 + from_lane<31>(v), r2 = r1 + from_lane<47>(v);
    return v + (lane < 16 ? 0 : lane < 32 ? r0 : lane < 48 ? r1 : r2);
}

// A logit as the selections compare it: NaN comes last (unordered, several would share a rank, and ranks below k
// would be left without an expert)
__device__ inline double ordered(double l) { return l == l ? l : -INFINITY; }

// Top-k selection by one wave: lane l holds logits l, l + 64, ... (NR of them, 64 NR >= E).  rank[i] becomes
// the position of logit lane + 64 i in the order (larger first, lower index first among equals) where that is
// below k, else MOE_MAX_EXPERTS; returns, in lane j < k, the index of rank j.
//
// k rounds of a maximum over 32-bit keys that order like the logits rounded to fp32 (six lane moves each);
// where several logits share the largest key, their fp64 values decide.  (Counting the rank of every fp64
// logit, by one wave for up to 32 experts and by all waves of a workgroup beyond, took 0.9 us for 16 experts,
// 2.8 us for 128, and 12.8 us for 128 experts and 8 tokens.)
template <int NR>
__device__ inline int select_topk(const double (&logit)[NR], int E, int k, int lane, int (&rank)[NR])
{
    constexpr int kNone = -2147483647 - 1;       // below the key of every number
    double l[NR];
    int key[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        l[i] = ordered(logit[i]);
        const int b = __float_as_int((float)l[i] + 0.f);     // (-0 and 0 are equal)
        key[i] = lane + 64 * i < E ? b ^ ((b >> 31) & 0x7fffffff) : kNone;
        rank[i] = MOE_MAX_EXPERTS;
    }
    int id = 0;
    for (int j = 0; j < k; ++j) {
        int m = key[0];
#pragma unroll
        for (int i = 1; i < NR; ++i) m = m > key[i] ? m : key[i];
        m = max(m);
        unsigned long long hit[NR];
        int hits = 0;
#pragma unroll
        for (int i = 0; i < NR; ++i) { hit[i] = __ballot(key[i] == m); hits += __popcll(hit[i]); }
        if (hits > 1) {
            double d = -INFINITY;
#pragma unroll
            for (int i = 0; i < NR; ++i) d = key[i] == m ? fmax(d, l[i]) : d;
            d = max(d);
#pragma unroll
            for (int i = 0; i < NR; ++i) hit[i] = __ballot(key[i] == m && l[i] == d);
        }
        int e = 0;
#pragma unroll
        for (int i = NR - 1; i >= 0; --i) e = hit[i] ? 64 * i + __ffsll((long long)hit[i]) - 1 : e;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const bool won = lane + 64 * i == e;
            key[i] = won ? kNone : key[i];
            rank[i] = won ? j : rank[i];
        }
        id = lane == j ? e : id;
    }
    return id;
}

// Rank counting for a top-k selection by several waves.  logit[0 .. E) and rank[0 .. E) live in
// LDS, rank zeroed.  The calling wave adds to rank[e] the number of logits e2 = first,
// first + stride, ... that come before logit e in the order (larger first, lower index first
// among equals); with every e2 covered by some wave, rank[] becomes the position of each logit in
// that strict order.  Lane l keeps logits l, l + 64, ... (NR of them, NR >= ceil(E / 64)) in
// registers; the logits e2 are broadcast reads, kBatch in flight, compared without branches
// (every comparison leaves a mask in scalar registers: a smaller batch where those are scarce).
template <int NR, int kBatch = 8>
__device__ inline void count_ranks(const double *logit, int32_t *rank, int E, int lane, int first, int stride)
{
    double mine[NR];
    int part[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int e = lane + 64 * i;
        mine[i] = ordered(logit[e < E ? e : E - 1]);
        part[i] = 0;
    }
    for (int e2 = first; e2 < E; e2 += kBatch * stride) {
        double v[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int idx = e2 + j * stride;
            v[j] = ordered(logit[idx < E ? idx : E - 1]);
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int idx = e2 + j * stride;
            const int live = idx < E ? 1 : 0;
#pragma unroll
            for (int i = 0; i < NR; ++i)
                part[i] += live & ((int)(v[j] > mine[i]) | ((int)(v[j] == mine[i]) & (int)(idx < lane + 64 * i)));
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int e = lane + 64 * i;
        if (e < E && part[i] != 0) atomicAdd(&rank[e], part[i]);
    }
}
__device__ inline void count_ranks(const double *logit, int32_t *rank, int E, int lane, int first, int stride)
{
    if (E <= 64) count_ranks<1>(logit, rank, E, lane, first, stride);
    else if (E <= 128) count_ranks<2>(logit, rank, E, lane, first, stride);
    else count_ranks<4>(logit, rank, E, lane, first, stride);
}

}  // namespace wave
}  // namespace moespeq
