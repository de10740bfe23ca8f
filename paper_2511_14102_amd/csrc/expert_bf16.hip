// bf16 SwiGLU expert kernels for the verify pass (and for the shared experts of the draft
// pass), gfx950.
//
// Paper section 3.4.4: after regrouping, all tokens of one expert are processed together, so
// an expert's weights are streamed from HBM exactly once per call however many of the K+1
// tokens chose it.  Section 2.3: the cost of verification is the union of the experts.
// With at most 16 tokens per expert the work is a [rows x K] x [K x <=16] contraction: the
// weights are the A operand of the 16x16x32 bf16 MFMA, stored pre-tiled so that one 16-byte
// load per lane fetches a whole A tile, and the tokens are the (zero padded) B operand.
// The kernels are bound by the weight stream; MFMA is idle most of the time by design.
#include "plan.h"
#include "stream.h"
#include "wave.h"

namespace moespeq {

namespace {

constexpr int kWaves = 4;          // K-split inside a workgroup
constexpr int kUnroll = 8;         // tiles in flight per wave and matrix

__device__ inline f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// h[row][16 rt .. + 15] = silu(Wg x) * (Wu x) for the rows (tokens) of one expert: 4 waves split K = H; lane (n, c) holds
// token n's inputs and, of its results, intermediate rows 4 c .. 4 c + 3.  row: the lane's row, kNoRow where token n is not
// the expert's.  kHiLo: also h - bf16(h) (rounded to bf16) to hb_lo, for callers that need h to ~16 bits.
struct GateUpSums { float v[kWaves][2][4][64]; };
template <bool kHiLo>
__device__ inline void gateup_tile(const char *gate, const char *up, const uint16_t *__restrict__ x, int row,
                                   uint16_t *__restrict__ hb, uint16_t *__restrict__ hb_lo, int H, int I, int rt, GateUpSums &s_red)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, c = lane >> 4;
    const int U = H / 32, ku0 = (wave * U) / kWaves, nt = ((wave + 1) * U) / kWaves - ku0;
    const bool live = row != kNoRow;
    const size_t first = ((size_t)rt * U + ku0) * 1024;
    const run_t rg = make_run(gate + first, nt * 1024), ru = make_run(up + first, nt * 1024);
    const uint16_t *xrow = x + (size_t)(live ? n : 0) * H + ku0 * 32 + c * 8;

    f32x4 cg = {0.f, 0.f, 0.f, 0.f}, cu = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < nt; k0 += kUnroll) {
        u32x4 a[kUnroll], b[kUnroll], xv[kUnroll];
#pragma unroll
        for (int i = 0; i < kUnroll; ++i) {
            a[i] = run_load16(rg, lane * 16u + (uint32_t)(k0 + i) * 1024u);
            b[i] = run_load16(ru, lane * 16u + (uint32_t)(k0 + i) * 1024u);
            xv[i] = live && k0 + i < nt ? *reinterpret_cast<const u32x4 *>(xrow + (k0 + i) * 32) : (u32x4){0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int i = 0; i < kUnroll; ++i) {
            cg = mfma16(a[i], xv[i], cg);
            cu = mfma16(b[i], xv[i], cu);
        }
    }

#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s_red.v[wave][0][i][lane] = cg[i];
        s_red.v[wave][1][i][lane] = cu[i];
    }
    __syncthreads();
    if (wave != 0 || !live) return;
    uint16_t out[4], out_lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float g = 0.f, v = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { g += s_red.v[w][0][i][lane]; v += s_red.v[w][1][i][lane]; }
        float h = g / (1.f + expf(-g)) * v;
        out[i] = f32_to_bf16_rne(h);
        if (kHiLo) out_lo[i] = f32_to_bf16_rne(h - __uint_as_float((uint32_t)out[i] << 16));
    }
    const size_t o = (size_t)row * I + rt * 16 + c * 4;
    *reinterpret_cast<uint2 *>(hb + o) = make_uint2((uint32_t)out[0] | ((uint32_t)out[1] << 16),
                                                    (uint32_t)out[2] | ((uint32_t)out[3] << 16));
    if (kHiLo)
        *reinterpret_cast<uint2 *>(hb_lo + o) = make_uint2((uint32_t)out_lo[0] | ((uint32_t)out_lo[1] << 16),
                                                           (uint32_t)out_lo[2] | ((uint32_t)out_lo[3] << 16));
}

// The routing weights of a verify call's rows: softmax over the experts, of the ones the plan's launch selected (ids in rank
// order).  One workgroup, one wave per token.
struct WeightArgs { const double *logits; const int32_t *ids; float *row_w; int T, E, k, S, renorm; };
__device__ inline void routing_weights(const WeightArgs &a)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int t = wave; t < a.T; t += kWaves) {
        double l[MOE_MAX_EXPERTS / 64], mx = -INFINITY, den = 0.0;
#pragma unroll
        for (int i = 0; i < MOE_MAX_EXPERTS / 64; ++i) {
            l[i] = lane + 64 * i < a.E ? a.logits[(size_t)t * a.E + lane + 64 * i] : -INFINITY;
            mx = fmax(mx, l[i]);
        }
        const double mine = lane < a.k ? a.logits[(size_t)t * a.E + a.ids[t * a.k + lane]] : -INFINITY;
        mx = wave::max(mx);
#pragma unroll
        for (int i = 0; i < MOE_MAX_EXPERTS / 64; ++i)
            if (64 * i < a.E) den += lane + 64 * i < a.E ? exp(l[i] - mx) : 0.0;
        den = wave::sum(den);
        const double p = lane < a.k ? exp(mine - mx) / den : 0.0, sel = wave::sum(p);
        if (lane < a.k) a.row_w[t * a.k + lane] = a.renorm ? (float)(p / sel) : (float)p;
    }
    if (tid < a.S * a.T) a.row_w[a.T * a.k + tid] = 1.f;
}

// The verify call's down launch counts its arrivals (two row tiles of every live expert) per 32 output columns in the tags of
// the draft kernels' exchange slots (16 bytes each, the tag in the last 8): counter i in the tag of slot i `spread`, as far
// apart as there is room, since atomics on one line are served one after another; the smallest workspace (8 KiB of slots) has
// room for the 2048 counters of the largest H at four to a tag (16 bits each; spread 0).  The gate/up launch clears the
// counters, whatever the workspace holds there (another layer's rows, where layers of different expert counts share it), and the
// last arrival leaves zeros, as the draft calls need them.
struct CombineArgs { unsigned long long *slots; uint16_t *y; int spread, T, k, S, accumulate; };
struct Counter { uint32_t *word; uint32_t shift; };
__device__ inline Counter counter_of(const CombineArgs &c, uint32_t i)
{
    const uint32_t slot = c.spread ? i * c.spread : i / 4, field = c.spread ? 0 : i % 4;
    return {reinterpret_cast<uint32_t *>(c.slots + 2 * slot + 1) + field / 2, 16 * (field % 2)};
}

// All counters to zero, by `workgroups` workgroups
__device__ inline void clear_counters(const CombineArgs &c, int n, int workgroup, int workgroups)
{
    for (int i = workgroup * kWaves * 64 + threadIdx.x; i < n; i += workgroups * kWaves * 64) *counter_of(c, i).word = 0u;
}

// grid.x = I / 16, grid.y = experts of the plan.  kHiLo: the shared experts of a draft call.  Otherwise the verify call;
// its grid has a row more, in front, for what only the down launch needs: the first workgroup computes the routing weights, the
// others clear the arrival counters.
template <bool kHiLo>
__global__ __launch_bounds__(kWaves * 64)
void bf16_gateup_kernel(const Plan *__restrict__ plan, const uint16_t *__restrict__ x, uint16_t *__restrict__ hb,
                        uint16_t *__restrict__ hb_lo, int H, int I, const WeightArgs w, const CombineArgs comb)
{
    __shared__ GateUpSums s_red;
    const int u = kHiLo ? blockIdx.y : (int)blockIdx.y - 1;
    if constexpr (!kHiLo) {
        if (u < 0) {
            if (blockIdx.x == 0) routing_weights(w);
            else clear_counters(comb, H / 32, blockIdx.x - 1, gridDim.x - 1);          // (I >= 64: at least four workgroups)
            return;
        }
    }
    const int row = plan->act_row[u][threadIdx.x & 15];              // (entries past the last are inside the plan)
    const char *gate = (const char *)plan->act_w0[u];
    if (u >= plan->n_active || !__any(row != kNoRow)) return;
    gateup_tile<kHiLo>(gate, gate + (size_t)I * H * 2, x, row, hb, hb_lo, H, I, blockIdx.x, s_red);
}

__device__ inline void load16_agent(const float *p, f32x4 &v)      // two 8-byte loads that the compiler may keep in flight
{
    const unsigned long long *q = reinterpret_cast<const unsigned long long *>(p);
    const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = (f32x4){__uint_as_float((uint32_t)lo), __uint_as_float((uint32_t)(lo >> 32)),
                __uint_as_float((uint32_t)hi), __uint_as_float((uint32_t)(hi >> 32))};
}

// What the last workgroup of 32 output columns does for them: y[t] (bf16) = the token's live rows in a fixed order, routed ones
// by rank, then shared ones.  One wave: lane (token, column quad) takes 4 columns of each half.
__device__ inline void combine_columns(const Plan *__restrict__ plan, const float *obuf, const CombineArgs &c, int H, int col0)
{
    const int lane = threadIdx.x & 63, t = lane & 15, T = c.T, k = c.k, rows = k + c.S;
    if (t >= T) return;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int col = col0 + 16 * half + (lane >> 4) * 4;
        uint2 *out = reinterpret_cast<uint2 *>(c.y + (size_t)t * H + col);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        if (c.accumulate) {
            const uint2 old = *out;
            acc = (f32x4){__uint_as_float(old.x << 16), __uint_as_float(old.x & 0xffff0000u),
                          __uint_as_float(old.y << 16), __uint_as_float(old.y & 0xffff0000u)};
        }
        constexpr int kBatch = 4;
        for (int j0 = 0; j0 < rows; j0 += kBatch) {
            f32x4 v[kBatch];
            int live[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int jj = j0 + j < rows ? j0 + j : rows - 1;
                const int row = t * (jj < k ? k : 1) + (jj < k ? jj : T * k + (jj - k) * T);
                live[j] = plan->row_live[row] & (j0 + j < rows ? 1 : 0);
                load16_agent(obuf + (size_t)row * H + col, v[j]);
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (live[j]) acc += v[j];
        }
        *out = make_uint2((uint32_t)f32_to_bf16_rne(acc.x) | ((uint32_t)f32_to_bf16_rne(acc.y) << 16),
                          (uint32_t)f32_to_bf16_rne(acc.z) | ((uint32_t)f32_to_bf16_rne(acc.w) << 16));
    }
}

// obuf[row, r] = row_w[row] * (Wd h[row])[r] for 16 values of r.
// grid.x = H / 16, grid.y = experts; block = 4 waves splitting K = I.
// kShared (the draft call's shared experts): the operand is hb + hb_lo (two MFMAs per tile), and
// instead of writing obuf the row's outputs are added to y[token] with fp32 atomics (y already holds
// the routed experts' sum, itself made of such atomics, so no combine launch is needed).
// Verify call: the rows leave at agent scope, and the last workgroup of 32 columns to arrive adds them up.  That costs this
// launch 1.8 us (phi shape, 5 tokens: 40.5 / 42.3; 8 tokens x 128 experts 23.3 / 25.0), 3.4 with two shared experts (dsv2lite, 6
// tokens: 29.6 / 33.0), and saves a launch of 4.0 to 4.8 us and the gap before it.  That holds a workgroup about a round trip
// longer, which the loads pay for: a wave's tiles past its last whole batch come in one batch too (one by one, 768
// inputs: 28.5 us for 8 tokens x 128 experts x 2048 outputs, now 25.0).
template <bool kShared>
__global__ __launch_bounds__(kWaves * 64)
void bf16_down_kernel(const Plan *__restrict__ plan, const uint16_t *__restrict__ hb, const uint16_t *__restrict__ hb_lo,
                      float *__restrict__ obuf, int H, int I, const CombineArgs comb)
{
    const int u = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, c = lane >> 4;
    const int n_active = plan->n_active, row = plan->act_row[u][n];      // (entries past the last are inside the plan)
    if constexpr (!kShared) {
        if (u == 0 && plan->n_live == 0) {                               // nobody else will write y
            if (wave == 0 && blockIdx.x % 2 == 0) combine_columns(plan, obuf, comb, H, blockIdx.x * 16);
            return;
        }
    }
    if (u >= n_active || !__any(row != kNoRow)) return;
    const int U = I / 32, ku0 = (wave * U) / kWaves, nt = ((wave + 1) * U) / kWaves - ku0;
    const bool live = row != kNoRow;
    const run_t rd = make_run((const char *)plan->act_w0[u] + (size_t)I * H * 4 + ((size_t)blockIdx.x * U + ku0) * 1024, nt * 1024);
    const size_t hoff = (size_t)(live ? row : 0) * I + ku0 * 32 + c * 8;
    const uint16_t *hrow = hb + hoff;
    const uint16_t *lrow = kShared ? hb_lo + hoff : nullptr;
    const u32x4 zero = {0u, 0u, 0u, 0u};

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < nt; k0 += kUnroll) {
        u32x4 a[kUnroll], hv[kUnroll], lv[kUnroll];
#pragma unroll
        for (int i = 0; i < kUnroll; ++i) {
            a[i] = run_load16(rd, lane * 16u + (uint32_t)(k0 + i) * 1024u);
            hv[i] = live && k0 + i < nt ? *reinterpret_cast<const u32x4 *>(hrow + (k0 + i) * 32) : zero;
            if (kShared) lv[i] = live && k0 + i < nt ? *reinterpret_cast<const u32x4 *>(lrow + (k0 + i) * 32) : zero;
        }
#pragma unroll
        for (int i = 0; i < kUnroll; ++i) {
            acc = mfma16(a[i], hv[i], acc);
            if (kShared) acc = mfma16(a[i], lv[i], acc);
        }
    }

    __shared__ float s_red[kWaves][4][64];
#pragma unroll
    for (int i = 0; i < 4; ++i) s_red[wave][i][lane] = acc[i];
    __syncthreads();
    if (wave != 0) return;
    f32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) v += s_red[w][i][lane];
        o[i] = v;
    }
    // D layout: lane holds rows 4 c .. 4 c + 3 of column n
    const int col = blockIdx.x * 16 + c * 4;
    if constexpr (kShared) {
        if (!live) return;
        float *yrow = obuf + (size_t)n * H + col;                        // obuf is y here
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __hip_atomic_fetch_add(yrow + i, o[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        if (live) {
            const float rw = plan->row_w[row];
            o *= rw;
            unsigned long long *p = reinterpret_cast<unsigned long long *>(obuf + (size_t)row * H + col);
            __hip_atomic_store(p, (unsigned long long)__float_as_uint(o.x) | ((unsigned long long)__float_as_uint(o.y) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(p + 1, (unsigned long long)__float_as_uint(o.z) | ((unsigned long long)__float_as_uint(o.w) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // the stores have been performed
        const Counter at = counter_of(comb, blockIdx.x / 2);
        const uint32_t all = 2u * (uint32_t)plan->n_live;
        uint32_t before = 0;
        if (lane == 0) before = __hip_atomic_fetch_add(at.word, 1u << at.shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (((__builtin_amdgcn_readfirstlane(before) >> at.shift) & 0xffffu) != all - 1u) return;
        if (lane == 0) __hip_atomic_fetch_sub(at.word, all << at.shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" ::: "memory");
        combine_columns(plan, obuf, comb, H, (blockIdx.x & ~1u) * 16);
    }
}

CombineArgs combine_args(const Shape &s, const VerifyCall &v)
{
    return {v.slots, (uint16_t *)v.y, (int)(v.slot_bytes / 16 / (s.H / 32)), s.T, s.k, s.S, v.accumulate};
}

}  // namespace

void launch_verify_gateup(const Shape &s, const VerifyCall &v, hipStream_t st)
{
    const WeightArgs w = {v.logits, v.plan->ids, v.plan->row_w, s.T, s.E, s.k, s.S, s.renorm};
    launch(bf16_gateup_kernel<false>, dim3(s.I / 16, 1 + s.S + (s.E < s.T * s.k ? s.E : s.T * s.k)), dim3(kWaves * 64), 0, st, v.plan,
           (const uint16_t *)v.x, (uint16_t *)v.hb, (uint16_t *)nullptr, s.H, s.I, w, combine_args(s, v));
}

void launch_verify_down(const Shape &s, const VerifyCall &v, hipStream_t st)
{
    const dim3 grid(s.H / 16, s.S + (s.E < s.T * s.k ? s.E : s.T * s.k)), block(kWaves * 64);
    launch(bf16_down_kernel<false>, grid, block, 0, st, v.plan, (const uint16_t *)v.hb, (const uint16_t *)nullptr, v.obuf, s.H, s.I,
           combine_args(s, v));
}

void launch_shared_gateup(const Shape &s, const Plan *plan, const void *x, void *hb, void *hb_lo, hipStream_t st)
{
    launch(bf16_gateup_kernel<true>, dim3(s.I / 16, s.S), dim3(kWaves * 64), 0, st, plan, (const uint16_t *)x, (uint16_t *)hb,
           (uint16_t *)hb_lo, s.H, s.I, WeightArgs{}, CombineArgs{});
}

void launch_shared_down_add(const Shape &s, const Plan *plan, const void *hb, const void *hb_lo, float *y, hipStream_t st)
{
    launch(bf16_down_kernel<true>, dim3(s.H / 16, s.S), dim3(kWaves * 64), 0, st, plan, (const uint16_t *)hb, (const uint16_t *)hb_lo,
           y, s.H, s.I, CombineArgs{});
}

}  // namespace moespeq
