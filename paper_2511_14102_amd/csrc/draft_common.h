// Shared pieces of the two draft-pass kernel files (gfx950): the arithmetic helpers of the int4
// path (code unpacking into exact bf16 integers, MFMA wrapper, scale / zero entries), agent-scope
// 16-byte accesses of the router exchange, and the kernels' argument block.
//
// Arithmetic (paper section 4.1.3: 4-bit weights in groups along the input dimension).
// W = (q - z) * s, so for one output row and one group G of inputs
//     sum_{c in G} W[c] v[c] = s * ( sum_c (128 + q[c]) v[c]  -  (z + 128) * sum_c v[c] ).
// 0x4300 is bf16 128.0 with a zero mantissa, so or-ing a code into mantissa bits 0-3 gives the
// bf16 value 128 + q exactly: unpacking is one shift and one and-or per pair of codes.  The
// products and sums are then done by the matrix cores (16x16x32 bf16 MFMA, fp32 accumulation):
// the unpacked codes of 16 weight rows are the B operand, the activations of up to 16 tokens the
// A operand.  Scale, zero and the 128 offset are applied once per group on the accumulators.
#pragma once
#include <type_traits>
#include "plan.h"
#include "stream.h"
#include "wave.h"

namespace moespeq {

namespace {

constexpr int kWaves = kDraftWaves;
constexpr int kThreads = kWaves * 64;
constexpr int kTicketGroups = 16;
constexpr uint32_t kMagic = 0x43004300u;      // bf16 pair (128, 128)

__device__ inline float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// Unpack constants.  Both are made opaque to the compiler (one in a scalar, one in a vector
// register) so that (a & mask) | magic has no literal operand and is selected as the single
// instruction v_and_or_b32.  It must be the compiler's own instruction, not inline assembly:
// the hazard recogniser does not see inline assembly as a VALU write, and an MFMA that read
// such a result directly got a stale operand (wrong results on the GPU).
struct UnpackConsts { uint32_t mask, magic; };
__device__ inline UnpackConsts unpack_consts() {
    UnpackConsts k = {0x000F000Fu, kMagic};
    asm volatile("" : "+s"(k.mask));
    asm volatile("" : "+v"(k.magic));
    return k;
}

// The 8 codes of one 32-bit word as 8 bf16 values 128 + code, in code order (an MFMA operand)
__device__ inline bf16x8 unpack8(uint32_t w, UnpackConsts k) {
    u32x4 r;
    r.x = (w & k.mask) | k.magic;
    r.y = ((w >> 4) & k.mask) | k.magic;
    r.z = ((w >> 8) & k.mask) | k.magic;
    r.w = ((w >> 12) & k.mask) | k.magic;
    return __builtin_bit_cast(bf16x8, r);
}

// ---- e4m3: products of codes with an intermediate h
// A code byte 0 .. 15 IS the e4m3 number q 2^-9 (below 8 a denormal), so the 8 codes of a word become operand bytes with
// two masks and a shift: codes 0, 4, 1, 5 in the first four bytes, 2, 6, 3, 7 in the others.
__device__ inline void unpack8_e4m3(uint32_t w, uint32_t mask, uint32_t &lo, uint32_t &hi) {
    lo = w & mask;
    hi = (w >> 4) & mask;
}
// h = 2^(byte - 127) (p0 + p1 / 16 + p2 / 256 + p3 / 4096), p_i e4m3, with one power of two for up to 128 h, which puts the largest
// in [128, 256).  What the planes leave of h: 4e-7 of the norm; two bf16 numbers left 2.5e-6.
//
// The matrix cores add the products of eight neighbouring bytes of an operand on one grid, 2^-13 of the largest one's exponent
// (measured, 16x16x32 and 16x16x128; the sums of eights meet in fp32).  So the first two planes of eight neighbouring h are rounded to a grid of 2^-10
// of the eight's largest exponent first: with codes below 16 their products then lie on the cores' grid and their sum is exact, and the next plane takes
// up what the grid left (what four bits leave, times 16, has no larger exponent than the value, so the grid is the same for
// both).  Without this: 7.6e-5 of a group's sum, with it 4e-7.
constexpr int kPlanes = 4, kPlaneShift = 4;
// from the largest magnitude: the scale byte, what h is multiplied by, and back.  (The largest of values that are not all finite may be
// any; the sums of the planes are then NaN, which takes all outputs of the token to NaN.)
struct PlaneScale {
    uint32_t byte;
    __device__ explicit PlaneScale(float largest) {
        const uint32_t e = __float_as_uint(largest) >> 23;
        byte = (e < 32u ? 32u : e < 254u ? e : 254u) - 7u;
    }
    __device__ float up() const { return __uint_as_float((254u - byte) << 23); }
    __device__ float down() const { return __uint_as_float(byte << 23); }
};
// 1.5 2^23 units of the grid of eight scaled h, the largest magnitude m.  The exponent is that of the largest value as it is
// rounded, to the grid and then to four bits: the next one from 1.9375 - 2^-11 on (one exponent too low cost such an eight's sum
// 1e-3 of it).  2^-8 at least.
__device__ inline float plane_grid(float m) {
    const uint32_t e = (__float_as_uint(m) + 0x81000u) >> 23;
    return __uint_as_float(((e > 119u ? e : 119u) + 13u) << 23 | 0x400000u);
}

// Computes a value here: a window slot may be refilled behind this point (into the same registers) though the
// value made from its old contents is used further down.  Left alone, the compiler makes the value where it
// is used, copies the slot's contents for that, and waits for all loads in flight at every such copy.
__device__ inline void compute_here(bf16x8 &v) {
    u32x4 u = __builtin_bit_cast(u32x4, v);
    asm volatile("" : "+v"(u));
    v = __builtin_bit_cast(bf16x8, u);
}
__device__ inline void compute_here(float &v) { asm volatile("" : "+v"(v)); }
__device__ inline void compute_here(uint64_t &v) { asm volatile("" : "+v"(v)); }

__device__ inline f32x4 mfma(u32x4 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), b, c, 0, 0, 0);
}

__device__ inline f32x4 mfma_e4m3(uint64_t a, uint64_t b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8((long)a, (long)b, c, 0, 0, 0);
}

// One 16-byte load at agent scope (served by the device's coherence point, not a stale cache line)
__device__ inline u32x4 load16_agent(const void *p) {
    u32x4 v;
    asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");
    return v;
}

// Two and four of them behind one wait (early-clobber outputs: an output must not take the place of
// an address that a later load of the block still needs)
__device__ inline void load16_agent(const void *const (&p)[1], u32x4 (&v)[1]) { v[0] = load16_agent(p[0]); }
__device__ inline void load16_agent(const void *const (&p)[2], u32x4 (&v)[2]) {
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]) : "v"(p[0]), "v"(p[1]) : "memory");
}
__device__ inline void load16_agent(const void *const (&p)[4], u32x4 (&v)[4]) {
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
                 "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]) : "memory");
}

__device__ inline void store16_agent(void *p, u32x4 v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}

// 1 KiB of device memory (16 bytes per lane, at the lane's address g) straight into LDS at byte
// offset lds_base (wave-uniform) + 16 * lane.  Issued as assembly on purpose: the compiler then
// does not know of the transfer and adds no waits of its own for it (it would wait for ALL vector
// memory operations before every barrier and every LDS read that follows); the caller orders the
// use of the data behind the arrival of a later load of the same wave (vector memory operations
// complete in order).  A load to LDS reads M0, and needs a wait state behind the scalar write of it: the
// compiler puts one there for its own loads, but does not look into assembly.
__device__ inline void load16_to_lds(const void *g, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"(g) : "memory");
}

struct FusedArgs {
    const uint16_t *wr;         // [E,H] bf16
    const float *bias;          // [E] or null
    const char *q;              // int4 codes blobs
    const char *sz;             // scale/zero blobs
    size_t stride_q, stride_sz;
    unsigned long long *slots;  // copies (exchange_copies_lg) x [T,E] x {logit bits, tag}; idle: tag = 0
    size_t replica_stride;      // in 8-byte units
    uint32_t *tickets;          // kTicketGroups + 1 counters; idle: 0
    uint32_t *status;           // set to 1 when a wait for the router result ran out of polls
    uint32_t spin_limit;        // polls of the router result before a workgroup gives up
    float *y;                   // [T,H] out, accumulated with atomics
    int32_t *ids_out;           // [T,k]
    float *conf_out;            // [T,k] or null
    Plan *plan;                 // filled for the shared-expert kernels when S > 0
    const char *shared;         // bf16 shared expert blobs
    size_t shared_stride;
    int T, H, E, I, k, g, S, renorm;
};

// ---- the router inside a draft call (both kernels)

// Workgroup b (numbered among the call's `nprod` router workgroups) reduces router rows b, b + nprod, ...
// for all T tokens and publishes each {logit, tag}.  The NW waves are shared out over the tokens, NW / T2
// of them (T2: T rounded up to a power of two) splitting H, so that a row costs one round of loads and
// one barrier however many tokens there are (one token after another took 6 us for 8 tokens).  fp64
// accumulation of exact fp32 products.  Before it publishes, the workgroup clears its share of y.
// ROWS = 2 (one token): it takes two neighbouring rows at a time, half of its waves each.  us per pass, one row / two: H = 2048, E = 128, 22
// routed workgroups 255 / 204; phi shape (E = 16) 191.5 / 193.5, which is what the room for other calls' workgroups costs (router_workgroups).
template <int NW, int ROWS>
__device__ inline void publish_router_rows(const uint16_t *__restrict__ xin, const FusedArgs &a, int b, int nprod,
                                           double (&s_part)[NW])
{
    constexpr int kTh = NW * 64, kRowWaves = NW / ROWS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = a.T, H = a.H, E = a.E, chunks = H / 8, lg = exchange_copies_lg(E);
    for (int i = b * kTh + tid; i < T * H; i += nprod * kTh)
        __hip_atomic_store(&a.y[i], 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int lt = T <= 1 ? 0 : (T <= 2 ? 1 : (T <= 4 ? 2 : 3));
    const int in_row = ROWS > 1 ? wave % kRowWaves : wave, t = in_row & ((1 << lt) - 1), part = in_row >> lt, step = (kRowWaves >> lt) * 64;
    const uint16_t *xt = xin + (size_t)(t < T ? t : T - 1) * H;
    for (int e = b * ROWS; e < E; e += nprod * ROWS) {
        // of the rows e, e + 1: the one to reduce, the one to publish (behind an odd last row, that one again, not published)
        const int reduced = ROWS > 1 && e + 1 < E ? wave / kRowWaves : 0, mine = ROWS > 1 ? (tid >> lg) % ROWS : 0;
        const uint16_t *row = a.wr + (size_t)(e + reduced) * H;
        const float bias = a.bias ? a.bias[ROWS > 1 && e + mine >= E ? e : e + mine] : 0.f;          // (here and not behind the barrier: a round trip to memory)
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        auto chunks_at = [&](int c0, auto batch) {           // (a position past the end counts as zeros)
            constexpr int kB = decltype(batch)::value;
            u32x4 xv[kB], wv[kB];
#pragma unroll
            for (int j = 0; j < kB; ++j) {
                const int c = c0 + j * step, cc = c < chunks ? c : chunks - 1;
                xv[j] = *reinterpret_cast<const u32x4 *>(xt + cc * 8);
                wv[j] = *reinterpret_cast<const u32x4 *>(row + cc * 8);
            }
#pragma unroll
            for (int j = 0; j < kB; ++j) {
                const bool in = c0 + j * step < chunks;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t xs = in ? xv[j][i] : 0u, ws = in ? wv[j][i] : 0u;
                    acc[i] += (double)(bf16_lo(xs) * bf16_lo(ws));       // bf16 x bf16 is exact in fp32
                    acc[i] += (double)(bf16_hi(xs) * bf16_hi(ws));
                }
            }
        };
        if (chunks <= step) chunks_at(part * 64 + lane, std::integral_constant<int, 1>{});
        else for (int c0 = part * 64 + lane; c0 - lane < chunks; c0 += 4 * step) chunks_at(c0, std::integral_constant<int, 4>{});
        const double sum = wave::sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
        if (lane == 0) s_part[wave] = sum;
        // every thread's clearing stores have been performed before the workgroup publishes (a
        // workgroup-scope release fence does not imply this wait; it is nearly free here, the loads
        // of the row were issued after the stores and have returned)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid < (T * ROWS) << lg && (ROWS == 1 || e + mine < E)) {        // thread (token or row, copy)
            const int tt = ROWS > 1 ? 0 : tid >> lg, rep = tid & ((1 << lg) - 1);
            double l = 0.0;
#pragma unroll
            for (int w = 0; w < kRowWaves; ++w) l += (w & ((1 << lt) - 1)) == tt ? s_part[mine * kRowWaves + w] : 0.0;
            l += (double)bias;
            // {logit, tag} leaves as ONE aligned 16-byte agent-scope store and is read with one
            // 16-byte load: a reader sees the tag only together with the logit
            const unsigned long long lb = (unsigned long long)__double_as_longlong(l);
            const u32x4 rec = {(uint32_t)lb, (uint32_t)(lb >> 32), 1u, 0u};
            store16_agent(a.slots + (size_t)rep * a.replica_stride + 2 * ((size_t)tt * E + e + mine), rec);
        }
        if (e + nprod * ROWS < E) __syncthreads();                  // s_part is written again
    }
}

// One wave polls the slots of token t until all are tagged and selects its top-k: ids in rank order
// (larger logit first, lower index first among equals) to ids[0 .. k), every logit and its rank
// (MOE_MAX_EXPERTS: not selected) to LDS for the softmax, which follows later, and the selected experts
// to the words of `mask` (unless null).  `logit` null: only the wait.  False: the wait ran out of polls.
template <int NR>                                // NR: 64 NR >= E
__device__ inline bool poll_and_select(const FusedArgs &a, int t, double *logit, int32_t *rank, int32_t *ids,
                                       unsigned long long *mask)
{
    const int lane = threadIdx.x & 63, E = a.E, k = a.k;
    const void *from[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int e = lane + 64 * i < E ? lane + 64 * i : E - 1;
        from[i] = a.slots + (size_t)(blockIdx.x & ((1u << exchange_copies_lg(E)) - 1u)) * a.replica_stride + 2 * ((size_t)t * E + e);
    }
    u32x4 v[NR];
    bool all = false;
    for (uint32_t spins = 1; spins < a.spin_limit; ++spins) {
        load16_agent(from, v);
        bool mine = true;
#pragma unroll
        for (int i = 0; i < NR; ++i) mine = mine && v[i].z == 1u;
        all = __all(mine);
        if (all) break;
        __builtin_amdgcn_s_sleep(2);
    }
    if (!all) return false;
    if (!logit) return true;
    double l[NR];
    int rk[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int e = lane + 64 * i;
        l[i] = __longlong_as_double((long long)(((unsigned long long)v[i].y << 32) | v[i].x));
        if (e < E) logit[e] = l[i];
    }
    const int id = wave::select_topk(l, E, k, lane, rk);
    if (lane < k) ids[lane] = id;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (lane + 64 * i < E) rank[lane + 64 * i] = rk[i];
        if (mask) {
            const unsigned long long sel = __ballot(rk[i] < k);
            if (lane == 0) atomicOr(&mask[i], sel);
        }
    }
    return true;
}
__device__ inline bool poll_and_select(const FusedArgs &a, int t, double *logit, int32_t *rank, int32_t *ids,
                                       unsigned long long *mask)
{
    if (a.E <= 64) return poll_and_select<1>(a, t, logit, rank, ids, mask);
    if (a.E <= 128) return poll_and_select<2>(a, t, logit, rank, ids, mask);
    return poll_and_select<4>(a, t, logit, rank, ids, mask);
}

// Tickets.  A wave draws one when its workgroup has finished polling; the holder of the last one puts the
// slots back to idle.  Two levels (kTicketGroups counters, then one) so that the returning atomics do not
// queue up on one address.  The counter's address goes through an opaque vector register: on a uniform
// address the compiler aggregates over the wave and reads the result back at once, which waits for
// everything the wave has in flight; like this the result is waited for where it is used.
__device__ inline uint32_t draw_ticket(uint32_t *counter) {
    uint64_t p = (uint64_t)counter;
    asm volatile("" : "+v"(p));
    return __hip_atomic_fetch_add((__attribute__((address_space(1))) uint32_t *)p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint32_t ticket_members(uint32_t b, uint32_t grid) { return (grid - b % kTicketGroups + kTicketGroups - 1) / kTicketGroups; }
__device__ inline uint32_t ticket_groups(uint32_t grid) { return grid < (uint32_t)kTicketGroups ? grid : (uint32_t)kTicketGroups; }
// `threads` threads, of which the calling one is number `me`, put slots and tickets back to idle
__device__ inline void reset_exchange(const FusedArgs &a, int me, int threads) {
    // (all copies of a slot by neighbouring threads: copy by copy, few experts' stores were sixteen rounds one after another at the
    // kernel's end; us per pass, copy by copy / now: H = 640, E = 6 219.5 / 209.7, H = 1280, E = 5 324.2 / 316.9)
    const int lg = exchange_copies_lg(a.E), n = (a.T * a.E) << lg;
    for (int i = me; i < n; i += threads)
        __hip_atomic_store(a.slots + (size_t)(i & ((1 << lg) - 1)) * a.replica_stride + 2 * (size_t)(i >> lg) + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (me <= kTicketGroups) __hip_atomic_store(a.tickets + me, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The softmax of a token whose logits and ranks the calling wave left in LDS: confidences and routing
// weights in rank order.  The selection compared the fp64 logits; the softmax values only have to be good
// to fp32, so they are computed in fp32 from the fp64 differences.
__device__ inline void finish_softmax(const FusedArgs &a, const double *logit, const int32_t *rank, float *conf, float *w)
{
    const int lane = threadIdx.x & 63, E = a.E, k = a.k;
    double mx = -INFINITY;
    for (int e = lane; e < E; e += 64) mx = fmax(mx, logit[e]);
    mx = wave::max(mx);
    float den = 0.f, sel = 0.f;
    for (int e = lane; e < E; e += 64) den += expf((float)(logit[e] - mx));
    den = wave::sum(den);
    for (int e = lane; e < E; e += 64) sel += rank[e] < k ? expf((float)(logit[e] - mx)) / den : 0.f;
    sel = wave::sum(sel);
    for (int e = lane; e < E; e += 64) {
        const int r = rank[e];
        if (r < k) {
            const float p = expf((float)(logit[e] - mx)) / den;
            conf[r] = p;
            w[r] = a.renorm ? p / sel : p;
        }
    }
}

// The plan that the shared experts' own kernels read (one workgroup writes it)
__device__ inline void write_shared_plan(const FusedArgs &a)
{
    Plan *p = a.plan;
    const int tid = threadIdx.x, n = a.T * a.k;
    if (tid < a.S * 16) {
        const int s = tid / 16, t = tid % 16;
        p->act_row[s][t] = t < a.T ? (uint8_t)(n + s * a.T + t) : kNoRow;
    }
    if (tid < a.S) p->act_w0[tid] = (uint64_t)(a.shared + (size_t)tid * a.shared_stride);
    if (tid == 0) p->n_active = a.S;
}

// Launch with `lds` bytes of dynamic LDS; beyond 48 KiB the limit has to be raised once per kernel.
template <typename K>
void launch_with_lds(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, const uint16_t *x,
                     const FusedArgs &a)
{
    static size_t raised = 0;                    // per instantiation
    if (lds > 48 * 1024 && lds > raised) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        raised = lds;
    }
    launch(kernel, grid, block, lds, st, x, a);
}

// workgroups of `kernel` (block threads, lds bytes of dynamic LDS) one compute unit holds at once
template <typename K>
int resident_per_cu(K kernel, int threads, size_t lds)
{
    if (lds > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds) != hipSuccess) return 0;
    return n;
}

inline FusedArgs fused_args(const Shape &s, const DraftFusedArgs &d)
{
    FusedArgs a;
    a.wr = (const uint16_t *)d.wr; a.bias = d.bias;
    a.q = (const char *)d.q; a.sz = (const char *)d.sz; a.stride_q = d.stride_q; a.stride_sz = d.stride_sz;
    a.slots = d.slots; a.replica_stride = d.replica_stride; a.tickets = d.tickets; a.y = d.y;
    a.status = d.status; a.spin_limit = d.spin_limit;
    a.ids_out = d.ids_out; a.conf_out = d.conf_out; a.plan = d.plan;
    a.shared = (const char *)d.shared; a.shared_stride = d.shared_stride;
    a.T = s.T; a.H = s.H; a.E = s.E; a.I = s.I; a.k = s.k; a.g = s.g; a.S = s.S; a.renorm = s.renorm;
    return a;
}

}  // namespace

}  // namespace moespeq
