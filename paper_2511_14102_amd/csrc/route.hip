// Router, top-k, softmax weights, token->expert histogram / permutation, execution plan and
// expert union kernels (gfx950).
//
// Paper section 2.1: the router turns a token's hidden state into a distribution over the
// experts and the top-k experts are selected, weighted by their scores.  Section 3.4.2: the
// gate stays 16-bit in the draft model because routing errors corrupt the lookahead, so the
// logits here are accumulated in fp64 (products of two bf16 values are exact), which keeps
// the selected ids identical to an exact evaluation unless two logits agree to ~1e-13.
// Section 3.4.4: assignments are regrouped per expert.  Section 2.3 / 3.2.2: union of the
// experts of a window and the part of it that is not resident.
#include "plan.h"
#include "wave.h"

namespace moespeq {

namespace {

constexpr int kRouteThreads = 1024;

// One workgroup per token: logits of all experts (one wave per expert row at a time), ranks of
// the logits counted by all waves, then wave 0 writes the k selected experts in rank order with
// their softmax weights.
__global__ __launch_bounds__(kRouteThreads)
void route_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wr,
                  const float *__restrict__ bias, int H, int E, int k, int renorm,
                  int32_t *__restrict__ ids, float *__restrict__ w, float *__restrict__ conf)
{
    __shared__ double s_logit[MOE_MAX_EXPERTS];
    __shared__ int32_t s_rank[MOE_MAX_EXPERTS];
    const int t = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nwave = kRouteThreads / 64;
    const uint16_t *xt = x + (size_t)t * H;
    const int chunks = H / 8;

    for (int e = wave; e < E; e += nwave) {
        const uint16_t *row = wr + (size_t)e * H;
        // eight independent partial sums instead of one chain of dependent fp64 additions; the
        // products are exact in fp32 (bf16 x bf16).  (The loop is bound by the instruction rate of
        // the one compute unit a token's workgroup runs on: batching the loads did not help.)
        double part[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int c = lane; c < chunks; c += 64) {
            uint4 xv = *reinterpret_cast<const uint4 *>(xt + c * 8);
            uint4 wv = *reinterpret_cast<const uint4 *>(row + c * 8);
            const uint32_t xs[4] = {xv.x, xv.y, xv.z, xv.w};
            const uint32_t ws[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                part[2 * i] += (double)(__uint_as_float(xs[i] << 16) * __uint_as_float(ws[i] << 16));
                part[2 * i + 1] += (double)(__uint_as_float(xs[i] & 0xffff0000u) * __uint_as_float(ws[i] & 0xffff0000u));
            }
        }
        double acc = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
        acc = wave::sum(acc);
        if (lane == 0) { s_logit[e] = acc + (bias ? (double)bias[e] : 0.0); s_rank[e] = 0; }
    }

    __syncthreads();
    // Rank of every logit under (larger first, lower index first among equals), counted by all
    // sixteen waves, each over its share of the experts (one wave alone needs microseconds for a
    // serial selection: about 16 clocks per instruction, and the count grows with E).  The order is
    // strict, so the ranks are a permutation and rank < k is the selection.
    wave::count_ranks(s_logit, s_rank, E, lane, wave, nwave);
    __syncthreads();
    if (wave != 0) return;
    double mine[4], pe[4];
    int rank[4];
    double mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = lane + 64 * i;
        const bool have = 64 * i < E && e < E;
        mine[i] = have ? s_logit[e] : -INFINITY;
        rank[i] = have ? s_rank[e] : MOE_MAX_EXPERTS;
        mx = fmax(mx, mine[i]);
    }
    mx = wave::max(mx);
    double den = 0.0, sel = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        pe[i] = rank[i] < MOE_MAX_EXPERTS ? exp(mine[i] - mx) : 0.0;
        den += pe[i];
    }
    den = wave::sum(den);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        pe[i] = pe[i] / den;
        sel += rank[i] < k ? pe[i] : 0.0;
    }
    sel = wave::sum(sel);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (rank[i] < k) {
            const size_t o = (size_t)t * k + rank[i];
            ids[o] = lane + 64 * i;
            const float c = (float)pe[i];
            if (conf) conf[o] = c;
            w[o] = renorm ? (float)(pe[i] / sel) : c;
        }
    }
}

// count / off / perm for n <= MOE_MAX_ASSIGN assignments over E experts; one workgroup of at least
// 256 threads, results in `count`, `off`, `perm` (global or shared memory), `ids` in LDS.
// Thread a owns assignment a: counts by LDS atomics, offsets by a scan in wave 0 (four experts per
// lane), and the place of a inside its expert is the number of earlier assignments with the same
// expert, counted over broadcast reads of ids (ascending a inside an expert: stable).  The loops
// of the first version (thread e scanning all assignments and all smaller experts, one dependent
// LDS read per step) took 12 us for 64 assignments over 128 experts.
__device__ inline void histogram_perm(const int32_t *ids, int n, int E, int32_t *count,
                                      int32_t *off, int32_t *perm, int32_t *s_count)
{
    __shared__ int32_t s_excl[MOE_MAX_EXPERTS + 1];
    const int tid = threadIdx.x;
    for (int e = tid; e < E; e += blockDim.x) s_count[e] = 0;
    __syncthreads();
    const int my_e = tid < n ? ids[tid] : -1;
    if (tid < n) atomicAdd(&s_count[my_e], 1);
    __syncthreads();
    if (tid < 64) {
        int c[4], sum = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 4 * tid + i;
            c[i] = e < E ? s_count[e] : 0;
            sum += c[i];
        }
        int incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(incl, d, 64);
            if (tid >= d) incl += v;
        }
        int base = incl - sum;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 4 * tid + i;
            if (e < E) s_excl[e] = base;
            base += c[i];
        }
        if (tid == 0) s_excl[E] = n;
    }
    __syncthreads();
    for (int e = tid; e <= E; e += blockDim.x) {
        off[e] = s_excl[e];
        if (e < E) count[e] = s_count[e];
    }
    if (tid < n) {
        int before = 0;
        for (int a = 0; a < n; a += 8) {
            int v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = ids[a + j < n ? a + j : n - 1];       // the same address in every lane
#pragma unroll
            for (int j = 0; j < 8; ++j) before += (int)(a + j < tid) & (int)(v[j] == my_e);
        }
        perm[s_excl[my_e] + before] = tid;
    }
    __syncthreads();
}

__global__ __launch_bounds__(256)
void perm_kernel(const int32_t *__restrict__ ids, int n, int E, int32_t *count, int32_t *off,
                 int32_t *perm)
{
    __shared__ int32_t s_ids[MOE_MAX_ASSIGN];
    __shared__ int32_t s_count[MOE_MAX_EXPERTS];
    for (int a = threadIdx.x; a < n; a += blockDim.x) s_ids[a] = ids[a];
    __syncthreads();
    histogram_perm(s_ids, n, E, count, off, perm, s_count);
}

// Builds the execution plan: histogram / permutation, the list of experts to run (shared
// experts at active indices [0, S), then present routed experts ascending), their weight
// pointers and row ranges, the per-row token / weight / live flags, and the missing list.  The ids and weights
// come from other workgroups of the launch: stored and loaded at agent scope.
template <typename V>
__device__ inline void put(V *p, V v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename V>
__device__ inline V get(const V *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ inline void plan_body(Plan *__restrict__ plan, int T, int E, int k, int S,
                 const char *pool, size_t slot_stride,
                 const int32_t *__restrict__ slot_of_expert,
                 const char *shared, size_t shared_stride, int flags,
                 int32_t *ids_out, int32_t *missing, int32_t *n_missing)
{
    __shared__ int32_t s_ids[MOE_MAX_ASSIGN];
    __shared__ int32_t s_count[MOE_MAX_EXPERTS];
    __shared__ int32_t s_slot[MOE_MAX_EXPERTS];
    __shared__ unsigned char s_listed[MOE_MAX_EXPERTS];
    __shared__ int32_t s_off[MOE_MAX_EXPERTS + 1];     // offsets and permutation stay in LDS for the
    __shared__ int32_t s_perm[MOE_MAX_ASSIGN];         // steps below; the plan gets a copy
    __shared__ int32_t s_nact, s_nmiss;
    const int n = T * k;
    const bool only_listed = (flags & MOE_VERIFY_ONLY_LISTED) != 0;

    for (int a = threadIdx.x; a < n; a += blockDim.x) {
        int id = get(&plan->ids[a]);
        s_ids[a] = id;
        if (ids_out) ids_out[a] = id;
    }
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        s_slot[e] = slot_of_expert[e];
        s_listed[e] = only_listed ? 0 : 1;
    }
    __syncthreads();
    if (only_listed) {
        int nin = *n_missing;
        nin = nin < 0 ? 0 : (nin > E ? E : nin);
        for (int i = threadIdx.x; i < nin; i += blockDim.x) {
            int e = missing[i];
            if (e >= 0 && e < E) s_listed[e] = 1;
        }
    }
    __syncthreads();
    histogram_perm(s_ids, n, E, plan->count, s_off, s_perm, s_count);
    for (int e = threadIdx.x; e <= E; e += blockDim.x) plan->off[e] = s_off[e];
    for (int i = threadIdx.x; i < n; i += blockDim.x) plan->perm[i] = s_perm[i];

    // shared experts: active slots [0, S), rows T*k + s*T + t
    for (int i = threadIdx.x; i < S * T; i += blockDim.x) {
        plan->row_tok[n + i] = i % T;
        plan->row_w[n + i] = 1.f;
        plan->row_live[n + i] = only_listed ? 0 : 1;
    }
    if ((int)threadIdx.x < S) {
        int s = threadIdx.x;
        plan->act_expert[s] = E + s;
        plan->act_off[s] = n + s * T;
        plan->act_cnt[s] = only_listed ? 0 : T;
        plan->act_w0[s] = (uint64_t)(shared + (size_t)s * shared_stride);
    }
    // routed experts: ordered compaction, 64 experts per step, by wave 0
    if (threadIdx.x < 64) {
        int nact = S, nmiss = 0;
        for (int base = 0; base < E; base += 64) {
            int e = base + threadIdx.x;
            bool used = e < E && s_count[e] > 0 && s_listed[e];
            bool present = used && s_slot[e] >= 0;
            bool absent = used && s_slot[e] < 0;
            unsigned long long bp = __ballot(present), ba = __ballot(absent);
            unsigned long long below = (1ull << threadIdx.x) - 1ull;
            if (present) {
                int u = nact + __popcll(bp & below);
                int slot = s_slot[e];
                plan->act_expert[u] = e;
                plan->act_off[u] = s_off[e];
                plan->act_cnt[u] = s_count[e];
                plan->act_w0[u] = (uint64_t)(pool + (size_t)slot * slot_stride);
            }
            if (absent) missing[nmiss + __popcll(ba & below)] = e;
            nact += __popcll(bp);
            nmiss += __popcll(ba);
        }
        if (threadIdx.x == 0) { s_nact = nact; s_nmiss = nmiss; }
    }
    __syncthreads();
    for (int pos = threadIdx.x; pos < n; pos += blockDim.x) {
        int a = s_perm[pos];
        int e = s_ids[a];
        plan->row_tok[pos] = a / k;
        plan->row_w[pos] = get(&plan->w[a]);
        plan->row_live[pos] = (s_listed[e] && s_slot[e] >= 0) ? 1 : 0;
    }
    if (threadIdx.x == 0) {
        plan->n_active = s_nact;
        plan->n_routed_active = s_nact - S;
        plan->n_rows = n + S * T;
        plan->n_missing = s_nmiss;
        if (n_missing) *n_missing = s_nmiss;
    }
}

struct PlanKernelArgs {
    Plan *plan; int T, E, k, S;
    const char *pool; size_t slot_stride;
    const int32_t *slot_of_expert; const char *shared; size_t shared_stride; int flags;
    int32_t *ids_out; int32_t *missing; int32_t *n_missing;
};

// Router and plan in one launch (the verify call).  Workgroup (b, t) reduces the router rows of
// experts 16 b .. 16 b + 15 for token t, one row per wave, and stores the fp64 logits at agent
// scope; the workgroup that arrives last for its token (a counter per token) has all of the
// token's logits in reach, ranks them, forms the softmax weights and stores ids / weights /
// confidences; the workgroup that arrives last of all builds the plan.  All counters live in the
// workspace, are zero between launches and are put back to zero by the last arrival.  (One
// workgroup per token computing all E rows took 25 us for 128 experts: the instruction rate of
// the one compute unit a token ran on.)
constexpr int kRouteBlock = kRouteThreads / 64;          // experts per workgroup: one per wave

__global__ __launch_bounds__(kRouteThreads)
void route_plan_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wr,
                       const float *__restrict__ bias, int H, int renorm, const PlanKernelArgs a,
                       double *logits, uint32_t *token_arrivals, uint32_t *arrivals)
{
    __shared__ double s_logit[MOE_MAX_EXPERTS];
    __shared__ int32_t s_rank[MOE_MAX_EXPERTS];
    __shared__ int s_last;
    const int t = blockIdx.y, E = a.E, k = a.k;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nblk = gridDim.x;
    const int e = blockIdx.x * kRouteBlock + wave;
    if (e < E) {
        const uint16_t *xt = x + (size_t)t * H, *row = wr + (size_t)e * H;
        // eight independent partial sums instead of one chain of dependent fp64 additions; the
        // products are exact in fp32 (bf16 x bf16)
        double part[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int c = lane; c < H / 8; c += 64) {
            uint4 xv = *reinterpret_cast<const uint4 *>(xt + c * 8);
            uint4 wv = *reinterpret_cast<const uint4 *>(row + c * 8);
            const uint32_t xs[4] = {xv.x, xv.y, xv.z, xv.w};
            const uint32_t ws[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                part[2 * i] += (double)(__uint_as_float(xs[i] << 16) * __uint_as_float(ws[i] << 16));
                part[2 * i + 1] += (double)(__uint_as_float(xs[i] & 0xffff0000u) * __uint_as_float(ws[i] & 0xffff0000u));
            }
        }
        double acc = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
        acc = wave::sum(acc);
        if (lane == 0) {
            acc += bias ? (double)bias[e] : 0.0;
            if (nblk > 1) __hip_atomic_store(&logits[(size_t)t * E + e], acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else { s_logit[e] = acc; s_rank[e] = 0; }
        }
    }
    if (nblk > 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // this thread's stores have been performed
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t n = __hip_atomic_fetch_add(&token_arrivals[t], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = n == (uint32_t)nblk - 1;
            if (s_last) __hip_atomic_store(&token_arrivals[t], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!s_last) return;
        for (int i = threadIdx.x; i < E; i += kRouteThreads) {
            s_logit[i] = __hip_atomic_load(&logits[(size_t)t * E + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_rank[i] = 0;
        }
    }
    __syncthreads();
    // Rank of every logit under (larger first, lower index first among equals), counted by all
    // sixteen waves, each over its share of the experts; the order is strict, so the ranks are a
    // permutation and rank < k is the selection.
    wave::count_ranks(s_logit, s_rank, E, lane, wave, kRouteThreads / 64);
    __syncthreads();
    if (wave == 0) {
        double mine[4], pe[4];
        int rank[4];
        double mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ei = lane + 64 * i;
            const bool have = 64 * i < E && ei < E;
            mine[i] = have ? s_logit[ei] : -INFINITY;
            rank[i] = have ? s_rank[ei] : MOE_MAX_EXPERTS;
            mx = fmax(mx, mine[i]);
        }
        mx = wave::max(mx);
        double den = 0.0, sel = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pe[i] = rank[i] < MOE_MAX_EXPERTS ? exp(mine[i] - mx) : 0.0;
            den += pe[i];
        }
        den = wave::sum(den);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pe[i] = pe[i] / den;
            sel += rank[i] < k ? pe[i] : 0.0;
        }
        sel = wave::sum(sel);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (rank[i] < k) {
                const size_t o = (size_t)t * k + rank[i];
                put(&a.plan->ids[o], (int32_t)(lane + 64 * i));
                put(&a.plan->w[o], renorm ? (float)(pe[i] / sel) : (float)pe[i]);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // this thread's stores have been performed
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t n = __hip_atomic_fetch_add(arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = n == gridDim.y - 1;
        if (s_last) __hip_atomic_store(arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!s_last) return;
    plan_body(a.plan, a.T, a.E, a.k, a.S, a.pool, a.slot_stride, a.slot_of_expert,
              a.shared, a.shared_stride, a.flags, a.ids_out, a.missing, a.n_missing);
}

// Router of a long run of tokens, first launch: partial logits [part][T][E] in fp64 over a share of H.  A
// workgroup takes 16 tokens, 16 experts and one of gridDim.z shares of the k-steps of 32 inputs, its four
// waves a quarter of that each, on the fp64 matrix cores (16x16x4): a lane loads 8 inputs of one token and of
// one expert row and feeds eight products.  Bound: those matrix instructions (64 cycles each) and the round
// trip in front of them; the shares are there to spread few tokens over the chip.  (One workgroup per token,
// re-reading all router rows for each, took 24.5 us for 333 tokens x 64 experts x 2048 inputs and 92 us for
// 4096 x 8 x 4096; now 12 and 26 us with the second launch.)
typedef __attribute__((ext_vector_type(4))) double f64x4;
constexpr int kLogitWaves = 4, kMaxParts = 8;

__global__ __launch_bounds__(kLogitWaves * 64)
void prefill_logits_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wr, int T, int H, int E,
                           double *__restrict__ parts, int32_t *__restrict__ count)
{
    __shared__ double s_part[kLogitWaves][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, c = lane >> 4;
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)           // the expert counts of the second launch
        for (int e = tid; e < E; e += kLogitWaves * 64) count[e] = 0;
    const int t = blockIdx.x * 16 + r, e = blockIdx.y * 16 + r;
    const uint16_t *xt = x + (size_t)(t < T ? t : T - 1) * H + c * 8;
    const uint16_t *row = wr + (size_t)(e < E ? e : E - 1) * H + c * 8;
    const int nk = H / 32, shares = gridDim.z * kLogitWaves, share = blockIdx.z * kLogitWaves + wave;
    const int k0 = (int)((long)nk * share / shares), k1 = (int)((long)nk * (share + 1) / shares);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    constexpr int kAhead = 4;                    // k-steps in flight; past the end the last one is loaded again
    uint4 xv[kAhead], wv[kAhead];
    auto load = [&](int slot, int k) {
        const int kk = k < nk ? k : nk - 1;
        xv[slot] = *reinterpret_cast<const uint4 *>(xt + kk * 32);
        wv[slot] = *reinterpret_cast<const uint4 *>(row + kk * 32);
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) load(i, k0 + i);
    for (int k = k0; k < k1; k += kAhead) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const uint32_t xs[4] = {xv[i].x, xv[i].y, xv[i].z, xv[i].w}, ws[4] = {wv[i].x, wv[i].y, wv[i].z, wv[i].w};
            if (k + i < k1) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)__uint_as_float(xs[j] << 16), (double)__uint_as_float(ws[j] << 16), acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)__uint_as_float(xs[j] & 0xffff0000u), (double)__uint_as_float(ws[j] & 0xffff0000u), acc, 0, 0, 0);
                }
            }
            load(i, k + i + kAhead);
        }
    }
    // fp64 results: lane (r, c) holds column r (expert) of rows (tokens) c, c + 4, c + 8, c + 12
#pragma unroll
    for (int i = 0; i < 4; ++i) s_part[wave][(4 * i + c) * 16 + r] = acc[i];
    __syncthreads();
    const int to = blockIdx.x * 16 + (tid >> 4), eo = blockIdx.y * 16 + (tid & 15);
    if (to < T && eo < E)
        parts[((size_t)blockIdx.z * T + to) * E + eo] = (s_part[0][tid] + s_part[1][tid]) + (s_part[2][tid] + s_part[3][tid]);
}

// Second launch: one wave per token adds the shares, selects the top-k, and forms the softmax; the workgroup
// then gives every assignment a place in its expert's list (list[expert T + place]; the order inside an expert is
// arbitrary: no result depends on it), with one addition to the expert's count for all its tokens.
template <int NR>
__device__ inline void prefill_topk(const double *__restrict__ parts, int nparts, const float *__restrict__ bias, int T, int E,
                                    int k, int renorm, int t, int lane, int32_t *ids, float *w, float *conf, int &id)
{
    double l[NR], v[NR][kMaxParts];
    int rank[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int e = lane + 64 * i < E ? lane + 64 * i : E - 1;
        l[i] = bias ? (double)bias[e] : 0.0;
        v[i][0] = parts[(size_t)t * E + e];
        if (nparts > 1) {                        // (all loads before the first sum; past the end the last share again)
#pragma unroll
            for (int p = 1; p < kMaxParts; ++p) v[i][p] = parts[((size_t)(p < nparts ? p : nparts - 1) * T + t) * E + e];
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        double sum = v[i][0];
#pragma unroll
        for (int p = 1; p < kMaxParts; ++p) sum += p < nparts ? v[i][p] : 0.0;
        l[i] += sum;
    }
    id = wave::select_topk(l, E, k, lane, rank);
    double mx = -INFINITY, den = 0.0, sel = 0.0, pe[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) mx = lane + 64 * i < E ? fmax(mx, l[i]) : mx;
    mx = wave::max(mx);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        pe[i] = lane + 64 * i < E ? exp(l[i] - mx) : 0.0;
        den += pe[i];
    }
    den = wave::sum(den);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        pe[i] = pe[i] / den;
        sel += rank[i] < k ? pe[i] : 0.0;
    }
    sel = wave::sum(sel);
    if (lane < k) ids[(size_t)t * k + lane] = id;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (rank[i] < k) {
            const size_t o = (size_t)t * k + rank[i];
            if (conf) conf[o] = (float)pe[i];
            w[o] = renorm ? (float)(pe[i] / sel) : (float)pe[i];
        }
    }
}

constexpr int kTopkTokens = 16;

__global__ __launch_bounds__(kTopkTokens * 64)
void prefill_topk_kernel(const double *__restrict__ parts, int nparts, const float *__restrict__ bias, int T, int E, int k,
                         int renorm, int32_t *__restrict__ ids, float *__restrict__ w, float *__restrict__ conf,
                         int32_t *__restrict__ count, int32_t *__restrict__ list)
{
    __shared__ int32_t s_count[MOE_MAX_EXPERTS], s_base[MOE_MAX_EXPERTS];
    const int tid = threadIdx.x, lane = tid & 63, t = blockIdx.x * kTopkTokens + (tid >> 6);
    for (int e = tid; e < E; e += kTopkTokens * 64) s_count[e] = 0;
    __syncthreads();
    int id = 0, place = 0;
    const bool mine = t < T && lane < k;
    if (t < T) {
        if (E <= 64) prefill_topk<1>(parts, nparts, bias, T, E, k, renorm, t, lane, ids, w, conf, id);
        else if (E <= 128) prefill_topk<2>(parts, nparts, bias, T, E, k, renorm, t, lane, ids, w, conf, id);
        else prefill_topk<4>(parts, nparts, bias, T, E, k, renorm, t, lane, ids, w, conf, id);
        if (mine) place = atomicAdd(&s_count[id], 1);
    }
    __syncthreads();
    for (int e = tid; e < E; e += kTopkTokens * 64) s_base[e] = s_count[e] > 0 ? atomicAdd(&count[e], s_count[e]) : 0;
    __syncthreads();
    if (mine) list[(size_t)id * T + s_base[id] + place] = t * k + lane;
}

// Union of expert ids: bitmask in shared memory, then ordered compaction by one wave.
__global__ __launch_bounds__(256)
void union_kernel(const int32_t *__restrict__ ids, int n_ids, int E,
                  const int32_t *__restrict__ slot, uint64_t *mask, int32_t *list,
                  int32_t *n_list, int32_t *missing, int32_t *n_missing)
{
    __shared__ unsigned int s_bits[MOE_MAX_EXPERTS / 32];
    if (threadIdx.x < MOE_MAX_EXPERTS / 32) s_bits[threadIdx.x] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n_ids; i += blockDim.x) {
        int e = ids[i];
        if (e >= 0 && e < E) atomicOr(&s_bits[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int words = (E + 63) / 64;
    if ((int)threadIdx.x < words)
        mask[threadIdx.x] = (uint64_t)s_bits[2 * threadIdx.x] | ((uint64_t)s_bits[2 * threadIdx.x + 1] << 32);
    int nl = 0, nm = 0;
    for (int base = 0; base < E; base += 64) {
        int e = base + threadIdx.x;
        bool in = e < E && ((s_bits[e >> 5] >> (e & 31)) & 1u);
        bool miss = in && slot && slot[e] < 0;
        unsigned long long bi = __ballot(in), bm = __ballot(miss);
        unsigned long long below = (1ull << threadIdx.x) - 1ull;
        if (in) list[nl + __popcll(bi & below)] = e;
        if (miss) missing[nm + __popcll(bm & below)] = e;
        nl += __popcll(bi);
        nm += __popcll(bm);
    }
    if (threadIdx.x == 0) { *n_list = nl; *n_missing = nm; }
}

}  // namespace

void launch_route(const Shape &s, const void *x, const void *wr, const float *bias,
                  int32_t *ids, float *w, float *conf, hipStream_t st)
{
    launch(route_kernel, dim3(s.T), dim3(kRouteThreads), 0, st,
                       (const uint16_t *)x, (const uint16_t *)wr, bias, s.H, s.E, s.k, s.renorm,
                       ids, w, conf);
}

// shares of H: enough workgroups to fill the chip twice, at least four k-steps per wave
constexpr int kLogitBlocks = 512;
static int most_parts(const Shape &s)
{
    const int most = s.H / 32 / (4 * kLogitWaves);
    return most < 1 ? 1 : (most < kMaxParts ? most : kMaxParts);
}
int prefill_logit_parts(const Shape &s)
{
    const int blocks = ((s.T + 15) / 16) * ((s.E + 15) / 16);
    const int want = kLogitBlocks / blocks, most = most_parts(s);
    return want < 1 ? 1 : (want < most ? want : most);
}

// The largest parts x T of any call with up to s.T tokens: the shares get fewer as the tokens get more, and a
// workspace made for many tokens has to hold a call with fewer.  With two or more shares parts x ceil(T / 16) x
// ceil(E / 16) is at most kLogitBlocks.
size_t prefill_logit_rows(const Shape &s)
{
    const size_t all = (size_t)s.T * most_parts(s), spread = (size_t)kLogitBlocks * 16 / ((s.E + 15) / 16);
    const size_t split = all < spread ? all : spread;
    return split > (size_t)s.T ? split : (size_t)s.T;
}

void launch_prefill_logits(const Shape &s, const void *x, const void *wr, double *parts, int32_t *count, hipStream_t st)
{
    launch(prefill_logits_kernel, dim3((s.T + 15) / 16, (s.E + 15) / 16, prefill_logit_parts(s)), dim3(kLogitWaves * 64), 0, st,
           (const uint16_t *)x, (const uint16_t *)wr, s.T, s.H, s.E, parts, count);
}

void launch_prefill_topk(const Shape &s, const double *parts, const float *bias, int32_t *ids, float *w, float *conf,
                         int32_t *count, int32_t *list, hipStream_t st)
{
    launch(prefill_topk_kernel, dim3((s.T + kTopkTokens - 1) / kTopkTokens), dim3(kTopkTokens * 64), 0, st, parts, prefill_logit_parts(s),
           bias, s.T, s.E, s.k, s.renorm, ids, w, conf, count, list);
}

void launch_perm(const Shape &s, const int32_t *ids, int32_t *count, int32_t *off,
                 int32_t *perm, hipStream_t st)
{
    launch(perm_kernel, dim3(1), dim3(256), 0, st, ids, s.T * s.k, s.E, count, off, perm);
}

static PlanKernelArgs plan_kernel_args(const Shape &s, const PlanArgs &a)
{
    PlanKernelArgs k;
    k.plan = a.plan; k.T = s.T; k.E = s.E; k.k = s.k; k.S = s.S;
    k.pool = (const char *)a.pool; k.slot_stride = a.slot_stride;
    k.slot_of_expert = a.slot_of_expert; k.shared = (const char *)a.shared; k.shared_stride = a.shared_stride;
    k.flags = a.flags; k.ids_out = a.ids_out; k.missing = a.missing; k.n_missing = a.n_missing;
    return k;
}

void launch_route_plan(const Shape &s, const void *x, const void *wr, const float *bias, const PlanArgs &a,
                       double *logits, uint32_t *token_arrivals, uint32_t *arrivals, hipStream_t st)
{
    const dim3 grid((s.E + kRouteBlock - 1) / kRouteBlock, s.T);
    launch(route_plan_kernel, grid, dim3(kRouteThreads), 0, st, (const uint16_t *)x, (const uint16_t *)wr,
           bias, s.H, s.renorm, plan_kernel_args(s, a), logits, token_arrivals, arrivals);
}

void launch_union(const int32_t *ids, int n_ids, int E, const int32_t *slot,
                  uint64_t *mask, int32_t *list, int32_t *n_list,
                  int32_t *missing, int32_t *n_missing, hipStream_t st)
{
    launch(union_kernel, dim3(1), dim3(256), 0, st, ids, n_ids, E, slot, mask, list,
                       n_list, missing, n_missing);
}

}  // namespace moespeq
