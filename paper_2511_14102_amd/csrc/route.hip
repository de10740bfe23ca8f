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
#include "stream.h"
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

template <typename V>
__device__ inline void put(V *p, V v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename V>
__device__ inline V get(const V *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Router and plan of the verify call.  One workgroup per expert row and up to eight tokens: its eight waves are shared out
// over the tokens, the waves of a token splitting H, and a wave keeps its loads of a batch in flight.  The workgroup
// that arrives last (a counter in the workspace, put back to zero) has all logits in reach: one wave per token selects,
// then the present experts are listed in ascending order behind the shared ones.  The softmax is not on this path: the
// gate/up launch computes the rows' weights on the side.  Ids and logits travel at agent scope.
// Bound: the launch and a chain of four round trips to memory (rows, stores, counter, logits).
// (A counter per token and another over all, the softmax and a permutation of the rows in the chain: 12.6 us for 8 tokens
// x 128 experts x 2048 inputs, now 9.0; 5 x 16 x 4096: 10.6 / 6.7.  Logits alone, each workgroup of the next launch
// finding its own expert's tokens in them: 4.8 us here, but 6 us more there, for the workgroups of experts nobody chose.)
constexpr int kVerifyWaves = 8;

struct VerifyRouteArgs {
    Plan *plan; int T, H, E, k, S;
    const char *pool; size_t slot_stride;
    const int32_t *slot_of_expert; const char *shared; size_t shared_stride; int only_listed;
    int32_t *ids_out; int32_t *missing; int32_t *n_missing;
    double *logits; uint32_t *arrivals;
};

template <int NR>                            // NR: 64 NR >= E
__device__ inline int select_of_token(const VerifyRouteArgs &a, int t, int lane)
{
    double l[NR];
    int rank[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) l[i] = get(&a.logits[(size_t)t * a.E + (lane + 64 * i < a.E ? lane + 64 * i : a.E - 1)]);
    return wave::select_topk(l, a.E, a.k, lane, rank);
}

__global__ __launch_bounds__(kVerifyWaves * 64)
void verify_route_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wr, const float *__restrict__ bias,
                         const VerifyRouteArgs a)
{
    __shared__ double s_part[kVerifyWaves];
    __shared__ __attribute__((aligned(16))) uint8_t s_row[MOE_MAX_EXPERTS][16];      // row of (expert, token)
    __shared__ uint32_t s_chosen[MOE_MAX_EXPERTS / 32], s_listed[MOE_MAX_EXPERTS / 32];
    __shared__ int s_last;
    const int T = a.T, H = a.H, E = a.E, k = a.k, S = a.S;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int e = blockIdx.x, t0 = blockIdx.y * kVerifyWaves, n = T - t0 < kVerifyWaves ? T - t0 : kVerifyWaves;
    const int lt = n <= 1 ? 0 : (n <= 2 ? 1 : (n <= 4 ? 2 : 3));
    const int t = wave & ((1 << lt) - 1), part = wave >> lt, step = (kVerifyWaves >> lt) * 64;
    const uint16_t *xt = x + (size_t)(t0 + (t < n ? t : n - 1)) * H, *row = wr + (size_t)e * H;
    const int chunks = H / 8;
    const float b = bias ? bias[e] : 0.f;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    constexpr int kB = 4;
    for (int c0 = part * 64 + lane; c0 - lane < chunks; c0 += kB * step) {
        uint4 xv[kB], wv[kB];
#pragma unroll
        for (int j = 0; j < kB; ++j) {
            const int c = c0 + j * step, cc = c < chunks ? c : chunks - 1;
            xv[j] = *reinterpret_cast<const uint4 *>(xt + cc * 8);
            wv[j] = *reinterpret_cast<const uint4 *>(row + cc * 8);
        }
#pragma unroll
        for (int j = 0; j < kB; ++j) {
            const bool in = c0 + j * step < chunks;              // (a position past the end counts as zeros)
            const uint32_t xs[4] = {xv[j].x, xv[j].y, xv[j].z, xv[j].w}, ws[4] = {wv[j].x, wv[j].y, wv[j].z, wv[j].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t xi = in ? xs[i] : 0u, wi = in ? ws[i] : 0u;
                acc[i] += (double)(__uint_as_float(xi << 16) * __uint_as_float(wi << 16));      // bf16 x bf16 is exact in fp32
                acc[i] += (double)(__uint_as_float(xi & 0xffff0000u) * __uint_as_float(wi & 0xffff0000u));
            }
        }
    }
    const double sum = wave::sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
    if (lane == 0) s_part[wave] = sum;
    __syncthreads();
    if (wave == 0) {
        if (lane < n) {
            double l = 0.0;
#pragma unroll
            for (int w = 0; w < kVerifyWaves; ++w) l += (w & ((1 << lt) - 1)) == lane ? s_part[w] : 0.0;
            put(&a.logits[(size_t)(t0 + lane) * E + e], l + (double)b);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // the stores have been performed
        if (lane == 0) {
            const uint32_t before = __hip_atomic_fetch_add(a.arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = before == gridDim.x * gridDim.y - 1;
        }
    }
    for (int i = tid; i < E * 4; i += kVerifyWaves * 64) reinterpret_cast<uint32_t *>(s_row)[i] = kNoRow * 0x01010101u;
    if (tid < MOE_MAX_EXPERTS / 32) { s_chosen[tid] = 0u; s_listed[tid] = a.only_listed ? 0u : ~0u; }
    __syncthreads();
    if (!s_last) return;
    if (tid == 0) put(a.arrivals, 0u);
    for (int tt = wave; tt < T; tt += kVerifyWaves) {
        const int id = E <= 64 ? select_of_token<1>(a, tt, lane) : E <= 128 ? select_of_token<2>(a, tt, lane) : select_of_token<4>(a, tt, lane);
        if (lane < k) {
            s_row[id][tt] = (uint8_t)(tt * k + lane);
            atomicOr(&s_chosen[id >> 5], 1u << (id & 31));
            a.plan->ids[tt * k + lane] = id;
            if (a.ids_out) a.ids_out[tt * k + lane] = id;
        }
    }
    if (a.only_listed) {
        int nin = *a.n_missing;
        nin = nin < 0 ? 0 : (nin > E ? E : nin);
        for (int i = tid; i < nin; i += kVerifyWaves * 64) {
            const int m = a.missing[i];
            if (m >= 0 && m < E) atomicOr(&s_listed[m >> 5], 1u << (m & 31));
        }
    }
    // shared experts: active indices [0, S), rows T k + s T + t; left out by a call for listed experts
    Plan *plan = a.plan;
    if (tid < S * 16) plan->act_row[tid / 16][tid % 16] = tid % 16 < T && !a.only_listed ? (uint8_t)(T * k + tid / 16 * T + tid % 16) : kNoRow;
    if (tid < S) plan->act_w0[tid] = (uint64_t)(a.shared + (size_t)tid * a.shared_stride);
    if (tid < S * T) plan->row_live[T * k + tid] = a.only_listed ? 0 : 1;
    __syncthreads();
    // routed experts: ordered compaction, 64 experts per step
    if (wave != 0) return;
    int nact = S, nmiss = 0;
    for (int base = 0; base < E; base += 64) {
        const int o = base + lane;
        const bool used = o < E && ((s_chosen[o >> 5] >> (o & 31)) & 1u);
        const bool listed = used && ((s_listed[o >> 5] >> (o & 31)) & 1u);
        const int slot = used ? a.slot_of_expert[o] : -1;
        const unsigned long long bp = __ballot(listed && slot >= 0), ba = __ballot(listed && slot < 0);
        const unsigned long long below = (1ull << lane) - 1ull;
        if (used) {
            const u32x4 rows = *reinterpret_cast<const u32x4 *>(s_row[o]);
            if (listed && slot >= 0) {
                const int u = nact + __popcll(bp & below);
                plan->act_w0[u] = (uint64_t)(a.pool + (size_t)slot * a.slot_stride);
                *reinterpret_cast<u32x4 *>(plan->act_row[u]) = rows;
            }
            for (int tt = 0; tt < T; ++tt) {
                const uint32_t row = s_row[o][tt];
                if (row != kNoRow) plan->row_live[row] = listed && slot >= 0 ? 1 : 0;
            }
        }
        if (listed && slot < 0) a.missing[nmiss + __popcll(ba & below)] = o;
        nact += __popcll(bp);
        nmiss += __popcll(ba);
    }
    if (lane == 0) {
        plan->n_active = nact;
        plan->n_live = a.only_listed ? nact - S : nact;
        *a.n_missing = nmiss;
    }
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

void launch_verify_route(const Shape &s, const void *x, const void *wr, const float *bias, const PlanArgs &p,
                         double *logits, uint32_t *arrivals, hipStream_t st)
{
    VerifyRouteArgs a;
    a.plan = p.plan; a.T = s.T; a.H = s.H; a.E = s.E; a.k = s.k; a.S = s.S;
    a.pool = (const char *)p.pool; a.slot_stride = p.slot_stride;
    a.slot_of_expert = p.slot_of_expert; a.shared = (const char *)p.shared; a.shared_stride = p.shared_stride;
    a.only_listed = (p.flags & MOE_VERIFY_ONLY_LISTED) ? 1 : 0;
    a.ids_out = p.ids_out; a.missing = p.missing; a.n_missing = p.n_missing;
    a.logits = logits; a.arrivals = arrivals;
    launch(verify_route_kernel, dim3(s.E, (s.T + kVerifyWaves - 1) / kVerifyWaves), dim3(kVerifyWaves * 64), 0, st,
           (const uint16_t *)x, (const uint16_t *)wr, bias, a);
}

void launch_union(const int32_t *ids, int n_ids, int E, const int32_t *slot,
                  uint64_t *mask, int32_t *list, int32_t *n_list,
                  int32_t *missing, int32_t *n_missing, hipStream_t st)
{
    launch(union_kernel, dim3(1), dim3(256), 0, st, ids, n_ids, E, slot, mask, list,
                       n_list, missing, n_missing);
}

}  // namespace moespeq
