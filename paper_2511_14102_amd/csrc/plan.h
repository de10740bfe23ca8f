// Internal: the per-call execution plan that the route/plan kernels leave in the workspace
// and that the expert kernels read, plus the host-side launcher prototypes of each .hip file.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include "../../include/moespeq.h"
#include "draft_rules.h"

namespace moespeq {

// Every kernel of the library is launched through launch().  When a timing pair is pending on
// this host thread (set by the profiling mode of the C ABI) the launch carries it: the runtime
// then stamps `start` / `stop` with the begin and end of the kernel's own execution, which is the
// duration a kernel trace reports, without the gaps an event recorded before and after would add.
struct LaunchTiming { hipEvent_t start, stop; };
extern thread_local LaunchTiming g_launch_timing;

template <typename K, typename... A>
inline void launch(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, A... args)
{
    if (g_launch_timing.stop) {
        const LaunchTiming t = g_launch_timing;
        g_launch_timing = LaunchTiming{nullptr, nullptr};
        hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, st, t.start, t.stop, 0, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds, st, args...);
    }
}

constexpr int kMaxRows = MOE_MAX_ASSIGN + MOE_MAX_TOKENS * MOE_MAX_SHARED;   // routed + shared rows
constexpr int kMaxActive = MOE_MAX_ASSIGN + MOE_MAX_SHARED;                   // distinct experts per call

// A "row" is one (token, expert) pair the bf16 expert kernels work on: assignment a = t k + j is row a, token t of
// shared expert s is row T k + s T + t.  Column t of an expert's matrix products is token t (T <= 16 columns of
// the MFMA), so the tokens of one expert run together (section 3.4.4) without being moved next to each other.
constexpr uint8_t kNoRow = 255;
static_assert(kMaxRows < kNoRow && MOE_MAX_TOKENS <= 16, "rows are bytes, tokens are MFMA columns");
struct Plan {
    int32_t n_active;                 // experts of the down launch: the shared ones, then the present routed ones, ascending
    int32_t n_live;                   // those of them that have tokens
    int32_t ids[MOE_MAX_ASSIGN];      // [T,k]
    uint64_t act_w0[kMaxActive];      // weights: bf16 blob
    alignas(16) uint8_t act_row[kMaxActive][16];     // row of token t, kNoRow: the token did not choose this expert
    float   row_w[kMaxRows];          // routing weight of a row (1 for shared)
    int32_t row_live[kMaxRows];       // 0: expert absent, the row's output must be skipped
};

// Workspace carve-up (byte offsets from a 256-byte aligned base).  [tickets, plan) must be
// zero between calls ("idle state"): moe_workspace_init establishes it, the draft kernel
// restores it.  Their sizes do not depend on T, so the idle region is the same for every call.
constexpr int kDraftSlotReplicas = 16;   // copies of the draft kernel's router-exchange slots that the workspace has room for (calls use exchange_copies_lg of them)
// inside the first block (the `tickets` block, kWsHeadBytes): the verify call's arrival counter and the
// draft calls' status word (0: fine, 1: a wait for the router result ran out of polls)
constexpr size_t kWsArrivalsOffset = 128, kWsStatusOffset = 192;
constexpr size_t kWsHeadBytes = 512;                     // size of that first block
constexpr uint32_t kDefaultSpinLimit = 1u << 22;

struct WsLayout {
    // tickets: one counter; slots: [MOE_MAX_DRAFT_TOKENS, E] x {fp64 logit, 64-bit tag} of the
    // draft kernel's router exchange; hb / hb_lo: bf16 intermediate and its bf16 remainder;
    // obuf: fp32 [rows,H] expert outputs
    size_t tickets, slots, slot_replica_bytes, plan, vlogits, hb, hb_lo, obuf, total;
};
WsLayout ws_layout(const moe_layer_desc &d, int max_tokens);

// route.hip
void launch_route(const Shape &s, const void *x, const void *wr, const float *bias,
                  int32_t *ids, float *w, float *conf, hipStream_t st);
void launch_perm(const Shape &s, const int32_t *ids, int32_t *count, int32_t *off,
                 int32_t *perm, hipStream_t st);
// a long run of tokens: partial logits [prefill_logit_parts][T][E] (and the expert counts cleared), then ids, weights,
// confidences, the experts' counts and their assignments list[expert T + place]
int prefill_logit_parts(const Shape &s);
size_t prefill_logit_rows(const Shape &s);       // rows of E logits the workspace holds for them: at least parts x T
void launch_prefill_logits(const Shape &s, const void *x, const void *wr, double *parts, int32_t *count, hipStream_t st);
void launch_prefill_topk(const Shape &s, const double *parts, const float *bias, int32_t *ids, float *w, float *conf,
                         int32_t *count, int32_t *list, hipStream_t st);
// the verify call's router and plan: fp64 logits [T, E], the plan but its row weights, the ids (plan->ids and ids_out) and
// the missing list; arrivals: a counter in the workspace, zero between launches
struct PlanArgs {
    Plan *plan;
    const void *pool; size_t slot_stride;
    const int32_t *slot_of_expert;
    const void *shared; size_t shared_stride;
    int flags;
    int32_t *ids_out;
    int32_t *missing; int32_t *n_missing;
};
void launch_verify_route(const Shape &s, const void *x, const void *wr, const float *bias, const PlanArgs &a,
                         double *logits, uint32_t *arrivals, hipStream_t st);
void launch_union(const int32_t *ids, int n_ids, int E, const int32_t *slot,
                  uint64_t *mask, int32_t *list, int32_t *n_list,
                  int32_t *missing, int32_t *n_missing, hipStream_t st);

// Work item of the draft call over a long run of tokens: up to prefill_chunk(s) assignments of one
// expert, list[first .. first + cnt), or (expert >= E: shared expert) tokens [first, first + cnt).
// Item i owns slots [64 i, 64 i + cnt); src: the item whose operand tiles of x it reads.
struct PrefillItem { int32_t expert, first, cnt, src; };
int prefill_chunk(const Shape &s);         // tokens of a full item: 64, or 32 for small calls
int prefill_max_items(const Shape &s);     // at most that many items
size_t prefill_item_room(const Shape &s);  // items the workspace has room for: no fewer than any call with fewer tokens needs

// draft_int4.hip (a call of 2 to 8 tokens) and draft_slice.hip (a call of one token)
struct DraftFusedArgs {
    const void *x, *wr; const float *bias;
    const void *q, *sz; size_t stride_q, stride_sz;
    int symmetric;                     // sz holds scale blobs (z = 8)
    int shared_inside;                 // the shared experts run in the call's launch
    OneTokenForm form;                 // of a call with one token (draft_form); more tokens: the persistent launch
    unsigned long long *slots; size_t replica_stride; uint32_t *tickets;
    uint32_t *status; uint32_t spin_limit;
    float *y; int32_t *ids_out; float *conf_out;
    Plan *plan; const void *shared; size_t shared_stride;
};
// slots: what draft_resident_slots returned for the call (more than one token: the persistent grid)
void launch_draft_fused(const Shape &s, const DraftFusedArgs &a, int n_cu, int slots, hipStream_t st);
// The form of the call's launch (a.form), once the rest of `a` is there
OneTokenForm draft_form(const Shape &s, const DraftFusedArgs &a, int n_cu);
// How many workgroups of the call's launch the device (n_cu compute units) holds at once; 0 if the ones that
// reduce the router rows would not all be running while the others wait for them
int draft_resident_slots(const Shape &s, const DraftFusedArgs &a, int n_cu);
// draft_slice.hip: the call with ONE token (router inside the launch) in a form of one or two (expert, slice) work items per
// workgroup
void launch_draft_one_token(const Shape &s, const DraftFusedArgs &a, hipStream_t st);
int draft_one_token_slots(const Shape &s, const DraftFusedArgs &a, OneTokenForm form, int n_cu);   // workgroups of it the device holds at once
void launch_zero(void *p, size_t bytes, hipStream_t st);
void launch_stream_read(const void *src, size_t bytes, int workgroups, void *sink, hipStream_t st);

// draft_prefill.hip: a routed run of tokens.  Byte sizes of the buffers a call with at most
// `items` work items needs, then the launches in order.
struct PrefillBuffers { size_t xt, x_sums, h, h_sums, h_scales, zeros, obuf; };
PrefillBuffers prefill_buffers(const moe_layer_desc &d, size_t items);
struct PrefillCall {
    const void *x;                     // [T,H] bf16
    const void *q, *sz; size_t stride_q, stride_sz; int symmetric;
    PrefillItem *items; int32_t *n_items;                          // written by the plan or the stage launch
    const int32_t *count, *list; int32_t *slot_of;
    const float *w_all;                // routing weight of every assignment [T k]
    void *xt, *x_sums, *h, *h_sums, *h_scales, *zeros; float *obuf;
    float *y;                          // [T,H] fp32, written (not accumulated)
    const void *shared; size_t shared_stride;                          // bf16 blobs of the shared experts
};
bool prefill_small(const Shape &s);        // the small form of the routing: launch_route, then
void launch_prefill_plan(const Shape &s, const int32_t *ids, const PrefillCall &p, hipStream_t st);
void launch_prefill_stage(const Shape &s, const PrefillCall &p, int max_items, hipStream_t st);
void launch_prefill_gateup(const Shape &s, const PrefillCall &p, int max_items, hipStream_t st);
void launch_prefill_down(const Shape &s, const PrefillCall &p, int max_items, hipStream_t st);
void launch_prefill_combine(const Shape &s, const PrefillCall &p, hipStream_t st);

// expert_bf16.hip
// The verify call's launches on the plan.  Gate/up also writes the rows' routing weights and clears the arrival counters of
// the next one; down: the products into obuf ([rows][H] fp32), and the last workgroup of every 32 output columns to arrive
// (counted in the tags of the exchange slots, zero after) writes y[t] (bf16) = (accumulate ? y[t] : 0) + the token's live rows
struct VerifyCall {
    Plan *plan;
    const void *x; const double *logits;
    void *hb; float *obuf;
    unsigned long long *slots; size_t slot_bytes;
    int accumulate; void *y;
};
void launch_verify_gateup(const Shape &s, const VerifyCall &v, hipStream_t st);
void launch_verify_down(const Shape &s, const VerifyCall &v, hipStream_t st);
// The draft call's shared experts on the plan of its launch: the intermediate is kept as a bf16 hi + lo pair, and each
// row's outputs are added to y[token] (fp32, [T,H]) with atomics
void launch_shared_gateup(const Shape &s, const Plan *plan, const void *x, void *hb, void *hb_lo, hipStream_t st);
void launch_shared_down_add(const Shape &s, const Plan *plan, const void *hb, const void *hb_lo, float *y, hipStream_t st);

}  // namespace moespeq
