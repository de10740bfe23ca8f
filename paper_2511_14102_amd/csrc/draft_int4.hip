// Draft-pass kernel for calls of two to eight tokens, and of one token with many work items: router, top-k and the SwiGLU FFN of the
// selected experts on group-wise int4 weights, dequantisation fused into the matrix products, ONE
// launch per call (gfx950).  (Other calls with one token run the kernel of draft_slice.hip.)
//
// Paper section 3.4.3: the draft pass has to avoid the launch and utilisation losses of
// per-expert small GEMMs (one monolithic expert-fused kernel); section 4.1.3: 4-bit weights in
// groups along the input dimension; section 3.3.1: (expert id, confidence) per token and layer
// is recorded for the lookahead buffer.  The arithmetic is described in draft_common.h.
//
// Work decomposition.  A work item is (expert, slice of 32 intermediate rows): the 32 gate and
// 32 up pre-activations (K = H split over the waves by groups), h = silu(gate) * up, and at
// once the product of h with the 32 matching columns of the down projection for all H outputs,
// added into y with fp32 atomics.  Nothing but the router result crosses workgroups.
//
// The launch is persistent: the grid never exceeds what the device holds at once, and the items
// are dealt evenly, a run of consecutive items per workgroup.  A wave's weight tiles of all its
// items form ONE stream (gate/up tiles of item 0, its down tiles, gate/up tiles of item 1, ...)
// that is read through a rolling window of tiles in flight, so the loads of an item's successor
// are under way while the item's own sums are reduced, h is formed and its down tiles are
// multiplied.  With several tokens a call has many items (every distinct expert of the call,
// I / 32 slices each) and this wins clearly over one workgroup per item.
//
// Bound: the weight stream at one workgroup per compute unit (phi shape, 4 tokens: 202 MB in 45 to 47 us, of which
// the start takes about 5 us), and with few tokens per expert also the vector work per tile.  What the stream
// needs is that its loads stay in flight: a window slot is unpacked and refilled at once, addresses are
// buffer offsets without clamps, and nothing under a branch counts on the vector memory counter (an empty slot's
// atomics go out of range instead).  us per call before these: phi 4 tokens 57.5, mixtral 3 tokens, symmetric
// 87 (now 70 to 78), qwen3 8 tokens 60.6 (now 36 to 37).
//
// Cross-workgroup protocol (one bounded wait, no cache flushes):
//   1. router row e is reduced by workgroup e (mod router_workgroups), which first clears its share of y
//      with agent-scope stores, waits for their completion, and then publishes the 16-byte
//      slot {logit, tag = 1} of every token as one 16-byte store (in a few copies);
//   2. every workgroup polls the slots with single 16-byte agent-scope loads until all are
//      tagged, then selects the top-k itself (identical in all workgroups) and draws a ticket;
//   3. y contributions (of an item, or of a workgroup's items of one expert) are agent-scope atomics, which land after the clearing stores because
//      the clearing completed before the slots were published;
//   4. the workgroup holding the last ticket (everybody has finished polling by then) clears
//      the tags and the ticket counters at its end, so the workspace is back in its idle state
//      when the kernel ends.  This also holds when the same launch is replayed from a HIP graph.
// The wait of step 2 needs the producing workgroups (the first min(E, grid) ones) to be running
// while the others poll: the grid never exceeds the number of compute units, and a workgroup
// fits a compute unit by itself, so on an otherwise idle device all are resident.  If the wait
// runs out (spin limit), the workgroup skips its items and workgroup 0 reports ids = -1.
#include "draft_common.h"

namespace moespeq {

namespace {

// MT: token capacity of the launch (2, 4 or 8); UPG: 32-code units per
// group (g / 32); SYM: symmetric format (scale blobs, z = 8); kWin:
// tiles a wave keeps in flight; SUMS: y is summed in LDS over a workgroup's items of one expert, sum_slots(MT) token slots of it.
template <int MT, int UPG, bool SYM, int kWin, bool SUMS>
__device__ __forceinline__ void draft_stream(const uint16_t *__restrict__ xin, const FusedArgs &a)
{
    __shared__ double s_part[kWaves];
    __shared__ int32_t s_ids[MOE_MAX_ASSIGN];
    __shared__ float s_w[MOE_MAX_ASSIGN];
    __shared__ float s_conf[MOE_MAX_ASSIGN];
    __shared__ unsigned long long s_mask[MOE_MAX_EXPERTS / 64];
    // rows and sums of an item are kept twice (item parity): an item's successor is set up while waves
    // may still be reading the item's own
    __shared__ int32_t s_row_a[2][MT];          // assignment index of each row (token slot) of the item
    __shared__ int32_t s_cnt[2];
    __shared__ float s_hsum[2][MT];
    __shared__ int32_t s_flag, s_last;
    __shared__ int32_t s_list[MOE_MAX_EXPERTS];  // the call's distinct experts, ascending
    __shared__ float s_red[kWaves][MT][64];      // partial gate/up sums [wave][token slot][row]
    __shared__ __attribute__((aligned(16))) uint16_t s_hhi[MT][32], s_hlo[MT][32];
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];   // x copy, its group sums, routing scratch

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = a.T, H = a.H, E = a.E, I = a.I, k = a.k, g = a.g;
    const int n = T * k;
    const int G = H / g;
    const int xstride = H + 8;                   // bf16 elements per token in LDS (+16 B against bank conflicts)
    uint16_t *s_x = reinterpret_cast<uint16_t *>(s_dyn);
    float *s_xsum = reinterpret_cast<float *>(s_dyn + (size_t)MT * xstride * 2);   // [MT][G]
    // routing scratch behind the group sums, used with many experts: logits [MT][E] (fp64), ranks
    const size_t logit_off = ((size_t)MT * xstride * 2 + (size_t)MT * G * 4 + 7) & ~(size_t)7;
    double *s_logit = reinterpret_cast<double *>(s_dyn + logit_off);
    int32_t *s_rank = reinterpret_cast<int32_t *>(s_dyn + logit_off + (size_t)MT * E * 8);

    // ---- 1. router rows owned by this workgroup
    const int nprod = router_workgroups(E, 1, gridDim.x);
    if ((int)blockIdx.x < nprod) publish_router_rows<kWaves, 1>(xin, a, blockIdx.x, nprod, s_part);
    if (tid == 0) s_flag = 1;
    if (tid < MOE_MAX_EXPERTS / 64) s_mask[tid] = 0ull;
    if (tid < 2 * MT) s_hsum[tid / MT][tid % MT] = 0.f;

    // ---- 1b. (while the router result travels) x goes to LDS, and its sum per group: 4 UPG neighbouring threads hold a group.
    // (Summed from LDS, by threads that found their token and group with divisions, this was 2.4 us of the start of a call with 4 tokens
    // of the phi shape and 3.5 us with 8 of the qwen3 shape, where the routing's result is there after 3 us; before / now with the shares of
    // split_items, us per pass: phi 380 / 373, mixtral, 3 tokens 281 / 277, qwen3 300 / 294; H = 3072, E = 24, 5 tokens 426 / 399.)
    const int nx = T * (H / 8);                  // pieces of eight values
    // (whole quotients of a dividend below 2^21 by a reciprocal: (i + 1/2) / d is at least 1 / 2d away from a whole number, and the rounding of
    // reciprocal and product, 1.5 x 2^-23 of it, is less.  i < 2^16 here, as H <= 2^16 and T <= 8; items < 2^19, as T k <= 128 and I / 32 <= 2^12.)
    const float per_token = 8.f * __builtin_amdgcn_rcpf((float)H);
    auto keep = [&](int i, u32x4 v) {
        float s = ((bf16_lo(v.x) + bf16_hi(v.x)) + (bf16_lo(v.y) + bf16_hi(v.y))) +
                  ((bf16_lo(v.z) + bf16_hi(v.z)) + (bf16_lo(v.w) + bf16_hi(v.w)));
        s += wave::move<wave::kSwap1>(s);
        s += wave::move<wave::kSwap2>(s);
        if constexpr (UPG > 1) s += wave::move<wave::kHalfMirror>(s);
        if constexpr (UPG > 2) s += wave::move<wave::kMirror>(s);
        if (i < nx) {
            *reinterpret_cast<u32x4 *>(s_x + (i + (int)(((float)i + 0.5f) * per_token)) * 8) = v;      // (rows are 8 elements longer than H)
            if (i % (4 * UPG) == 0) s_xsum[i / (4 * UPG)] = s;
        }
    };
    constexpr int kBatch = MT < 4 ? MT : 4;
    for (int i0 = tid; i0 - tid < nx; i0 += kBatch * kThreads) {
        u32x4 v[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) v[j] = *reinterpret_cast<const u32x4 *>(xin + (size_t)(i0 + j * kThreads < nx ? i0 + j * kThreads : nx - 1) * 8);
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (i0 - tid + j * kThreads < nx) keep(i0 + j * kThreads, v[j]);
    }
    __syncthreads();

    const int nslice = I / 32;
    const float per_slice = __builtin_amdgcn_rcpf((float)nslice), per_workgroup = __builtin_amdgcn_rcpf((float)gridDim.x);     // (while the router result travels; exact as above)
    const int U = H / 32;
    const int r = lane & 15, c = lane >> 4;                  // MFMA lane coordinates
    const UnpackConsts uk = unpack_consts();
    const uint32_t lane_off = (uint32_t)lane * 16u;
    constexpr int kEpl = SYM ? 2 : 1;                        // groups (row tiles) per 256-byte block of entries
    const int nrt = H / 64;
    // ---- this wave's share of every item: gate/up tiles u0 .. u1 (K = H split over the waves by
    // groups; the symmetric format keeps two groups / row tiles in one block of entries: whole
    // pairs per wave), padded to whole windows, then its down row tiles r0 .. r1, padded likewise.
    const int g0 = ((wave * (G / kEpl)) / kWaves) * kEpl, g1 = (((wave + 1) * (G / kEpl)) / kWaves) * kEpl;
    const int u0 = g0 * UPG, u1 = g1 * UPG;
    const int nt = u1 - u0;
    const int ntp = (nt + kWin - 1) / kWin * kWin;
    const int r0 = ((wave * (nrt / kEpl)) / kWaves) * kEpl, r1 = (((wave + 1) * (nrt / kEpl)) / kWaves) * kEpl;
    const int ndw = r1 - r0;
    const int ndp = (ndw + kWin - 1) / kWin * kWin;
    const int Lw = ntp + ndp;                                // stream positions of this wave per item
    // One item: expert and slice, and the addresses of this wave's two runs of tiles.  codes:
    // [gate|up tiles (slice, ku)] then [down tiles (slice, rt)], 64 lanes x 16 B each; scale/zero:
    // [gate|up (slice, group)] then [down (group of I, rt)], one 256-byte block of entries per
    // group (row tile), or per pair of them (symmetric format).
    struct Item {
        const char *szb;
        const char *gu_run, *dn_run;     // this wave's first gate/up tile and first down tile of the slice
        int u, slice, expert;            // u: rank of the expert among the call's distinct experts
    };
    // where item idx sits (no routing needed) ...
    auto item_pos = [&](Item &it, int idx) {
        it.u = __builtin_amdgcn_readfirstlane((int)(((float)idx + 0.5f) * per_slice));
        it.slice = idx - it.u * nslice;
    };
    auto item_after = [&](Item &it, const Item &prev) {     // ... and its successor, without a division
        const bool wrap = prev.slice + 1 == nslice;
        it.u = wrap ? prev.u + 1 : prev.u;
        it.slice = wrap ? 0 : prev.slice + 1;
    };
    // ... and its addresses, once the experts are known
    auto item_addr = [&](Item &it, int expert) {
        it.expert = expert;
        const char *qb = a.q + (size_t)it.expert * a.stride_q;
        it.szb = a.sz + (size_t)it.expert * a.stride_sz;
        it.gu_run = qb + ((size_t)it.slice * U + u0) * 1024;
        it.dn_run = qb + ((size_t)nslice * U + (size_t)it.slice * nrt + r0) * 1024;
    };
    // One window of this wave's stream: kWin positions from q0 (a multiple of kWin, counted from the start of
    // item `cur`; positions from Lw on belong to `nxt`).  Parts are padded to whole windows, so a window
    // lies inside one part and is a run that ends with the part.  EVERY load of the stream is
    // unconditional: past the end of a part, and past the last item (`more` false), it returns zeros and
    // moves nothing (the compiler counts the loads in flight in program order; a load under a branch
    // makes it wait for more of them than it needs, and a second copy of a loop body without the loads
    // costs a full wait where the copies meet).
    auto window_run = [&](const Item &cur, const Item &nxt, bool more, int q0) {
        const bool wrap = q0 >= Lw;
        const int qq = wrap ? q0 - Lw : q0;
        const char *gu = wrap ? nxt.gu_run : cur.gu_run, *dn = wrap ? nxt.dn_run : cur.dn_run;
        const int j = qq - ntp;
        const char *base = qq < ntp ? gu + (size_t)qq * 1024 : dn + (size_t)j * 1024;
        const int room = qq < ntp ? nt - qq : ndw - j;
        return make_run(base, room > 0 && (!wrap || more) ? (uint32_t)room * 1024u : 0u);
    };

    // Scale / zero entries do not travel through registers: a wave copies the entries of its own
    // groups (row tiles) of an item straight into LDS (16-byte loads that write LDS, 1 KiB per
    // instruction, no destination registers and so nothing the compiler has to keep alive across
    // the item loop) BEFORE it requests any tile they belong to: the down entries as the item's gate/up
    // part begins, the successor's gate/up entries as the item's down part begins, when the wave has
    // used the ones in their place.  Vector memory operations complete in order, so once a tile has
    // arrived, so have its entries; an entry is read only behind the use of such a tile.  (A wave without
    // tiles in one of the parts requests the other part's tiles too early for this and waits.)
    const int ngl = (g1 - g0) / kEpl, ndl = (r1 - r0) / kEpl;          // 256-byte blocks of this wave
    const int gl_max = (G / kEpl + kWaves - 1) / kWaves, dl_max = (nrt / kEpl + kWaves - 1) / kWaves;
    const int eb_gu = (gl_max + 3) / 4 * 1024, eb_dn = (dl_max + 3) / 4 * 1024;
    const size_t ent_off = (logit_off + (size_t)MT * E * 12 + 15) & ~(size_t)15;
    unsigned char *s_ent = s_dyn + ent_off + (size_t)wave * (eb_gu + eb_dn);                  // [gate/up | down]
    // Sums of y over this workgroup's items of one expert: kAcc token slots of H outputs, each wave's own columns
    float *s_y = reinterpret_cast<float *>(s_dyn + ent_off + (size_t)kWaves * (eb_gu + eb_dn));
    const uint32_t s_ent_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)s_ent);   // LDS byte address
    auto request_blocks = [&](const char *src, int blocks, uint32_t dst) {
        for (int op = 0; op * 4 < blocks; ++op) {
            const int off = op * 1024 + (int)lane_off;
            const int lim = blocks * 256 - 16;
            load16_to_lds(src + (off < lim ? off : lim), dst + op * 1024);
        }
        if (ngl == 0 || ndl == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    auto request_gu_entries = [&](const Item &it) {
        request_blocks(it.szb + ((size_t)it.slice * (G / kEpl) + g0 / kEpl) * 256, ngl, s_ent_addr);
    };
    auto request_dn_entries = [&](const Item &it) {
        request_blocks(it.szb + ((size_t)nslice * (G / kEpl) + (size_t)((it.slice * 32) / g) * (nrt / kEpl) + r0 / kEpl) * 256,
                       ndl, s_ent_addr + eb_gu);
    };
    // entry of row block d, row r in block `unit` (counted from the wave's first) of part 0 gate/up, 1 down;
    // `odd`: the second group (row tile) of a pair in the symmetric format
    auto entry = [&](int part, int unit, int odd, int d) -> uint32_t {
        const unsigned char *p = s_ent + part * eb_gu + unit * 256 + r * 16;
        if constexpr (SYM) return *reinterpret_cast<const uint16_t *>(p + odd * 8 + d * 2);
        else return *reinterpret_cast<const uint32_t *>(p + d * 4);
    };
    auto scale_of = [](uint32_t e) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(e & 0xffff)); };
    auto zero_of = [](uint32_t e) { return SYM ? 136.f : (float)__builtin_bit_cast(_Float16, (uint16_t)(e >> 16)) + 128.f; };
    // Orders what follows behind the arrival of a tile: `b` is made from the tile's words, so the wait for the
    // tile's load precedes this point, and no memory access is moved across it.
    auto behind_tile = [](const bf16x8 &b) { asm volatile("" : : "v"(__builtin_bit_cast(u32x4, b)) : "memory"); };
    const uint32_t cm1 = 0u - (uint32_t)(c & 1), cm2 = 0u - (uint32_t)(c >> 1);
    auto mix = [](float a, float b, uint32_t m) { return __uint_as_float((__float_as_uint(b) & m) | (__float_as_uint(a) & ~m)); };
    auto pick4 = [&](float v0, float v1, float v2, float v3) { return mix(mix(v0, v1, cm1), mix(v2, v3, cm1), cm2); };   // v_c
    auto pick2 = [&](float v0, float v1) { return mix(v0, v1, cm2); };                                                // v_(c / 2)
    constexpr uint32_t kPastY = 0x80000000u;     // beyond any y, also with a tile's offset added
    const run_t y_run = make_run((const char *)a.y, (uint32_t)(T * H) * 4u);
    // rows (token slots) of an item: the assignments with its expert, ascending; one wave
    auto item_rows = [&](int expert, int par) {
        int cnt = 0;
        for (int base = 0; base < n; base += 64) {
            const int aidx = base + lane;
            const bool hit = aidx < n && s_ids[aidx] == expert;
            const unsigned long long b = __ballot(hit);
            if (hit) {
                const int pos = cnt + __popcll(b & ((1ull << lane) - 1ull));
                if (pos < MT) s_row_a[par][pos] = aidx;
            }
            cnt += __popcll(b);
        }
        if (lane == 0) s_cnt[par] = cnt < MT ? cnt : MT;
    };

    // Work split: the items (distinct experts ascending, I / 32 slices each) are dealt evenly, n / G
    // each, the last n % G workgroups one more (the first ones, which reduce the router rows, begin later: us per pass, the
    // first / the last ones, phi, 4 tokens 367.4 / 363.9, qwen3, 8 tokens 299.9 / 292.3; H = 384, E = 5, I = 3200, 2 tokens 223.0 / 214.0).
    int it_begin = 0, it_end = 0;
    Item cur, nxt;
    auto split_items = [&](int n_items) {
        const uint32_t it_q = (uint32_t)__builtin_amdgcn_readfirstlane((int)(((float)n_items + 0.5f) * per_workgroup)), it_r = (uint32_t)n_items - it_q * gridDim.x;
        const uint32_t fewer = gridDim.x - it_r;              // workgroups without one more
        it_begin = (int)(blockIdx.x * it_q + (blockIdx.x > fewer ? blockIdx.x - fewer : 0u));
        it_end = it_begin + (int)it_q + (blockIdx.x >= fewer ? 1 : 0);
        item_pos(cur, it_begin);
        if (it_begin + 1 < it_end) item_after(nxt, cur);
        else nxt = cur;
    };

    // ---- 2. wave t polls the slots of token t (bounded) and selects its top-k
    if (wave < T) {                              // T <= kWaves
        const bool got = poll_and_select(a, wave, s_logit + wave * E, s_rank + wave * E, s_ids + wave * k, s_mask);
        if (!got && lane == 0) {                 // gave up: the call fails, and says so in the workspace
            s_flag = 0;
            __hip_atomic_store(a.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    const bool ok = s_flag != 0;
    // the softmax of wave t's token, off the path to the first weight load
    auto softmax = [&]() {
        if (wave < T && ok) finish_softmax(a, s_logit + wave * E, s_rank + wave * E, s_conf + wave * k, s_w + wave * k);
    };
    // This workgroup will not look at the slots again: its last wave draws a ticket (the holder of the last one
    // puts the slots back to idle, at its own end).
    uint32_t ticket = 0xffffffffu, ticket2 = 0xffffffffu;
    if (tid == kThreads - 64) ticket = draw_ticket(a.tickets + blockIdx.x % kTicketGroups);
    auto second_ticket = [&]() {
        if (lane == 0 && ticket == ticket_members(blockIdx.x, gridDim.x) - 1) ticket2 = draw_ticket(a.tickets + kTicketGroups);
    };

    // ---- 3. this workgroup's items: the distinct experts ascending, I / 32 slices each.  Every wave lists the
    // experts for itself (the same values in the same places, so no barrier is needed).
    int n_experts_used = 0;
    for (int wd = 0; wd * 64 < E; ++wd) {
        const unsigned long long mk = s_mask[wd];
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)mk), hi = __builtin_amdgcn_readfirstlane((uint32_t)(mk >> 32));
        const int below = n_experts_used + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
        if (((lane < 32 ? lo : hi) >> (lane & 31)) & 1u) s_list[below] = wd * 64 + lane;
        n_experts_used += __popc(lo) + __popc(hi);
    }
    auto nth_expert = [&](int u) { return __builtin_amdgcn_readfirstlane(s_list[u]); };
    split_items(ok ? n_experts_used * nslice : 0);
    if (it_begin < it_end) {
        item_addr(cur, nth_expert(cur.u));
        if (it_begin + 1 < it_end) item_addr(nxt, nth_expert(nxt.u));
        else nxt = cur;
        // ---- 3a. the first entries and the first window of weight loads go out before anything
        // else of the item is set up: every microsecond of bookkeeping behind them is hidden by
        // their latency
        u32x4 win[kWin];
        if (Lw > 0) {
            request_gu_entries(cur);
            const run_t w0 = window_run(cur, nxt, it_begin + 1 < it_end, 0);
#pragma unroll
            for (int i = 0; i < kWin; ++i) win[i] = run_load16(w0, lane_off + (uint32_t)i * 1024u);
        }
        if (wave == kWaves - 1) item_rows(cur.expert, 0);
        softmax();
        constexpr int kAcc = sum_slots(MT);
        if constexpr (SUMS) {
#pragma unroll
            for (int sl = 0; sl < kAcc; ++sl)
                for (int rt = r0; rt < r1; ++rt) s_y[sl * H + rt * 64 + lane] = 0.f;
        }
        __syncthreads();

        for (int it = it_begin; it < it_end; ++it) {
            const int par = (it - it_begin) & 1;
            const bool last = it + 1 == it_end;
            const int cnt = __builtin_amdgcn_readfirstlane(s_cnt[par]);
            auto token_of = [&](int slot) { return s_row_a[par][slot < cnt ? slot : 0] / k; };   // (slots >= cnt repeat slot 0)
            if (Lw > 0) request_dn_entries(cur);
            {
                // A row m is token slot m % MT, so lane group c holds, for each of its slots, the sums of all four row
                // blocks, and finishes only some of them: with up to four slots block c of every slot, with eight
                // slots blocks 2 (c / 2), 2 (c / 2) + 1 of slots 4 (c % 2) ...  (Every lane group finishing all four blocks
                // of its own slots, most of them empty, was twice the vector work.)
                constexpr int NI = MT < 4 ? MT : 4;                  // slots per lane
                constexpr int NB = MT > 4 ? 2 : 1;                   // row blocks per lane
                const int slot0 = MT > 4 ? 4 * (c & 1) : 0, block0 = MT > 4 ? 2 * (c >> 1) : c;
                const uint16_t *xrow = s_x + token_of(r % MT) * xstride + c * 8;
                const float *xs_of[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i) xs_of[i] = s_xsum + token_of(slot0 + i) * G;
                float tot[NB][NI];
                f32x4 acc[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int bb = 0; bb < NB; ++bb)
#pragma unroll
                    for (int i = 0; i < NI; ++i) tot[bb][i] = 0.f;
                u32x4 xa = *reinterpret_cast<const u32x4 *>(xrow + (nt > 0 ? u0 : 0) * 32);
                // one window; kGuard: some of its tiles may lie past the wave's run (the padding of the last window)
                // and are skipped.  Full windows carry no per-tile tests.
                auto gu_window = [&](int base, auto guarded) {
                    constexpr bool kGuard = decltype(guarded)::value;
                    const run_t wr = window_run(cur, nxt, !last, base + kWin);
#pragma unroll
                    for (int i = 0; i < kWin; ++i) {
                        const int ku = u0 + base + i;
                        // The tile's four words are unpacked first, then the window slot is refilled (into the
                        // registers the words just left), then come the products.  Left alone, the scheduler gathers
                        // the refills behind the whole window's arithmetic.
                        bf16x8 b0 = unpack8(win[i].x, uk), b1 = unpack8(win[i].y, uk), b2 = unpack8(win[i].z, uk), b3 = unpack8(win[i].w, uk);
                        compute_here(b0); compute_here(b1); compute_here(b2); compute_here(b3);
                        __builtin_amdgcn_sched_barrier(0);
                        win[i] = run_load16(wr, lane_off + (uint32_t)i * 1024u);
                        __builtin_amdgcn_sched_barrier(0);
                        if (!kGuard || ku < u1) {
                            const u32x4 xn = *reinterpret_cast<const u32x4 *>(xrow + (ku + 1 < u1 ? ku + 1 : ku) * 32);
                            acc[0] = mfma(xa, b0, acc[0]);
                            acc[1] = mfma(xa, b1, acc[1]);
                            acc[2] = mfma(xa, b2, acc[2]);
                            acc[3] = mfma(xa, b3, acc[3]);
                            xa = xn;
                            if (i % UPG == UPG - 1) {                 // end of a group: scale / zero / offset
                                const int gi = ku / UPG;
                                behind_tile(b0);
#pragma unroll
                                for (int bb = 0; bb < NB; ++bb) {
                                    const uint32_t ev = entry(0, (gi - g0) / kEpl, gi & 1, block0 + bb);
                                    const float sc = scale_of(ev), zp = zero_of(ev);
#pragma unroll
                                    for (int j = 0; j < NI; ++j) {
                                        const float v = MT > 4 ? pick2(acc[bb][j], acc[bb + 2][j]) : pick4(acc[0][j], acc[1][j], acc[2][j], acc[3][j]);
                                        tot[bb][j] += sc * (v - zp * xs_of[j][gi]);
                                    }
                                }
#pragma unroll
                                for (int d = 0; d < 4; ++d) acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
                            }
                        }
                    }
                };
                int base = 0;
                for (; base + kWin <= nt; base += kWin) gu_window(base, std::false_type{});
                if (base < ntp) gu_window(base, std::true_type{});
                // the window now holds this wave's first down tiles (or, for a wave without down tiles, the
                // successor's first gate/up tiles)
#pragma unroll
                for (int bb = 0; bb < NB; ++bb)
#pragma unroll
                    for (int i = 0; i < NI; ++i) s_red[wave][slot0 + i][(block0 + bb) * 16 + r] = tot[bb][i];
            }
            __syncthreads();
            // h for (token slot, row): rows 0-31 of the sums are gate rows, 32-63 the matching up rows
            if (tid < 32 * cnt) {
                const int slot = tid >> 5, row = tid & 31;
                float gsum = 0.f, usum = 0.f;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) { gsum += s_red[w][slot][row]; usum += s_red[w][slot][row + 32]; }
                const float h = gsum / (1.f + expf(-gsum)) * usum;
                const uint16_t hi = f32_to_bf16_rne(h);
                const uint16_t lo = f32_to_bf16_rne(h - __uint_as_float((uint32_t)hi << 16));
                s_hhi[slot][row] = hi;
                s_hlo[slot][row] = lo;
                // sum of the represented h over the slice, per token: 16 lanes add up in a fixed order, and the
                // slot's two sums meet in LDS (two addends commute, so the result does not depend on order)
                float hs = __uint_as_float((uint32_t)hi << 16) + __uint_as_float((uint32_t)lo << 16);
                hs = wave::row_sum(hs);
                if ((row & 15) == 0) atomicAdd(&s_hsum[par][slot], hs);
            }
            // the last wave (it has the smallest part, if any, in the sums above) sets up the successor's rows and
            // clears the successor's h sums; the other copy of both is still being read
            if (wave == kWaves - 1) {
                if (it == it_begin) second_ticket();
                if (!last) item_rows(nxt.expert, par ^ 1);
                if (lane < MT) s_hsum[par ^ 1][lane] = 0.f;
            }
            __syncthreads();

            // ---- down: this wave's row tiles, all H outputs of the slice's 32 columns.
            // The hi and the lo part of h of a token slot are two A rows, so one MFMA yields both products.  The 16 A
            // rows have room for more: the tile's row block bl gets its own copy of the h rows at A rows
            // bl * kRs .. (all other rows zero), and the kBpa MFMAs of kBpa row blocks accumulate into ONE D
            // tile, whose lane group(s) bl then hold row block bl.  Two slots take four row blocks: the whole
            // tile (64 outputs) in one D register pair per slot, one 64-lane atomic per slot and tile.  Most items
            // have one or two tokens: those are always done, slots 2-3 and 4-7 (two row blocks at a time) only
            // where the item has them.
            if (Lw > 0 && !last) request_gu_entries(nxt);
            if (Lw > 0 && ndw > 0) {
                auto h_rows = [&](int first, auto bpa_c, u32x4 *hab) {
                    constexpr int kBpa = decltype(bpa_c)::value, kRs = 16 / kBpa;
                    const int within = r % kRs, slot = first + (within >> 1);
                    const bool used = kBpa == 4 ? within < 4 : true;
                    const u32x4 hv = *reinterpret_cast<const u32x4 *>((within & 1) ? &s_hlo[slot & (MT - 1)][c * 8] : &s_hhi[slot & (MT - 1)][c * 8]);
#pragma unroll
                    for (int bl = 0; bl < kBpa; ++bl) {
                        const bool on = used && slot < cnt && r / kRs == bl;
                        hab[bl] = (u32x4){on ? hv.x : 0u, on ? hv.y : 0u, on ? hv.z : 0u, on ? hv.w : 0u};
                    }
                };
                // what the lane's two slots need: their sums of h, weights, and offsets in y.  An empty slot's outputs go
                // past the end of y, where an addition is dropped: no branch, so that the compiler can count
                // the atomics between the loads (it counts none under a branch, and each wait for a tile then also
                // waits for tiles requested behind it).
                struct Out { float hsum[2], w[2]; uint32_t off[2]; };
                auto outs = [&](int slot0, int block) {
                    Out o;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int t = slot0 + i, slot = t < cnt ? t : 0;
                        const int arow = s_row_a[par][slot];
                        o.hsum[i] = t < cnt ? s_hsum[par][slot] : 0.f;
                        o.w[i] = t < cnt ? s_w[arow] : 0.f;
                        o.off[i] = t < cnt ? (uint32_t)((arow / k) * H + block * 16 + r) * 4u : kPastY;
                    }
                    return o;
                };
                constexpr std::integral_constant<int, 4> four{};
                constexpr std::integral_constant<int, 2> two{};
                u32x4 ha[4], hb[MT > 2 ? 4 : 1], hc[MT > 4 ? 2 : 1];
                const Out oa = outs(0, c);
                Out ob, oc;
                h_rows(0, four, ha);
                if constexpr (MT > 2) { h_rows(2, four, hb); ob = outs(2, c); }
                if constexpr (MT > 4) { h_rows(4, two, hc); oc = outs(4 + 2 * (c & 1), c >> 1); }
                auto add = [&](const Out &o, f32x4 d, uint32_t ev, uint32_t toff) {
                    const float sc = scale_of(ev), zp = zero_of(ev);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(sc * ((d[2 * j] + d[2 * j + 1]) - zp * o.hsum[j]) * o.w[j],
                                                                        y_run, (int)(o.off[j] + toff), 0, 0);
                };
                // slots sl, sl + 1 (block c of the row tile: lane = output): onto `old` in LDS, or added to y at once.  (The
                // sums are each wave's own, so they are read and written: an atomic addition in LDS takes 160 clocks.)
                auto add_slots = [&](int sl, const Out &o, f32x4 d, uint32_t ev, uint32_t toff, int rt, const float *old) {
                    if constexpr (!SUMS) add(o, d, ev, toff);
                    else if (rt < r1) {
                        const float sc = scale_of(ev), zp = zero_of(ev);
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            s_y[(sl + j) * H + rt * 64 + lane] = old[j] + sc * ((d[2 * j] + d[2 * j + 1]) - zp * o.hsum[j]) * o.w[j];
                    }
                };
                for (int j0 = 0; j0 < ndw; j0 += kWin) {
                    const run_t wr = window_run(cur, nxt, !last, ntp + j0 + kWin);
#pragma unroll
                    for (int i = 0; i < kWin; ++i) {
                        const int rt = r0 + j0 + i, rt_in = rt < r1 ? rt : r1 - 1;
                        bf16x8 b[4] = {unpack8(win[i].x, uk), unpack8(win[i].y, uk), unpack8(win[i].z, uk), unpack8(win[i].w, uk)};
                        compute_here(b[0]); compute_here(b[1]); compute_here(b[2]); compute_here(b[3]);
                        __builtin_amdgcn_sched_barrier(0);
                        win[i] = run_load16(wr, lane_off + (uint32_t)i * 1024u);
                        __builtin_amdgcn_sched_barrier(0);
                        behind_tile(b[0]);
                        const uint32_t toff = rt < r1 ? (uint32_t)rt * 256u : kPastY / 2;    // (padding: dropped as well)
                        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                        const uint32_t ev = entry(1, (rt_in - r0) / kEpl, rt_in & 1, c);
                        float old[4] = {0.f, 0.f, 0.f, 0.f};
                        if constexpr (SUMS) { old[0] = s_y[rt_in * 64 + lane]; old[1] = s_y[H + rt_in * 64 + lane]; }
                        add_slots(0, oa, mfma(ha[3], b[3], mfma(ha[2], b[2], mfma(ha[1], b[1], mfma(ha[0], b[0], zero)))), ev, toff, rt, old);
                        if (MT > 2 && cnt > 2) {
                            if constexpr (SUMS && kAcc > 2) { old[2] = s_y[2 * H + rt_in * 64 + lane]; old[3] = s_y[3 * H + rt_in * 64 + lane]; }
                            const f32x4 d = mfma(hb[3], b[3], mfma(hb[2], b[2], mfma(hb[1], b[1], mfma(hb[0], b[0], zero))));
                            if constexpr (!SUMS || kAcc > 2) add_slots(2, ob, d, ev, toff, rt, old + 2);
                            else add(ob, d, ev, toff);
                        }
                        if constexpr (MT > 4) {
                            if (cnt > 4) {
#pragma unroll
                                for (int q = 0; q < 2; ++q)
                                    add(oc, mfma(hc[1], b[2 * q + 1], mfma(hc[0], b[2 * q], zero)),
                                        entry(1, (rt_in - r0) / kEpl, rt_in & 1, 2 * q + (c >> 1)), toff + q * 128u);
                            }
                        }
                    }
                }
            }
            // the last item of this expert: its sums leave, and all slots start again (an empty slot's products are zeros, but
            // not times an infinite scale)
            if (SUMS && (last || nxt.expert != cur.expert)) {
                for (int sl = 0; sl < kAcc; ++sl) {
                    const uint32_t off = (uint32_t)((s_row_a[par][sl < cnt ? sl : 0] / k) * H + lane) * 4u;
                    for (int rt = r0; rt < r1; ++rt) {
                        float *p = &s_y[sl * H + rt * 64 + lane];
                        if (sl < cnt) __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(*p, y_run, (int)(off + (uint32_t)rt * 256u), 0, 0);
                        *p = 0.f;
                    }
                }
            }
            cur = nxt;
            if (it + 2 < it_end) { item_after(nxt, cur); item_addr(nxt, nth_expert(nxt.u)); }
        }
    } else {
        softmax();
        if (wave == kWaves - 1) second_ticket();
        __syncthreads();
    }

    // ---- 4. the workgroup that holds the last ticket puts the workspace back to idle, all waves together (8 tokens x
    // 128 experts are 16384 stores: 256 rounds of one wave)
    if (tid == kThreads - 64) s_last = ticket2 == ticket_groups(gridDim.x) - 1;
    __syncthreads();
    if (s_last) reset_exchange(a, tid, kThreads);

    // ---- 5. workgroup 0 reports the routing (and the plan the shared-expert kernels read)
    if (blockIdx.x != 0) return;
    for (int i = tid; i < n; i += kThreads) {
        a.ids_out[i] = ok ? s_ids[i] : -1;
        if (a.conf_out) a.conf_out[i] = ok ? s_conf[i] : 0.f;
    }
    if (a.S > 0) write_shared_plan(a);
}

template <int MT, int UPG, bool SYM, int kWin>
__global__ __launch_bounds__(kThreads, kWaves / 4)
void draft_stream_kernel(const uint16_t *__restrict__ xin, const FusedArgs a) { draft_stream<MT, UPG, SYM, kWin, false>(xin, a); }

// Many items per workgroup: y summed in LDS.  Added to y item by item, the atomics sit between the weight loads, which
// complete in order behind them.  us per call, added at once / summed: phi shape, 4 tokens 48.7 / 43.3, 8 tokens 74.3 / 67.4,
// mixtral, 3 tokens, symmetric 88.0 / 76.7, 1 token 43.8 / 39.6.  With one or two short items per workgroup the sums only cost
// (24 experts, H = 3072, I = 640, 7 tokens: 44.8 / 46.0), and so they do with the window of four (qwen3 shape, 8 tokens: 38.2 / 40.1).
template <int MT, int UPG, bool SYM>
__global__ __launch_bounds__(kThreads, kWaves / 4)
void draft_stream_sums_kernel(const uint16_t *__restrict__ xin, const FusedArgs a) { draft_stream<MT, UPG, SYM, 8, true>(xin, a); }

__global__ __launch_bounds__(256)
void zero_kernel(uint32_t *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

// Plain streaming read of `tiles` 1 KiB tiles with the access shape of the weight stream above:
// every wave owns a contiguous run of tiles, a lane takes 16 bytes of a tile, kWin non-temporal
// loads in flight per lane, every load unconditional (past the end of the run it repeats the
// last tile: a load under a branch would make the compiler drain the window at every step).
// The words are folded so that the loads cannot be dropped; the fold is stored only when it
// equals a value that memory holding real data will not produce.
template <int kWin>
__global__ __launch_bounds__(512, 2)
void stream_read_kernel(const u32x4 *__restrict__ src, size_t tiles, uint32_t *sink)
{
    const int lane = threadIdx.x & 63;
    const size_t nwaves = (size_t)gridDim.x * 8;
    const size_t wave = (size_t)blockIdx.x * 8 + (threadIdx.x >> 6);
    const size_t per = (tiles + nwaves - 1) / nwaves;
    const size_t first = wave * per;
    const size_t mine = first >= tiles ? 0 : (tiles - first < per ? tiles - first : per);
    if (mine == 0) return;
    const u32x4 *q = src + first * 64 + lane;
    u32x4 win[kWin];
    uint32_t fold = 0;
#pragma unroll
    for (int i = 0; i < kWin; ++i) win[i] = __builtin_nontemporal_load(q + ((size_t)i < mine ? (size_t)i : mine - 1) * 64);
    for (size_t b = 0; b < mine; b += kWin) {
#pragma unroll
        for (int i = 0; i < kWin; ++i) {
            const size_t t = b + i;
            const u32x4 v = win[i];
            const size_t nx = t + kWin < mine ? t + kWin : mine - 1;
            win[i] = __builtin_nontemporal_load(q + nx * 64);
            if (t < mine) fold ^= v.x ^ v.y ^ v.z ^ v.w;
        }
    }
    if (fold == 0x9E3779B9u) sink[0] = fold;
}

// One workgroup per compute unit: two that share a unit are slower, also where they fit its registers (phi
// shape, 2 tokens: 37.6 us against 41.6 with two, qwen3 19.2 / 20.6; 4 tokens, held to 128 registers: 52.7 / 60.4; all on the
// form without sums of y in LDS).
constexpr int kMaxPerCu = 1;

// go(kernel, bytes of dynamic LDS) with the instantiation for a call
template <int MT, int UPG, bool SYM, typename F>
void stream_kernel_m(const Shape &s, int n_cu, F go)
{
    const size_t lds = draft_dynamic_lds(MT, s.H, s.g, s.E, SYM), sums = sum_lds(s, MT, SYM, n_cu);
    if (sums) go(draft_stream_sums_kernel<MT, UPG, SYM>, lds + sums);
    else if (stream_window(s, SYM) == 8) go(draft_stream_kernel<MT, UPG, SYM, 8>, lds);
    else go(draft_stream_kernel<MT, UPG, SYM, 4>, lds);
}
template <int UPG, bool SYM, typename F>
void stream_kernel_g(const Shape &s, int n_cu, F go)
{
    if (s.T <= 2) stream_kernel_m<2, UPG, SYM>(s, n_cu, go);
    else if (s.T <= 4) stream_kernel_m<4, UPG, SYM>(s, n_cu, go);
    else stream_kernel_m<8, UPG, SYM>(s, n_cu, go);
}
template <bool SYM, typename F>
void stream_kernel_t(const Shape &s, int n_cu, F go)
{
    if (s.g == 32) stream_kernel_g<1, SYM>(s, n_cu, go);
    else if (s.g == 64) stream_kernel_g<2, SYM>(s, n_cu, go);
    else stream_kernel_g<4, SYM>(s, n_cu, go);
}
template <typename F>
void stream_kernel(const Shape &s, bool sym, int n_cu, F go)
{
    if (sym) stream_kernel_t<true>(s, n_cu, go);
    else stream_kernel_t<false>(s, n_cu, go);
}

}  // namespace

OneTokenForm draft_form(const Shape &s, const DraftFusedArgs &d, int n_cu)
{
    if (s.T > 1) return kPersistent;
    return one_token_form(s, d.symmetric != 0, d.shared_inside != 0, n_cu, [&] { return draft_one_token_slots(s, d, kSingleItems, n_cu); });
}

// The launch shapes: one token, one workgroup per item or two, dispatched in order, so the first ones, which
// reduce the router rows, are resident together when that many fit on the device at once; more tokens,
// a grid of as many workgroups as the device holds at once.
int draft_resident_slots(const Shape &s, const DraftFusedArgs &d, int n_cu)
{
    if (d.form != kPersistent) {
        const int items = d.form == kPairsOfItems ? 2 : 1, slots = draft_one_token_slots(s, d, d.form, n_cu);
        return router_workgroups(s.E, items, s.k * (s.I / 32) / items) <= slots ? slots : 0;
    }
    int per = 0;
    stream_kernel(s, d.symmetric != 0, n_cu, [&](auto kernel, size_t lds) { per = resident_per_cu(kernel, kThreads, lds); });
    return (per < kMaxPerCu ? per : kMaxPerCu) * n_cu;
}

void launch_draft_fused(const Shape &s, const DraftFusedArgs &d, int n_cu, int slots, hipStream_t st)
{
    if (d.form != kPersistent) { launch_draft_one_token(s, d, st); return; }
    const FusedArgs a = fused_args(s, d);
    // never more workgroups than there can be items
    const int maxu = s.E < s.T * s.k ? s.E : s.T * s.k;
    const long items = (long)maxu * (s.I / 32);
    const dim3 grid((unsigned)(items < slots ? items : slots)), block(kThreads);
    stream_kernel(s, d.symmetric != 0, n_cu, [&](auto kernel, size_t lds) {
        launch_with_lds(kernel, grid, block, lds, st, (const uint16_t *)d.x, a);
    });
}

void launch_stream_read(const void *src, size_t bytes, int workgroups, void *sink, hipStream_t st)
{
    launch(stream_read_kernel<8>, dim3(workgroups), dim3(512), 0, st, (const u32x4 *)src,
                       bytes / 1024, (uint32_t *)sink);
}

void launch_zero(void *p, size_t bytes, hipStream_t st)
{
    const size_t n = bytes / 4;
    int blocks = (int)((n + 255) / 256);
    blocks = blocks > 1024 ? 1024 : (blocks < 1 ? 1 : blocks);
    launch(zero_kernel, dim3(blocks), dim3(256), 0, st, (uint32_t *)p, n);
}

}  // namespace moespeq
