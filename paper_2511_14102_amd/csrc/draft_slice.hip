// Draft-pass kernel for a call with ONE token: router, top-k and the SwiGLU FFN of the selected
// experts on group-wise int4 weights in one launch, one or two work items per workgroup (gfx950).
// (Calls of two to eight tokens, and of one with many long items, run the persistent kernel of
// draft_int4.hip, longer runs of tokens the grouped contraction of draft_prefill.hip.)
//
// Paper section 3.4.3 (one expert-fused kernel instead of per-expert small GEMMs), section 4.1.3
// (4-bit weights in groups along the input dimension), section 3.3.1 (expert id and confidence
// for the lookahead buffer).  The arithmetic is described in draft_common.h, the
// cross-workgroup protocol of the router exchange in draft_int4.hip (the same here).
//
// Work decomposition ("slice fusion").  A work item is (expert, slice of 32 intermediate
// rows): eight waves compute the 32 gate and 32 up pre-activations (K = H split over them
// by groups), h = silu(gate) * up, and immediately multiply h into the 32 matching
// columns of the down projection for all H outputs, which are added into y with
// fp32 atomics.  With one token a call has k I / 32 items (400 on the phi shape); a workgroup has one of them, or two
// (slice_pairs).  Long rows and two items per unit and more run the persistent kernel (one_token_streams).
//
// Bound: a chain of round trips to memory up to the first weight load (x and router rows, exchange, selection:
// about 3 us), then the weight stream (84 MB in about 14 us on the phi shape), then the chain of additions to y (slice_pairs).
#include "draft_common.h"

namespace moespeq {

namespace {

// UPG: 32-code units per group (g / 32); SYM: symmetric format (scale blobs, z = 8); SHARED: the shared
// experts run in this launch (without them the kernel is smaller: its start is a chain of code that runs once); ITEMS: one item
// per workgroup, or two neighbours (of one expert), eight waves each, whose outputs are added up in LDS; PLANES: the down part multiplies e4m3 planes of h
template <int UPG, bool SYM, bool SHARED, int ITEMS, bool PLANES>
__device__ __forceinline__ void draft_one_token(const uint16_t *__restrict__ xin, const FusedArgs &a)
{
    // tiles a wave keeps in flight (rolling window): two workgroups per compute unit leave 128 VGPRs per
    // wave, and with an entry per tile (g = 32) a window of 8 spills
    constexpr int kWin = UPG == 1 ? 6 : 8;
    constexpr int kSzWin = kWin / UPG;
    constexpr int kAll = kThreads * ITEMS;
    __shared__ double s_part[kWaves * ITEMS];
    __shared__ int32_t s_ids[MOE_MAX_TOPK];
    __shared__ float s_w[MOE_MAX_TOPK], s_conf[MOE_MAX_TOPK];
    __shared__ int32_t s_ok;
    __shared__ float s_red[ITEMS][kWaves][64];       // partial gate/up sums
    // h, each wave's own copy: its four e4m3 planes of 32 bytes (a shared expert's: 16 bf16 values and their remainders)
    __shared__ __attribute__((aligned(16))) uint16_t s_h[ITEMS][kWaves][2][32];
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];   // x, its group sums, logits, ranks, two items' outputs

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // eight waves to an item: `wave` of them, `half`: which item
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % kWaves, half = ITEMS > 1 ? __builtin_amdgcn_readfirstlane(tid >> 9) : 0;
    const bool wave0 = __builtin_amdgcn_readfirstlane(tid >> 6) == 0;
    const int H = a.H, E = a.E, I = a.I, k = a.k;
    const int G = H / (32 * UPG), U = H / 32, nslice = I / 32;
    uint16_t *s_x = reinterpret_cast<uint16_t *>(s_dyn);
    double *s_logit = reinterpret_cast<double *>(s_dyn + (size_t)H * 2);
    int32_t *s_rank = reinterpret_cast<int32_t *>(s_logit + E);
    float *s_xsum = reinterpret_cast<float *>(s_rank + E);
    float *s_y = s_xsum + G;                                 // [ITEMS][H], two items only
    const int r = lane & 15, c = lane >> 4;                  // MFMA lane coordinates

    // this thread's first piece of x, on its way while the router rows are reduced
    u32x4 xr = *reinterpret_cast<const u32x4 *>(xin + (tid < H / 8 ? tid : H / 8 - 1) * 8);

    // ---- 1. which work item.  The first workgroups reduce the router rows; workgroups are dispatched in order, so
    // they are running before any other waits for them.  Behind them the shared experts' items, which start at
    // once, then the other routed items, which wait for the routing.
    const int n_sh = SHARED ? a.S * (I / 16) / ITEMS : 0, n_routed = (int)gridDim.x - n_sh;
    const int nprod = router_workgroups(E, ITEMS, n_routed);
    const int b = blockIdx.x;
    const bool shared = SHARED && b >= nprod && b < nprod + n_sh;
    if (b < nprod) publish_router_rows<kWaves * ITEMS, ITEMS>(xin, a, b, nprod, s_part);
    uint32_t ticket = 0xffffffffu, ticket2 = 0xffffffffu;
    auto first_ticket = [&]() { if (lane == 0) ticket = draw_ticket(a.tickets + b % kTicketGroups); };
    auto stage_x = [&]() {
        if (tid < H / 8) *reinterpret_cast<u32x4 *>(s_x + tid * 8) = xr;
        for (int i = tid + kAll; i < H / 8; i += kAll)
            *reinterpret_cast<u32x4 *>(s_x + i * 8) = *reinterpret_cast<const u32x4 *>(xin + i * 8);
        __syncthreads();
    };
    auto give_up = [&]() {
        if (lane == 0) __hip_atomic_store(a.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // Tickets: wave 0 draws the workgroup's when it has polled.  The holder of the last one puts the
    // workspace back to idle (at its own end: nothing waits for it).
    auto second_ticket = [&]() {
        if (lane == 0 && ticket == ticket_members(b, gridDim.x) - 1) ticket2 = draw_ticket(a.tickets + kTicketGroups);
    };
    auto reset_if_last = [&]() {
        if (__any(ticket2 == ticket_groups(gridDim.x) - 1)) reset_exchange(a, lane, 64);
    };

    // An output of an item: added to y, or kept until both items of the workgroup have theirs
    auto add_output = [&](int at, float v) {
        if constexpr (ITEMS > 1) s_y[half * H + at] = v;
        else __hip_atomic_fetch_add(&a.y[at], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto add_both = [&]() {
        if constexpr (ITEMS > 1) {
            __syncthreads();
            for (int i = tid; i < H; i += kAll) __hip_atomic_fetch_add(&a.y[i], s_y[i] + s_y[H + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };

    if constexpr (SHARED) if (shared) {
        // ---- 2. an item of a shared expert: 16 intermediate rows (a gate and an up tile of 16 x 32 bf16 per
        // k-step), then their 16 columns of the down projection: half of a 16 x 32 tile, so a load takes the
        // halves of two tiles, and one MFMA multiplies both (the A rows of one tile's half are zero in the
        // other's k positions).  The stream and its window are the routed items'.
        const int nth = (b - nprod) * ITEMS + half, sh = nth / (I / 16), row16 = nth % (I / 16);
        const char *blob = a.shared + (size_t)sh * a.shared_stride;
        const char *gate = blob + (size_t)row16 * U * 1024, *up = gate + (size_t)I * H * 2;
        const uint32_t rstep = (uint32_t)(I / 32) * 1024;            // from one output row tile to the next
        const char *down = blob + (size_t)I * H * 4 + (size_t)(row16 / 2) * 1024;
        const uint32_t lane_off = lane * 16u;
        const uint32_t dlane = (uint32_t)(c >> 1) * 2 * rstep + (uint32_t)(((row16 & 1) * 2 + (c & 1)) * 16 + r) * 16u;
        const int k0 = (wave * U) / kWaves, nt = ((wave + 1) * U) / kWaves - k0;
        const int ntp = (2 * nt + kWin - 1) / kWin * kWin;           // gate/up loads, padded to whole windows
        const int ngrp = H / 64;                                     // groups of four row tiles: two loads each
        const int q0 = (wave * ngrp) / kWaves, nd = 2 * (((wave + 1) * ngrp) / kWaves - q0);
        // gate and up tiles of a k-step are I H 2 bytes apart: two runs; a pair of down loads is 4 rstep from the next
        const run_t g_run = make_run(gate + (size_t)k0 * 1024, nt * 1024), u_run = make_run(up + (size_t)k0 * 1024, nt * 1024);
        const run_t d_run = make_run(down + (size_t)4 * q0 * rstep, nd > 0 ? 2 * nd * rstep - (uint32_t)(row16 / 2) * 1024 : 0);
        auto pair_load = [&](bool into_down, int p, u32x4 &v, u32x4 &w) {      // loads p, p + 1 of a part
            const uint32_t off = into_down ? dlane + 2u * (uint32_t)p * rstep : lane_off + (uint32_t)p * 512u;
            v = run_load16(into_down ? d_run : g_run, off);
            w = run_load16(into_down ? d_run : u_run, off + (into_down ? rstep : 0u));
        };
        u32x4 win[kWin];
#pragma unroll
        for (int i = 0; i < kWin; i += 2) pair_load(ntp == 0, i, win[i], win[i + 1]);
        stage_x();
        const uint16_t *xrow = s_x + c * 8;
        f32x4 ag = {0.f, 0.f, 0.f, 0.f}, au = {0.f, 0.f, 0.f, 0.f};
        for (int base = 0; base < ntp; base += kWin) {
            const bool into_down = base + kWin >= ntp;
#pragma unroll
            for (int i = 0; i < kWin; i += 2) {
                const int kk = (base + i) / 2;
                const bf16x8 wg = __builtin_bit_cast(bf16x8, win[i]), wu = __builtin_bit_cast(bf16x8, win[i + 1]);
                if (kk < nt) {                       // (the padding of the last window is skipped)
                    const u32x4 xa = *reinterpret_cast<const u32x4 *>(xrow + (k0 + kk) * 32);
                    ag = mfma(xa, wg, ag);
                    au = mfma(xa, wu, au);
                }
                __builtin_amdgcn_sched_barrier(0);
                pair_load(into_down, (into_down ? 0 : base + kWin) + i, win[i], win[i + 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // all 16 A rows are the token: every lane group holds the same sums
        if (c < 2) s_red[half][wave][lane] = c == 0 ? ag[0] : au[0];
        if (wave0) {
            // the outputs may be added once y has been cleared, which every router workgroup does before it publishes
            const bool ok = poll_and_select(a, 0, nullptr, nullptr, nullptr, nullptr);
            first_ticket();
            if (!ok) give_up();
            if (lane == 0) s_ok = ok;
        }
        __syncthreads();
        {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v += s_red[half][w][lane & 31];
            const float u = __shfl_xor(v, 16);
            const float h = v / (1.f + expf(-v)) * u;
            const uint16_t hi = f32_to_bf16_rne(h);
            if (lane < 16) {
                s_h[half][wave][0][lane] = hi;
                s_h[half][wave][1][lane] = f32_to_bf16_rne(h - __uint_as_float((uint32_t)hi << 16));
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (wave0) second_ticket();
        if (s_ok) {
            // A rows 4 q, 4 q + 1 hold h and its remainder for the tile whose outputs lane group q gets:
            // groups 0, 2 from the halves of a pair's first load, 1, 3 from its second
            u32x4 ha[2];
            {
                const u32x4 hv = *reinterpret_cast<const u32x4 *>(&s_h[half][wave][r & 1][(c & 1) * 8]);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const bool on = (r & 3) < 2 && ((r >> 2) & 1) == j && (r >> 3) == (c >> 1);
                    ha[j] = (u32x4){on ? hv.x : 0u, on ? hv.y : 0u, on ? hv.z : 0u, on ? hv.w : 0u};
                }
            }
            auto down_pass = [&](int d0, auto reload) {
#pragma unroll
                for (int i = 0; i < kWin; i += 2) {
                    f32x4 o = {0.f, 0.f, 0.f, 0.f};
                    o = mfma(ha[0], __builtin_bit_cast(bf16x8, win[i]), o);
                    o = mfma(ha[1], __builtin_bit_cast(bf16x8, win[i + 1]), o);
                    if constexpr (decltype(reload)::value) {
                        __builtin_amdgcn_sched_barrier(0);
                        pair_load(true, d0 + kWin + i, win[i], win[i + 1]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (d0 + i < nd)
                        add_output((q0 + (d0 + i) / 2) * 64 + lane, o[0] + o[1]);
                }
            };
            int d0 = 0;
            for (; d0 + kWin < nd; d0 += kWin) down_pass(d0, std::true_type{});
            down_pass(d0, std::false_type{});
            add_both();
        }
        if (wave0) reset_if_last();
        return;
    }

    // ---- 3. a routed item: slice `slice` of the u-th ranked expert.  What does not depend on the expert is computed
    // while the router result travels.
    const int item = (b < nprod ? b : b - n_sh) * ITEMS + half;
    const int u = item / nslice, slice = item % nslice;
    const UnpackConsts uk = unpack_consts();
    const uint32_t lane_off = (uint32_t)lane * 16u;
    const int nrt = H / 64;
    constexpr int kEpl = SYM ? 2 : 1;                        // groups (row tiles) per 16-byte unit of entries
    // This wave's tile stream: its gate/up tiles u0 .. u1 (K = H split over the waves by groups; the
    // symmetric format keeps two groups in a unit: whole pairs), padded to whole windows, then its down row
    // tiles r0 .. r1 (their loads do not depend on h).  A rolling window of kWin tiles is in flight.  EVERY
    // load of the stream is unconditional: the compiler counts the loads in flight in program order, and a
    // load under a branch makes it wait for all of them wherever it needs one, which empties the window.
    const int u0 = ((wave * (G / kEpl)) / kWaves) * kEpl * UPG, u1 = (((wave + 1) * (G / kEpl)) / kWaves) * kEpl * UPG;
    const int nt = u1 - u0;
    const int ntp = (nt + kWin - 1) / kWin * kWin;
    const int r0 = ((wave * (nrt / kEpl)) / kWaves) * kEpl, r1 = (((wave + 1) * (nrt / kEpl)) / kWaves) * kEpl;
    const int ndw = r1 - r0;
    // codes: [gate|up tiles (slice, ku)] then [down tiles (slice, rt)], 64 lanes x 16 B each; the wave's two runs:
    const size_t gu_off = ((size_t)slice * U + u0) * 1024, dn_off = ((size_t)nslice * U + (size_t)slice * nrt + r0) * 1024;
    // scale/zero: 16 B = the 4 row blocks' (s, z) of lane row r; [gate|up (slice, group)] then [down (group of I, rt)]
    // (symmetric format: 16 B = the 4 row blocks' s of row r for two groups / two row tiles).  With one token all
    // 16 A rows hold it, so every lane group ends up with the same sums: lane group c finishes row block c
    // only and loads that block's entry itself.
    const uint32_t ent_lane = (uint32_t)((SYM ? r * 8 : r * 4) + c) * (SYM ? 2u : 4u);
    const size_t gent_off = ((size_t)slice * (G / kEpl) + u0 / (UPG * kEpl)) * 256;
    const size_t dent_off = ((size_t)nslice * (G / kEpl) + (size_t)(slice / UPG) * (nrt / kEpl) + r0 / kEpl) * 256;

    stage_x();
    // sums of x per group: 16 threads each
    for (int i = tid; i < G * 16; i += kAll) {
        constexpr int kPer = 2 * UPG;
        const uint16_t *src = s_x + i * kPer;
        float v = 0.f;
#pragma unroll
        for (int j = 0; j < kPer; ++j) v += __uint_as_float((uint32_t)src[j] << 16);
        v = wave::row_sum(v);
        if ((i & 15) == 0) s_xsum[i >> 4] = v;
    }

    // ---- 4. wave 0 polls the slots (bounded) and selects the top-k
    if (wave0) {
        const bool got = poll_and_select(a, 0, s_logit, s_rank, s_ids, nullptr);
        if (!got) give_up();                     // the call fails, and says so in the workspace
        if (lane == 0) s_ok = got;
    }
    __syncthreads();
    const bool ok = s_ok != 0;
    if (ok) {
        // ---- 5. the first window of weight loads goes out at once
        const int ex = __builtin_amdgcn_readfirstlane(s_ids[u]);
        const char *qb = a.q + (size_t)ex * a.stride_q, *sz = a.sz + (size_t)ex * a.stride_sz;
        const run_t gu_run = make_run(qb + gu_off, nt * 1024), dn_run = make_run(qb + dn_off, ndw * 1024);
        const run_t gent_run = make_run(sz + gent_off, nt / (UPG * kEpl) * 256), dent_run = make_run(sz + dent_off, ndw / kEpl * 256);
        auto entry = [&](run_t run, int t) {                 // of the run's t-th group or row tile
            if constexpr (SYM) return run_load2(run, ent_lane + (uint32_t)((t >> 1) * 256 + (t & 1) * 8));
            else return run_load4(run, ent_lane + (uint32_t)t * 256u);
        };
        auto scale_of = [](uint32_t e) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(e & 0xffff)); };
        auto zero_of = [](uint32_t e) { return SYM ? 136.f : (float)__builtin_bit_cast(_Float16, (uint16_t)(e >> 16)) + 128.f; };
        const uint32_t cm1 = 0u - (uint32_t)(c & 1), cm2 = 0u - (uint32_t)(c >> 1);
        auto of_my_block = [&](float v0, float v1, float v2, float v3) {   // v_c, chosen with bit masks
            const uint32_t lo = (__float_as_uint(v1) & cm1) | (__float_as_uint(v0) & ~cm1);
            const uint32_t hi = (__float_as_uint(v3) & cm1) | (__float_as_uint(v2) & ~cm1);
            return __uint_as_float((hi & cm2) | (lo & ~cm2));
        };
        // (an entry follows the last tile of its group)
        u32x4 win[kWin];
        uint32_t gent[kSzWin], dpe[kWin];
        {
            const run_t first = nt > 0 ? gu_run : dn_run;
#pragma unroll
            for (int i = 0; i < kWin; ++i) {
                win[i] = run_load16(first, lane_off + (uint32_t)i * 1024u);
                if (i % UPG == UPG - 1) gent[i / UPG] = entry(gent_run, i / UPG);
            }
        }
        // the ticket goes out behind the first loads: they would wait for it (loads and returning atomics complete in
        // order, and hundreds of tickets are drawn at about the same time)
        if (wave0) first_ticket();
        // the softmax, off the path to the first weight load
        if (wave0) finish_softmax(a, s_logit, s_rank, s_conf, s_w);

        // ---- 6. gate and up
        const uint16_t *xrow = s_x + c * 8;
        f32x4 acc[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
        float tot = 0.f;
        u32x4 xa = *reinterpret_cast<const u32x4 *>(xrow + (nt > 0 ? u0 : 0) * 32);
        // one window; kGuard: some of its tiles may lie past the wave's run (the padding of the last window)
        // and are skipped.  Full windows carry no per-tile tests.
        auto gu_window = [&](int base, auto guarded) {
            constexpr bool kGuard = decltype(guarded)::value;
            const bool into_down = base + kWin >= ntp;
            const run_t run = into_down ? dn_run : gu_run;
            const uint32_t off = lane_off + (into_down ? 0u : (uint32_t)(base + kWin) * 1024u);
#pragma unroll
            for (int i = 0; i < kWin; ++i) {
                const int ku = u0 + base + i;
                // The tile's words are unpacked first, then the window slot is refilled, then come the products.  Left
                // alone, the scheduler gathers the refills behind the whole window's arithmetic.
                bf16x8 b0 = unpack8(win[i].x, uk), b1 = unpack8(win[i].y, uk), b2 = unpack8(win[i].z, uk), b3 = unpack8(win[i].w, uk);
                compute_here(b0); compute_here(b1); compute_here(b2); compute_here(b3);
                __builtin_amdgcn_sched_barrier(0);
                win[i] = run_load16(run, off + (uint32_t)i * 1024u);
                float sc = 0.f, zp = 0.f;
                if (i % UPG == UPG - 1) {
                    sc = scale_of(gent[i / UPG]);
                    zp = zero_of(gent[i / UPG]);
                    compute_here(sc); compute_here(zp);
                    gent[i / UPG] = entry(gent_run, (base + kWin) / UPG + i / UPG);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (!kGuard || ku < u1) {
                    const u32x4 xn = *reinterpret_cast<const u32x4 *>(xrow + (ku + 1 < u1 ? ku + 1 : ku) * 32);
                    acc[0] = mfma(xa, b0, acc[0]);
                    acc[1] = mfma(xa, b1, acc[1]);
                    acc[2] = mfma(xa, b2, acc[2]);
                    acc[3] = mfma(xa, b3, acc[3]);
                    xa = xn;
                    if (i % UPG == UPG - 1) {                 // end of a group: scale / zero / offset
                        tot += sc * (of_my_block(acc[0][0], acc[1][0], acc[2][0], acc[3][0]) - zp * s_xsum[ku / UPG]);
#pragma unroll
                        for (int d = 0; d < 4; ++d) acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
                    }
                }
            }
        };
        {
            int base = 0;
            for (; base + kWin <= nt; base += kWin) gu_window(base, std::false_type{});
            if (base < ntp) gu_window(base, std::true_type{});
        }
        // the window now holds this wave's first down tiles; their entries follow
#pragma unroll
        for (int i = 0; i < kWin; ++i) dpe[i] = entry(dent_run, i);
        s_red[half][wave][lane] = tot;
        if (wave0) second_ticket();
        __syncthreads();

        // ---- 7. h of the slice's 32 rows, in every wave: lanes 0-31 hold the gate rows, 32-63 the up rows; then 8. down: this wave's
        // row tiles, all H outputs of the slice's 32 columns.  A rows 4 bl .. 4 bl + 3 hold the parts of h for row block bl of the
        // tile (all other rows zero), and the four MFMAs of a tile accumulate into ONE D tile whose lane group bl then holds row block
        // bl: the tile's 64 outputs, one 64-lane atomic per tile.
        // Where the weight stream is through before the last barrier, this is all that is left but the additions, and vector work bounds it.  Long
        // rows: h as four e4m3 planes (draft_common.h), whose products take codes as they stand: 12 instructions per tile
        // unpack them (28 as bf16, for h as two bf16 numbers), and an e4m3 product keeps the vector ALU waiting 10 clocks (15).  The cut into planes is some 45 instructions
        // more, in every wave of the unit, so a wave needs three row tiles to gain.  (Both in one kernel spill.)  us per pass, two bf16 numbers / planes: phi shape (eight
        // tiles a wave), 8 layers 192.5 / 186.9, qwen15 (four), 16 445.3 / 442.3, H = 1728 249.7 / 246.7, H = 1280 324.2 / 325.7, H = 640 219.5 / 222.3; qwen3 as single items (four) 225 / 225, H = 512 152 / 154.
        {
            constexpr bool kAsPlanes = PLANES;
            uint8_t *h_bytes = reinterpret_cast<uint8_t *>(&s_h[half][wave][0][0]);
            float hsum, down = 1.f;
            {
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) v += s_red[half][w][lane];
                const float other = __shfl_xor(v, 32);
                if constexpr (kAsPlanes) {
                    const float gate = lane < 32 ? v : other, up = lane < 32 ? other : v;
                    const float h = gate / (1.f + expf(-gate)) * up;                 // (lanes 32-63 do and write the same once more: no masks)
                    float m = fabsf(h);
                    m = fmaxf(m, wave::move<wave::kSwap1>(m));
                    m = fmaxf(m, wave::move<wave::kSwap2>(m));
                    m = fmaxf(m, wave::move<wave::kHalfMirror>(m));                  // of the row's eight
                    const float row = fmaxf(m, wave::move<wave::kMirror>(m));
                    const PlaneScale scale(fmaxf(wave::from_lane<0>(row), wave::from_lane<16>(row)));
                    down = scale.down();
                    const float hu = h * scale.up(), grid = plane_grid(m * scale.up());
                    uint8_t *at = h_bytes + ((lane & 24) | ((lane & 3) << 1) | ((lane >> 2) & 1));       // the byte order of a word's codes
                    float left = hu;
#pragma unroll
                    for (int p = 0; p < kPlanes; ++p) {
                        const float step = (float)(1 << (p * kPlaneShift));
                        const float t = p < 2 ? fmaf(left, step, grid) - grid : left * step;
                        const int b = __builtin_amdgcn_cvt_pk_fp8_f32(t, t, 0, false);
                        at[p * 32] = (uint8_t)b;
                        left = fmaf(__builtin_amdgcn_cvt_f32_fp8(b, 0), -1.f / step, left);              // (exact)
                    }
                    hsum = wave::sum(hu - left) * (0.5f / 512.f);                    // of what the planes hold (twice); a code byte is q 2^-9
                } else {
                    const float h = v / (1.f + expf(-v)) * other;
                    const uint16_t hi = f32_to_bf16_rne(h);
                    const uint16_t lo = f32_to_bf16_rne(h - __uint_as_float((uint32_t)hi << 16));
                    if (lane < 32) { s_h[half][wave][0][lane] = hi; s_h[half][wave][1][lane] = lo; }
                    const float hs = __uint_as_float((uint32_t)hi << 16) + __uint_as_float((uint32_t)lo << 16);   // the represented h
                    hsum = wave::sum(lane < 32 ? hs : 0.f);
                }
                __builtin_amdgcn_wave_barrier();
            }
            const float rw = s_w[u] * (kAsPlanes ? 512.f : 1.f);

            typedef std::conditional_t<kAsPlanes, uint64_t, u32x4> a_t;
            typedef std::conditional_t<kAsPlanes, uint64_t, bf16x8> b_t;
            a_t ha[4];
#pragma unroll
            for (int bl = 0; bl < 4; ++bl) {
                if constexpr (kAsPlanes) {
                    const uint64_t hv = *reinterpret_cast<const uint64_t *>(h_bytes + (r & 3) * 32 + c * 8);
                    ha[bl] = (r >> 2) == bl ? hv : 0ull;
                } else {
                    const u32x4 hv = *reinterpret_cast<const u32x4 *>(&s_h[half][wave][r & 1][c * 8]);
                    const bool on = (r & 3) < 2 && (r >> 2) == bl;
                    ha[bl] = (u32x4){on ? hv.x : 0u, on ? hv.y : 0u, on ? hv.z : 0u, on ? hv.w : 0u};
                }
            }
            uint32_t mask = 0x0f0f0f0fu;
            asm volatile("" : "+s"(mask));
            auto operand = [&](uint32_t w) -> b_t {
                if constexpr (kAsPlanes) {
                    uint32_t lo, hi;
                    unpack8_e4m3(w, mask, lo, hi);
                    return (uint64_t)hi << 32 | lo;
                } else return unpack8(w, uk);
            };
            // one pass over the window; kReload: the slot is refilled with the tile kWin further on; the last pass
            // refills nothing
            auto down_pass = [&](int j0, auto reload) {
                constexpr bool kReload = decltype(reload)::value;
#pragma unroll
                for (int i = 0; i < kWin; ++i) {
                    const int rt = r0 + j0 + i;
                    float sc = scale_of(dpe[i]), zp = zero_of(dpe[i]) - (kAsPlanes ? 128.f : 0.f);
                    b_t b0 = operand(win[i].x), b1 = operand(win[i].y), b2 = operand(win[i].z), b3 = operand(win[i].w);
                    if constexpr (kReload) {
                        compute_here(b0); compute_here(b1); compute_here(b2); compute_here(b3);
                        compute_here(sc); compute_here(zp);
                        __builtin_amdgcn_sched_barrier(0);
                        win[i] = run_load16(dn_run, lane_off + (uint32_t)(j0 + kWin + i) * 1024u);
                        dpe[i] = entry(dent_run, j0 + kWin + i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (rt < r1) {
                        f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
                        float val;
                        if constexpr (kAsPlanes) {
                            o = mfma_e4m3(ha[0], b0, o);
                            o = mfma_e4m3(ha[1], b1, o);
                            o = mfma_e4m3(ha[2], b2, o);
                            o = mfma_e4m3(ha[3], b3, o);
                            constexpr float kStep = 1.f / (1 << kPlaneShift);
                            const float sum = fmaf(fmaf(fmaf(o[3], kStep, o[2]), kStep, o[1]), kStep, o[0]);
                            val = sc * (sum - zp * hsum) * rw * down;
                        } else {
                            o = mfma(ha[0], b0, o);
                            o = mfma(ha[1], b1, o);
                            o = mfma(ha[2], b2, o);
                            o = mfma(ha[3], b3, o);
                            val = sc * ((o[0] + o[1]) - zp * hsum) * rw;
                        }
                        add_output(rt * 64 + lane, val);
                    }
                }
            };
            int j0 = 0;
            for (; j0 + kWin < ndw; j0 += kWin) down_pass(j0, std::true_type{});
            down_pass(j0, std::false_type{});
        }
        add_both();
    } else if (wave0) {
        first_ticket();
        second_ticket();
    }

    // ---- 9. workgroup 0 reports the routing
    if (wave0) reset_if_last();
    if (b != 0) return;
    if (!SHARED && a.S > 0) write_shared_plan(a);
    if (!ok) { if (tid < k) { a.ids_out[tid] = -1; if (a.conf_out) a.conf_out[tid] = 0.f; } return; }
    if (tid < k) {
        a.ids_out[tid] = s_ids[tid];
        if (a.conf_out) a.conf_out[tid] = s_conf[tid];
    }
}

// 4 waves per SIMD: two workgroups of one item per compute unit, or one of two
template <int UPG, bool SYM, bool SHARED>
__global__ __launch_bounds__(kThreads, 4)
void draft_fused_kernel(const uint16_t *__restrict__ xin, const FusedArgs a) { draft_one_token<UPG, SYM, SHARED, 1, false>(xin, a); }
template <int UPG, bool SYM, bool SHARED>
__global__ __launch_bounds__(2 * kThreads, 4)
void draft_pair_kernel(const uint16_t *__restrict__ xin, const FusedArgs a) { draft_one_token<UPG, SYM, SHARED, 2, false>(xin, a); }
// pairs with long rows, from which the cut of h into planes gains (three row tiles per wave)
constexpr int kPlanesFromH = 1536;
template <int UPG, bool SYM, bool SHARED>
__global__ __launch_bounds__(2 * kThreads, 4)
void draft_pair_planes_kernel(const uint16_t *__restrict__ xin, const FusedArgs a) { draft_one_token<UPG, SYM, SHARED, 2, true>(xin, a); }

template <int UPG, bool SYM, bool SHARED, typename F>
void slice_kernel(int H, bool pairs, F go)           // go(kernel, items per workgroup)
{
    if (!pairs) go(draft_fused_kernel<UPG, SYM, SHARED>, 1);
    else if (H < kPlanesFromH) go(draft_pair_kernel<UPG, SYM, SHARED>, 2);
    else go(draft_pair_planes_kernel<UPG, SYM, SHARED>, 2);
}
template <bool SYM, bool SHARED, typename F>
void slice_kernel(int H, int g, bool pairs, F go)
{
    if (g == 32) slice_kernel<1, SYM, SHARED>(H, pairs, go);
    else if (g == 64) slice_kernel<2, SYM, SHARED>(H, pairs, go);
    else slice_kernel<4, SYM, SHARED>(H, pairs, go);
}
template <typename F>
void slice_kernel(const Shape &s, const DraftFusedArgs &d, OneTokenForm form, F go)
{
    const bool pairs = form == kPairsOfItems;
    if (d.symmetric) { if (d.shared_inside) slice_kernel<true, true>(s.H, s.g, pairs, go); else slice_kernel<true, false>(s.H, s.g, pairs, go); }
    else { if (d.shared_inside) slice_kernel<false, true>(s.H, s.g, pairs, go); else slice_kernel<false, false>(s.H, s.g, pairs, go); }
}

}  // namespace

// one token: router inside the launch, a work item per (selected expert, slice) and per 16 rows of
// every shared expert
void launch_draft_one_token(const Shape &s, const DraftFusedArgs &d, hipStream_t st)
{
    const FusedArgs a = fused_args(s, d);
    slice_kernel(s, d, d.form, [&](auto kernel, int items) {
        const int grid = (a.k * (a.I / 32) + (d.shared_inside ? a.S * (a.I / 16) : 0)) / items;      // (I is a multiple of 64: even counts)
        launch_with_lds(kernel, dim3(grid), dim3(kThreads * items), slice_dynamic_lds(a.H, a.g, a.E, items), st, (const uint16_t *)d.x, a);
    });
}

int draft_one_token_slots(const Shape &s, const DraftFusedArgs &d, OneTokenForm form, int n_cu)
{
    int per = 0;
    slice_kernel(s, d, form, [&](auto kernel, int items) {
        per = resident_per_cu(kernel, kThreads * items, slice_dynamic_lds(s.H, s.g, s.E, items));
    });
    return per * n_cu;
}

}  // namespace moespeq
