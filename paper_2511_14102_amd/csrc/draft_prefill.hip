// Draft pass over a long run of tokens (gfx950): the int4 experts as a grouped small-M
// contraction (paper section 3.4.3, the prefill side of the prefill / decode split; int4 weights
// of section 4.1.3).  The tokens are routed first; every expert's assignments are cut into work
// items of up to 64, and each expert's weights are streamed once per item:
//
//   prefill_logits_kernel, prefill_topk_kernel (route.hip)  the routing, and every expert's assignments;
//                          small calls: route_kernel and prefill_plan_kernel
//   prefill_stage_kernel   the items (a shared expert's are the tokens in order, in front of the
//                          others), their tokens gathered into MFMA operand tiles (zero padded), and
//                          each group's sum for the zero points
//   prefill_tile_kernel<gate/up>  one workgroup per (item, four slices of 32 intermediate rows):
//                          per slice 64 pre-activations (32 gate, 32 up) x 64 tokens over all of
//                          H, h = silu(gate) * up written as operand tiles of a bf16 value and
//                          its bf16 remainder, plus the group sums of h
//   prefill_tile_kernel<down>     one workgroup per (item, four tiles of 64 output rows): those
//                          rows x 64 tokens over all of I, written to a per-slot fp32 buffer
//   prefill_combine_kernel y[t] = sum over the token's k assignments of weight x slot output, and
//                          over the shared experts of theirs
//
// No kernel adds into memory another workgroup writes: every output element has one owner, so
// the result does not depend on the order in which workgroups run.
//
// The tile kernel.  Each of its four waves owns one 64-row weight tile per k-step of 32 inputs
// (four row blocks of 16, one word of a lane's 16 bytes each) and all token blocks of the item.
// A code is unpacked once per workgroup, straight into the MFMA operand registers of the only
// wave that needs it; the token operand tiles are shared by the four waves and go from memory to
// LDS without passing through registers.  An operand tile read from LDS feeds four MFMAs: with two
// row blocks per wave the four SIMDs would ask LDS for 128 bytes a clock, all it delivers.
//
// Pipeline.  Operand tiles: stages of SK k-steps in four LDS buffers, requested three stages ahead,
// one barrier per stage.  Codes: a rolling window of eight k-steps in registers, refilled as it is
// consumed.  Every load is unconditional (past the end it repeats the last tile, and operand tiles
// of k-steps past the end are zeros): a load inside a branch makes the compiler wait for ALL loads in
// flight where the branch joins.  The four LDS buffers are four arrays on purpose: the compiler
// then knows which transfer a read of LDS depends on and does not wait for the later ones.
//
// Shared experts stay bf16 (section 3.4.2).  Their items run in the same launches, through a loop
// of the same form: a wave's 64 weight rows are four bf16 tiles per k-step instead of one tile of
// codes, which need no unpacking and no scales.  (As chunks of 16 tokens through the verify
// call's kernels, three launches each, they took 410 of the 605 us of a layer of the dsv2lite shape
// with 333 tokens.)
//
// The down part with groups of 128 (run_e4m3) runs on the 16x16x128 e4m3 products, which take a whole group at twice the rate: a
// code byte is an e4m3 number as it stands (three vector instructions per word of codes instead of eight), h is a sum of four e4m3
// planes with one power of two per token and group, which are as many operand bytes and as much time on the matrix cores as two bf16
// numbers, in half as many instructions, and hold more of h.  A product keeps the vector ALU waiting 22 of its 32 clocks (measured alone: clocks = 22 + 4 per
// vector instruction beside it, 32 at least), a bf16 product 15 of 16.  us of the down launch, two bf16 numbers / this: phi shape, 512 tokens 152 / 138, dsv2lite, 333 57.4 / 53.5;
// mixtral, 4096 1794 / 1727 (where the clock falls to 1.6 GHz: power); the cut into planes is nothing measurable of the gate/up launch.
// (x as two planes in the gate/up part, whose cut took 5, 6 and 16 us of the stage launch: 192 / 183, 71 / 70 and 2206 / 2091 us, but two planes do not hold every bf16 x, and
// with a third one where they do not it was no gain.)
//
// Arithmetic.  Codes become the exact bf16 integers 16 + q; a group's products are summed by the
// matrix cores (16x16x32 bf16, fp32 accumulate), starting at -24 (sum of the group's x), so that the sum
// is that of (q - 8) x, and enter the totals with one fused multiply-add by the group's scale.  What the
// zero points differ from 8 is one more contraction, over groups instead of inputs:
//   total = sum_G s_G acc_G + sum_G s_G (z_G - 8) / 24 (-24 x the sum of the group's x).
// Both factors of the second sum are fp32 numbers cut into three bf16 pieces (exactly; of the nine
// products of pieces all but the smallest are kept, 2^-30 of the term), eight k positions per
// group, so that it runs on the matrix cores as well: a sixteenth of the k-steps (g = 128) instead of
// a second multiply-add per group on the vector ALU, which the unpacking and the scales already load.
// It is added every four groups, so that the totals never hold more than four groups' share of it: added up
// behind the loop, and without the start at -24 sums, the totals of activations with a mean grew to 23.5 s
// times the sum of all x before they cancelled (x of mean 0.3 sigma, H = 4096, g = 32: error of y 4.0e-5; now
// 2.5e-6; h >= 0 over I = 8192: 1.1e-4, now 2.8e-6).  The start costs one LDS read per group and token block
// (mixtral shape, 4096 tokens: 2 % of the call).
//
// Bound and figures (gate/up and down kernel; first form: two row blocks per wave, operand tiles through
// registers, offset 128, two multiply-adds per group).  Many tokens per expert: the matrix cores.
// mixtral shape, 4096 tokens: 2221 and 1703 us (under the profiler; the whole call 3685, with h as two bf16 numbers, column by column 3741; the clock falls to 1.6 to 1.8 GHz)
// (first form: 3750 and 2933 us).  phi shape, 512 tokens:
// 182 and 127 us (406 and 261), the matrix cores busy 29 and 44 % of it and the vector ALU 46 and 28 %: between the two bounds, a
// wave waits for its turn at an instruction 38 % of its time and for data 19 %.  Few tokens per expert: the weight stream.
// dsv2lite shape, 333 tokens (31 per expert), with its shared experts in the same launches: 66 and 49 us for 219 and 110 MB (routed
// experts alone, first form: 99 and 66); matrix cores 23 and 31 %, waiting for data 22 and 28 %.
#include <hip/hip_runtime.h>
#include "draft_common.h"

namespace moespeq {

namespace {

constexpr int kItemTokens = 64;                   // slots of an item: four token blocks of 16
constexpr int kTileThreads = 256, kTileWaves = 4;
constexpr int kXcds = 8;
// The items, in segments: the shared experts' and full ones; then what is left of the experts' runs, by its token blocks of 16:
// four, three, two or one.  n_items: their count, then each segment's.  Where prefill_by_size does not choose this order, all
// items are in the first segment, expert by expert.
constexpr int kSegments = 4;
// Factor of a stored group sum: takes 16 + q (bf16 codes) or q (e4m3 codes) to q - 8
constexpr float kOffset = -24.f, kOffsetE4m3 = -8.f;

// Items of an expert in the first segment (lg: log2 of an item's tokens), and the segment of its last item (0: it has none elsewhere)
__device__ inline int head_items(int assignments, int lg, bool by_size) {
    return (assignments + (by_size ? 0 : (1 << lg) - 1)) >> lg;
}
__device__ inline int rest_segment(int assignments, int head, int lg) {
    const int left = assignments - (head << lg);
    return left <= 0 ? 0 : left > 48 ? 1 : left > 32 ? 2 : 3;
}

struct TileArgs {
    const char *q, *sz;              // int4 codes / scale(-zero) blobs of the routed experts
    size_t stride_q, stride_sz;
    const PrefillItem *items;
    const int32_t *n_items;          // [1 + segments]
    const char *act;                 // operand tiles of x, nk 4 KiB an item, or of h, twice that (layouts: below)
    const char *act_sums;            // group sums times the offset, fp32 [(item 4 nz + group) 64 + token]; nz = ceil(groups / 4)
    const char *act_scales;          // h, g = 128: a group's power of two, a byte each [((item nz + group / 4) 64 + token) 4 + group % 4]
    const char *zeros;               // 4 KiB of zeros
    char *h, *h_sums, *h_scales;     // gate/up: out, the same layouts over I
    float *obuf;                     // down: out [item 64 + token][H]
    const char *shared;              // bf16 blobs of the shared experts (experts E, E + 1, ...)
    size_t shared_stride;
    int H, I, E, segments, block;
    bool striped;
};

// The 8 codes of one word as 8 bf16 values 16 + code: 0x4180 is bf16 16.0, and a code in mantissa
// bits 3-6 adds itself (one unit there is 16 / 128).  The smaller offset costs one shift more than
// 128 + code and leaves 1/8 of its rounding error in the sums.
__device__ inline UnpackConsts unpack16_consts() {
    UnpackConsts k = {0x00780078u, 0x41804180u};
    asm volatile("" : "+s"(k.mask));
    asm volatile("" : "+v"(k.magic));
    return k;
}
__device__ inline bf16x8 unpack8_16(uint32_t w, UnpackConsts k) {
    u32x4 r;
    r.x = ((w << 3) & k.mask) | k.magic;
    r.y = ((w >> 1) & k.mask) | k.magic;
    r.z = ((w >> 5) & k.mask) | k.magic;
    r.w = ((w >> 9) & k.mask) | k.magic;
    return __builtin_bit_cast(bf16x8, r);
}

// ---- g = 128, down part: 16x16x128 products of e4m3 codes with h as e4m3 planes (draft_common.h), whose scale is a byte that
// the matrix cores apply
typedef __attribute__((ext_vector_type(8))) int i32x8;
// the scales of the code bytes (2^9) per plane, the plane's step in them
constexpr uint32_t kCodeScales = 136u | (136u - kPlaneShift) << 8 | (136u - 2 * kPlaneShift) << 16 | (136u - 3 * kPlaneShift) << 24;

__device__ inline float largest8(const float (&v)[8])
{
    float m = fabsf(v[0]);
#pragma unroll
    for (int j = 1; j < 8; ++j) m = fmaxf(m, fabsf(v[j]));
    return m;
}

// Eight h of a k-step (v, scaled; m: the largest of them) as planes; returns the sum of what the planes hold (scaled)
__device__ inline float split_planes(float (&v)[8], float m, uint32_t (&out)[kPlanes][2])
{
    const float grid = plane_grid(m);
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += v[j];
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
        const float up = (float)(1 << (p * kPlaneShift)), down = -1.f / up;
        float t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = p < 2 ? fmaf(v[j], up, grid) - grid : v[j] * up;
        int lo = __builtin_amdgcn_cvt_pk_fp8_f32(t[0], t[4], 0, false), hi = __builtin_amdgcn_cvt_pk_fp8_f32(t[2], t[6], 0, false);
        lo = __builtin_amdgcn_cvt_pk_fp8_f32(t[1], t[5], lo, true);
        hi = __builtin_amdgcn_cvt_pk_fp8_f32(t[3], t[7], hi, true);
        out[p][0] = (uint32_t)lo;
        out[p][1] = (uint32_t)hi;
        const auto a = __builtin_amdgcn_cvt_pk_f32_fp8(lo, false), b = __builtin_amdgcn_cvt_pk_f32_fp8(lo, true);
        const auto c = __builtin_amdgcn_cvt_pk_f32_fp8(hi, false), d = __builtin_amdgcn_cvt_pk_f32_fp8(hi, true);
        const float held[8] = {a[0], b[0], c[0], d[0], a[1], b[1], c[1], d[1]};
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = fmaf(held[j], down, v[j]);       // (exact)
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) sum -= v[j];
    return sum;
}

// the bytes of a scale word by which operands A and B are multiplied have to be constants of the instruction
template <int SA, int SB>
__device__ inline f32x4 mfma_e4m3(i32x8 a, i32x8 b, f32x4 c, uint32_t scale_a, uint32_t scale_b) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, SA, (int)scale_a, SB, (int)scale_b);
}

// f(0), f(1), .. f(N - 1) with constants
template <typename F, int... I>
__device__ __forceinline__ void each(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void each(F &&f) { each(f, std::make_integer_sequence<int, N>{}); }

// An fp32 value as three bf16 pieces (upper halves of p[0..2], exact), in the order in which the
// two factors of the group-sum contraction pair up over eight k positions:
//   factor:  a1 a1 a1 a2 a2 a3 a2 a3      sum:  b1 b2 b3 b1 b2 b1 b3 b2
__device__ inline void three_pieces(float v, uint32_t p[3]) {
    p[0] = __float_as_uint(v) & 0xffff0000u;
    const float r1 = v - __uint_as_float(p[0]);
    p[1] = __float_as_uint(r1) & 0xffff0000u;
    p[2] = __float_as_uint(r1 - __uint_as_float(p[1])) & 0xffff0000u;
}
__device__ inline u32x4 factor_operand(float v) {
    uint32_t p[3];
    three_pieces(v, p);
    const uint32_t a3a2 = p[2] | (p[1] >> 16);
    return (u32x4){p[0] | (p[0] >> 16), p[1] | (p[0] >> 16), a3a2, a3a2};
}
__device__ inline u32x4 sum_operand(float v) {
    uint32_t p[3];
    three_pieces(v, p);
    return (u32x4){p[1] | (p[0] >> 16), p[0] | (p[2] >> 16), p[0] | (p[1] >> 16), p[1] | (p[2] >> 16)};
}

// scale / zero entries of the four row blocks of one lane row and group
template <bool SYM> struct Entry;
template <> struct Entry<false> {
    u32x4 w;
    __device__ static Entry load(const char *p) { return {*reinterpret_cast<const u32x4 *>(p)}; }
    __device__ float scale(int d) const { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w[d] & 0xffff)); }
    __device__ float zero(int d) const { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w[d] >> 16)); }
};
template <> struct Entry<true> {
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
    u32x2 w;
    __device__ static Entry load(const char *p) { return {*reinterpret_cast<const u32x2 *>(p)}; }
    __device__ float scale(int d) const { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w[d >> 1] >> (16 * (d & 1)))); }
};

typedef __attribute__((address_space(3))) void *lvoid;

template <bool DOWN, bool SYM, int KPG>            // KPG: k-steps per group (g / 32)
__global__ __launch_bounds__(kTileThreads, 2)
void prefill_tile_kernel(TileArgs a)
{
    constexpr int NP = DOWN ? 2 : 1;               // operand planes (h and its remainder)
    constexpr int SK = DOWN ? 2 : 4;               // k-steps per stage
    constexpr int kWin = 8;                        // k-steps of codes in flight
    constexpr int kZeroStages = 4 * KPG / SK;      // stages per four groups
    constexpr int kSums = SK * NP * 4 * 1024;      // one stage of operand tiles, then the sums of the groups that begin in it
    constexpr int kBuf = kSums + 1024;
    constexpr int kRow = 36;                       // of h in LDS: 32 columns and 16 bytes against bank conflicts
    __shared__ __align__(1024) unsigned char s_x0[kBuf];
    __shared__ __align__(1024) unsigned char s_x1[kBuf];
    __shared__ __align__(1024) unsigned char s_x2[kBuf];
    __shared__ __align__(1024) unsigned char s_x3[kBuf];

    const int H = a.H, I = a.I;
    const int nk = DOWN ? I / 32 : H / 32, G = nk / KPG, nz = (G + 3) / 4;
    const int tiles = DOWN ? H / 64 : I / 32, cols = (tiles + kTileWaves - 1) / kTileWaves;
    // Workgroups go to the XCDs in turn.  The item list is in segments of falling size (the smallest workgroups come last); a segment's
    // (item, column) pairs are in blocks of `block` items, column by column in a block, so that the items of one expert, neighbours in the list, read
    // its weight tiles, and the columns of an item its operand tiles, through one L2 at about the same time.  XCD x takes the x-th contiguous eighth of a segment's
    // pairs, or (striped) of every block's, where an eighth of the segment would leave an XCD too few experts.  prefill_blocks says which.
    int n[kSegments];                                                    // (all counts by one load)
#pragma unroll
    for (int seg = 0; seg < kSegments; ++seg) n[seg] = a.n_items[1 + seg];
    const int xcd = (int)blockIdx.x % kXcds, block = a.block, of_block = (cols * block + kXcds - 1) / kXcds;      // pairs of a whole block that an XCD takes
    int at = (int)blockIdx.x / kXcds, seg_items = n[0], first_item = 0;
    auto per_xcd = [&](int items) {
        const int whole = a.striped ? items / block : 0;
        return whole * of_block + (cols * (items - whole * block) + kXcds - 1) / kXcds;
    };
    int per = per_xcd(seg_items);
    if (a.segments > 1) {                                                // (without: H = 512, 201 tokens 50.7 / 50.0 us)
#pragma unroll
        for (int seg = 1; seg < kSegments; ++seg) {
            const bool past = at >= per;
            at -= past ? per : 0;
            first_item += past ? seg_items : 0;
            seg_items = past ? n[seg] : seg_items;
            per = per_xcd(seg_items);
        }
    }
    if (at >= per) return;
    int blk, in_blk, end = cols * block;                                 // which block of the segment; which pair of it, below `end`
    if (a.striped) {
        blk = at / of_block;
        const int left = seg_items - blk * block, share = left < block ? (cols * left + kXcds - 1) / kXcds : of_block;
        // (in turn, since the last share of a block is the smallest)
        const int eighth = (xcd + blk) % kXcds;
        in_blk = eighth * share + at - blk * of_block;
        end = (eighth + 1) * share;
    } else {
        blk = (xcd * per + at) / (cols * block);
        in_blk = xcd * per + at - blk * cols * block;
    }
    const int left = seg_items - blk * block, wide = left < block ? left : block;
    if (left <= 0 || in_blk >= end || in_blk >= cols * wide) return;
    const int col = in_blk / wide, item = first_item + blk * block + in_blk - col * wide;
    const PrefillItem it = a.items[item];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, c = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const UnpackConsts uk = unpack16_consts();
    const bool mine = col * kTileWaves + wave < tiles;               // a wave past the end repeats the last tile
    const int tile = mine ? col * kTileWaves + wave : tiles - 1;

    const bool routed = it.expert < a.E;
    const char *wq = a.q + (size_t)it.expert * a.stride_q +
                     (DOWN ? (size_t)(I / 32) * (H / 32) * 1024 + (size_t)tile * 1024 : (size_t)tile * (H / 32) * 1024);
    const size_t wstep = DOWN ? (size_t)(H / 64) * 1024 : 1024;
    auto load_codes = [&](int k) {
        const char *p = wq + (size_t)(k < nk ? k : nk - 1) * wstep;
        return *reinterpret_cast<const u32x4 *>(p + lane * 16);
    };
    // symmetric format: 8-byte halves of the 16-byte units (two groups, or two row tiles)
    const char *szb = a.sz + (size_t)it.expert * a.stride_sz +
                      (DOWN ? (size_t)(I / 32) * (H / (32 * KPG)) * (SYM ? 128 : 256) : 0);
    auto entry_at = [&](int grp) {
        const int gi = grp < G ? grp : G - 1;
        size_t off;
        if constexpr (!SYM) off = (DOWN ? (size_t)gi * (H / 64) + tile : (size_t)tile * G + gi) * 256 + r * 16;
        else if constexpr (DOWN) off = ((size_t)gi * (H / 128) + tile / 2) * 256 + r * 16 + (tile % 2) * 8;
        else off = ((size_t)tile * (G / 2) + gi / 2) * 256 + r * 16 + (gi % 2) * 8;
        return Entry<SYM>::load(szb + off);
    };
    auto buffer = [&](auto j) -> unsigned char * {
        if constexpr (decltype(j)::value == 0) return s_x0;
        else if constexpr (decltype(j)::value == 1) return s_x1;
        else if constexpr (decltype(j)::value == 2) return s_x2;
        else return s_x3;
    };
    const int my_k = DOWN ? wave >> 1 : wave;                        // the k-step (and plane) of a stage this wave requests
    const char *tiles_of_item = a.act + (size_t)(DOWN ? 2 * item : it.src) * nk * 4096;
    const char *act = tiles_of_item + (DOWN && (wave & 1) ? (size_t)nk * 4096 : 0);       // bf16: [k-step][tb], h and then its remainder

    // this wave's operand tiles of stage n into buffer j
    auto request = [&](int n, auto j, auto ntb_c) {
        const int k = n * SK + my_k;
        // (chosen with a mask: a branch here would cut the stage into several scheduling regions)
        const char *from = act + (size_t)k * 4096;
        const char *src = a.zeros + ((from - a.zeros) & (k < nk ? ~(ptrdiff_t)0 : (ptrdiff_t)0));
        // Buffer loads, not global ones: after a FLAT-encoded load to LDS the compiler waits for ALL LDS
        // reads in flight wherever it needs one.
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, 4096, 0x00027000);
        unsigned char *dst = buffer(j) + wave * 4096;
#pragma unroll
        for (int tb = 0; tb < decltype(ntb_c)::value; ++tb)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lvoid)(dst + tb * 1024), 16, lane * 16, tb * 1024, 0, 0);
    };
    // the sums of the groups that begin in stage n into buffer j (the waves share them out, or repeat them)
    constexpr int kBegin = SK > KPG ? SK / KPG : 1;
    auto request_sums = [&](int n, auto j) {
        const int grp = n * SK / KPG + wave % kBegin;
        const char *src = a.act_sums + ((size_t)item * nz * 4 + (grp < 4 * nz ? grp : 4 * nz - 1)) * 256;
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, 256, 0x00027000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lvoid)(buffer(j) + kSums + wave % kBegin * 256), 4, lane * 4, 0, 0, 0);
    };
    // The start of a stage: its operand tiles are in their buffer once this wave's own transfers have landed
    // and the workgroup has met.  Issued behind those transfers (vector memory operations complete in
    // order): the weights of three stages, and the transfers of two (and some entries and sums, not counted).
    auto begin_stage = [&](auto ntb_c, auto stage_loads) {
        constexpr int kLater = 3 * decltype(stage_loads)::value + 2 * decltype(ntb_c)::value;
        static_assert(kLater < 64, "vmcnt");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt((kLater & 15) | ((kLater >> 4) << 14) | 0x0f70);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    const int ns = (nk + SK - 1) / SK;
    constexpr std::integral_constant<int, 0> k0{};
    constexpr std::integral_constant<int, 1> k1{};
    constexpr std::integral_constant<int, 2> k2{};
    constexpr std::integral_constant<int, 3> k3{};

    // h of a routed item, g = 128: the workgroup's 128 columns are a group, this wave's 32 its k-step `wave`.  s_h: [token][column]
    auto finish_e4m3 = [&](auto ntb_c, const float *s_h) {
        constexpr int NTB = decltype(ntb_c)::value;
        float (*s_max)[kItemTokens] = reinterpret_cast<float (*)[kItemTokens]>(s_x1 + kSums);
        float (*s_sum)[kItemTokens] = reinterpret_cast<float (*)[kItemTokens]>(s_x0 + kSums);
        auto load = [&](int tb, float (&h)[8]) {                  // token r of the block, columns 8 c ..
            const f32x4 h0 = *reinterpret_cast<const f32x4 *>(&s_h[(16 * tb + r) * kRow + 8 * c]);
            const f32x4 h1 = *reinterpret_cast<const f32x4 *>(&s_h[(16 * tb + r) * kRow + 8 * c + 4]);
#pragma unroll
            for (int j = 0; j < 4; ++j) { h[j] = h0[j]; h[j + 4] = h1[j]; }
        };
        float m8[NTB];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
            float h[8];
            load(tb, h);
            m8[tb] = largest8(h);
            float m = fmaxf(m8[tb], __shfl_xor(m8[tb], 16));
            m = fmaxf(m, __shfl_xor(m, 32));
            if (c == 0) s_max[wave][16 * tb + r] = m;
        }
        __syncthreads();
        const int GI = I / 128;
        char *out = a.h + ((size_t)item * GI + col) * 32768 + (wave >> 1) * 1024 + lane * 16 + (wave & 1) * 8;
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
            float h[8];
            load(tb, h);
            const int tok = 16 * tb + r;
            const PlaneScale gs(fmaxf(fmaxf(s_max[0][tok], s_max[1][tok]), fmaxf(s_max[2][tok], s_max[3][tok])));
            const float up = gs.up();
#pragma unroll
            for (int j = 0; j < 8; ++j) h[j] *= up;
            uint32_t planes[4][2];
            float sum = split_planes(h, m8[tb] * up, planes) * gs.down();
#pragma unroll
            for (int p = 0; p < 4; ++p)
                *reinterpret_cast<uint2 *>(out + tb * 8192 + p * 2048) = make_uint2(planes[p][0], planes[p][1]);
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            if (c == 0) {
                s_sum[wave][tok] = sum;
                if (wave == 0) a.h_scales[(((size_t)item * ((GI + 3) / 4) + col / 4) * kItemTokens + tok) * 4 + col % 4] = (char)gs.byte;
            }
        }
        __syncthreads();
        // the group's sums; the last column of workgroups also clears what is left of the last tile of four groups
        const int tok = tid & 63, gi = col + (tid >> 6);
        const bool pad = gi >= GI && gi / 4 == (GI - 1) / 4;
        if (tok < 16 * NTB && (gi == col || pad)) {
            const float v = gi == col ? (s_sum[0][tok] + s_sum[1][tok]) + (s_sum[2][tok] + s_sum[3][tok]) : 0.f;
            reinterpret_cast<float *>(a.h_sums)[((size_t)item * ((GI + 3) / 4) * 4 + gi) * kItemTokens + tok] = kOffsetE4m3 * v;
        }
    };

    // The results of an item: lane (r, c) holds, per row block d and token block, row 16 d + r of tokens
    // 4 c + i.
    auto finish = [&](auto ntb_c, auto &tot) {
        constexpr int NTB = decltype(ntb_c)::value;
        if constexpr (DOWN) {
            if (!mine) return;
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int tok = 16 * tb + 4 * c + i;
                    if (tok < it.cnt) {
                        float *o = a.obuf + ((size_t)item * kItemTokens + tok) * H + 64 * tile + r;
#pragma unroll
                        for (int d = 0; d < 4; ++d) o[16 * d] = tot[d][tb][i];
                    }
                }
        } else {
            // h of 16 tokens x 32 columns through this wave's own LDS area: lane (token, chunk) then
            // holds h of columns 8 chunk .. 8 chunk + 7, the operand layout
            __builtin_amdgcn_s_waitcnt(0x0f70);                       // transfers requested past the end
            __syncthreads();
            float (*s_hsum)[kItemTokens] = reinterpret_cast<float (*)[kItemTokens]>(s_x0 + kSums);
            float *s_h = reinterpret_cast<float *>(wave == 0 ? s_x0 : wave == 1 ? s_x1 : wave == 2 ? s_x2 : s_x3);
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) {
#pragma unroll
                for (int dd = 0; dd < 2; ++dd)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float gate = tot[dd][tb][i], up = tot[dd + 2][tb][i];
                        s_h[(16 * tb + 4 * c + i) * kRow + 16 * dd + r] = gate / (1.f + expf(-gate)) * up;
                    }
            }
            __builtin_amdgcn_wave_barrier();
            if (KPG == 4 && routed) { finish_e4m3(ntb_c, s_h); return; }
            char *h_of_item = a.h + (size_t)item * (I / 32) * 8192 + (size_t)tile * 4096;
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) {
                const f32x4 h0 = *reinterpret_cast<const f32x4 *>(&s_h[(16 * tb + r) * kRow + 8 * c]);
                const f32x4 h1 = *reinterpret_cast<const f32x4 *>(&s_h[(16 * tb + r) * kRow + 8 * c + 4]);
                uint32_t hi[4], lo[4];
                float sum = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float h = j < 4 ? h0[j & 3] : h1[j & 3];
                    const uint32_t hb = f32_to_bf16_rne(h);
                    const uint32_t lb = f32_to_bf16_rne(h - __uint_as_float(hb << 16));
                    sum += __uint_as_float(hb << 16) + __uint_as_float(lb << 16);
                    if (j & 1) { hi[j >> 1] |= hb << 16; lo[j >> 1] |= lb << 16; }
                    else { hi[j >> 1] = hb; lo[j >> 1] = lb; }
                }
                if (mine) {
                    char *t = h_of_item + tb * 1024 + lane * 16;
                    *reinterpret_cast<u32x4 *>(t) = (u32x4){hi[0], hi[1], hi[2], hi[3]};
                    *reinterpret_cast<u32x4 *>(t + (size_t)(I / 32) * 4096) = (u32x4){lo[0], lo[1], lo[2], lo[3]};
                }
                sum += __shfl_xor(sum, 16);
                sum += __shfl_xor(sum, 32);
                if (c == 0) s_hsum[wave][16 * tb + r] = sum;
            }
            __syncthreads();
            if (!routed) return;
            // group sums of h: the workgroup's 128 columns hold 4 / KPG whole groups; the last column of
            // workgroups also clears what is left of the last tile of four groups
            const int tok = tid & 63, pos = tid >> 6;
            const int GI = I / (32 * KPG), gi = col * (4 / KPG) + pos;
            const bool real = pos < 4 / KPG && gi < GI;
            const bool pad = gi >= GI && gi / 4 == (GI - 1) / 4 && col == cols - 1;
            if (tok < 16 * NTB && (real || pad)) {
                float v = 0.f;
                if (real) {
#pragma unroll
                    for (int w = 0; w < KPG; ++w) v += s_hsum[(pos * KPG + w) & 3][tok];
                }
                reinterpret_cast<float *>(a.h_sums)[((size_t)item * ((GI + 3) / 4) * 4 + gi) * kItemTokens + tok] = kOffset * v;
            }
        }
    };

    // an item of a routed expert with NTB token blocks (a compile-time count: no branch inside a stage)
    auto run = [&](auto ntb_c) {
        constexpr int NTB = decltype(ntb_c)::value;
        constexpr int EW = KPG == 1 || (KPG == 2 && NTB < 4) ? 4 : 2;     // groups of entries in flight (four more spill)
        f32x4 tot[4][NTB], acc[4][NTB];
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) tot[d][tb] = acc[d][tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
        u32x4 win[kWin];                           // codes of k-steps k .. k + 7, slot k % 8
        bf16x8 wb[2][4];                           // operands of k-step k and, as it is unpacked, k + 1
        Entry<SYM> ent[EW];
        float sc[4] = {0.f, 0.f, 0.f, 0.f};        // scales of the group that ended last
        // The zero points of four groups: lane group c keeps the entries and the sums of the c-th.
        // (past the tile's last group its entries are read again: the sums there are zeros)
        Entry<SYM> ze;
        float zs[NTB];
        const uint32_t zstep = DOWN ? (uint32_t)(H / 64) * 256 : 256;
        const char *z_run = szb + (size_t)tile * (DOWN ? 1 : G) * 256, *s_run = a.act_sums + (size_t)item * nz * 1024;
        auto load_zeros = [&](int q) {
            if constexpr (!SYM) {
                const uint32_t grp = 4 * q + c, off = (grp < (uint32_t)G ? grp : G - 1) * zstep + r * 16;
                ze.w = *reinterpret_cast<const u32x4 *>(z_run + off);
                const char *sums = s_run + (size_t)(q < nz ? q : nz - 1) * 1024;
#pragma unroll
                for (int tb = 0; tb < NTB; ++tb)
                    zs[tb] = *reinterpret_cast<const float *>(sums + (uint32_t)((c * kItemTokens + r) * 4) + tb * 64);
            }
        };
        auto add_scaled_rows = [&](int d, int tb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) tot[d][tb][i] = fmaf(sc[d], acc[d][tb][i], tot[d][tb][i]);
            asm volatile("" : "+v"(tot[d][tb]));       // here and not further down, or acc could not be used again
        };
        auto add_scaled = [&](int tb) {
#pragma unroll
            for (int d = 0; d < 4; ++d) add_scaled_rows(d, tb);
        };
        // The last token block's share of the group before is added here, in front of its zero points, as the other blocks'
        // was: a token's sums are the same bits in every block of an item.
        auto add_zeros = [&]() {
            if constexpr (!SYM) {
                bf16x8 zx[NTB];
#pragma unroll
                for (int tb = 0; tb < NTB; ++tb) zx[tb] = __builtin_bit_cast(bf16x8, sum_operand(zs[tb]));
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const bf16x8 f = __builtin_bit_cast(bf16x8, factor_operand(ze.scale(d) * ((ze.zero(d) - 8.f) * (-1.f / kOffset))));
                    add_scaled_rows(d, NTB - 1);
#pragma unroll
                    for (int tb = 0; tb < NTB; ++tb)
                        tot[d][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zx[tb], f, tot[d][tb], 0, 0, 0);
                }
            }
        };

        // One stage: the buffer that everybody has left takes the operand tiles three stages further on.
        // The stage is a row of blocks, one per operand tile: the LDS read three tiles ahead, a share of
        // the next k-step's unpacking, the scaling of the token block before (its products are complete
        // by then), and the tile's four MFMAs, so that the vector ALU and LDS work under the matrix
        // cores.  The barriers between blocks keep the scheduler from gathering all reads of a stage in
        // front, for which there are no registers.
        auto stage = [&](int n, auto j) {
            constexpr int J = decltype(j)::value;
            constexpr int kFirst = J * SK;         // position in the four stages of a loop trip
            constexpr int NB = NTB * NP, F = SK * NB, kA = 4;
            begin_stage(ntb_c, std::integral_constant<int, SK>{});
            const unsigned char *buf = buffer(j);
            u32x4 xa[kA];
            constexpr int kF = 2;                  // (three spill with g = 64)
            f32x4 from[kF];                        // where the products of a group start
            auto read = [&](int f) {               // tile f of the stage: k-step, token block, plane
                const int s = f / NB, tb = f % NB / NP, p = f % NP;
                xa[f % kA] = *reinterpret_cast<const u32x4 *>(&buf[((s * NP + p) * 4 + tb) * 1024 + lane * 16]);
            };
            auto read_sums = [&](int f) {
                const int s = f / NB, tb = f % NB / NP, p = f % NP;
                if ((kFirst + s) % KPG == 0 && p == 0)
                    from[f % kF] = *reinterpret_cast<const f32x4 *>(&buf[kSums + (s / KPG) * 256 + (16 * tb + 4 * c) * 4]);
            };
#pragma unroll
            for (int f = 0; f < kA - 1 && f < F; ++f) {
                read(f);
                if (f < kF - 1) read_sums(f);
            }
            request(n + 3, std::integral_constant<int, (J + 3) & 3>{}, ntb_c);
            if constexpr ((J + 3) * SK % KPG == 0) request_sums(n + 3, std::integral_constant<int, (J + 3) & 3>{});
            constexpr bool kZeros = !SYM && J % kZeroStages == 0;
            if constexpr (kZeros) {
                add_zeros();
                load_zeros(n / kZeroStages + 1);
            }
#pragma unroll
            for (int f = 0; f < F; ++f) {
                const int s = f / NB, t = f % NB, tb = t / NP, p = t % NP;
                const int pos = kFirst + s;
                const bool begins = pos % KPG == 0, ends = (pos + 1) % KPG == 0;      // of a group
                __builtin_amdgcn_sched_barrier(0);
                if (f + kA - 1 < F) read(f + kA - 1);
                if (f + kF - 1 < F) read_sums(f + kF - 1);
                if (begins && t == 0 && !(kZeros && s == 0)) add_scaled(NTB - 1);     // of the group before
                if (ends && t == 0) {
                    constexpr int kGroups = 4 * SK / KPG;
                    static_assert(kGroups % EW == 0, "the slot of a group has to be the same in every loop trip");
                    const int slot = (pos / KPG) % EW;
#pragma unroll
                    for (int d = 0; d < 4; ++d) sc[d] = ent[slot].scale(d);
                    ent[slot] = entry_at((n * SK + s) / KPG + EW);
                }
                const int nx = (pos + 1) % kWin;
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    if (d * NB / 4 == t) wb[(s + 1) & 1][d] = unpack8_16(win[nx][d], uk);
                if (t == NB - 1) win[nx] = load_codes(n * SK + s + 1 + kWin);
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    acc[d][tb] = mfma(xa[f % kA], wb[s & 1][d], begins && p == 0 ? from[f % kF] : acc[d][tb]);
                if (ends && p == 0 && tb > 0) add_scaled(tb - 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        request(0, k0, ntb_c);
        request_sums(0, k0);
        request(1, k1, ntb_c);
        if constexpr (SK % KPG == 0) request_sums(1, k1);
        request(2, k2, ntb_c);
        request_sums(2, k2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kWin; ++i) win[i] = load_codes(i);
#pragma unroll
        for (int i = 0; i < EW; ++i) ent[i] = entry_at(i);
        load_zeros(0);
        // the first stages' transfers have fewer operations behind them than the steady state counts on
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0070);
#pragma unroll
        for (int d = 0; d < 4; ++d) wb[0][d] = unpack8_16(win[0][d], uk);
        win[0] = load_codes(kWin);
        for (int n = 0; ; n += 4) {                // exits between the stages, for few k-steps (H = 256: gate/up 9.1 -> 7.6 us)
            stage(n, k0);
            if (n + 1 >= ns) break;
            stage(n + 1, k1);
            if (n + 2 >= ns) break;
            stage(n + 2, k2);
            if (n + 3 >= ns) break;
            stage(n + 3, k3);
            if (n + 4 >= ns) break;
        }
        // every last stage ends a group (k-steps past the end are zeros)
        add_scaled(NTB - 1);
        finish(ntb_c, tot);
    };

    // an item of a routed expert, down part, g = 128, on 16x16x128 products of e4m3 operands: one product per plane, row block and token block takes a
    // whole group.  A stage is NTB x 4 KiB of operand tiles, half of a group of h (in order: token block, plane, halves of a lane's 32 bytes).
    auto run_e4m3 = [&](auto ntb_c) {
        constexpr int NTB = decltype(ntb_c)::value, NPL = kPlanes;
        constexpr int SPG = 2;                     // stages per group
        constexpr int FS = 2 * NTB;                // operand tiles of 2 KiB per stage
        constexpr int W = 2;                       // groups of codes in flight
        f32x4 tot[4][NTB], acc[2][4];              // acc: products of a token block, and of the one before until they are scaled
        u32x4 win[4 * W];                          // codes: group n's in slots 4 (n % W) ..
        i32x8 wb[4];                               // operands of the group's row blocks
        Entry<SYM> ent[2], ze;
        float sc[4] = {0.f, 0.f, 0.f, 0.f}, zs[NTB];
        uint32_t ts[NTB], tn[NTB];                 // scales of the tokens' groups, a byte each: this four, the next
        uint32_t mask = 0x0f0f0f0fu, code_scales = kCodeScales;
        asm volatile("" : "+s"(mask));
        asm volatile("" : "+v"(code_scales));
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            acc[0][d] = acc[1][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) tot[d][tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
        const int stages = G * SPG;
        const char *scales = a.act_scales + (size_t)item * nz * 256, *s_run = a.act_sums + (size_t)item * nz * 1024;
        const char *z_run = szb + (size_t)tile * 256;
        const uint32_t zstep = (uint32_t)(H / 64) * 256;
        auto request_stage = [&](int n, auto j) {
            const int in = n < stages ? n : stages - 1;
            const char *src = tiles_of_item + (size_t)(in / SPG) * (SPG * 16384) + (in % SPG) * (NTB * 4096) + wave * (NTB * 1024);
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, NTB * 1024, 0x00027000);
            unsigned char *dst = buffer(j) + wave * (NTB * 1024);
#pragma unroll
            for (int i = 0; i < NTB; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lvoid)(dst + i * 1024), 16, lane * 16, i * 1024, 0, 0);
            const auto sums = __builtin_amdgcn_make_buffer_rsrc((void *)(s_run + (size_t)(in / SPG) * 256), 0, 256, 0x00027000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(sums, (lvoid)(buffer(j) + kSums), 4, lane * 4, 0, 0, 0);
        };
        // scales, and entries and sums of the zero points, of the q-th four groups (past the last: of the last again, the sums there are zeros)
        auto load_four = [&](int q) {
            const int in = q < nz ? q : nz - 1;
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) tn[tb] = *reinterpret_cast<const uint32_t *>(scales + in * 256 + (uint32_t)(r * 4) + tb * 64);
            if constexpr (!SYM) {
                const uint32_t grp = 4 * q + c, off = (grp < (uint32_t)G ? grp : G - 1) * zstep + r * 16;
                ze.w = *reinterpret_cast<const u32x4 *>(z_run + off);
#pragma unroll
                for (int tb = 0; tb < NTB; ++tb)
                    zs[tb] = *reinterpret_cast<const float *>(s_run + (size_t)in * 1024 + (uint32_t)((c * kItemTokens + r) * 4) + tb * 64);
            }
        };
        auto add_scaled_rows = [&](int d, int tb, const f32x4 &v) {
#pragma unroll
            for (int i = 0; i < 4; ++i) tot[d][tb][i] = fmaf(sc[d], v[i], tot[d][tb][i]);
            asm volatile("" : "+v"(tot[d][tb]));
        };
        auto unpack = [&](int slot, int d) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                uint32_t lo, hi;
                unpack8_e4m3(win[slot * 4 + s][d], mask, lo, hi);
                wb[d][2 * s] = (int)lo;
                wb[d][2 * s + 1] = (int)hi;
            }
            asm volatile("" : "+v"(wb[d]));
        };
        auto stage = [&](int grp, auto j) {        // j: stage of a trip of four groups
            constexpr int J = decltype(j)::value, Q = J / SPG, HALF = J % SPG;
            constexpr int B0 = J & 3;
            // issued behind the transfers that this stage needs: those of two stages (NTB + 1 each), and four loads of codes at the end
            // and one of entries at the start of each group
            constexpr int kLater = 2 * (NTB + 1) + (HALF == 0 ? 9 : 6);
            static_assert(kLater < 64, "vmcnt");
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt((kLater & 15) | ((kLater >> 4) << 14) | 0x0f70);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            const unsigned char *buf = buffer(std::integral_constant<int, B0>{});
            constexpr int kA = 3;
            u32x4 xa[kA][2];
            f32x4 from[2];
            auto read = [&](int fs) {
                xa[fs % kA][0] = *reinterpret_cast<const u32x4 *>(&buf[fs * 2048 + lane * 16]);
                xa[fs % kA][1] = *reinterpret_cast<const u32x4 *>(&buf[fs * 2048 + 1024 + lane * 16]);
            };
            auto read_sums = [&](int tb) { from[tb & 1] = *reinterpret_cast<const f32x4 *>(&buf[kSums + (16 * tb + 4 * c) * 4]); };
            constexpr int F0 = HALF * FS;          // tile of the group with which the stage begins
            read(0);
            if (F0 % NPL == 0) read_sums(F0 / NPL);
            read(1);
            request_stage(grp * SPG + HALF + 3, std::integral_constant<int, (B0 + 3) & 3>{});
            if constexpr (J == 0) {
                // the last token block's share of the group before comes in front of the zero points, as the other blocks' did: a token's
                // sums are the same bits in every block of an item
                if constexpr (!SYM) {
                    bf16x8 zx[NTB];
#pragma unroll
                    for (int tb = 0; tb < NTB; ++tb) zx[tb] = __builtin_bit_cast(bf16x8, sum_operand(zs[tb]));
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const bf16x8 f = __builtin_bit_cast(bf16x8, factor_operand(ze.scale(d) * ((ze.zero(d) - 8.f) * (-1.f / kOffsetE4m3))));
                        add_scaled_rows(d, NTB - 1, acc[1][d]);
#pragma unroll
                        for (int tb = 0; tb < NTB; ++tb)
                            tot[d][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zx[tb], f, tot[d][tb], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int tb = 0; tb < NTB; ++tb) ts[tb] = tn[tb];
                load_four(grp / 4 + 1);
            }
            each<FS>([&](auto fc) {
                constexpr int fs = decltype(fc)::value, f = F0 + fs, tb = f / NPL, p = f % NPL;
                constexpr int A = (Q * NTB + tb) & 1;      // of acc, token blocks in turn (4 NTB of them in a trip)
                __builtin_amdgcn_sched_barrier(0);
                if (fs + 2 < FS) read(fs + 2);
                if (fs + 1 < FS && (f + 1) % NPL == 0) read_sums(tb + 1);
                const i32x8 x8 = __builtin_bit_cast(i32x8, xa[fs % kA]);
                const bool before = p == 1 && (tb > 0 || SYM || J != 0);
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    acc[A][d] = mfma_e4m3<Q, p>(x8, wb[d], p == 0 ? from[tb & 1] : acc[A][d], ts[tb], code_scales);
                    if (before) add_scaled_rows(d, tb > 0 ? tb - 1 : NTB - 1, acc[A ^ 1][d]);
                    if (f == NTB * NPL - 1) unpack((Q + 1) % W, d);
                }
                if (f == 1) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) sc[d] = ent[Q % 2].scale(d);
                    ent[Q % 2] = entry_at(grp + 2);
                }
                if (f == NTB * NPL - 1) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int s = 0; s < 4; ++s) win[(Q + 1) % W * 4 + s] = load_codes(4 * (grp + 1 + W) + s);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        request_stage(0, k0);
        request_stage(1, k1);
        request_stage(2, k2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < W; ++g)
#pragma unroll
            for (int s = 0; s < 4; ++s) win[g * 4 + s] = load_codes(4 * g + s);
        ent[0] = entry_at(0);
        ent[1] = entry_at(1);
        load_four(0);
        // the first stages' transfers have fewer operations behind them than the steady state counts on
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0070);
#pragma unroll
        for (int d = 0; d < 4; ++d) unpack(0, d);
#pragma unroll
        for (int s = 0; s < 4; ++s) win[s] = load_codes(4 * W + s);
        auto group = [&](int grp, auto q) {
            constexpr int Q = decltype(q)::value;
            stage(grp, std::integral_constant<int, Q * SPG>{});
            stage(grp, std::integral_constant<int, Q * SPG + 1>{});
        };
        for (int grp = 0; ; grp += 4) {
            group(grp, k0);
            if (grp + 1 >= G) break;
            group(grp + 1, k1);
            if (grp + 2 >= G) break;
            group(grp + 2, k2);
            if (grp + 3 >= G) break;
            group(grp + 3, k3);
            if (grp + 4 >= G) break;
        }
        // (the last group's place in a trip says which half of acc holds its last token block)
        const bool odd = NTB % 2 == 1 && (G & 1);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            f32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = odd ? acc[0][d][i] : acc[1][d][i];
            add_scaled_rows(d, NTB - 1, v);
        }
        finish(ntb_c, tot);
    };

    // an item of a shared expert: the same loop over bf16 weight tiles
    auto run_shared = [&](auto ntb_c) {
        constexpr int NTB = decltype(ntb_c)::value;
        constexpr int kWinS = 4;                   // k-steps of weights in flight
        // row block d: gate or up rows 32 tile + 16 (d % 2) .., or output rows 64 tile + 16 d ..
        const char *blob = a.shared + (size_t)(it.expert - a.E) * a.shared_stride;
        const char *rows[4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
            rows[d] = DOWN ? blob + (size_t)I * H * 4 + (size_t)(4 * tile + d) * nk * 1024
                           : blob + (size_t)(d / 2) * I * H * 2 + (size_t)(2 * tile + d % 2) * nk * 1024;
        auto load_weights = [&](int k, int d) {
            return *reinterpret_cast<const u32x4 *>(rows[d] + (size_t)(k < nk ? k : nk - 1) * 1024 + lane * 16);
        };
        f32x4 acc[4][NTB];
        u32x4 win[kWinS][4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) acc[d][tb] = (f32x4){0.f, 0.f, 0.f, 0.f};
        auto stage = [&](int n, auto j) {
            constexpr int J = decltype(j)::value;
            constexpr int kFirst = J * SK;
            constexpr int NB = NTB * NP, F = SK * NB, kA = 4;
            begin_stage(ntb_c, std::integral_constant<int, 4 * SK>{});
            const unsigned char *buf = buffer(j);
            u32x4 xa[kA];
            auto read = [&](int f) {
                const int s = f / NB, tb = f % NB / NP, p = f % NP;
                xa[f % kA] = *reinterpret_cast<const u32x4 *>(&buf[((s * NP + p) * 4 + tb) * 1024 + lane * 16]);
            };
#pragma unroll
            for (int f = 0; f < kA - 1 && f < F; ++f) read(f);
            request(n + 3, std::integral_constant<int, (J + 3) & 3>{}, ntb_c);
#pragma unroll
            for (int f = 0; f < F; ++f) {
                const int s = f / NB, t = f % NB, tb = t / NP;
                const int slot = (kFirst + s) % kWinS;
                __builtin_amdgcn_sched_barrier(0);
                if (f + kA - 1 < F) read(f + kA - 1);
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    acc[d][tb] = mfma(xa[f % kA], __builtin_bit_cast(bf16x8, win[slot][d]), acc[d][tb]);
                if (t == NB - 1) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) win[slot][d] = load_weights(n * SK + s + kWinS, d);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        request(0, k0, ntb_c);
        request(1, k1, ntb_c);
        request(2, k2, ntb_c);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kWinS; ++i)
#pragma unroll
            for (int d = 0; d < 4; ++d) win[i][d] = load_weights(i, d);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0070);
        for (int n = 0; n < ns; n += 4) {
            stage(n, k0);
            stage(n + 1, k1);
            stage(n + 2, k2);
            stage(n + 3, k3);
        }
        finish(ntb_c, acc);
    };
    const int ntb = (it.cnt + 15) >> 4;
    auto by_blocks = [&](auto &&go) {
        if (ntb == 4) go(std::integral_constant<int, 4>{});
        else if (ntb == 3) go(std::integral_constant<int, 3>{});
        else if (ntb == 2) go(std::integral_constant<int, 2>{});
        else go(std::integral_constant<int, 1>{});
    };
    if (!routed) by_blocks(run_shared);
    else if constexpr (DOWN && KPG == 4) by_blocks(run_e4m3);
    else by_blocks(run);
}

// Gathers the tokens of token block (item, tb) into operand tiles [(item nk + u) 4 + tb]: lane
// (token, chunk) of tile u holds x[token][32 u + 8 chunk .. + 7]; positions past the item's count
// hold zeros.  (The shared experts read one copy.)  Also the group sums x -24, [(item 4 nz + group) 64 + token].  One wave per
// (block, four tiles): 128 inputs, whole groups.
// Which item that is: kPlanned: prefill_plan_kernel has written the items; else it follows from the experts'
// counts (the shared experts' S ceil(T / chunk) items come first, then the routed ones in their segments; expert
// e's assignments are list[e T ..]); each workgroup sums the counts up for itself, the first one also writes the items,
// and a block's first workgroup the slots of its assignments.  The first workgroup also writes the tile of zeros.
// kBySize: in segments by size; else all in the first one, without the work for the others.  Every workgroup finds its item
// first, so that counts: sums over the experts by lane moves, two words a wave (lane permutes, ballots and a word per
// segment, in every call: this launch for dsv2lite, 333 tokens 8.9 / 7.8 us; qwen3, 333 tokens 11.1 / 9.6; H = 448, 618 tokens 6.1 / 5.2).
template <int KPG, bool kPlanned, bool kBySize>
__global__ __launch_bounds__(256)
void prefill_stage_kernel(const uint16_t *__restrict__ x, const int32_t *__restrict__ count, const int32_t *__restrict__ list,
                          PrefillItem *__restrict__ items, int32_t *__restrict__ n_items, int32_t *__restrict__ slot_of,
                          char *__restrict__ xt, char *__restrict__ sums, char *__restrict__ zeros, int T, int H, int k, int E, int S, int lg)
{
    const int chunk = 1 << lg, item = blockIdx.x >> (lg - 4), tb = blockIdx.x & ((chunk >> 4) - 1), tid = threadIdx.x;
    const bool first = blockIdx.x == 0 && blockIdx.y == 0;
    if (first) *reinterpret_cast<u32x4 *>(zeros + tid * 16) = (u32x4){0u, 0u, 0u, 0u};
    PrefillItem it;
    if constexpr (kPlanned) {
        const int n = *n_items;                      // (both loads at once: items past the last are inside the buffer)
        it = items[item];
        if ((item >= n) | (16 * tb >= it.cnt) | (it.src != item)) return;
    } else {
        __shared__ __align__(16) int32_t s_head[4], s_rest[4];         // per wave of 64 experts: items in the first and in the other segments
        __shared__ PrefillItem s_item;
        const int chunks = (T + chunk - 1) >> lg, wave = tid >> 6, lane = tid & 63;
        if (tid == 0) s_item = PrefillItem{0, 0, 0, -1};
        // thread e: expert e's items are [begin, begin + head) and, in segment `seg`, item `rest`.  (The counts of the
        // other segments travel as three fields of ten bits.)
        const int cnt = tid < E ? count[tid] : 0;
        const int head = head_items(cnt, lg, kBySize), seg = kBySize ? rest_segment(cnt, head, lg) : 0;
        const int field = 10 * (seg - 1), incl = wave::prefix_sum(head, lane), rests = kBySize ? wave::prefix_sum(seg ? 1 << field : 0, lane) : 0;
        if (lane == 63) {
            s_head[wave] = incl;
            if constexpr (kBySize) s_rest[wave] = rests;
        }
        __syncthreads();
        auto of_waves = [&](const int32_t *p, int &below, int &all) {
            const int4 n = *reinterpret_cast<const int4 *>(p);
            below = (wave > 0 ? n.x : 0) + (wave > 1 ? n.y : 0) + (wave > 2 ? n.z : 0);
            all = n.x + n.y + n.z + n.w;
        };
        int begin, total, rest = 0, n_seg[kSegments] = {0, 0, 0, 0};
        of_waves(s_head, begin, total);
        begin += S * chunks + incl - head;
        total += S * chunks;
        n_seg[0] = total;
        if constexpr (kBySize) {
            int below, all;
            of_waves(s_rest, below, all);
            if (seg) rest = total + ((below + rests) >> field & 1023) - 1;
#pragma unroll
            for (int g = 1; g < kSegments; ++g) {
                n_seg[g] = all >> 10 * (g - 1) & 1023;
                total += n_seg[g];
                rest += seg > g ? n_seg[g] : 0;
            }
        }
        auto chunk_of = [&](int j, int at) {             // of this thread's expert
            return PrefillItem{tid, tid * T + j * chunk, cnt - j * chunk < chunk ? cnt - j * chunk : chunk, at};
        };
        auto shared_item = [&](int i) {
            const int j = i % chunks;
            return PrefillItem{E + i / chunks, j * chunk, T - j * chunk < chunk ? T - j * chunk : chunk, j};
        };
        if (item >= begin && item < begin + head) s_item = chunk_of(item - begin, item);
        if (seg != 0 && item == rest) s_item = chunk_of(head, item);
        if (tid == 0 && item < S * chunks) s_item = shared_item(item);
        if (first) {
            for (int i = tid; i < S * chunks; i += 256) items[i] = shared_item(i);
            for (int j = 0; j < head; ++j) items[begin + j] = chunk_of(j, begin + j);
            if (seg != 0) items[rest] = chunk_of(head, rest);
            if (tid == 0) {
                n_items[0] = total;
#pragma unroll
                for (int g = 0; g < (kBySize ? kSegments : 1); ++g) n_items[1 + g] = n_seg[g];
            }
        }
        __syncthreads();
        if (item >= total) return;
        it = s_item;
        if (blockIdx.y == 0 && tid < 16 && it.expert < E && 16 * tb + tid < it.cnt)
            slot_of[list[it.first + 16 * tb + tid]] = item * kItemTokens + 16 * tb + tid;
    }
    if (16 * tb >= it.cnt || it.src != item) return;
    const int nk = H / 32, u4 = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (u4 * 4 >= nk) return;
    const int lane = threadIdx.x & 63, tok16 = lane & 15, part = lane >> 4, pos = 16 * tb + tok16;
    const int at = it.first + (pos < it.cnt ? pos : 0);
    const int token = it.expert < E ? list[at] / k : at;
    float s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int u = u4 * 4 + j;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (u < nk && pos < it.cnt) v = *reinterpret_cast<const u32x4 *>(x + (size_t)token * H + 32 * u + 8 * part);
        if (u < nk) *reinterpret_cast<u32x4 *>(xt + (((size_t)item * nk + u) * 4 + tb) * 1024 + lane * 16) = v;
        s[j] = ((bf16_lo(v.x) + bf16_hi(v.x)) + (bf16_lo(v.y) + bf16_hi(v.y))) +
               ((bf16_lo(v.z) + bf16_hi(v.z)) + (bf16_lo(v.w) + bf16_hi(v.w)));
        s[j] += __shfl_xor(s[j], 16);
        s[j] += __shfl_xor(s[j], 32);
    }
    // group `part` of this wave's 4 / KPG groups; the wave with the last inputs also clears what is left
    // of the last tile of four groups
    const int G = nk / KPG, gi = u4 * (4 / KPG) + part;
    const bool real = part < 4 / KPG && gi < G, last = u4 * 4 + 4 >= nk;
    if (real || (last && gi >= G && gi / 4 == (G - 1) / 4)) {
        float v = 0.f;
        if (real) {
            if constexpr (KPG == 4) v = (s[0] + s[1]) + (s[2] + s[3]);
            else if constexpr (KPG == 2) v = part == 0 ? s[0] + s[1] : s[2] + s[3];
            else v = part == 0 ? s[0] : part == 1 ? s[1] : part == 2 ? s[2] : s[3];
        }
        reinterpret_cast<float *>(sums)[((size_t)item * ((G + 3) / 4) * 4 + gi) * kItemTokens + 16 * tb + tok16] = kOffset * v;
    }
}

// y[t][:] = sum_j w[t k + j] * obuf[slot_of[t k + j]][:], j ascending, then the shared experts' rows
__global__ __launch_bounds__(256)
void prefill_combine_kernel(const float *__restrict__ obuf, const int32_t *__restrict__ slot_of,
                            const float *__restrict__ w_all, float *__restrict__ y, int H, int k, int S, int chunk)
{
    const int t = blockIdx.x, col = (blockIdx.y * 256 + threadIdx.x) * 4;
    if (col >= H) return;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < k; ++j) {
        const int a = t * k + j;
        const f32x4 v = *reinterpret_cast<const f32x4 *>(obuf + (size_t)slot_of[a] * H + col);
        const float w = w_all[a];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = fmaf(w, v[i], acc[i]);
    }
    const int chunks = ((int)gridDim.x + chunk - 1) / chunk;                               // items of one shared expert
    for (int sh = 0; sh < S; ++sh)
        acc += *reinterpret_cast<const f32x4 *>(obuf + ((size_t)(sh * chunks + t / chunk) * kItemTokens + t % chunk) * H + col);
    *reinterpret_cast<f32x4 *>(y + (size_t)t * H + col) = acc;
}

// Sorts the n = T k assignments by expert (the order inside an expert is arbitrary: no result
// depends on it, a row's sums do not depend on the other rows of its item), cuts every expert's
// run into items of at most `chunk` and records the slot (item x 64 + position) of every assignment.
// The first S ceil(T / chunk) items are the shared experts', over the tokens in order.  One workgroup.
__global__ __launch_bounds__(1024)
void prefill_plan_kernel(const int32_t *__restrict__ ids, int n, int E, int T, int S, int lg, bool by_size,
                         int32_t *__restrict__ list, int32_t *__restrict__ slot_of,
                         PrefillItem *__restrict__ items, int32_t *__restrict__ n_items)
{
    __shared__ int32_t s_count[MOE_MAX_EXPERTS], s_off[MOE_MAX_EXPERTS], s_fill[MOE_MAX_EXPERTS],
        s_item0[MOE_MAX_EXPERTS], s_rest[MOE_MAX_EXPERTS];
    const int chunk = 1 << lg, chunks = (T + chunk - 1) >> lg;
    for (int i = threadIdx.x; i < S * chunks; i += blockDim.x) {
        const int j = i % chunks;
        items[i] = PrefillItem{E + i / chunks, j * chunk, T - j * chunk < chunk ? T - j * chunk : chunk, j};
    }
    for (int e = threadIdx.x; e < E; e += blockDim.x) { s_count[e] = 0; s_fill[e] = 0; }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) atomicAdd(&s_count[ids[i]], 1);
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int off = 0, item = S * chunks;
        for (int g = 0; g < (by_size ? kSegments : 1); ++g) {
            const int first = g == 0 ? 0 : item;
            for (int base = 0; base < E; base += 64) {
                const int cnt = base + lane < E ? s_count[base + lane] : 0;
                const int head = head_items(cnt, lg, by_size), mine = g == 0 ? head : rest_segment(cnt, head, lg) == g ? 1 : 0;
                // (assignments of all experts, in the first round: at most 2^16; items: at most 2^11 + 2^8)
                const int incl = wave::prefix_sum((g == 0 ? cnt : 0) | mine << 18, lane);
                if (g == 0 && base + lane < E) s_off[base + lane] = off + (incl & 0x3ffff) - cnt;
                if (mine > 0) (g == 0 ? s_item0 : s_rest)[base + lane] = item + (incl >> 18) - mine;
                const int all = __builtin_amdgcn_readlane(incl, 63);
                off += all & 0x3ffff;
                item += all >> 18;
            }
            if (lane == 0) n_items[1 + g] = item - first;
        }
        if (lane == 0) n_items[0] = item;
    }
    __syncthreads();
    auto item_of = [&](int e, int j) { return j < head_items(s_count[e], lg, by_size) ? s_item0[e] + j : s_rest[e]; };
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int e = ids[i];
        const int idx = atomicAdd(&s_fill[e], 1);
        list[s_off[e] + idx] = i;
        slot_of[i] = item_of(e, idx >> lg) * kItemTokens + (idx & (chunk - 1));
    }
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int cnt = s_count[e];
        for (int j = 0; j * chunk < cnt; ++j) {
            PrefillItem it;
            it.expert = e; it.first = s_off[e] + j * chunk;
            it.cnt = cnt - j * chunk < chunk ? cnt - j * chunk : chunk;
            it.src = item_of(e, j);
            items[it.src] = it;
        }
    }
}

template <bool DOWN, bool SYM>
void launch_tile_g(const TileArgs &t, int g, int tiles, int max_items, hipStream_t st)
{
    const size_t pairs = (size_t)((tiles + kTileWaves - 1) / kTileWaves) * max_items;
    // (each segment is rounded up, and each block where those are striped)
    const dim3 grid((unsigned)(((pairs + kXcds - 1) / kXcds + t.segments - 1 + (t.striped ? max_items / t.block + t.segments : 0)) * kXcds)), block(kTileThreads);
    if (g == 32) launch(prefill_tile_kernel<DOWN, SYM, 1>, grid, block, 0, st, t);
    else if (g == 64) launch(prefill_tile_kernel<DOWN, SYM, 2>, grid, block, 0, st, t);
    else launch(prefill_tile_kernel<DOWN, SYM, 4>, grid, block, 0, st, t);
}

template <bool DOWN>
void launch_tile(const TileArgs &t, bool sym, int g, int tiles, int max_items, hipStream_t st)
{
    if (sym) launch_tile_g<DOWN, true>(t, g, tiles, max_items, st);
    else launch_tile_g<DOWN, false>(t, g, tiles, max_items, st);
}

}  // namespace

// workgroups of the tile launches per item: the down launch's, and the larger of the two
static int down_columns(const Shape &s) { return (s.H / 64 + kTileWaves - 1) / kTileWaves; }
static int prefill_columns(const Shape &s)
{
    const int gate = (s.I / 32 + kTileWaves - 1) / kTileWaves, down = down_columns(s);
    return gate > down ? gate : down;
}

// sum over experts of ceil(count / chunk) <= n / chunk + number of experts that occur
static int items_of(const Shape &s, int chunk)
{
    const int n = s.T * s.k;
    return n / chunk + (s.E < n ? s.E : n) + s.S * ((s.T + chunk - 1) / chunk);
}

// A launch that leaves compute units empty gets items of 32 tokens: as long as those are at most one workgroup per
// unit.  us per call, items of 64 / of 32 (workgroups of 32, upper bound): H = 256, I = 512, E = 8, k = 2, 421 tokens
// (136) 38.5 / 32.7; H = 384, I = 384, k = 5, 274 tokens (150) 39.2 / 34.4; H = 2048, I = 1408, E = 4, a shared
// expert, 200 tokens (253) 72.5 / 60.2, 400 tokens (462) 78.7 / 85.2.  With more columns 32 still wins beyond the line
// (H = 1024, I = 2048, 300 tokens, 416: 65.8 / 55.9), the more evenly the 64s fill the units the less.
constexpr int kSmallGrid = 256;
int prefill_chunk(const Shape &s) { return (long)prefill_columns(s) * items_of(s, 32) <= kSmallGrid ? 32 : 64; }
// Largest items first, where a launch has few rounds of workgroups (two a compute unit), so that it ends with short ones and a unit
// that takes two workgroups takes a long and a short one.  Not where that counts little: beyond three and a half rounds
// (upper bound of either launch), where the parting of an expert's items, which read the same weights, counts more; where the down
// launch leaves units empty; and where all items are alike: runs of less than a token block and no shared experts.
// us per call, expert by expert / largest first (gate/up and down workgroups, upper bound):
//   phi shape, 512 tokens (1600, 512)       348 / 324       dsv2lite, 333 tokens (1177, 856)        156 / 147
//   phi shape, 600 tokens (1700, 544)       374 / 354       ..., 700 tokens (1661, 1208)            229 / 224
//   even popularity, 600 tokens             397 / 375       H = 1472, E = 20, k = 6, 2 shared, 294 (342, 342)   82.4 / 72.0
//   mixtral, 200 tokens (1568, 224)         368 / 360       H = 4096, E = 4, I = 12288, k = 4, 200 (1536, 256)  393 / 385
// and outside: mixtral, 283 tokens (1792, 256) 405 / 425; dsv2lite, 1200 (2354, 1712) 322 / 335; qwen3, 1500 (1890, 2520) 298 / 314;
// H = 1280, E = 7, I = 7296, k = 1, 4 shared, 27 tokens (627, 55) 149 / 152; H = 256, E = 109, I = 1920, k = 6, 40 tokens
// (1680, 112) 57.0 / 58.8.  Inside it can lose (H = 2112, I = 512, E = 15, k = 1, 2 shared, 2024 tokens (440, 990) 122.9 / 125.7),
// above the line it can win (zipf popularity, H = 1088, E = 96, 378 tokens (3562, 685) 196 / 173).
static bool prefill_by_size(const Shape &s)
{
    const long items = items_of(s, kItemTokens);
    const bool alike = s.S == 0 && s.T * s.k < 16 * s.E;
    return prefill_chunk(s) == kItemTokens && prefill_columns(s) * items < 7 * 256 && down_columns(s) * items > 200 && !alike;
}
static int prefill_lg(const Shape &s) { return prefill_chunk(s) == 32 ? 5 : 6; }
int prefill_max_items(const Shape &s) { return items_of(s, prefill_chunk(s)); }
size_t prefill_item_room(const Shape &s)
{
    const int items = prefill_max_items(s), small = kSmallGrid / prefill_columns(s);
    return prefill_chunk(s) == 32 || items > small ? items : small;
}

PrefillBuffers prefill_buffers(const moe_layer_desc &d, size_t m)
{
    PrefillBuffers b;
    b.xt = m * (d.hidden / 32) * 4096;
    b.x_sums = m * ((d.hidden / d.group_size + 3) / 4) * 1024;
    b.h = m * (d.inter / 32) * 8192;
    b.h_sums = m * ((d.inter / d.group_size + 3) / 4) * 1024;
    b.h_scales = d.group_size == 128 ? b.h_sums / 4 : 0;
    b.zeros = 4096;
    b.obuf = m * kItemTokens * d.hidden * 4;
    return b;
}

// Small calls: one workgroup per token routes (route_kernel) and one workgroup sorts (prefill_plan_kernel); larger
// ones: the two launches of route.hip, and the stage launch finds the items.  us of the three launches, small
// form / large form: 421 tokens of the tiny shape (H = 256, E = 8, k = 2; 1.7 million here) 11 / 14, 1703
// tokens (7 million) 18 / 15, phi shape, 512 tokens (34 million) 28 / 20, dsv2lite, 333 (46 million) 40 / 22.
bool prefill_small(const Shape &s) { return (long)s.T * ((long)s.E * s.H + 1024L * s.k) < (4L << 20); }

void launch_prefill_plan(const Shape &s, const int32_t *ids, const PrefillCall &p, hipStream_t st)
{
    launch(prefill_plan_kernel, dim3(1), dim3(1024), 0, st, ids, s.T * s.k, s.E, s.T, s.S, prefill_lg(s), prefill_by_size(s), (int32_t *)p.list, p.slot_of, p.items, p.n_items);
}

void launch_prefill_stage(const Shape &s, const PrefillCall &p, int max_items, hipStream_t st)
{
    const int lg = prefill_lg(s);
    const dim3 grid(max_items << (lg - 4), (s.H / 32 + 15) / 16), block(256);
    auto go = [&](auto kernel) {
        launch(kernel, grid, block, 0, st, (const uint16_t *)p.x, p.count, p.list, p.items, p.n_items, p.slot_of, (char *)p.xt,
               (char *)p.x_sums, (char *)p.zeros, s.T, s.H, s.k, s.E, s.S, lg);
    };
    auto of_group = [&](auto planned, auto by_size) {
        constexpr bool kPlanned = decltype(planned)::value, kBySize = decltype(by_size)::value;
        if (s.g == 32) go(prefill_stage_kernel<1, kPlanned, kBySize>);
        else if (s.g == 64) go(prefill_stage_kernel<2, kPlanned, kBySize>);
        else go(prefill_stage_kernel<4, kPlanned, kBySize>);
    };
    if (prefill_small(s)) of_group(std::true_type{}, std::false_type{});
    else if (prefill_by_size(s)) of_group(std::false_type{}, std::true_type{});
    else of_group(std::false_type{}, std::false_type{});
}

static TileArgs tile_args(const Shape &s, const PrefillCall &p)
{
    TileArgs t;
    t.q = (const char *)p.q; t.sz = (const char *)p.sz; t.stride_q = p.stride_q; t.stride_sz = p.stride_sz;
    t.items = p.items; t.n_items = p.n_items; t.zeros = (const char *)p.zeros;
    t.h = (char *)p.h; t.h_sums = (char *)p.h_sums; t.h_scales = (char *)p.h_scales; t.obuf = p.obuf;
    t.shared = (const char *)p.shared; t.shared_stride = p.shared_stride;
    t.H = s.H; t.I = s.I; t.E = s.E; t.segments = prefill_by_size(s) ? kSegments : 1;
    return t;
}

// The order of the (item, column) pairs.  Blocks of two items: an XCD then has a few experts to itself, whose weights and x it alone reads.
// Where experts are wide and so few, blocks of eight and an eighth of each to every XCD: x is then read by all XCDs, which costs less than
// leaving some of them with other amounts of work (shared experts, short rests).  us per pass, items of all experts column by column as it was / blocks of two /
// eight, striped:  dsv2lite, 333 tokens 570 / 556 / 571; 1200 1290 / 1226 / 1280; qwen3, 512 629 / 599 / 625; qwen15, 700 874 / 840 / 878; H = 1024, E = 24, I = 2048, 900
// 481 / 453 / 474; phi, 512 609 / 610 / 600, 2048 1793 / 1744 / 1732; phi, 150 423 / 425 / 413; mixtral, 512 605 / 613 / 589, 4096 3455 / 3594 / 3331; H = 2048, E = 6, I = 4096, a shared
// expert, 2500 1312 / 1344 / 1285.  In the down launch the two differ by less than 1 %, and h is as many bytes as the weights: blocks of two.  Also striped, in both
// launches: many rounds of short routed items behind the shared experts' long ones, which one XCD would have to itself (H = 1728, E = 102, I = 1984, k = 8, two
// shared, 292 tokens 238 / 278 / 234).
static void prefill_blocks(TileArgs &t, const Shape &s, bool down)
{
    const bool short_behind_shared = s.S > 0 && s.T * s.k < kItemTokens * s.E && (long)prefill_columns(s) * items_of(s, kItemTokens) >= 7 * 256;
    t.striped = (!down && t.I >= 4096) || short_behind_shared;
    t.block = t.striped ? 8 : 2;
}

void launch_prefill_gateup(const Shape &s, const PrefillCall &p, int max_items, hipStream_t st)
{
    TileArgs t = tile_args(s, p);
    prefill_blocks(t, s, false);
    t.act = (const char *)p.xt; t.act_sums = (const char *)p.x_sums; t.act_scales = nullptr;
    launch_tile<false>(t, p.symmetric != 0, s.g, s.I / 32, max_items, st);
}

void launch_prefill_down(const Shape &s, const PrefillCall &p, int max_items, hipStream_t st)
{
    TileArgs t = tile_args(s, p);
    prefill_blocks(t, s, true);
    t.act = (const char *)p.h; t.act_sums = (const char *)p.h_sums; t.act_scales = (const char *)p.h_scales;
    launch_tile<true>(t, p.symmetric != 0, s.g, s.H / 64, max_items, st);
}

void launch_prefill_combine(const Shape &s, const PrefillCall &p, hipStream_t st)
{
    launch(prefill_combine_kernel, dim3(s.T, (s.H / 4 + 255) / 256), dim3(256), 0, st,
           (const float *)p.obuf, p.slot_of, p.w_all, p.y, s.H, s.k, s.S, prefill_chunk(s));
}

}  // namespace moespeq
