// The rules by which a draft call is laid out, on its sizes and the device's compute units alone: plain C++ (host code and
// kernels share them, and the CPU tests compile them by themselves).
#pragma once
#include <stddef.h>

namespace moespeq {

struct Shape {
    int T, H, E, I, k, S, g, renorm;
};

constexpr int kDraftWaves = 8;                           // of a workgroup, or of an item where a workgroup has two
constexpr size_t kDraftLds = (size_t)(160 - 20) * 1024;  // dynamic LDS: 160 KiB per workgroup less the kernels' static arrays

// Workgroups that reduce the router rows, the first ones of the launch, `rows` rows at a time each, for all tokens.  All workgroups
// wait for them, so calls on several streams that are dispatched together, each on its part of the units, go on only if one of
// them has all of these running: few of them, however many tokens there are.  (A row's tokens shared out over up to the whole
// grid shortened the start of a call, qwen3 shape, 8 tokens, 128 / 256 workgroups 37.5 / 36.5 us, and let two such calls wait for each other
// until their polls ran out.)
constexpr int router_workgroups(int E, int rows, int workgroups) {
    const int n = (E + rows - 1) / rows;
    return n < workgroups ? n : workgroups;
}

// Copies of the router's results that a call publishes, 2 to the power of this; workgroup b polls copy b mod their number, so that the polls of
// hundreds of workgroups do not all land on one address.  A copy is a 16-byte store per logit, four of them to a line of memory that
// different workgroups write, which the last reader clears again: with many experts that costs more than the polls.  us per pass, sixteen / four copies (one
// token; E): 72 210 / 200, 100 190 / 179, 128 (qwen3) 232 / 220, 256 230 / 212; 8 tokens, E = 128 283 / 274 (two copies 275, one 277).  E <= 64, sixteen / eight / four:
// dsv2lite 271.3 / 272.4 / 272.9, phi 187.7 / 186.5 / 185.4, qwen15 442 / 440 / 437, E = 32 164.5 / 162.5 / 163.2; E = 8, H = 8192 177.2 / 177.5 / 171, mixtral 156.7 / 158.3 / 157.6.
constexpr int exchange_copies_lg(int E) { return E > 64 ? 2 : E >= 16 ? 3 : 4; }

// ---- calls of two to eight tokens (draft_int4.hip)

// Token slots of y that a workgroup sums in LDS
constexpr int sum_slots(int MT) { return MT == 4 ? 4 : 2; }

// Tiles a wave keeps in flight: eight, or four where padding the two parts of an item to whole windows of eight
// would add more than a fifth to the stream's positions (an empty position is a load that is not in
// flight).  8 against 4: phi shape (16 and 8 tiles per part and wave), 4 tokens 43.3 / 50.4 us (without the sums of y, which the
// window of four does not have, 48.7 / 50.4), 2 tokens 36.7 / 38.4; qwen3 shape (8 and 4), 8 tokens 41.5 / 37.4, 2 tokens 20.8 /
// 19.1.  Windows of 12 and 16 only add padding (phi, 4 tokens, when 8 took 52.7 us: 58.3 and 59.4).
inline int stream_window(const Shape &s, bool sym)
{
    const int epl = sym ? 2 : 1;
    const int nt = (s.H / s.g / epl + kDraftWaves - 1) / kDraftWaves * epl * (s.g / 32);
    const int nd = (s.H / 64 / epl + kDraftWaves - 1) / kDraftWaves * epl;
    auto positions = [&](int w) { return (nt + w - 1) / w * w + (nd + w - 1) / w * w; };
    return positions(8) * 5 > positions(4) * 6 ? 4 : 8;
}

// dynamic LDS: the bf16 copy of x (padded rows), its per-group sums, the routing scratch (fp64
// logits and ranks), and per wave the scale / zero entries of its groups and row tiles of one
// item (whole KiB each)
inline size_t draft_dynamic_lds(int MT, int H, int g, int E, bool sym, int entry_copies = 1)
{
    const int nw = kDraftWaves;
    size_t lds = ((size_t)MT * (H + 8) * 2 + (size_t)MT * (H / g) * 4 + 7) & ~(size_t)7;
    lds += (size_t)MT * E * 12;
    lds = (lds + 15) & ~(size_t)15;
    const int epl = sym ? 2 : 1;
    const int gl_max = (H / g / epl + nw - 1) / nw, dl_max = (H / 64 / epl + nw - 1) / nw;
    lds += (size_t)entry_copies * nw * ((size_t)((gl_max + 3) / 4) + (size_t)((dl_max + 3) / 4)) * 1024;
    return lds;
}

// and behind it the sums of y: from two items per workgroup on, in calls with the window of eight, where they fit (0: no sums)
inline size_t sum_lds(const Shape &s, int MT, bool sym, int n_cu)
{
    const int maxu = s.E < s.T * s.k ? s.E : s.T * s.k;
    const size_t sums = (size_t)sum_slots(MT) * s.H * 4;
    if ((long)maxu * (s.I / 32) < 2L * n_cu || stream_window(s, sym) != 8) return 0;
    return draft_dynamic_lds(MT, s.H, s.g, s.E, sym) + sums <= kDraftLds ? sums : 0;
}

// ---- calls of one token (draft_slice.hip, and draft_int4.hip where there are many long items)

// dynamic LDS of a one-token workgroup: x, the fp64 logits and the ranks, the sums of x per group, the outputs of two items
inline size_t slice_dynamic_lds(int H, int g, int E, int items) { return (size_t)H * 2 + (size_t)E * 12 + (size_t)(H / g) * 4 + (items > 1 ? (size_t)H * 8 : 0); }

// whether the LDS of a call with that many tokens fits
inline bool draft_fits(const Shape &s, int tokens, bool sym)
{
    if (tokens <= 1) return slice_dynamic_lds(s.H, s.g, s.E, 1) <= kDraftLds;
    const int MT = tokens <= 2 ? 2 : (tokens <= 4 ? 4 : 8);
    // (the limit callers know counts the entries twice; one copy is kept)
    const size_t entries = draft_dynamic_lds(MT, s.H, s.g, s.E, sym) - draft_dynamic_lds(MT, s.H, s.g, s.E, sym, 0);
    return draft_dynamic_lds(MT, s.H, s.g, s.E, sym) + entries <= kDraftLds;
}

// Items per workgroup.  Every item adds to all of y, and fp32 additions to one address follow each other at 25 ns (400 workgroups
// adding to the same 4096 floats take 13.8 us, to four copies of them 7.9, without adding 3.8), so that n items cannot
// end less than n x 25 ns after the first one, and beyond 256 items some units have two, whose second one also starts late: its
// loads wait until the first one's have returned.  Two items in one workgroup halve the chain and start together.  Below two
// items per unit they leave units empty: up to one item per unit that costs more than the shorter chain saves (at exactly one with long
// rows and no shared experts inside), beyond it less.  With long items not beyond two per unit, where a second
// round of workgroups costs more than the chain.  us per call, single / paired (items):
//   H = 4096: 224 18.5 / 19.6, 256 20.0 / 20.0, 320 23.7 / 21.5, 384 25.7 / 24.7, 576 38.9 / 47.0, 768 44.4 / 49.8
//   H = 2048: 192 14.6 / 17.1, 224 14.3 / 15.1, 240 15.0 / 15.2, 320 18.8 / 16.4, 504 24.4 / 20.6, 624 30.9 / 28.7, 768 35.6 / 28.9
//   H = 512: 240 13.0 / 12.6, 504 21.1 / 15.8, 768 26.0 / 17.9
//   256 items, groups of 32: H = 1024 14.6 / 13.8, 2048 16.9 / 17.1, 4096 20.6 / 22.2, 5120 24.1 / 25.4, 7168 28.3 / 30.5; groups of
//   128: H = 1024 14.5 / 13.6, 2048 16.0 / 15.8, 4096 21.0 / 20.7, 5120 22.8 / 23.6, 7168 28.0 / 28.1; 128 of them
//   shared ones': H = 2048 15.1 / 13.5, 4096 20.9 / 20.4; 264 items: H = 8192 38.0 / 30.0
inline bool slice_pairs(const Shape &s, bool shared_inside, int n_cu)
{
    const int items = s.k * (s.I / 32) + (shared_inside ? s.S * (s.I / 16) : 0), routed = s.k * (s.I / 32) / 2;
    // (a unit holds one workgroup of two items: those that reduce the router rows have to be running together)
    return (items > n_cu || (items == n_cu && (s.H < 2048 || shared_inside))) && (items <= 2 * n_cu || s.H <= 2048) && router_workgroups(s.E, 2, routed) <= n_cu &&
           slice_dynamic_lds(s.H, s.g, s.E, 2) <= kDraftLds;
}

// Whether a one-token call runs its shared experts in its own launch: up to three 16-row items per compute unit, or one per 256 of
// H where that is more; as pairs of items up to seven, or one per 128.  Beyond, items are many and short, a workgroup's start costs
// more than two launches, and the bf16 kernels take them.  us per call inside as pairs / in their own launches (256 units):
//   items per unit   H = 256       H = 512       H = 1024      H = 1536      H = 2048
//   4   (S = 4)      28.1 / 29.8                 35.1 / 35.1
//   5.5 (S = 4)      37.7 / 41.5   40.1 / 44.9   48.5 / 53.5
//   7   (S = 2)      39.8 / 50.7                 49.0 / 58.4
//   8   (S = 4)      48.8 / 47.7                 50.9 / 54.9
//   12  (S = 4)                                                99.5 / 106.0
//   14  (S = 4)                    71.7 / 67.2   78.8 / 77.5                 142.2 / 147.5
// With one routed expert beside four shared ones and short rows the two sides lie close together from five per unit on, and inside
// is the slower one where its workgroups fill their rounds badly: the line is five.  The same two sides, S = 4, k = 1: H = 256, 5 per unit
// 26.4 / 26.9, 6 30.9 / 29.9, 7 35.1 / 33.2; H = 768, 6 36.9 / 36.9, 7 40.5 / 41.6; H = 1024, 5 34.0 / 36.9, 6 42.3 / 41.1, 8 51.6 / 50.9; H = 1280, 8
// 58.2 / 63.3; H = 2048, 14 131 / 136; k = 2, H = 256, 7 36.9 / 39.4; S = 3, k = 1, H = 256, 7 36.0 / 39.7.
// As single items (their chain of additions is twice as long) beyond the first line, with eight experts chosen, whose routed items
// leave the persistent launch as well: H = 2304, 10 per unit 180 / 168, 14 per unit 248 / 223; H = 3072, 14 289 / 256; H = 3456, 14 297 / 286.
inline bool draft_shared_inside(const Shape &s, int n_cu)
{
    const long items = (long)s.S * (s.I / 16);
    if (s.T != 1 || s.S == 0) return false;
    if (items <= 3L * n_cu || items * 256 <= (long)n_cu * s.H) return true;
    const bool few_routed = 4 * s.k <= s.S && s.H <= 1024;
    return (few_routed ? items <= 5L * n_cu : items <= 7L * n_cu || items * 128 <= (long)n_cu * s.H) && slice_pairs(s, true, n_cu);
}

// One token through the persistent kernel: from two items per compute unit on, where the launch carries no shared
// experts and the kernel's two copies of x fit LDS, if it sums y in LDS (long rows); without the sums only where pairs of items
// make between one and one and a half rounds of long workgroups.  us per call, persistent / pairs (items):
// H = 4096 (with the sums): 512 27.4 / 27.8, 600 30.9 / 40.9; H = 2304, 576 27.4 / 33.0; H = 2048: 512 23.9 / 20.1, 640 27.7 / 29.5,
// 768 30.2 / 30.1, 1024 37.2 / 33.4; H = 1024: 512 21.9 / 17.2, 640 25.7 / 25.2, 1024 34.6 / 28.0; H = 320, 1870 56.2 / 39.9.
inline bool can_stream_one_token(const Shape &s, bool sym, bool shared_inside, int n_cu)
{
    return s.k * (s.I / 32) >= 2 * n_cu && !shared_inside && draft_fits(s, 2, sym);
}
inline bool one_token_streams(const Shape &s, bool sym, bool shared_inside, int n_cu)
{
    const int items = s.k * (s.I / 32);
    if (!can_stream_one_token(s, sym, shared_inside, n_cu)) return false;
    return s.H > 2048 || sum_lds(s, 2, sym, n_cu) > 0 || (s.H > 1024 && items > 2 * n_cu && items < 3 * n_cu);
}

// The form of a call of one token.  `single_slots()`: workgroups of single items that the device holds at once.  Where those that
// reduce the router rows are more (many experts on few units), the persistent launch, whose own always fit, takes what it can.
enum OneTokenForm { kSingleItems, kPairsOfItems, kPersistent };
template <typename F>
inline OneTokenForm one_token_form(const Shape &s, bool sym, bool shared_inside, int n_cu, F single_slots)
{
    if (one_token_streams(s, sym, shared_inside, n_cu)) return kPersistent;
    if (slice_pairs(s, shared_inside, n_cu)) return kPairsOfItems;
    if (can_stream_one_token(s, sym, shared_inside, n_cu) && single_slots() < router_workgroups(s.E, 1, s.k * (s.I / 32))) return kPersistent;
    return kSingleItems;
}

}  // namespace moespeq
