"""Measured workloads of the MoE draft / verify layer.

A case is one pass of a serving program through a stack of `layers` distinct MoE layers (each with
its own weights, so that they come from device memory and not from a cache), by its `kind`:

  draft    one moe_draft_layer_int4 call per layer over `tokens` tokens (1: the canonical draft step,
           2-8: several branches or requests drafted together)
  verify   one moe_verify_layer_bf16 call per layer over the K + 1 = `tokens` tokens of a window, all
           experts resident, slots in permuted order
  prefill  one moe_draft_prefill_int4 call per layer over a prompt of `tokens` tokens
  cycle    per layer: K = tokens - 1 one-token draft calls, the expert union of the window, and the
           verify call over all tokens (the step that bench.py times)

Shapes are those of the repository's workload list (synth/configs.py); draw() adds generic ones.
Weights are drawn in the packed form that a program keeps after loading: bf16 blobs of N(0, 0.02)
values, int4 codes with the distribution that round-to-nearest quantisation of such values gives."""
import math

import torch

from paper_2511_14102_amd import binding as B

STD = 0.02                                            # of router and expert weights
RANGE = {32: 4.14, 64: 4.74, 128: 5.33}               # expected range of a group of normal values, in std


def _case(name, kind, tokens, layers, hidden, experts, inter, top_k, group, shared=0, symmetric=False,
          routing="plain"):
    c = dict(kind=kind, tokens=tokens, layers=layers, hidden=hidden, experts=experts, inter=inter, top_k=top_k,
             group=group, shared=shared, symmetric=symmetric, routing=routing)
    return c if name is None else dict(c, name=name)


TINY = dict(hidden=256, experts=8, inter=512, top_k=2, group=32)
PHI = dict(hidden=4096, experts=16, inter=6400, top_k=2, group=128, routing="zipf")
MIXTRAL = dict(hidden=4096, experts=8, inter=14336, top_k=2, group=128)
QWEN3 = dict(hidden=2048, experts=128, inter=768, top_k=8, group=64, routing="ar1")
DSV2LITE = dict(hidden=2048, experts=64, inter=1408, top_k=6, group=128, shared=2)
QWEN15 = dict(hidden=2048, experts=60, inter=1408, top_k=4, group=128, shared=4, routing="ar1")


def listed():
    return [
        # the smallest work: a whole speculative cycle of a layer that costs nothing but latency and launches
        _case("cycle_tiny_4", "cycle", 4, 4, **TINY),
        # the canonical draft step, one token: few large experts with skewed popularity ...
        _case("draft_phi_1", "draft", 1, 8, **PHI),
        # ... many small experts ...
        _case("draft_qwen3_1", "draft", 1, 16, **QWEN3),
        # ... and shared experts beside the routed ones
        _case("draft_dsv2lite_1", "draft", 1, 16, **DSV2LITE),
        # several branches or requests drafted in one call: ordinary, an odd number of tokens with the
        # symmetric weight format, and the most tokens a call takes over many small experts
        _case("draft_phi_4", "draft", 4, 8, **PHI),
        _case("draft_mixtral_3_symmetric", "draft", 3, 4, symmetric=True, **MIXTRAL),
        _case("draft_qwen3_8", "draft", 8, 8, **QWEN3),
        # verification of a window of 5 and of 8 tokens
        _case("verify_phi_5", "verify", 5, 4, **PHI),
        _case("verify_qwen3_8", "verify", 8, 8, **QWEN3),
        # prompts: ordinary; ragged, with shared experts; the longest over the largest layer
        _case("prefill_phi_512", "prefill", 512, 2, **PHI),
        _case("prefill_dsv2lite_333", "prefill", 333, 4, **DSV2LITE),
        _case("prefill_mixtral_4096", "prefill", 4096, 1, **MIXTRAL),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng):
    """A listed shape, or a generic one inside their ranges (sizes in the layer's granularity)."""
    if rng.random() < 0.4:
        s = dict(rng.choice([TINY, PHI, MIXTRAL, QWEN3, DSV2LITE, QWEN15]))
    else:
        group = rng.choice([32, 64, 128])
        unit = max(64, group)
        experts = _log_uniform(rng, 4, 128)
        s = dict(hidden=unit * _log_uniform(rng, max(1, 256 // unit), 4096 // unit), experts=experts,
                 inter=unit * _log_uniform(rng, max(1, 384 // unit), 14336 // unit),
                 top_k=rng.randint(1, min(8, experts)), group=group,
                 shared=rng.choice([0, 0, 0, 1, 2, 4]), routing=rng.choice(["plain", "zipf", "ar1"]))
    symmetric_fits = s["hidden"] % 128 == 0 and (s["hidden"] // s["group"]) % 2 == 0
    return dict(s, symmetric=symmetric_fits and rng.random() < 0.25)


def draw(rng):
    largest = work(listed()[-1])
    while True:
        kind = rng.choice(["draft", "draft", "draft", "verify", "verify", "prefill", "prefill", "cycle"])
        s = _draw_shape(rng)
        if kind == "draft":
            tokens = rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 7, 8])
        elif kind == "prefill":
            tokens = _log_uniform(rng, 17, 4096)
        else:
            tokens = rng.randint(2, 16 if kind == "verify" else 9)
        if kind in ("verify", "cycle") and tokens * s["top_k"] > 128:
            continue
        one = _case(None, kind, tokens, 1, **s)
        # as many layers as keep a pass from living in a cache, within 12 GiB of weights
        weights = _weight_bytes(one)
        if weights > 12 << 30:
            continue
        layers = min(16, max(1, round((768 << 20) / work(one)["bytes"])), (12 << 30) // weights)
        case = dict(one, layers=layers)
        w = work(case)
        if kind in ("draft", "cycle") and B.draft_call_fits(_desc(case), tokens if kind == "draft" else 1) != 0:
            continue
        if w["bytes"] > 2 * largest["bytes"] or w["flops"] > 0.25 * largest["flops"]:
            continue
        return case


def _desc(c):
    d = B.LayerDesc()
    d.hidden, d.n_experts, d.inter, d.top_k = c["hidden"], c["experts"], c["inter"], c["top_k"]
    d.n_shared, d.group_size, d.renormalize = c["shared"], c["group"], 1
    return d


def _int4_bytes(c):
    p = 3 * c["hidden"] * c["inter"]
    return p // 2 + p // c["group"] * (2 if c["symmetric"] else 4)


def _bf16_bytes(c):
    return 6 * c["hidden"] * c["inter"]


def _weight_bytes(c):
    """Of one layer, as prepare() lays it out."""
    n = c["shared"] * _bf16_bytes(c)
    if c["kind"] != "verify":
        n += c["experts"] * _int4_bytes(c)
    if c["kind"] in ("verify", "cycle"):
        n += c["experts"] * _bf16_bytes(c)
    return n


def _distinct(c, tokens):
    """Expected number of distinct experts that `tokens` tokens choose."""
    E, k = c["experts"], c["top_k"]
    pi = [(e + 1.0) ** -1.1 if c["routing"] == "zipf" else 1.0 for e in range(E)]
    total = sum(pi)
    return min(float(E), max(float(k), sum(1.0 - (1.0 - p / total) ** (k * tokens) for p in pi)))


def work(case):
    """Every distinct expert's weights, the shared experts', the router and the activations once."""
    c, T, H, E, k, S = case, case["tokens"], case["hidden"], case["experts"], case["top_k"], case["shared"]
    expert_flops = 6.0 * H * c["inter"]

    def call(tokens, int4):
        out = tokens * (H * (4 if int4 else 2) + 8 * k)
        b = _distinct(c, tokens) * (_int4_bytes(c) if int4 else _bf16_bytes(c)) + S * _bf16_bytes(c)
        return b + E * H * 2 + tokens * H * 2 + out, tokens * ((k + S) * expert_flops + 2.0 * E * H)

    calls = {"draft": [call(T, True)], "prefill": [call(T, True)], "verify": [call(T, False)],
             "cycle": [call(1, True)] * (T - 1) + [call(T, False)]}[c["kind"]]
    return {"bytes": c["layers"] * sum(b for b, _ in calls), "flops": c["layers"] * sum(f for _, f in calls)}


def tolerance(case):
    """Expert ids, counts and masks are whole numbers and exact.  fp32 sums of int4 products with a
    16-bit intermediate: the draft and the prefill kernels, which add in different orders, differ on
    the same inputs by 2e-6 to 8e-6 (largest difference 2.8e-5).  bf16 results (verify): against
    64-bit sums 2.4e-3 (largest difference 8.8e-3).  Four to five times that."""
    return {"rel": 1e-2, "max": 4e-2} if case["kind"] in ("verify", "cycle") else {"rel": 4e-5, "max": 1.5e-4}


def _int4_codes(nbytes, group, gen):
    """Packed codes of RTN-quantised normal values (two a byte): bytes picked from a table of such pairs."""
    scale = RANGE[group] / 15.0
    pair = torch.randn((65536, 2), device="cuda", generator=gen).div_(scale).add_(7.5).round_().clamp_(0, 15).to(torch.uint8)
    table = pair[:, 0] | (pair[:, 1] << 4)
    out = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    for a in range(0, nbytes, 1 << 27):
        n = min(1 << 27, nbytes - a)
        out[a:a + n] = table.index_select(0, torch.randint(0, 65536, (n,), dtype=torch.int32, device="cuda", generator=gen))
    return out


def _int4_scales(nbytes, c, gen):
    n = nbytes // (2 if c["symmetric"] else 4)
    if c["symmetric"]:
        s = STD * RANGE[c["group"]] / 14.0
        return torch.randn(n, device="cuda", generator=gen).mul_(0.08 * s).add_(s).clamp_(0.5 * s, 1.5 * s).half()
    s = STD * RANGE[c["group"]] / 15.0
    scale = torch.randn(n, device="cuda", generator=gen).mul_(0.08 * s).add_(s).clamp_(0.5 * s, 1.5 * s).half()
    zero = torch.randn(n, device="cuda", generator=gen).mul_(0.8).add_(7.5).round_().clamp_(0, 15).half()
    return torch.stack([scale, zero], dim=-1).contiguous()


def _tokens(c, T, gen):
    x = torch.randn((T, c["hidden"]), device="cuda", generator=gen)
    if c["routing"] == "ar1":                          # neighbouring tokens share part of their routing
        for t in range(1, T if T <= 64 else 64):
            x[t] = 0.56 * x[t - 1] + math.sqrt(1 - 0.56 ** 2) * x[t]
    return x.bfloat16()


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    H, E, k, S, T, N = c["hidden"], c["experts"], c["top_k"], c["shared"], c["tokens"], c["layers"]
    st = {"case": c, "desc": _desc(c), "ctx": B.Context(torch.cuda.current_device()), "layers": []}
    desc = st["desc"]
    draft = c["kind"] != "verify"
    verify = c["kind"] in ("verify", "cycle")
    q_bytes, bf16_bytes = B.int4_expert_q_bytes(desc), B.bf16_expert_bytes(desc)
    sz_bytes = B.int4_expert_scale_bytes(desc) if c["symmetric"] else B.int4_expert_sz_bytes(desc)
    st["strides"] = (q_bytes, sz_bytes, bf16_bytes)
    if c["kind"] == "prefill":
        st["workspace"] = torch.empty(B.prefill_workspace_bytes(desc, T), dtype=torch.uint8, device="cuda")
    else:
        st["workspace"] = torch.empty(B.workspace_bytes(desc, T), dtype=torch.uint8, device="cuda")
        st["ctx"].workspace_init(st["workspace"])

    def bf16(n):
        return torch.empty(n // 2, dtype=torch.bfloat16, device="cuda").normal_(0.0, STD, generator=gen)

    out = {}
    Td = T - 1 if c["kind"] == "cycle" else T
    if draft:
        out["y"] = torch.zeros((N, Td, H), dtype=torch.float32, device="cuda")
        out["ids"] = torch.zeros((N, Td, k), dtype=torch.int32, device="cuda")
        out["conf"] = torch.zeros((N, Td, k), dtype=torch.float32, device="cuda")
    if verify:
        out["y_verify"] = torch.zeros((N, T, H), dtype=torch.bfloat16, device="cuda")
        out["ids_verify"] = torch.zeros((N, T, k), dtype=torch.int32, device="cuda")
        out["n_missing"] = torch.zeros((N, 1), dtype=torch.int32, device="cuda")
    if c["kind"] == "cycle":
        out["union_mask"] = torch.zeros((N, (E + 63) // 64), dtype=torch.int64, device="cuda")
        out["union_list"] = torch.zeros((N, E), dtype=torch.int32, device="cuda")
        out["union_n"] = torch.zeros((N, 1), dtype=torch.int32, device="cuda")
    st["out"] = out
    st["missing"] = torch.zeros(E, dtype=torch.int32, device="cuda")
    st["union_missing"] = (torch.zeros(E, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    for n in range(N):
        L = {"x": _tokens(c, T, gen), "bias": None, "shared": None}
        L["router"] = torch.randn((E, H), device="cuda", generator=gen).mul_(STD).bfloat16()
        if c["routing"] == "zipf":
            rank = torch.randperm(E, device="cuda", generator=gen).float() + 1.0
            pi = rank ** -1.1
            L["bias"] = torch.log(pi / pi.sum()).contiguous()
        if S:
            L["shared"] = bf16(S * bf16_bytes)
        if draft:
            L["q"] = _int4_codes(E * q_bytes, c["group"], gen)
            L["sz"] = _int4_scales(E * sz_bytes, c, gen)
        if verify:
            L["pool"] = bf16(E * bf16_bytes)
            L["slots"] = torch.randperm(E, device="cuda", generator=gen).to(torch.int32)
        for name, t in out.items():
            L[name] = t[n]
        if c["kind"] == "cycle":                       # each drafted token's views, as a decoding loop keeps them
            L["steps"] = [(L["x"][t:t + 1], L["y"][t:t + 1], L["ids"][t:t + 1], L["conf"][t:t + 1]) for t in range(T - 1)]
        st["layers"].append(L)
    return st


def _draft(st, L, x, T, y, ids, conf):
    q, sz, _ = st["strides"]
    st["ctx"].draft_layer_int4(st["desc"], x, L["router"], L["bias"], L["q"], L["sz"], q, sz, L["shared"], T,
                               y, ids, conf, st["workspace"], symmetric=st["case"]["symmetric"])


def _verify(st, L, T):
    st["ctx"].verify_layer_bf16(st["desc"], L["x"], L["router"], L["bias"], L["pool"], st["strides"][2], L["slots"],
                                L["shared"], T, 0, L["y_verify"], L["ids_verify"], st["missing"], L["n_missing"],
                                st["workspace"])


def run(st):
    c = st["case"]
    kind, T = c["kind"], c["tokens"]
    for L in st["layers"]:
        if kind == "draft":
            _draft(st, L, L["x"], T, L["y"], L["ids"], L["conf"])
        elif kind == "verify":
            _verify(st, L, T)
        elif kind == "prefill":
            q, sz, _ = st["strides"]
            st["ctx"].draft_prefill_int4(st["desc"], L["x"], L["router"], L["bias"], L["q"], L["sz"], q, sz, L["shared"],
                                         T, L["y"], L["ids"], L["conf"], st["workspace"], symmetric=c["symmetric"])
        else:
            for x, y, ids, conf in L["steps"]:
                _draft(st, L, x, 1, y, ids, conf)
            st["ctx"].expert_union(L["ids"], L["ids"].numel(), c["experts"], L["slots"], L["union_mask"], L["union_list"],
                                   L["union_n"], *st["union_missing"])
            _verify(st, L, T)
    return st["out"]
