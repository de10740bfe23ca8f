"""The draft call's own router and its shared experts at their edges.

Selection: expert counts around the 64-expert words, k up to E, logits that are equal, that differ
only below fp32 and that are -inf; ids against the oracle, exactly.  Shared experts of a one-token
call: hidden sizes with fewer k-steps or row tiles than waves, with a ragged last window and with more
than one window of down tiles; y against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as orc
from synth.configs import LayerConfig
from tests.common import oracle_arrays, oracle_draft, rel_err
from tests.draft_rules import rules
from tests.gpu_common import TOL_DRAFT, build_layer, say, to_np, tokens_with_clear_routing

pytestmark = pytest.mark.gpu

from paper_2511_14102_amd import binding as B          # noqa: E402
from paper_2511_14102_amd.harness import DeviceLayer   # noqa: E402


@pytest.mark.parametrize("E,k", [(1, 1), (8, 8), (63, 3), (65, 16), (128, 8), (129, 5), (256, 16)])
def test_selection_edges(E, k):
    cfg = LayerConfig(71, "sel%d" % E, 64, E, 64, k, 32, 0, 1)
    ctx = B.Context(0)
    L = synth.make_layer(cfg, 0)
    rng = np.random.default_rng(E)
    # integer logits from a narrow range: many exact ties; half the experts sit at 2^30, where fp32
    # cannot tell neighbouring integers apart
    router = rng.integers(-1, 2, (E, 64)).astype(np.float32)
    router[:, 0] = 2.0 ** 15 * rng.integers(0, 2, E)
    L["router"] = torch.from_numpy(router).to(torch.bfloat16)
    x = rng.integers(-1, 2, (8, 64)).astype(np.float32)
    x[:, 0] = 2.0 ** 15
    x[7] = 0.0                                             # all logits equal
    x = torch.from_numpy(x).to(torch.bfloat16)
    bias = np.zeros(E, np.float32)
    bias[rng.permutation(E)[: E // 2]] = -np.inf
    for b in (None, bias):
        L["router_bias"] = None if b is None else torch.from_numpy(b)
        D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False)
        A = oracle_arrays(L)
        ids, _, conf, _ = orc.route(orc.bits(x), A["router"], A["bias"], k, True)
        for T in (1, 3, min(8, 128 // k)):
            say("selection E", E, "k", k, "T", T, "bias" if b is not None else "")
            xs = x[8 - T:]
            r = D.draft(xs.cuda())
            torch.cuda.synchronize()
            assert np.array_equal(to_np(r["ids"]), ids[8 - T:])
            np.testing.assert_allclose(to_np(r["conf"]), conf[8 - T:], rtol=2e-6, atol=1e-30)
    ctx.close()


@pytest.mark.parametrize("H,I,g,S", [(64, 64, 32, 1), (192, 128, 64, 4), (320, 192, 32, 2), (2304, 128, 128, 1), (1088, 320, 64, 3)])
def test_one_token_with_shared_experts(H, I, g, S):
    cfg = LayerConfig(72, "sh%d" % H, H, 6, I, 2, g, S, 1)
    ctx = B.Context(0)
    L = synth.make_layer(cfg, 0)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=2, verify=False)
    x = tokens_with_clear_routing(cfg, A, 3, step=4)
    ref = oracle_draft(A, x)
    for t in range(3):
        say("shared H", H, "I", I, "g", g, "S", S, "token", t)
        r = D.draft(x[t:t + 1].cuda())
        torch.cuda.synchronize()
        assert np.array_equal(to_np(r["ids"]), ref["ids"][t:t + 1])
        assert rel_err(to_np(r["y"]), ref["y"][t:t + 1]) <= TOL_DRAFT
    ctx.close()


def one_token_form(cfg):
    """(whether the shared experts run inside, the form) of a one-token call on 256 units: 0 single items, 1 pairs, 2 persistent."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the forms are stated for 256 compute units")
    shape = (cfg.hidden, cfg.n_experts, cfg.inter, cfg.top_k, cfg.group_size, cfg.n_shared)
    inside = rules().rule_shared_inside(*shape, 256)
    return bool(inside), rules().rule_one_token_form(*shape, inside, 256, 512)


@pytest.mark.parametrize("H,I,k,g,S,form", [(128, 8192, 2, 32, 0, (False, 1)), (576, 8192, 2, 64, 0, (False, 1)), (128, 8192, 2, 32, 2, (True, 1)),
                                            (128, 8192, 1, 32, 4, (False, 1)), (1088, 5120, 4, 32, 0, (False, 2)), (2304, 8192, 2, 64, 0, (False, 2))])
def test_one_token_with_many_items(H, I, k, g, S, form):
    """256 to 640 work items of routed experts, then three tokens: short rows run as pairs, with two shared experts inside and with
    four, which are more 16-row items than the call's own launch takes; longer rows run in the persistent kernel, without sums of y in LDS and with."""
    cfg = LayerConfig(73, "many%d" % H, H, 4, I, k, g, S, 1)
    assert one_token_form(cfg) == form
    ctx = B.Context(0)
    for symmetric in (False, True):
        if symmetric and B.int4_expert_scale_bytes(B.LayerDesc.from_config(cfg)) == 0:
            continue
        L = synth.make_layer(cfg, 0, symmetric=symmetric)
        A = oracle_arrays(L)
        D = DeviceLayer(ctx, cfg, L, max_tokens=3, verify=False, symmetric=symmetric)
        x = tokens_with_clear_routing(cfg, A, 3, step=6)
        ref = oracle_draft(A, x)
        for t0, t1 in ((0, 1), (1, 2), (0, 3)):
            say("many items H", H, "S", S, "symmetric" if symmetric else "", "tokens", t0, t1)
            r = D.draft(x[t0:t1].cuda())
            torch.cuda.synchronize()
            assert np.array_equal(to_np(r["ids"]), ref["ids"][t0:t1])
            assert rel_err(to_np(r["y"]), ref["y"][t0:t1]) <= TOL_DRAFT
    ctx.close()


@pytest.mark.parametrize("g", [32, 64, 128])
def test_stream_windows_of_eight(g):
    """H = 2304: 9 to 12 gate/up and 4 to 6 down tiles per wave, ragged parts under the window of eight (the other
    small shapes of these group sizes run the window of four)."""
    cfg = LayerConfig(79, "win%d" % g, 2304, 5, 128, 2, g, 0, 1)
    ctx = B.Context(0)
    for symmetric in (False, True):
        L = synth.make_layer(cfg, 0, symmetric=symmetric)
        A = oracle_arrays(L)
        D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False, symmetric=symmetric)
        x = tokens_with_clear_routing(cfg, A, 8, step=3)
        ref = oracle_draft(A, x)
        for T in (2, 3, 8):
            say("window of eight g", g, "symmetric" if symmetric else "", "T", T)
            r = D.draft(x[:T].cuda())
            torch.cuda.synchronize()
            assert np.array_equal(to_np(r["ids"]), ref["ids"][:T])
            assert rel_err(to_np(r["y"]), ref["y"][:T]) <= TOL_DRAFT
    ctx.close()


@pytest.mark.parametrize("H,I,E,k,g,S", [(64, 4096, 3, 2, 32, 0), (320, 2048, 4, 4, 64, 0), (2112, 2752, 5, 3, 64, 0), (1024, 4160, 6, 4, 32, 0),
                                         (320, 2048, 8, 8, 64, 0), (576, 5120, 6, 5, 64, 0),
                                         (512, 2048, 4, 1, 64, 2), (2304, 1024, 8, 8, 128, 2), (192, 8192, 3, 2, 64, 2),
                                         (192, 1024, 128, 1, 64, 4), (64, 1024, 67, 2, 32, 4), (1088, 2048, 9, 1, 32, 4)])
def test_one_token_with_pairs_of_items(H, I, E, k, g, S):
    """Calls of one token with 256 work items and more, which run two items per workgroup: fewer row tiles or groups than waves, ragged
    shares of both, exactly 256 and 512 items, more than two per unit (520 and 800, short rows), and shared experts beside the routed ones; two router rows to a
    workgroup, an odd last one, and several rounds of them (128 and 67 experts over 16 and 32 routed workgroups)."""
    cfg = LayerConfig(81, "pair%d" % H, H, E, I, k, g, S, 1)
    assert one_token_form(cfg) == (S > 0, 1)
    ctx = B.Context(0)
    for symmetric in (False, True):
        if symmetric and B.int4_expert_scale_bytes(B.LayerDesc.from_config(cfg)) == 0:
            continue
        L = synth.make_layer(cfg, 0, symmetric=symmetric)
        A = oracle_arrays(L)
        D = DeviceLayer(ctx, cfg, L, max_tokens=1, verify=False, symmetric=symmetric)
        x = tokens_with_clear_routing(cfg, A, 2, step=6)
        ref = oracle_draft(A, x)
        for t in (0, 1, 0):
            say("pairs H", H, "I", I, "S", S, "symmetric" if symmetric else "", "token", t)
            r = D.draft(x[t:t + 1].cuda())
            torch.cuda.synchronize()
            assert np.array_equal(to_np(r["ids"]), ref["ids"][t:t + 1])
            assert rel_err(to_np(r["y"]), ref["y"][t:t + 1]) <= TOL_DRAFT
    ctx.close()


@pytest.mark.parametrize("H,E,T,g", [(192, 16, 8, 32), (3136, 60, 7, 64), (2176, 100, 5, 128), (1088, 200, 3, 32), (64, 256, 8, 32), (4224, 5, 2, 128)])
def test_router_rows_shared_out_by_tokens(H, E, T, g):
    """A workgroup's waves shared out over the tokens of its router row, a power of two of them or fewer; x in one round of a
    workgroup's loads and in several, the last one ragged."""
    cfg = LayerConfig(80, "rows%d" % E, H, E, 256, min(8, E), g, 0, 1)
    ctx = B.Context(0)
    L = build_layer(cfg)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=T, verify=False)
    x = tokens_with_clear_routing(cfg, A, T, step=5)
    ref = oracle_draft(A, x)
    say("router rows H", H, "E", E, "T", T)
    for again in range(2):                                 # (the second call finds the exchange slots as the first left them)
        r = D.draft(x.cuda())
        torch.cuda.synchronize()
        assert np.array_equal(to_np(r["ids"]), ref["ids"])
        assert rel_err(to_np(r["y"]), ref["y"]) <= TOL_DRAFT
    ctx.close()


@pytest.mark.parametrize("H,I,k,S,g,inside", [(1024, 8192, 1, 2, 128, True),
                                              (256, 7168, 2, 4, 64, True), (256, 7232, 2, 4, 64, False),
                                              (1024, 8192, 2, 4, 64, True), (1024, 8256, 2, 4, 64, False),
                                              (2304, 9216, 2, 4, 64, True), (2304, 9280, 2, 4, 64, False)])
def test_shared_experts_on_the_line_run_inside(H, I, k, S, g, inside):
    """On 256 units: as many 16-row items as H has 256s per unit; seven per unit, as pairs, and one step more; as many as H has 128s, and
    one step more; rows too long for pairs, on the line of single items (9 per unit) and one step beyond.  Up to the line the call's own launch
    runs the shared experts and no launch of the bf16 kernels is made; beyond, the routed experts run alone (as pairs, or in the persistent
    launch) and leave the plan for the bf16 kernels."""
    cfg = LayerConfig(74, "line", H, 2, I, k, g, S, 1)
    assert one_token_form(cfg)[0] == inside
    ctx = B.Context(0)
    L = build_layer(cfg)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=1, verify=False)
    x = tokens_with_clear_routing(cfg, A, 1, step=2)
    ref = oracle_draft(A, x)
    say("line of shared experts H", H, "I", I)
    ctx.profile_enable(True)
    r = D.draft(x.cuda())
    torch.cuda.synchronize()
    launches = {name: n for name, (_, n) in ctx.profile_read().items()}
    ctx.profile_enable(False)
    assert np.array_equal(to_np(r["ids"]), ref["ids"])
    assert rel_err(to_np(r["y"]), ref["y"]) <= TOL_DRAFT
    assert launches["draft_fused_kernel"] == 1 and launches["bf16_gateup_kernel"] == (0 if inside else 1)
    ctx.close()


@pytest.mark.parametrize("H,g,S", [(1472, 32, 0), (1536, 32, 0), (1600, 64, 0), (1536, 128, 0), (1472, 64, 2), (1536, 64, 2), (1600, 32, 2)])
def test_pairs_around_the_line_of_long_rows(H, g, S):
    """Pairs carry h as two bf16 numbers up to H = 1472 and as four e4m3 planes from 1536 on (three row tiles per wave; at 1600 one wave has four): 272 items, and
    128 with two shared experts of 128 each beside them."""
    cfg = LayerConfig(83, "line%d" % H, H, 4, 4352 if S == 0 else 2048, 2, g, S, 1)
    assert one_token_form(cfg) == (S > 0, 1)
    ctx = B.Context(0)
    for symmetric in (False, True):
        if symmetric and B.int4_expert_scale_bytes(B.LayerDesc.from_config(cfg)) == 0:
            continue
        L = synth.make_layer(cfg, 0, symmetric=symmetric)
        A = oracle_arrays(L)
        D = DeviceLayer(ctx, cfg, L, max_tokens=1, verify=False, symmetric=symmetric)
        x = tokens_with_clear_routing(cfg, A, 2, step=6)
        ref = oracle_draft(A, x)
        for t in (0, 1, 0):
            say("line H", H, "g", g, "S", S, "symmetric" if symmetric else "", "token", t)
            r = D.draft(x[t:t + 1].cuda())
            torch.cuda.synchronize()
            assert np.array_equal(to_np(r["ids"]), ref["ids"][t:t + 1])
            assert rel_err(to_np(r["y"]), ref["y"][t:t + 1]) <= TOL_DRAFT
    ctx.close()
