"""The grouped contraction of the prefill call at the edges of its tiles: k-steps that do not fill a
stage, group sums that do not fill a tile of four groups, slices and row tiles that do not fill a
workgroup's four, and items of 1 to 32 (small calls) or 64 tokens (whole and ragged token blocks,
several items per expert), for every group size and both weight formats."""
import numpy as np
import pytest
import torch

import synth
from synth.configs import LayerConfig
from tests.common import oracle_arrays, oracle_draft, rel_err
from tests.gpu_common import TOL_DRAFT, Guarded, build_layer, say, to_np, tokens_with_clear_routing

pytestmark = pytest.mark.gpu

from paper_2511_14102_amd import binding as B          # noqa: E402
from paper_2511_14102_amd.harness import DeviceLayer   # noqa: E402

SHAPES = [
    #            idx  name    H    E   I   k   g  S  renorm
    LayerConfig(61, "p64", 64, 3, 64, 1, 32, 0, 1),        # fewer k-steps than one stage, one row tile
    LayerConfig(62, "p192", 192, 5, 320, 2, 64, 2, 1),     # 3 and 5 groups, 10 slices, two shared experts
    LayerConfig(63, "p320", 320, 2, 192, 2, 32, 0, 0),     # 10 groups, every token in both experts
    LayerConfig(64, "p640", 640, 4, 384, 2, 128, 0, 1),    # 5 and 3 groups, 12 slices
    LayerConfig(65, "p256", 256, 40, 128, 3, 128, 0, 1),   # many experts with a token or two
]


@pytest.mark.parametrize("cfg", SHAPES, ids=[c.name for c in SHAPES])
def test_prefill_tile_edges(cfg):
    ctx = B.Context(0)
    sizes = (1, 15, 33, 64, 150)
    for symmetric in (False, True):
        if symmetric and B.int4_expert_scale_bytes(B.LayerDesc.from_config(cfg)) == 0:
            continue
        L = synth.make_layer(cfg, 0, symmetric=symmetric)
        A = oracle_arrays(L)
        D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False, symmetric=symmetric)
        x = tokens_with_clear_routing(cfg, A, max(sizes), step=3, kind="iid")
        ref = oracle_draft(A, x)
        for T in sizes:
            say("prefill", cfg.name, "symmetric" if symmetric else "", "T", T)
            r = D.prefill(x[:T].cuda())
            torch.cuda.synchronize()
            assert np.array_equal(to_np(r["ids"]), ref["ids"][:T])
            assert rel_err(to_np(r["y"]), ref["y"][:T]) <= TOL_DRAFT
    ctx.close()


WIDE = [
    #            idx  name    H    E   I    k   g  S  renorm    (enough weight columns for items of 64 tokens)
    LayerConfig(76, "w32", 384, 5, 1280, 2, 32, 0, 1),     # 12 and 40 groups, 6 row tiles
    LayerConfig(77, "w64", 256, 5, 1344, 2, 64, 1, 1),     # 4 and 21 groups, 42 slices, a shared expert
    LayerConfig(78, "w128", 640, 5, 1152, 2, 128, 0, 1),   # 5 and 9 groups, 36 slices, 10 row tiles
    LayerConfig(79, "v128", 256, 5, 1280, 2, 128, 2, 0),   # 2 and 10 groups, both formats
]


@pytest.mark.parametrize("cfg", WIDE, ids=[c.name for c in WIDE])
def test_prefill_long_items(cfg):
    """Items of up to 64 tokens: the experts' counts leave items of one to four token blocks."""
    ctx = B.Context(0)
    blocks = set()
    for symmetric in (False, True):
        if symmetric and B.int4_expert_scale_bytes(B.LayerDesc.from_config(cfg)) == 0:
            continue
        L = synth.make_layer(cfg, 0, symmetric=symmetric)
        A = oracle_arrays(L)
        D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False, symmetric=symmetric)
        x = tokens_with_clear_routing(cfg, A, 477, step=9, kind="iid")
        ref = oracle_draft(A, x)
        for T in (400, 431, 477):
            say("prefill", cfg.name, "symmetric" if symmetric else "", "T", T)
            r = D.prefill(x[:T].cuda())
            torch.cuda.synchronize()
            assert np.array_equal(to_np(r["ids"]), ref["ids"][:T])
            assert rel_err(to_np(r["y"]), ref["y"][:T]) <= TOL_DRAFT
            blocks |= {(c % 64 + 15) // 16 for c in np.bincount(ref["ids"][:T].ravel(), minlength=5)}
    assert blocks >= {1, 2, 3, 4}
    ctx.close()


ROUTED = [
    #            idx  name    H    E   I   k   g  S  renorm     (large enough for the two-launch routing)
    LayerConfig(66, "r70", 320, 70, 64, 3, 32, 0, 1),      # ragged token and expert blocks, k-steps that do not fill a share
    LayerConfig(67, "r130", 192, 130, 64, 4, 64, 1, 0),    # more than 128 experts, a shared expert
    LayerConfig(68, "r5", 2112, 5, 64, 5, 64, 2, 1),       # few experts, shares of H, every token in every expert
    LayerConfig(80, "r72", 512, 72, 1024, 6, 128, 1, 1),   # more than 64 experts with one to four token blocks left
    LayerConfig(70, "r4160", 4160, 4, 64, 2, 64, 0, 1),    # the most shares of H (8 x 4 waves), 130 k-steps over them
]


@pytest.mark.parametrize("cfg", ROUTED, ids=[c.name for c in ROUTED])
def test_prefill_routing_edges(cfg):
    ctx = B.Context(0)
    L = synth.make_layer(cfg, 0)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False)
    x = tokens_with_clear_routing(cfg, A, 421, step=5, kind="iid")
    ref = oracle_draft(A, x)
    ws = Guarded(max(B.prefill_workspace_bytes(D.desc, T) for T in (257, 420, 421)))
    D._prefill_ws = ws.view                                # (one workspace for all of them)
    for T in (257, 420, 421):
        say("prefill routing", cfg.name, "T", T)
        assert B.prefill_workspace_bytes(D.desc, T) <= B.prefill_workspace_bytes(D.desc, 421)
        r = D.prefill(x[:T].cuda())
        torch.cuda.synchronize()
        assert ws.intact() and D._prefill_ws is ws.view
        assert np.array_equal(to_np(r["ids"]), ref["ids"][:T])
        np.testing.assert_allclose(to_np(r["conf"]), ref["conf"][:T], rtol=2e-6)
        assert rel_err(to_np(r["y"]), ref["y"][:T]) <= TOL_DRAFT
    ctx.close()


@pytest.mark.parametrize("H,I,g,symmetric", [(4096, 128, 32, False), (4096, 128, 128, False), (4096, 128, 64, True),
                                             (128, 8192, 32, False), (256, 8192, 128, True)])
def test_prefill_sums_of_tokens_with_a_mean(H, I, g, symmetric):
    """The zero points are cancelled as the sums grow: with activations that have a mean (x: 0.3 of its
    deviation; h where H is small: up = gate, so that h >= 0) the long-run call is as close to the 64-bit sums as the draft call, which cancels them group by
    group.  (Cancelled behind all groups, the error was several times as large.)  Both keep h as two bf16 numbers, so
    most of either error is that rounding; an eighth more than the draft call's leaves room for the order of the sums."""
    cfg = LayerConfig(69, "mean%d" % H, H, 4, I, 2, g, 0, 1)
    ctx = B.Context(0)
    L = synth.make_layer(cfg, 0, symmetric=symmetric)
    if H < I:
        for n in ("q_", "s_", "z_"):
            L[n + "up"] = L[n + "gate"]
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=4, verify=False, symmetric=symmetric)
    x = (tokens_with_clear_routing(cfg, A, 48, step=7, kind="iid").float() + 0.3).bfloat16()
    ref = oracle_draft(A, x)["y"]
    err = lambda y: np.linalg.norm(y - ref) / np.linalg.norm(ref)
    long_run = err(to_np(D.prefill(x.cuda())["y"]))
    short = err(np.concatenate([to_np(D.draft(x[t:t + 4].cuda())["y"]) for t in range(0, 48, 4)]))
    say("prefill %.3e draft %.3e" % (long_run, short))
    assert long_run <= 1.125 * short
    ctx.close()


@pytest.mark.parametrize("g", [32, 64, 128])
@pytest.mark.parametrize("symmetric", [False, True])
def test_prefill_magnitudes(g, symmetric):
    """Tokens far from unit size, with values far from each other in a group, with groups of zeros, and with an infinite value.  Every finite
    token is as close to the 64-bit sums as one of N(0,1): x is exact, h has at least 16 significant bits (2.5e-6 of its norm), and the fp32 sums
    of 1280 and 640 products leave less than that: together below 1e-5 of a token's y."""
    cfg = LayerConfig(94, "mag%d" % g, 1280, 3, 640, 2, g, 0, 1)      # 10 and 5 groups of 128
    ctx = B.Context(0)
    L = synth.make_layer(cfg, 0, symmetric=symmetric)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=4, verify=False, symmetric=symmetric)
    x = tokens_with_clear_routing(cfg, A, 75, step=19, kind="iid").float()
    gen = torch.Generator().manual_seed(5)
    for t in range(0, 40):
        x[t] *= 2.0 ** (t - 20)
    for t in range(40, 50):                                          # one value far above the rest of its group
        x[t, 7 + 128 * (t - 40)] *= 300.0
    x[50:60, 128:256] = 0.0
    x[60:65] *= 2.0 ** torch.randint(-9, 3, (5, cfg.hidden), generator=gen)
    x[65:70, ::100] *= 100.0
    x[70] = 0.0
    x = x.bfloat16()
    ref = oracle_draft(A, x)
    x[74, 300] = float("inf")
    say("prefill magnitudes", g, "symmetric" if symmetric else "")
    r = D.prefill(x.cuda())
    y = to_np(r["y"])
    same = [t for t in range(74) if t != 70 and np.array_equal(to_np(r["ids"])[t], ref["ids"][t])]
    assert len(same) == 73 and not np.any(y[70])
    err = np.linalg.norm(y[same] - ref["y"][same], axis=1) / np.linalg.norm(ref["y"][same], axis=1)
    say("   worst token %.3e" % err.max())
    assert err.max() <= 1e-5
    assert np.isnan(y[74]).all()
    ctx.close()


PLACES = [
    #            idx  name     H    E   I   k  g    S  renorm
    (LayerConfig(86, "q32", 384, 3, 384, 2, 32, 0, 1), 150),       # items of 32 tokens, 12 groups
    (LayerConfig(87, "q64", 640, 5, 1344, 2, 64, 1, 1), 431),      # items of 64, 10 and 21 groups, a shared expert
    (LayerConfig(88, "q128", 1152, 5, 1280, 2, 128, 0, 1), 400),   # 9 and 10 groups
]


@pytest.mark.parametrize("cfg,T", PLACES, ids=[c[0].name for c in PLACES])
def test_prefill_does_not_depend_on_a_tokens_place(cfg, T):
    """A token's y, ids and confidences are the same bits wherever it stands in the prompt, and so in its experts' items
    (the place there is drawn from a counter, so that calls on the same prompt differ in it)."""
    ctx = B.Context(0)
    for symmetric in (False, True):
        if symmetric and B.int4_expert_scale_bytes(B.LayerDesc.from_config(cfg)) == 0:
            continue
        D = DeviceLayer(ctx, cfg, synth.make_layer(cfg, 0, symmetric=symmetric), max_tokens=8, verify=False, symmetric=symmetric)
        x = synth.make_tokens(cfg, T, step=13, kind="iid").cuda()
        first = D.prefill(x)
        for seed in range(3):
            perm = torch.randperm(T, generator=torch.Generator().manual_seed(seed)).cuda()
            say("prefill", cfg.name, "symmetric" if symmetric else "", "order", seed)
            r = D.prefill(x[perm].contiguous())
            torch.cuda.synchronize()
            for n in ("ids", "conf", "y"):
                assert torch.equal(r[n], first[n][perm]), n
    ctx.close()


ORDERS = [
    #            idx  name      H    E   I    k  g   S  renorm     tokens, largest items first, items by the sorting kernel
    (LayerConfig(89, "o768", 768, 72, 1024, 6, 128, 1, 1), 421, True, False),     # every kind of rest, a shared expert
    (LayerConfig(90, "o4096s", 4096, 8, 128, 2, 64, 4, 1), 120, True, True),
    (LayerConfig(91, "o4096", 4096, 16, 64, 2, 32, 0, 1), 300, True, False),      # no shared experts
    (LayerConfig(92, "o128", 128, 48, 4096, 8, 32, 0, 1), 300, False, False),     # more than three and a half rounds
    (LayerConfig(93, "o192", 192, 20, 8192, 2, 64, 1, 1), 280, False, True),
    (LayerConfig(95, "o1280", 1280, 20, 4096, 1, 128, 0, 1), 1500, True, False),  # largest first, in striped blocks
]


@pytest.mark.parametrize("cfg,T,by_size,sorted_by_kernel", ORDERS, ids=[c[0].name for c in ORDERS])
def test_prefill_orders_of_the_items(cfg, T, by_size, sorted_by_kernel):
    """Items of 64 tokens in both orders, from the stage kernel and from the sorting kernel, with runs of no and of several
    whole items and rests of one to four token blocks (experts of falling popularity)."""
    cols = max(-(-cfg.inter // 128), -(-cfg.hidden // 256))
    items = lambda n: T * cfg.top_k // n + min(cfg.n_experts, T * cfg.top_k) + cfg.n_shared * -(-T // n)
    assert cols * items(32) > 256                          # items of 64
    assert (cols * items(64) < 1792 and -(-cfg.hidden // 256) * items(64) > 200
            and (cfg.n_shared > 0 or T * cfg.top_k >= 16 * cfg.n_experts)) == by_size
    assert (T * (cfg.n_experts * cfg.hidden + 1024 * cfg.top_k) < 4 << 20) == sorted_by_kernel
    ctx = B.Context(0)
    L = build_layer(cfg, bias="zipf")
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False)
    x = tokens_with_clear_routing(cfg, A, T, step=17, kind="iid")
    ref = oracle_draft(A, x)
    counts = np.bincount(ref["ids"].ravel(), minlength=cfg.n_experts)
    say("prefill", cfg.name, "T", T, "counts", counts.tolist())
    assert counts.max() > 64 and counts.min() < 16 and len({(c % 64 + 15) // 16 for c in counts} - {0}) >= 3
    ws = Guarded(B.prefill_workspace_bytes(D.desc, T))
    D._prefill_ws = ws.view
    for _ in range(2):
        ws.view.fill_(0xff)
        r = D.prefill(x.cuda())
        torch.cuda.synchronize()
        assert ws.intact() and np.array_equal(to_np(r["ids"]), ref["ids"])
        assert rel_err(to_np(r["y"]), ref["y"]) <= TOL_DRAFT
    ctx.close()
