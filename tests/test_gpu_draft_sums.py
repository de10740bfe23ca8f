"""Draft calls of several tokens that sum y in LDS over a workgroup's items: items of two experts in one workgroup, items of one
to eight tokens, row tiles that do not fill a window, a hidden size whose sums do not fit LDS, and infinite scales."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as orc
from synth.configs import LayerConfig
from tests.common import oracle_arrays, oracle_draft, rel_err
from tests.gpu_common import TOL_DRAFT, build_layer, say, to_np, tokens_with_clear_routing

pytestmark = pytest.mark.gpu

from paper_2511_14102_amd import binding as B          # noqa: E402
from paper_2511_14102_amd.harness import DeviceLayer   # noqa: E402

CASES = [
    #            idx  name       H     E  I     k  g    S  renorm
    # 88 slices an expert: up to three items a workgroup, across experts (2 tokens: too few items for sums)
    (LayerConfig(81, "d3072", 3072, 8, 2816, 2, 128, 0, 1), (2, 3, 8)),
    # 33 row tiles over eight waves; many tokens in an expert (1 token: too few items)
    (LayerConfig(82, "d2112", 2112, 2, 9856, 1, 32, 1, 1), (1, 2, 4, 5)),
    (LayerConfig(83, "d6144", 6144, 6, 2816, 2, 128, 0, 1), (3,)),          # the sums of four slots do not fit
]


@pytest.mark.parametrize("cfg,tokens", CASES, ids=[c[0].name for c in CASES])
def test_draft_sums(cfg, tokens):
    ctx = B.Context(0)
    L = build_layer(cfg)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False)
    x = tokens_with_clear_routing(cfg, A, max(tokens), step=11)
    ref = oracle_draft(A, x)
    for T in tokens:
        say("draft", cfg.name, "T", T)
        r = D.draft(x[:T].cuda())
        torch.cuda.synchronize()
        assert np.array_equal(to_np(r["ids"]), ref["ids"][:T])
        assert rel_err(to_np(r["y"]), ref["y"][:T]) <= TOL_DRAFT
    ctx.close()


def test_draft_sums_of_an_expert_with_infinite_scales():
    """A workgroup's items 306 and 307 are the one-token expert 0's and its item 308 is expert 1's: nothing of
    expert 0, whose scales are infinite, stays in the sums of a token slot that it leaves empty."""
    cfg = LayerConfig(84, "d2112inf", 2112, 2, 9856, 1, 32, 0, 1)
    ctx = B.Context(0)
    L = build_layer(cfg)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False)
    x = tokens_with_clear_routing(cfg, A, 16, step=12)
    ids = orc.route(orc.bits(x), A["router"], A["bias"], 1, 1)[0].reshape(-1)
    a, b = int(np.flatnonzero(ids == 0)[0]), int(np.flatnonzero(ids == 1)[0])
    x = x[[a, b, b]].contiguous()
    ref = oracle_draft(A, x)
    D.sz_blob[:D.sz_bytes].view(torch.float16).fill_(float("inf"))
    say("draft", cfg.name, "tokens", a, b)
    r = D.draft(x.cuda())
    torch.cuda.synchronize()
    assert np.array_equal(to_np(r["ids"]), ref["ids"])
    assert not np.isfinite(to_np(r["y"])[0]).any()
    assert rel_err(to_np(r["y"])[1:], ref["y"][1:]) <= TOL_DRAFT
    ctx.close()


FORMATS = [
    #            idx  name       H     E  I     k  g   S  renorm   (33 and 34 row tiles over eight waves, 130 slices an expert)
    (LayerConfig(94, "d64", 2112, 4, 4160, 2, 64, 0, 1), False),
    (LayerConfig(95, "d64s", 2176, 4, 4160, 2, 64, 0, 1), True),
    (LayerConfig(96, "d32s", 2176, 4, 4160, 2, 32, 0, 1), True),
    (LayerConfig(97, "d128s", 3328, 4, 4224, 2, 128, 1, 1), True),
]


def summed(cfg, T, symmetric):
    """The rule of the library: two items a compute unit, and a window of eight tiles that is no more than a fifth padding."""
    epl, up = 2 if symmetric else 1, lambda a, b: -(-a // b)
    gate = up(cfg.hidden // cfg.group_size // epl, 8) * epl * (cfg.group_size // 32)
    down = up(cfg.hidden // 64 // epl, 8) * epl
    positions = lambda w: up(gate, w) * w + up(down, w) * w
    items = min(cfg.n_experts, T * cfg.top_k) * (cfg.inter // 32)
    return items >= 2 * torch.cuda.get_device_properties(0).multi_processor_count and positions(8) * 5 <= positions(4) * 6


@pytest.mark.parametrize("cfg,symmetric", FORMATS, ids=[c[0].name for c in FORMATS])
def test_draft_sums_of_the_formats(cfg, symmetric):
    """Group sizes and formats that the other cases leave out, two, three and four, and up to eight tokens."""
    ctx = B.Context(0)
    L = synth.make_layer(cfg, 0, symmetric=symmetric, quant_device="cuda:0")
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=8, verify=False, symmetric=symmetric)
    x = tokens_with_clear_routing(cfg, A, 8, step=14)
    ref = oracle_draft(A, x)
    for T in (2, 3, 4, 5, 8):
        assert summed(cfg, T, symmetric)
        say("draft", cfg.name, "T", T)
        r = D.draft(x[:T].cuda())
        torch.cuda.synchronize()
        assert np.array_equal(to_np(r["ids"]), ref["ids"][:T])
        assert rel_err(to_np(r["y"]), ref["y"][:T]) <= TOL_DRAFT
    ctx.close()
