"""Draft calls of several tokens that sum y in LDS over a workgroup's items: items of two experts in one workgroup, items of one
to eight tokens, row tiles that do not fill a window, a hidden size whose sums do not fit LDS, and infinite scales."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from synth.configs import LayerConfig
from tests.common import oracle_arrays, oracle_draft, rel_err
from tests.gpu_common import TOL_DRAFT, build_layer, say, to_np, tokens_with_clear_routing

pytestmark = pytest.mark.gpu

from paper_2511_14102_amd import binding as B          # noqa: E402
from paper_2511_14102_amd.harness import DeviceLayer   # noqa: E402

CASES = [
    #            idx  name       H     E  I     k  g    S  renorm
    (LayerConfig(81, "d3072", 3072, 8, 2816, 2, 128, 0, 1), (2, 3, 8)),     # 88 slices an expert: three items a workgroup, across experts
    (LayerConfig(82, "d2112", 2112, 2, 9856, 1, 32, 1, 1), (1, 2, 4, 5)),   # 33 row tiles over eight waves; many tokens in an expert
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
