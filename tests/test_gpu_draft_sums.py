"""Draft calls of several tokens that sum y in LDS over a workgroup's items: items of two experts in one workgroup, items of one
to eight tokens, row tiles that do not fill a window, and a hidden size whose sums do not fit LDS."""
import numpy as np
import pytest
import torch

from synth.configs import LayerConfig
from tests.common import oracle_arrays, oracle_draft, rel_err
from tests.gpu_common import TOL_DRAFT, build_layer, say, to_np, tokens_with_clear_routing

pytestmark = pytest.mark.gpu

from paper_2511_14102_amd import binding as B          # noqa: E402
from paper_2511_14102_amd.harness import DeviceLayer   # noqa: E402

CASES = [
    #            idx  name       H     E  I     k  g    S  renorm
    (LayerConfig(81, "d3072", 3072, 8, 2816, 2, 128, 0, 1), (2, 3, 8)),     # 88 slices an expert: three items a workgroup, across experts
    (LayerConfig(82, "d3136", 3136, 3, 128, 2, 64, 1, 1), (1, 2, 4, 5)),    # 49 row tiles over eight waves; most tokens in every expert
    (LayerConfig(83, "d6144", 6144, 4, 256, 2, 128, 0, 1), (2, 3)),         # the sums of four slots do not fit
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
