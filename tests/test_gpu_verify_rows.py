"""The verify call where its launches can go wrong: one and two blocks of tokens in the router, more experts than a wave
has lanes, K shares that are no whole batches of tiles, nothing to add up, and arrival counters that share a tag (more
columns than the smallest workspace has exchange slots)."""
import numpy as np
import pytest
import torch

from synth.configs import LayerConfig
import synth
from tests.common import oracle_arrays, oracle_verify, rel_err
from tests.gpu_common import TOL_VERIFY, say, to_np, tokens_with_clear_routing

pytestmark = pytest.mark.gpu

from paper_2511_14102_amd import binding as B          # noqa: E402
from paper_2511_14102_amd.harness import DeviceLayer   # noqa: E402

CASES = [
    #            idx  name          H      E    I    k  g   S  renorm
    (LayerConfig(61, "v64", 64, 3, 64, 1, 32, 0, 1), (1, 16)),
    (LayerConfig(62, "v256e", 128, 256, 64, 8, 64, 0, 1), (9, 16)),
    (LayerConfig(63, "v448", 448, 20, 384, 3, 64, 4, 0), (8, 9)),
    (LayerConfig(64, "v32768", 32768, 2, 64, 1, 64, 0, 1), (2,)),
]


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def idle(D):
    n = B.workspace_idle_bytes(D.desc)
    tags = D.workspace[512:n].view(torch.int64).reshape(-1, 2)[:, 1]
    return int(D.workspace[:512].count_nonzero().item()) == 0 and int(tags.count_nonzero().item()) == 0


@pytest.mark.parametrize("cfg,tokens", CASES, ids=[c[0].name for c in CASES])
def test_verify_rows(ctx, cfg, tokens):
    E, S = cfg.n_experts, cfg.n_shared
    L = synth.make_layer(cfg, 0, quantize=False)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=max(tokens), draft=False)
    table = D.slot_of_expert.clone()
    for T in tokens:
        say("verify", cfg.name, "T", T)
        x = tokens_with_clear_routing(cfg, A, T, step=3 + T)
        ref = oracle_verify(A, x)
        r = D.verify(x.cuda())
        torch.cuda.synchronize()
        assert np.array_equal(to_np(r["ids"]), ref["ids"]) and int(r["n_missing"].item()) == 0
        assert rel_err(to_np(r["y"]), ref["y"]) <= TOL_VERIFY
        assert idle(D)
        # no routed expert resident: only the shared experts' terms, every chosen expert reported ...
        D.slot_of_expert.fill_(-1)
        part = oracle_verify(A, x, present=np.zeros(E, np.uint8))
        r0 = D.verify(x.cuda(), y=torch.full((T, cfg.hidden), 7.0, dtype=torch.bfloat16, device="cuda"))
        torch.cuda.synchronize()
        chosen = sorted(set(ref["ids"].reshape(-1).tolist()))
        nm = int(r0["n_missing"].item())
        assert to_np(r0["missing"])[:nm].tolist() == chosen
        if S:
            assert rel_err(to_np(r0["y"]), part["y"]) <= TOL_VERIFY
        else:
            assert int(r0["y"].count_nonzero().item()) == 0
        # ... a call for listed experts with none of them resident adds nothing and lists them again ...
        before = r0["y"].clone()
        D.verify(x.cuda(), flags=B.MOE_VERIFY_ACCUMULATE | B.MOE_VERIFY_ONLY_LISTED, y=r0["y"])
        torch.cuda.synchronize()
        assert torch.equal(r0["y"], before) and to_np(D.missing)[:int(D.n_missing.item())].tolist() == chosen
        # ... and with all of them resident completes y
        D.slot_of_expert.copy_(table)
        D.verify(x.cuda(), flags=B.MOE_VERIFY_ACCUMULATE | B.MOE_VERIFY_ONLY_LISTED, y=r0["y"])
        torch.cuda.synchronize()
        assert int(D.n_missing.item()) == 0 and idle(D)
        assert rel_err(to_np(r0["y"]), ref["y"]) <= TOL_VERIFY


def test_verify_layers_of_different_expert_counts_share_a_workspace(ctx):
    """The rows of the layer of few experts lie where the other layer's exchange slots, and the arrival counters in their
    tags, are."""
    cfgs = (LayerConfig(85, "v2", 448, 2, 384, 1, 64, 0, 1), LayerConfig(63, "v448", 448, 20, 384, 3, 64, 4, 0))
    layers = []
    for cfg in cfgs:
        L = synth.make_layer(cfg, 0, quantize=False)
        A = oracle_arrays(L)
        x = tokens_with_clear_routing(cfg, A, 9, step=5)
        layers.append((DeviceLayer(ctx, cfg, L, max_tokens=9, draft=False), x.cuda(), oracle_verify(A, x)))
    ws = max((D.workspace for D, _, _ in layers), key=lambda w: w.numel())
    assert B.workspace_idle_bytes(layers[0][0].desc) < B.workspace_idle_bytes(layers[1][0].desc)
    ctx.workspace_init(ws)
    for D, x, ref in layers * 3:
        say("verify", D.cfg.name)
        D.workspace = ws
        r = D.verify(x, y=torch.full((9, 448), 7.0, dtype=torch.bfloat16, device="cuda"))
        torch.cuda.synchronize()
        assert np.array_equal(to_np(r["ids"]), ref["ids"]) and rel_err(to_np(r["y"]), ref["y"]) <= TOL_VERIFY
