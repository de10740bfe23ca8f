"""A token of NaNs: its logits are all NaN.  Every call still selects k distinct experts for it (the lists
behind the routing are indexed by them), its output is NaN, and the other tokens' results are theirs."""
import numpy as np
import pytest
import torch

import synth
from synth.configs import LayerConfig
from tests.common import oracle_arrays, oracle_draft, oracle_verify, rel_err
from tests.gpu_common import TOL_DRAFT, TOL_VERIFY, say, to_np, tokens_with_clear_routing

pytestmark = pytest.mark.gpu

from paper_2511_14102_amd import binding as B          # noqa: E402
from paper_2511_14102_amd.harness import DeviceLayer   # noqa: E402


def _check(r, ref, bad, k, E, tol):
    ids, y = to_np(r["ids"]), to_np(r["y"])
    good = [t for t in range(len(ids)) if t not in bad]
    if good:
        assert np.array_equal(ids[good], ref["ids"][good])
        assert rel_err(y[good], ref["y"][good]) <= tol
    for t in bad:
        assert len(set(ids[t].tolist())) == k and ids[t].min() >= 0 and ids[t].max() < E
        assert np.isnan(y[t]).all()


@pytest.mark.parametrize("E,k", [(8, 3), (130, 5)])
def test_token_of_nans(E, k):
    cfg = LayerConfig(75, "nan%d" % E, 256, E, 64, k, 32, 0, 1)
    ctx = B.Context(0)
    L = synth.make_layer(cfg, 0)
    A = oracle_arrays(L)
    D = DeviceLayer(ctx, cfg, L, max_tokens=8)
    x = tokens_with_clear_routing(cfg, A, 600, step=8, kind="iid")
    clean_d, clean_v = oracle_draft(A, x), oracle_verify(A, x[:8])
    for t in (1, 70, 333, 599):
        x[t] = float("nan")
    xd = x.cuda()
    for T, bad in ((1, []), (3, [1]), (8, [1])):
        say("draft E", E, "T", T)
        _check(D.draft(xd[:T]), {n: v[:T] for n, v in clean_d.items()}, bad, k, E, TOL_DRAFT)
    say("draft of the token alone")
    _check(D.draft(xd[1:2]), {n: v[1:2] for n, v in clean_d.items()}, [0], k, E, TOL_DRAFT)
    say("verify E", E)
    _check(D.verify(xd[:8]), clean_v, [1], k, E, TOL_VERIFY)
    for T, bad in ((40, [1]), (600, [1, 70, 333, 599])):              # both forms of the prefill call's routing
        say("prefill E", E, "T", T)
        _check(D.prefill(xd[:T]), {n: v[:T] for n, v in clean_d.items()}, bad, k, E, TOL_DRAFT)
    ctx.close()
