"""The size rules of the draft calls on devices of several sizes (no GPU)."""
import pytest

from tests.draft_rules import rules

UNITS = (32, 64, 128, 256)


@pytest.mark.parametrize("n_cu", UNITS)
@pytest.mark.parametrize("E", (1, 5, 8, 10, 16, 60, 64, 100, 128, 200, 256))
def test_calls_on_several_streams_cannot_stop_each_other(n_cu, E):
    """Every workgroup of a draft call waits for the call's router workgroups.  Of `calls` calls of several tokens that are
    dispatched at the same time, one workgroup to a unit, one holds at least n_cu / calls units: with E <= n_cu / calls all of
    its router workgroups run, it ends, and its units go to the others."""
    for grid in (1, n_cu // 2, n_cu):
        assert rules().rule_router_workgroups(E, 1, grid) <= min(E, grid)
    calls = n_cu // E
    assert calls == 0 or rules().rule_router_workgroups(E, 1, n_cu) <= n_cu // calls


@pytest.mark.parametrize("n_cu", UNITS)
@pytest.mark.parametrize("E", (1, 5, 8, 10, 16, 60, 64, 67, 100, 128, 200, 256))
def test_pairs_leave_as_much_room_as_single_items(n_cu, E):
    """One-token calls: a unit holds two workgroups of one item or one of a pair, so a pair's workgroup has to do for two router rows
    what two of single items do, at once: as many calls go on together (an odd last row has a unit's half for itself)."""
    single, pair = rules().rule_router_workgroups(E, 1, 10 ** 6), rules().rule_router_workgroups(E, 2, 10 ** 6)
    assert single == E
    calls = 2 * n_cu // (E + E % 2)
    assert calls == 0 or pair <= n_cu // calls


SHAPES = [(H, E, I, k, g, 0) for H in (256, 1024, 2048, 2304, 4096) for E in (8, 64, 65, 100, 128, 200, 256) for I in (512, 768, 1408, 4096, 14336)
          for k in (1, 2, 8) for g in (64, 128)]


@pytest.mark.parametrize("n_cu", UNITS)
def test_one_token_calls_with_two_items_per_unit_are_never_refused(n_cu):
    """The persistent launch takes every such call without shared experts whose two copies of x fit LDS; another form is
    chosen only where the device holds its router workgroups at once (two of single items to a unit, one of a pair)."""
    r = rules()
    seen = set()
    for H, E, I, k, g, S in SHAPES:
        if k * (I // 32) < 2 * n_cu or not r.rule_fits(H, E, I, k, g, S, 2):
            continue
        form = r.rule_one_token_form(H, E, I, k, g, S, 0, n_cu, 2 * n_cu)
        seen.add(form)
        if form < 2:
            items, room = (1, 2 * n_cu) if form == 0 else (2, n_cu)
            assert r.rule_router_workgroups(E, items, k * (I // 32) // items) <= room, (H, E, I, k, g, form)
    assert 2 in seen and 1 in seen


@pytest.mark.parametrize("n_cu", UNITS)
def test_many_shared_items_run_inside_only_as_pairs(n_cu):
    """The line up to which shared experts run in a one-token call's own launch was measured with pairs of items; where the call
    runs single items (long rows, more than two items per unit), it is three per unit, or one per 256 of H."""
    r = rules()
    inside = outside = 0
    for H in range(256, 4097, 128):
        for I in (512, 1408, 4096, 7168, 10240, 14336):
            for S in (1, 2, 4):
                for k in (1, 2, 8):
                    items = S * (I // 16)
                    if not r.rule_shared_inside(H, 64, I, k, 128, S, n_cu):
                        outside += 1
                        assert items > 3 * n_cu and items * 256 > n_cu * H
                    elif items > 3 * n_cu and items * 256 > n_cu * H:
                        inside += 1
                        assert r.rule_one_token_form(H, 64, I, k, 128, S, 1, n_cu, 2 * n_cu) == 1, (H, I, S, k)
    assert inside and outside


@pytest.mark.parametrize("H,I,k,S,inside", [(256, 5120, 1, 4, True), (256, 6144, 1, 4, False), (256, 7168, 1, 4, False), (512, 7168, 1, 4, False),
                                            (1024, 6144, 1, 4, False), (1024, 8192, 1, 4, False), (1280, 8192, 1, 4, True), (2048, 16384, 1, 4, True),
                                            (256, 7168, 2, 4, True), (1024, 8192, 2, 4, True), (256, 9536, 1, 3, True), (256, 14336, 1, 2, True)])
def test_shared_experts_beside_one_routed(H, I, k, S, inside):
    """Four shared experts beside one routed and short rows: beyond five items per unit (256 units) their own launches are faster."""
    assert bool(rules().rule_shared_inside(H, 8, I, k, 64, S, 256)) == inside


@pytest.mark.parametrize("n_cu", UNITS)
def test_one_item_per_unit_runs_single_items(n_cu):
    """With exactly one item per unit and long rows single items fill the device and pairs half of it; one more item and some unit
    would have two."""
    r = rules()
    k = 4
    I = n_cu // k * 32
    for H, form in ((1024, 1), (2048, 0), (4096, 0), (8192, 0)):
        assert r.rule_one_token_form(H, 8, I, k, 64, 0, 0, n_cu, 2 * n_cu) == form
        assert r.rule_one_token_form(H, 8, I + 64, k, 64, 0, 0, n_cu, 2 * n_cu) == 1
        assert r.rule_one_token_form(H, 8, I - 64, k, 64, 0, 0, n_cu, 2 * n_cu) == 0
        if n_cu >= 64:                                     # half of the items a shared expert's
            assert r.rule_one_token_form(H, 8, I // 2, k, 64, 2, 1, n_cu, 2 * n_cu) == 1
