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
