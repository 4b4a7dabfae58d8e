"""Sizes that the host decides before any launch: what a plan of slots says
against what its handles take, and the padding of positions to units of
work."""
import pytest

from farmnet import synth
from paper_1502_02908_amd import sim as S
from paper_1502_02908_amd.serve import plan_slots


def network(n_nodes, n_days, seed):
    return synth.sise3_network(n_nodes=n_nodes, n_days=n_days, seed=seed, age_days=(10, 30), e1_per_node_day=0.02)


@pytest.mark.parametrize("slot_lanes", [64, 16])
@pytest.mark.parametrize("budget", [4 << 20, 40 << 20, 300 << 20, 2000 << 20])
def test_planned_slots_take_the_planned_bytes(slot_lanes, budget):
    # sizes whose units of work change with the columns (up to 32,768 nodes x
    # columns and past it), and a network of fewer positions than a list of
    # long chains has room for
    nets = [network(30, 60, 1), network(1000, 90, 2), network(4000, 40, 3), network(9001, 20, 4)]
    demand = [1, 2, 3, 4]
    per_col = 64 // slot_lanes
    slots, taken = plan_slots(nets, budget, demand, slot_lanes=slot_lanes)
    for net, n, nbytes, w in zip(nets, slots, taken, demand):
        share = budget * w / sum(demand)
        assert n % per_col == 0 and n >= per_col
        assert nbytes == S.SlotHandle.workspace_bytes(net, n, slot_lanes)
        assert nbytes <= share or n == per_col
        if n < 256 * per_col:  # no room is left for another column
            assert S.SlotHandle.workspace_bytes(net, n + per_col, slot_lanes) > share
