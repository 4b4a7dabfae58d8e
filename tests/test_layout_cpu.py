"""Sizes that the host decides before any launch: what a plan of slots says
against what its handles take, and the padding of positions to units of
work."""
import ctypes as C
import dataclasses

import numpy as np
import pytest

from farmnet import synth
import paper_1502_02908_amd as P
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


def packed_bytes(problems, **opts):
    structs = [S._marshal(p) for p in problems]
    arr = (C.POINTER(S.sim_problem) * len(problems))(*[C.pointer(s) for s, _ in structs])
    o = S.sim_device_opts()
    for k, v in opts.items():
        setattr(o, k, v)
    return int(P.lib().sim_workspace_bytes_batch(arr, len(problems), C.byref(o)))


@pytest.mark.parametrize("sizes,reps,unit", [
    ([50] * 6000, 1, 64),              # a unit for every network, whatever all of them hold together
    ([130] * 2400, 1, 256),
    ([100000] + [50] * 5000, 1, 256),
    ([8192] * 100, 1, 512),            # four herds of each network have units of their own
    ([20] * 1000, 64, 32),
    ([100] * 200, 64, 64),
    ([30000] + [20] * 500, 100, 64),
])
def test_small_packed_networks_are_not_padded_to_large_units(sizes, reps, unit):
    nets = {n: network(n, 5, n).with_replicates(reps) for n in set(sizes)}
    problems = [nets[n] for n in sizes]
    # (a unit's days take 12 bytes each: room for six units more a network)
    assert 0 < packed_bytes(problems) <= packed_bytes(problems, tile_nodes=unit) + 400 * len(sizes)


@pytest.mark.parametrize("n_nodes,regions,reps,unit", [(300000, 1000, 1, 512), (100000, 400, 64, 128)])
def test_regions_are_not_padded_to_large_units(n_nodes, regions, reps, unit):
    p = network(n_nodes, 3, 5).with_replicates(reps)
    p = dataclasses.replace(p, n_regions=regions, region=np.arange(n_nodes, dtype=np.int32) % regions)
    assert 0 < packed_bytes([p]) <= packed_bytes([p], tile_nodes=unit)


def test_many_small_networks_with_replicates_are_accepted():
    # 330,000 herds by 256 replicates: with 512 positions for each network of
    # 20 herds the lanes would pass 2^31
    p = dataclasses.replace(synth.flip_model(n_nodes=20, S0=1, I0=1, n_days=1)).with_replicates(256)
    assert packed_bytes([p] * 16500) > 0


def test_tuner_times_no_schedule_twice():
    # heavy_herds has a sign only, and few_chains is read by replicate tiles
    # (and the persistent launch) only
    from paper_1502_02908_amd.tune import LANE_CANDIDATES, TILE_CANDIDATES
    lanes = [{k: v for k, v in c.items() if k not in ("few_chains", "heavy_herds")} for c in LANE_CANDIDATES]
    tiles = [{k: -1 if k == "heavy_herds" else v for k, v in c.items() if not (k == "heavy_herds" and v >= 0)}
             for c in TILE_CANDIDATES]
    for candidates in (lanes, tiles):
        assert all(c not in candidates[:j] for j, c in enumerate(candidates))
