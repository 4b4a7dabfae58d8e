"""The walks of SSA chains on the GPU against the oracle, bit for bit, at the
sizes where a walk or a unit changes: herds whose chains are walked by a
segment of a wavefront, a wavefront or a workgroup; unit sizes from 64 to 1024
nodes; more private events in a unit than threads; and models of three to
eight compartments, with and without a second reactant."""
import dataclasses

import numpy as np
import pytest

from farmnet import synth
from oracle import oracle as O
import paper_1502_02908_amd as P

from .gpu_common import assert_parity, gpu_run, say

pytestmark = pytest.mark.gpu


def check(p, **kw):
    g = gpu_run(p, **kw)
    assert_parity(g, O.run(p, threads=8))
    return g


@pytest.mark.parametrize("classes", [1, 3])
def test_chains_of_every_length(classes):
    # herds of 1 to 40,000 animals at one transition per animal and day: the
    # attempts expected run across the bounds of the three walks (48, 256), of
    # a round (8, 16, 64, 1024) and of the summed head of a chain (64)
    make = synth.flip_model if classes == 1 else synth.flip_classes
    p = make(n_nodes=120, S0=0, I0=0, n_days=3)
    sizes = [1, 2, 7, 8, 9, 15, 16, 17, 40, 47, 48, 49, 60, 64, 66, 128, 250, 256, 260, 900, 1020, 1030, 2100, 40000]
    p.u0 = np.ascontiguousarray(p.u0)
    for i, n in enumerate(sizes):
        p.u0[5 * i % 120 + i % 5, i % p.n_comp] = n
    p.record_days = np.array([0, 2], np.int32)
    say(f"[walks] lengths classes={classes}")
    check(p)


@pytest.mark.parametrize("n_nodes", [1, 63, 64, 65, 1000, 16385, 32769, 70000, 262145])
def test_unit_sizes(n_nodes):
    # 64 positions a unit up to 16,384 nodes, then 128, 256, 512 and 1024
    p = synth.sise3_network(n_nodes=n_nodes, n_days=4, seed=91, u=10.0, seeded_frac=0.2, seeded_I=0.3, age_days=(1, 2))
    p.v0[:] = 5.0
    p.record_days = np.array([0, 3], np.int32)
    say(f"[walks] unit sizes n_nodes={n_nodes}")
    check(p)


@pytest.mark.parametrize("density", [14.0, 24.0])
def test_private_events_around_the_workgroup_size(density):
    # a unit of 64 nodes with about 900 and 1,500 private events a day: the
    # tasks run in LDS up to 1,024 and on global memory past that
    p = synth.sise3_network(n_nodes=256, n_days=12, seed=92, age_days=(2, 5), median=400.0, e1_per_node_day=density)
    p.record_days = np.array([0, 11], np.int32)
    check(p)


def chain_model(n_comp, n_nodes, n_days, bimolecular, seed):
    """Compartments 0 -> 1 -> ... -> n_comp - 1 -> 0, the first step forced by
    phi (or by the count of compartment 1), births, deaths and movements."""
    base = synth.sis_network(n_nodes=n_nodes, n_days=n_days, seed=seed, p_exit=0.02, p_enter=0.02, p_ext=0.01)
    S = np.zeros((n_comp, n_comp), np.int32)
    for k in range(n_comp):
        S[k, k] -= 1
        S[(k + 1) % n_comp, k] += 1
    u0 = np.zeros((n_nodes, n_comp), np.int32)
    u0[:, :2] = base.u0
    u0[::5, 1] += 7
    u0[3] = 3000
    E = np.ones((n_comp, 2), np.int32)
    E[1:, 0] = 0
    phi = np.zeros(n_comp, np.int32)
    phi[0] = 0 if bimolecular else 1
    coef = np.full((1, n_comp), 0.3)
    r2 = None
    if bimolecular:
        coef[0, 0] = 0.001
        r2 = np.full(n_comp, -1, np.int32)
        r2[0] = 1
    return dataclasses.replace(base, n_comp=n_comp, n_trans=n_comp, u0=u0, S=S, reactant=np.arange(n_comp, dtype=np.int32),
                               uses_phi=phi, coef=coef, reactant2=r2, phi_I_mask=0b10, phi_N_mask=(1 << n_comp) - 1,
                               E=E, N=np.zeros((n_comp, 0), np.int32), name="chain")


@pytest.mark.parametrize("n_comp,bimolecular,reps", [(3, False, 1), (4, True, 1), (5, False, 1), (8, True, 1),
                                                     (3, True, 5), (7, False, 3)])
def test_general_models(n_comp, bimolecular, reps):
    p = chain_model(n_comp, 150, 8, bimolecular, 93)
    if reps > 1:
        p = p.with_replicates(reps, replicate_id=np.arange(reps, dtype=np.uint32) + 9)
    p.record_days = np.array([0, 7], np.int32)
    say(f"[walks] general n_comp={n_comp} bimolecular={bimolecular} reps={reps}")
    g = check(p)
    assert g["transitions"].sum() > 1000


@pytest.mark.parametrize("n_comp,tile_nodes", [(2, 0), (3, 256), (8, 0), (8, 512)])
def test_level_events_in_the_next_day(n_comp, tile_nodes):
    # days of up to 512 level events on up to 768 nodes run in the next day's
    # launch (or the closing one), larger days in launches of their own: the
    # days here lie on both sides, and the run is cut so that the closing
    # launch gets either kind
    p = synth.sis_network(n_nodes=1500, n_days=10, seed=94, p_exit=0.02, p_enter=0.02, p_ext=0.33)
    if n_comp > 2:
        p = dataclasses.replace(chain_model(n_comp, 1500, 10, False, 94),
                                **{k: v for k, v in vars(p).items() if k.startswith("ev_")})
    p.record_days = np.array([0, 4, 9], np.int32)
    move = p.ev_dest >= 0
    n = [len(set(p.ev_node[move & (p.ev_day == d)]) | set(p.ev_dest[move & (p.ev_day == d)])) for d in range(10)]
    say(f"[walks] level events n_comp={n_comp} tile_nodes={tile_nodes}: {min(n)} to {max(n)} nodes moved between a day")
    assert min(n) < 768 < max(n)
    check(p, chunks=[1, 2, 1, 3, 1, 1, 1], tile_nodes=tile_nodes)


@pytest.mark.parametrize("kw", [dict(), dict(tile_nodes=512, heavy_herds=-1), dict(tile_nodes=8, heavy_herds=40)])
def test_replicate_tiles_with_more_long_chains_than_listed(kw):
    # 200 herds by 64 replicates, every chain of some 60 attempts: past the
    # 4,096 of a list of long chains the rest are walked in place; with
    # heavy_herds=-1 none is listed; chunks swap the lists' counters
    p = synth.flip_classes(n_nodes=200, S0=10, I0=10, n_days=4)
    p.u0 = np.ascontiguousarray(p.u0)
    p.u0[::40, 0] = 900
    p = p.with_replicates(64, replicate_id=np.arange(64, dtype=np.uint32) + 3)
    p.record_days = np.array([0, 3], np.int32)
    say(f"[walks] long chains in tiles {kw}")
    check(p, chunks=[1, 2, 1], **kw)


@pytest.mark.parametrize("model,reps,large", [("flip", 2, 3), ("flip3", 64, 2), ("flip3", 64, 3), ("flip", 100, 2),
                                              ("4", 3, 2), ("8", 3, 2)])
def test_longest_chains_of_replicate_tiles(model, reps, large):
    # from 8,192 positions on, chains of 2,048 attempts or more are walked by a
    # workgroup each while at most 128 of them are listed: 6, 128 and 9 chains,
    # and 192 and 200 of which each gets a wavefront
    if model in "48":
        p = chain_model(int(model), 8300, 2, model == "8", 96)
        p.u0[:large] = 0
        p.u0[:large, 2] = [12000, 9000][:large]
        p.v0[:] = 0.5
    else:
        p = (synth.flip_model if model == "flip" else synth.flip_classes)(n_nodes=8300, S0=1, I0=0, n_days=2)
        p.u0[[100, 4000, 8299][:large], 0] = [3000, 2600, 5000][:large]
    p = p.with_replicates(reps, replicate_id=np.arange(reps, dtype=np.uint32) + 5)
    p.record_days = np.array([1], np.int32)
    say(f"[walks] longest chains of tiles {model} reps={reps}, {large} herds")
    g = check(p, chunks=[1, 1])
    assert (g["max_transitions"] > 2048).all()


def test_longest_chains_of_slots():
    # the same in the slots of two requests, the second a step behind
    net = synth.flip_classes(n_nodes=8300, S0=1, I0=0, n_days=3)
    net.u0[[100, 8299], 0] = [3000, 2600]
    out = {}
    H = P.SlotHandle(net, 2, slot_lanes=32)
    try:
        for step in range(5):
            if step < 2:
                n = 20 - 13 * step
                ids = np.arange(n, dtype=np.uint32) + 40 * step
                H.start(step, 3 - step, np.ones((n, 6)), np.ones(n), np.full((n, 4), 0.1), ids)
            for slot in H.step():
                n = 20 - 13 * slot
                rec = [np.zeros((3 - slot, n), np.int32), np.zeros((3 - slot, n), np.int64), np.zeros((3 - slot, n, 6), np.int64)]
                H.fetch(slot, *rec)
                while not H.query(slot):
                    pass
                out[slot] = rec, H.state(slot, n)
    finally:
        H.close()
    assert sorted(out) == [0, 1]
    for slot, (rec, (u, v)) in out.items():
        n = 20 - 13 * slot
        p = net.truncated(3 - slot).with_replicates(n, coef=np.ones((n, 6)), alpha=np.ones(n), beta=np.full((n, 4), 0.1),
                                                    replicate_id=np.arange(n, dtype=np.uint32) + 40 * slot)
        o = O.run(p, threads=8)
        for a, k in zip(rec, ("prevalence", "transitions", "totals")):
            assert np.array_equal(a, o[k]), (slot, k)
        assert np.array_equal(u, o["u"]) and np.array_equal(v.view(np.int64), o["v"].view(np.int64))


@pytest.mark.parametrize("n_comp,reps", [(3, 1), (8, 1), (4, 3)])
def test_draws_computed_ahead(n_comp, reps):
    # movements and deaths of 1 to 9 animals from three compartments or more,
    # around the six (two in a private task) draws computed ahead
    p = chain_model(n_comp, 400, 6, False, 98)
    p.u0[:, :] += 60
    n = np.array([1, 2, 3, 5, 6, 7, 9], np.int32)
    p.ev_n = np.where(p.ev_kind == 1, p.ev_n, n[np.arange(p.n_events) % 7]).astype(np.int32)
    p = p.with_replicates(reps)
    p.record_days = np.array([0, 5], np.int32)
    say(f"[walks] draws ahead n_comp={n_comp} reps={reps}: {p.n_events} events")
    check(p, chunks=[1, 3, 2])


@pytest.mark.parametrize("n_nodes,tile,density,pre", [(512, 512, 2.1, 0), (512, 512, 2.6, 1), (77000, 256, 2.3, 0)])
def test_private_events_past_the_workgroup_size(n_nodes, tile, density, pre):
    # units of 512 and 256 herds with up to about 1,100, 1,300 and 600 private
    # events a day: past the 1,024 threads of a workgroup (512 in the third,
    # of 301 units) the tasks run on global memory, below them in LDS
    p = synth.sise3_network(n_nodes=n_nodes, n_days=6 if n_nodes > 1000 else 12, seed=99, age_days=(1, 3), median=400.0,
                            e1_per_node_day=density)
    p.phi_pre_events = pre
    p.record_days = np.array([0, p.n_days - 1], np.int32)
    threads = 512 if n_nodes > 1000 else 1024
    move = p.ev_dest >= 0
    a_day = np.bincount(p.ev_day[~move], minlength=p.n_days) / (n_nodes / tile)
    say(f"[walks] private events {n_nodes} herds: {a_day.min():.0f} to {a_day.max():.0f} a unit and day")
    assert a_day.min() < threads < a_day.max()
    check(p, tile_nodes=tile)


@pytest.mark.parametrize("n_nodes,classes", [(16, 1), (4800, 3), (9600, 1)])
@pytest.mark.parametrize("large", [3, 4])
def test_several_workgroup_chains_in_a_unit(n_nodes, classes, large):
    # units of 16 herds, three of them with 1,100 to 6,000 attempts a day: the
    # workgroup walks one after another (of 1,024, 512 and 256 threads); of
    # four, each gets a wavefront
    p = (synth.flip_model if classes == 1 else synth.flip_classes)(n_nodes=n_nodes, S0=1, I0=0, n_days=2)
    big = np.random.default_rng(3).integers(1100, 6000, large * (n_nodes // 16))
    p.u0[np.random.default_rng(4).permutation(n_nodes)[:len(big)], 0] = big
    p.record_days = np.array([1], np.int32)
    say(f"[walks] {large} long chains in each of {n_nodes // 16} units")
    check(p, tile_nodes=16, group_min_attempts=64, group_herds=-1)


@pytest.mark.parametrize("least", [8, 4096])
def test_threshold_of_the_workgroup_walk(least):
    p = synth.sise3_network(n_nodes=9000, n_days=30, seed=100, u=10.0, age_days=(10, 20))
    p.record_days = np.array([29], np.int32)
    say(f"[walks] group_min_attempts={least}")
    check(p, group_min_attempts=least)


@pytest.mark.parametrize("n_nodes,reps", [(1, 1), (1, 2), (8200, 2)])
def test_too_many_transitions_in_a_day(n_nodes, reps):
    # a herd whose chain passes 2^24 transitions, walked by a workgroup of the
    # day kernel, a wavefront and a workgroup of the long chains' launch: the
    # run reports it, and the handle goes on from another state
    p = synth.flip_model(n_nodes=n_nodes, S0=3, I0=3, n_days=2).with_replicates(reps)
    u = np.broadcast_to(p.u0, (reps,) + p.u0.shape).copy()
    v = np.zeros((reps, n_nodes))
    over = u.copy()
    over[reps - 1, 0] = 12_000_000
    say(f"[walks] past the limit of transitions n_nodes={n_nodes} reps={reps}")
    with P.Simulator(p) as sim:
        sim.set_state(over, v, 0)
        sim.run(2)
        with pytest.raises(P.SimError) as e:
            sim.sync()
        assert e.value.code == P.SIM_ELIMIT and f"replicate {reps - 1}" in str(e.value)
        sim.set_state(u, v, 0)
        sim.run(2)
        g = sim.trajectory()
    o = O.run(p, threads=8)
    for k in ("transitions", "totals", "prevalence", "max_transitions"):
        assert np.array_equal(g[k], o[k]), k
