"""Units of work on the GPU against the oracle, bit for bit: networks packed in
one handle that fill units of their own sizes, the units of the general
models of more than four compartments, and large networks whose herds are
walked by their owners' lanes."""
import dataclasses

import numpy as np
import pytest

from farmnet import synth
from oracle import oracle as O
import paper_1502_02908_amd as P

from .gpu_common import assert_parity, gpu_run, say
from .test_gpu_walks import chain_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,reps", [([3, 4, 5, 64, 65, 300] * 60, 1), ([9000] + [20] * 300, 1), ([3, 5, 20, 21, 130] * 12, 64)])
def test_packed_networks_of_uneven_sizes(sizes, reps):
    # small networks beside each other and beside a large one (with herds that
    # have units of their own), every one against its own run of the oracle
    coef, alpha, beta = synth.prior_draws(reps, seed=6)
    probs = []
    for j, n in enumerate(sizes):
        p = synth.sise3_network(n_nodes=n, n_days=6, seed=600 + j, u=5.0, seeded_frac=0.3, seeded_I=0.3, age_days=(1, 3),
                                e1_per_node_day=0.5, e2_per_node_day=0.2)
        p.v0[:] = 2.0
        p.record_days = np.array([5], np.int32)
        probs.append(p.with_replicates(reps, coef=coef, alpha=alpha, beta=beta))
    say(f"[units] {len(sizes)} networks, {sum(sizes)} herds, {reps} replicates")
    with P.Simulator(probs) as sim:
        sim.run(0)
        g = sim.trajectory()
        u, v, _ = sim.get_state()
    at = 0
    for j, p in enumerate(probs):
        rows, herds = slice(j * reps, (j + 1) * reps), slice(at, at + p.n_nodes)
        at += p.n_nodes
        one = {k: g[k][:, rows] for k in ("prevalence", "transitions", "totals", "max_transitions")}
        one.update({k: g[k][:, :, herds] for k in ("snap_u", "snap_v")}, u=u[:, herds], v=v[:, herds])
        assert_parity(one, O.run(p, threads=8))


@pytest.mark.parametrize("n_comp,n_nodes,kw", [(5, 700, {}), (8, 2100, dict(tile_nodes=512)), (8, 140000, {})])
def test_large_general_models(n_comp, n_nodes, kw):
    # units of 4, of as many positions as a workgroup of these models has
    # threads, and of 256
    p = chain_model(n_comp, n_nodes, 3, n_comp == 8, 95)
    p.record_days = np.array([2], np.int32)
    say(f"[units] general model of {n_comp}, {n_nodes} herds {kw}")
    assert_parity(gpu_run(p, **kw), O.run(p, threads=8))


def widespread(model, n_nodes, n_days, frac, seed):
    """A network in which a herd has a chain with probability frac."""
    if model == "sis":
        p = synth.sis_network(n_nodes=n_nodes, n_days=n_days, seed=seed, seeded_frac=frac, seeded_I=0.3)
    elif model.startswith("sise3"):
        p = synth.sise3_network(n_nodes=n_nodes, n_days=n_days, seed=seed, u=4.0, seeded_frac=frac, seeded_I=0.3, age_days=(1, 2),
                                e2_per_node_day=1e-3 if model == "sise3 levels" else 235.0 / 37221.0)
        p.phi_pre_events = int(model == "sise3 pre")
    else:
        p = chain_model(int(model), n_nodes, n_days, False, seed)
        p.u0[np.random.default_rng(seed).random(n_nodes) >= frac] = 0
        keep = np.zeros(p.n_events, bool)
        p = dataclasses.replace(p, **{k: v[keep] for k, v in vars(p).items() if k.startswith("ev_")})
    p.record_days = np.array([n_days - 1], np.int32)
    return p


@pytest.mark.parametrize("frac", [0.375, 1.0])
@pytest.mark.parametrize("model,n_nodes,tile", [("sis", 66000, 0), ("sis", 132001, 0), ("sise3", 66000, 0), ("sise3", 66100, 256),
                                                ("sise3 levels", 66000, 0), ("sise3 pre", 132001, 0), ("3", 66000, 0),
                                                ("8", 66000, 0)])
def test_herds_walked_by_their_owners(model, n_nodes, tile, frac):
    # units of 512 and 1024 positions in workgroups of 1,024 threads, and more
    # units of 256 than fill the chip with those: wavefronts of 64 herds hold 24
    # chains on average, on both sides of the number that they walk themselves,
    # and 64, of which the last eight and the longest start again in segments
    p = widespread(model, n_nodes, 3, frac, 97)
    say(f"[units] owners {model} {n_nodes} herds, {frac} of them with a chain")
    g = gpu_run(p, tile_nodes=tile)
    assert_parity(g, O.run(p, threads=8))
    assert g["transitions"][0].sum() > 0.1 * frac * n_nodes
