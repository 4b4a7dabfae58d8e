"""Units of work on the GPU against the oracle, bit for bit: networks packed in
one handle that fill units of their own sizes, and the units of the general
models of more than four compartments."""
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
    # units of 4 and of 512 positions, as many as a workgroup of these models
    # has threads (140,000 herds would fill 1,024 each otherwise)
    p = chain_model(n_comp, n_nodes, 3, n_comp == 8, 95)
    p.record_days = np.array([2], np.int32)
    say(f"[units] general model of {n_comp}, {n_nodes} herds {kw}")
    assert_parity(gpu_run(p, **kw), O.run(p, threads=8))
