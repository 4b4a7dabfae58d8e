"""The work whose speed is measured: calls that a program makes through the
package's public entry points, over the range of networks, models, replicate
counts and device options in use.

A case names its inputs by plain sizes; the network, its event list and its
parameters follow from the case and a seed. Kinds of case:

  trajectory  one handle, one trajectory: the state is set, the horizon is run,
              records and the final state are read back;
  fit         one evaluation of the fitting study: replicates of one network
              with their own parameters, run over the horizon, with the daily
              regional sums and the goal function against a reference;
  packed      several networks of different sizes in one handle, one
              trajectory each;
  slots       a resident network that runs replicates of new parameter vectors
              in its slots;
  serve       the request loop over several resident networks.
"""
import dataclasses
import math

import numpy as np
import torch

import paper_1502_02908_amd as P
from farmnet import EXTERNAL, synth
from paper_1502_02908_amd.serve import Server

REGIONS = 21  # the fitting study's regions


def listed():
    return [
        # the smallest network in use (plain SIS, 1,000 herds): a day is little
        # work, so what a day costs besides its work shows here
        {"name": "sis 1k x 365", "kind": "trajectory", "model": "sis", "nodes": 1000, "days": 365, "u": 1.0, "tile": 0},
        # the smallest network a request names, three age classes
        {"name": "sise3 1k x 365", "kind": "trajectory", "model": "sise3", "nodes": 1000, "days": 365, "u": 1.0, "tile": 0},
        # the national network over a year: the ordinary call
        {"name": "sise3 37k x 365", "kind": "trajectory", "model": "sise3", "nodes": 37000, "days": 365, "u": 1.0, "tile": 0},
        # the same with ten times the rates: long chains in the largest herds
        {"name": "sise3 37k x 120 u=10", "kind": "trajectory", "model": "sise3", "nodes": 37221, "days": 120, "u": 10.0, "tile": 0},
        # the scale-up: a million herds, a hub of many hundred thousand animals
        {"name": "sise3 1m x 60", "kind": "trajectory", "model": "sise3", "nodes": 1000000, "days": 60, "u": 1.0, "tile": 0},
        # the SSA-heavy synthetic model (about 2,000 transitions per node and
        # day) with the tile width that the tuner picks for it
        {"name": "flip 1k x 50 tiles", "kind": "trajectory", "model": "flip", "nodes": 1000, "days": 50, "u": 1.0, "tile": 4},
        # a model outside the paired S <-> I form: S -> I -> R -> S
        {"name": "sir 5k x 120", "kind": "trajectory", "model": "sir", "nodes": 5000, "days": 120, "u": 1.0, "tile": 0},
        # one goal evaluation of the fitting study
        {"name": "fit 64 x 1k x 60", "kind": "fit", "nodes": 1000, "days": 60, "reps": 64, "u": 1.0},
        # uneven networks of one model advanced together
        {"name": "packed 12 x 1k-20k x 90", "kind": "packed", "instances": 12, "lo": 1000, "hi": 20000, "days": 90},
        # many replicates of the national network: 256 in four slots
        {"name": "slots 37k x 256 x 40", "kind": "slots", "nodes": 37000, "days": 40, "slots": 4, "lanes": 64, "last": 64},
        # a queue of requests of mixed sizes, horizons and replicate counts
        {"name": "serve 24 requests", "kind": "serve", "lo": 1000, "hi": 16000, "days": 90, "requests": 24, "lanes": 16, "stream": 5},
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["trajectory"] * 6 + ["fit", "fit", "packed", "slots", "slots", "serve"])
    if kind == "trajectory":
        model = rng.choice(["sis", "sise3", "sise3", "sise3", "flip", "sir"])
        nodes = log(200, 300000) if model == "sise3" else log(200, 2000) if model == "flip" else log(200, 20000)
        days = min(log(20, 365), max(20, 10000000 // nodes))
        if model == "flip":
            days = min(days, 60)
        u = round(math.exp(rng.uniform(0.0, math.log(10.0))), 2) if model == "sise3" and nodes <= 50000 else 1.0
        return {"kind": kind, "model": model, "nodes": nodes, "days": days, "u": u,
                "tile": rng.choice([0, 4, 4, 8, 16]) if model == "flip" else 0}
    if kind == "fit":
        reps = rng.choice([2, 10, 20, 40, 64, 100])
        return {"kind": kind, "nodes": log(300, 4000), "days": log(20, 60), "reps": reps, "u": round(rng.uniform(1.0, 4.0), 2)}
    if kind == "packed":
        return {"kind": kind, "instances": rng.randint(3, 14), "lo": log(200, 1000), "hi": log(4000, 20000), "days": log(20, 90)}
    lanes = rng.choice([16, 32, 64])
    if kind == "slots":
        slots = rng.randint(1, 3) * (64 // lanes)
        return {"kind": kind, "nodes": log(500, 37000), "days": log(10, 40), "slots": slots, "lanes": lanes,
                "last": rng.randint(1, lanes)}
    return {"kind": kind, "lo": log(500, 2000), "hi": log(4000, 12000), "days": log(30, 80),
            "requests": rng.randint(6, 20), "lanes": rng.choice([16, 32]), "stream": rng.randint(1, 1000)}


def farm(nodes, days, seed, u=1.0, grown=730):
    """A farm network in mid-life: every herd already holds what it would have
    received by movements over `grown` days, a tenth of the herds are infected,
    and phi stands at its balance with the infected fraction. Short horizons
    age their animals early so that the aging events occur in them."""
    p = synth.sise3_network(n_nodes=nodes, n_days=days, seed=seed, u=u, seeded_frac=0.1, seeded_I=0.3,
                            age_days=(100, 400) if days > 150 else (10, 30), record_days=np.array([days - 1]))
    mv = p.ev_kind == EXTERNAL
    got = np.zeros((nodes, 3))
    np.add.at(got, (p.ev_dest[mv], p.ev_select[mv] - 1), p.ev_n[mv])
    more = np.rint(got * (grown / days)).astype(np.int32)
    infected = np.where((p.u0[:, 1::2].sum(axis=1) > 0)[:, None] | (more.sum(axis=1) > 2000)[:, None],
                        np.rint(0.3 * more).astype(np.int32), 0)
    p.u0[:, 0::2] += more - infected
    p.u0[:, 1::2] += infected
    p.v0[:] = p.u0[:, 1::2].sum(axis=1) / np.maximum(p.u0.sum(axis=1), 1) / 0.04
    return p


def sis(nodes, days, seed):
    return synth.sis_network(n_nodes=nodes, n_days=days, seed=seed, seeded_frac=0.1, seeded_I=0.3,
                             record_days=np.array([days - 1]))


def sir(nodes, days, seed):
    base = synth.sis_network(n_nodes=nodes, n_days=days, seed=seed, p_exit=0.01, p_enter=0.01, p_ext=0.005,
                             record_days=np.array([days - 1]))
    u0 = np.zeros((nodes, 3), np.int32)
    u0[:, :2] = base.u0
    u0[::7, 1] += 5
    return dataclasses.replace(
        base, n_comp=3, n_trans=3, u0=u0, S=np.array([[-1, 0, 1], [1, -1, 0], [0, 1, -1]], np.int32),
        reactant=np.array([0, 1, 2], np.int32), uses_phi=np.array([1, 0, 0], np.int32),
        coef=np.array([[0.3, 0.2, 0.05]]), phi_I_mask=0b010, phi_N_mask=0b111,
        E=np.array([[1, 1], [0, 1], [0, 1]], np.int32), N=np.zeros((3, 0), np.int32), name="sir")


def one_network(case, seed):
    nodes, days = case["nodes"], case["days"]
    if case.get("model") == "sis":
        return sis(nodes, days, seed)
    if case.get("model") == "sir":
        return sir(nodes, days, seed)
    if case.get("model") == "flip":
        return dataclasses.replace(synth.flip_model(n_nodes=nodes, n_days=days, seed=seed), record_days=np.array([days - 1]))
    return farm(nodes, days, seed, case.get("u", 1.0))


def sizes(case, n):
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** (j / max(1, n - 1)))) for j in range(n)]


class State:
    pass


def prepare(case, seed):
    st = State()
    st.case = dict(case)
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    seed = int(rng.integers(1 << 30))
    if kind == "trajectory":
        st.p = one_network(case, seed)
        st.sim = P.Simulator(st.p, tile_nodes=case["tile"])
        st.u, st.v = st.p.u0[None], st.p.v0[None]
    elif kind == "fit":
        base = farm(case["nodes"], case["days"], seed, case["u"])
        reps = case["reps"]
        coef, alpha, beta = synth.prior_draws(reps, seed=seed + 1)
        reg = rng.choice(REGIONS, size=base.n_nodes, p=rng.dirichlet(np.full(REGIONS, 0.7))).astype(np.int32)
        reg[rng.random(base.n_nodes) < 0.05] = -1
        st.p = dataclasses.replace(base.with_replicates(reps, coef=coef * case["u"], alpha=alpha, beta=beta),
                                   n_regions=REGIONS, region=reg)
        st.sim = P.Simulator(st.p)
        st.u = np.ascontiguousarray(np.broadcast_to(st.p.u0, (reps,) + st.p.u0.shape))
        st.v = np.ascontiguousarray(np.broadcast_to(st.p.v0, (reps,) + st.p.v0.shape))
        here = np.zeros((REGIONS, 6), np.int64)
        np.add.at(here, reg[reg >= 0], st.p.u0[reg >= 0])
        st.reference = np.ascontiguousarray(np.broadcast_to(here, (case["days"], REGIONS, 6)))
    elif kind == "packed":
        n = case["instances"]
        coef, alpha, beta = synth.prior_draws(n, seed=seed + 1)
        probs = [farm(m, case["days"], seed + 2 + j).with_replicates(1, coef=coef[j:j + 1], alpha=alpha[j:j + 1], beta=beta[j:j + 1])
                 for j, m in enumerate(sizes(case, n))]
        st.sim = P.Simulator(probs)
        st.u = np.concatenate([q.u0 for q in probs])[None]
        st.v = np.concatenate([q.v0 for q in probs])[None]
    elif kind == "slots":
        st.p = dataclasses.replace(farm(case["nodes"], case["days"], seed), record_days=None)
        st.handle = P.SlotHandle(st.p, case["slots"], slot_lanes=case["lanes"])
        st.work, st.buf = [], []
        for j in range(case["slots"]):
            n = case["last"] if j == case["slots"] - 1 else case["lanes"]
            st.work.append(synth.prior_draws(n, seed=seed + 1 + j) + (np.arange(n, dtype=np.uint32) + 64 * j,))
            pin = dict(pin_memory=torch.cuda.is_available())
            D = case["days"]
            st.buf.append((torch.empty(D, n, dtype=torch.int32, **pin), torch.empty(D, n, dtype=torch.int64, **pin),
                           torch.empty(D, n, 6, dtype=torch.int64, **pin)))
    else:
        nets = [dataclasses.replace(farm(m, case["days"], seed + j), record_days=None) for j, m in enumerate(sizes(case, 3))]
        st.server = Server(nets, [4 * (64 // case["lanes"])] * 3, slot_lanes=case["lanes"])
        # the stream (networks, horizons, replicate counts) belongs to the case, the parameters to the seed
        st.requests = synth.serving_requests(n_requests=case["requests"], horizon=(case["days"] // 3, case["days"]), seed=case["stream"])
        for q in st.requests:
            q["coef"], q["alpha"], q["beta"] = synth.prior_draws(q["n_rep"], seed=seed + 3 + q["rid"])
    return st


def run(st):
    case = st.case
    kind = case["kind"]
    if kind in ("trajectory", "fit", "packed"):
        st.sim.set_state(st.u, st.v, 0)
        st.sim.run(0)
        out = st.sim.trajectory()
        if kind == "fit":
            out["goal"] = np.array(st.sim.goal(st.reference))
        return out
    if kind == "slots":
        for j, (coef, alpha, beta, rid) in enumerate(st.work):
            st.handle.start(j, case["days"], coef, alpha, beta, rid)
        done = 0
        while done < case["slots"]:
            for j in st.handle.step():
                st.handle.fetch(j, *st.buf[j])
                done += 1
        for j in range(case["slots"]):
            while not st.handle.query(j):
                pass
        return [[b.numpy().copy() for b in bufs] for bufs in st.buf]
    results, _ = st.server.serve(st.requests, realtime=False)
    results.sort(key=lambda r: r.rid)
    return {"prevalence": np.concatenate([r.prevalence.ravel() for r in results]),
            "transitions": np.concatenate([r.transitions.ravel() for r in results])}


def work(case):
    """The state in and out once, every event read once (its seven fields) and
    the records written once; per node and day one attempt of the direct
    method (its random numbers, -log, waiting time and rates), or as many as
    the synthetic model is known to take, and the phi update."""
    kind, days = case["kind"], case["days"]
    comps = {"sis": 2, "flip": 2, "sir": 3}.get(case.get("model"), 6)
    if kind == "trajectory":
        nets, reps = [case["nodes"]], 1
    elif kind == "fit":
        nets, reps = [case["nodes"]], case["reps"]
    elif kind == "packed":
        nets, reps = sizes(case, case["instances"]), 1
    elif kind == "slots":
        nets, reps = [case["nodes"]], (case["slots"] - 1) * case["lanes"] + case["last"]
    else:
        # requests spread over the networks, half the replicates and two
        # thirds of the horizon on average
        nets, reps, days = sizes(case, 3), case["requests"] * 32 / 3, days * 2 / 3
    n = sum(nets)
    per_day = {"sis": 0.005, "flip": 0.0, "sir": 0.025}.get(case.get("model"), 3942.0 / 37221.0)
    regions = REGIONS if kind == "fit" else 0
    sets = reps * (len(nets) if kind == "packed" else 1)
    attempts = 2100.0 if case.get("model") == "flip" else 1.0
    return {"bytes": float(2 * n * reps * (4 * comps + 8) + 28 * n * per_day * days + days * sets * (16 + 8 * comps * (1 + regions))),
            "flops": float(n * reps * days * (50.0 * attempts + 10.0))}


# --- the same trajectory in plain numpy (binary64) --------------------------

def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon et al., SC'11) on arrays of counter words."""
    m32 = np.uint64(0xFFFFFFFF)
    x = [np.asarray(c, np.uint64) for c in (c0, c1, c2, c3)]
    k0, k1 = int(k0), int(k1)
    for _ in range(10):
        a, c = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        x = [(c >> np.uint64(32)) ^ x[1] ^ np.uint64(k0), c & m32, (a >> np.uint64(32)) ^ x[3] ^ np.uint64(k1), a & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x


def _uniform(lo, hi):
    w = (hi << np.uint64(32)) | lo
    return ((w >> np.uint64(11)) | np.uint64(1)).astype(np.float64) * 2.0 ** -53


def _ssa_day(p, x, phi, d):
    """Gillespie's direct method on every node over one day; transitions per node."""
    fired = np.zeros(p.n_nodes, np.int64)
    clock = np.zeros(p.n_nodes)
    scale = np.where(p.uses_phi[None, :] != 0, p.coef[0] * phi[:, None], p.coef[0])
    live, k, draws = np.arange(p.n_nodes), 0, 16
    while len(live):
        o = _philox(np.arange(k, k + draws)[None, :], live[:, None], np.uint64(d), np.uint64(0), p.seed, p.replicate_id[0])
        wait, pick = -np.log(_uniform(o[0], o[1])), _uniform(o[2], o[3])
        row = np.arange(len(live))
        for q in range(draws):
            i = live[row]
            cum = np.cumsum(scale[i] * x[i][:, p.reactant], axis=1)
            lam = cum[:, -1]
            with np.errstate(divide="ignore"):
                t = clock[i] + wait[row, q] / lam
            go = t < 1.0
            row, i, cum, lam = row[go], i[go], cum[go], lam[go]
            if not len(row):
                break
            clock[i] = t[go]
            j = (cum < (pick[row, q] * lam)[:, None]).sum(axis=1)
            x[i] += p.S.T[j]
            fired[i] += 1
        live, k = live[row], k + draws
    return fired


def _event(p, x, g, d):
    """Event g of the list on day d: the individuals are drawn one by one."""
    kind, node, n = int(p.ev_kind[g]), int(p.ev_node[g]), int(p.ev_n[g])
    sel = [c for c in range(p.n_comp) if p.E[c, p.ev_select[g]]]
    if kind == 1:  # enter
        x[node, sel[0]] += n
        return
    take = [0] * p.n_comp
    left = {c: int(x[node, c]) for c in sel}
    for q in range(n):
        if q % 2 == 0:
            o = [int(w) for w in _philox(q // 2, g, d, 1, p.seed, p.replicate_id[0])]
        bits = (o[1] << 32 | o[0]) if q % 2 == 0 else (o[3] << 32 | o[2])
        at = bits * sum(left.values()) >> 64
        for c in sel:
            if at < left[c]:
                break
            at -= left[c]
        left[c] -= 1
        take[c] += 1
    to = node if kind == 2 else int(p.ev_dest[g])
    for c in sel:
        x[node, c] -= take[c]
        if kind >= 2:
            x[to, c + (int(p.N[c, p.ev_shift[g]]) if p.ev_shift[g] >= 0 else 0)] += take[c]


def exact(case, seed):
    """Small trajectories, day by day in numpy; larger ones, where that takes
    minutes, have none (their outputs but phi are whole numbers)."""
    if case["kind"] != "trajectory" or case["model"] not in ("sis", "sise3", "sir"):
        return None
    if case["nodes"] > 2000 or case["nodes"] * case["days"] > 400000 or case["u"] > 4.0:
        return None
    p = one_network(case, int(np.random.default_rng(seed).integers(1 << 30)))
    infected = np.array([(p.phi_I_mask >> c) & 1 for c in range(p.n_comp)], bool)
    x, phi = p.u0.astype(np.int64), p.v0.copy()
    D = p.n_days
    out = dict(prevalence=np.zeros((D, 1), np.int32), transitions=np.zeros((D, 1), np.int64),
               totals=np.zeros((D, 1, p.n_comp), np.int64), max_transitions=np.zeros((D, 1), np.int32))
    first = np.searchsorted(p.ev_day, np.arange(D + 1))
    for d in range(D):
        fired = _ssa_day(p, x, phi, d)
        for g in range(first[d], first[d + 1]):
            _event(p, x, g, d)
        I, N = x[:, infected].sum(axis=1), x.sum(axis=1)
        y = d % 365
        beta = p.beta[0, 0 if y <= 91 else 1 if y <= 182 else 2 if y <= 273 else 3]
        phi = (1.0 - beta) * phi + p.alpha[0] * np.where(N > 0, I / np.maximum(N, 1), 0.0)
        out["prevalence"][d, 0] = (I > 0).sum()
        out["transitions"][d, 0] = fired.sum()
        out["totals"][d, 0] = x.sum(axis=0)
        out["max_transitions"][d, 0] = fired.max()
    out["snap_u"], out["snap_v"] = x[None, None].astype(np.int32), phi[None, None]
    return out
