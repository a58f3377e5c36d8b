"""Performance cases of the decoder: what its users run, through the public
entry points of ``paper_2509_17837_amd.decoder``.

Four kinds of work make up a user's program:

``syndrome``  the syndromes of a Monte Carlo batch of sampled errors;
``greedy``    greedy-matching references alone (the greedy decoder, and the
              first stage of a decode);
``decode``    the whole decoder on a batch: one syndrome or many, both
              lattices, colour-class or random-site steps, annealing or
              replica exchange, through a plain call, kept buffers or a
              captured graph;
``anneal``    the chains from references the caller already has;
``serve``     single-syndrome requests through the serving loop.

Sizes are those of the repository's workloads (``inputs.WORKLOADS``), of its
tests, and of the paper's Monte Carlo (N_SA = 1..100 references per syndrome);
long schedules and batches are cut where a pass would take seconds.
"""
import numpy as np
import torch

from paper_2509_17837_amd import _lib as X
from paper_2509_17837_amd import decoder as D

LAYOUT = {"rotated": X.ROTATED, "planar": X.PLANAR}
NOISE = {"ratio": X.BIAS_RATIO, "paper": X.BIAS_PAPER}
SCHEDULE = {"linear": X.SCHED_LINEAR, "geometric": X.SCHED_GEOMETRIC, "paper_log": X.SCHED_PAPER_LOG}
MODE = {"random": X.GREEDY_RANDOM, "same": X.GREEDY_SAME, "boundary": X.GREEDY_BOUNDARY}
GREEDY_SEED, ANNEAL_SEED = 2001, 3001

# what a decode is when a case does not say otherwise
DECODE = dict(kind="decode", layout="rotated", noise="ratio", schedule="geometric", b0=0.05, b1=10.0, order="colour",
              ladder=0, ladder_lo=0.5, ladder_hi=10.0, mode="random", via="call", chains=False)


def listed():
    return [
        # Monte Carlo: the syndromes of 10^6 sampled errors on the paper's own lattice
        dict(name="syndrome_planar_d9_1e6", kind="syndrome", layout="planar", d="9", p="0.15", eta="5", noise="paper",
             n=1_000_000),
        # the greedy decoder's references on a large lattice: an odd batch, the paper's N_SA = 10
        dict(name="greedy_d21", kind="greedy", layout="rotated", d="21", p="0.15", eta="10", noise="ratio", n=1021,
             reps=10, mode="random"),
        # one syndrome in hand, the answer awaited: latency (the serving workload's replicas and sweeps)
        dict(DECODE, name="decode_one_d11", d="11", p="0.12", eta="10", n=1, reps=16, sweeps=1000),
        # the smallest workload: d = 3, one reference, four chains a syndrome
        dict(DECODE, name="decode_d3_small", d="3", p="0.15", eta="10", n=1000, reps=1, sweeps=200, schedule="linear",
             b0=0.1, b1=5.0),
        # the headline throughput workload: four error rates in one call, buffers kept between calls
        dict(DECODE, name="decode_d11_bias100", d="11", p="0.10,0.15,0.20,0.25", eta="100", n=2048, reps=32,
             sweeps=2000, via="kept"),
        # uneven distances in one call
        dict(DECODE, name="decode_mixed_d5_21", d="5,9,13,17,21", p="0.18", eta="10", n=256, reps=64, sweeps=5000,
             via="kept"),
        # the largest lattice
        dict(DECODE, name="decode_d31_large", d="31", p="0.20", eta="10", n=512, reps=128, sweeps=2000, b0=0.02,
             b1=20.0, via="kept"),
        # the paper's Monte Carlo, six noise settings in one captured decode
        dict(DECODE, name="decode_planar_paper_d9", layout="planar", noise="paper", d="9", p="0.10,0.15", eta="1,5,10",
             n=2048, reps=10, sweeps=100, schedule="paper_log", b0=0.9, b1=1.0, via="graph"),
        # the same with the chain as the paper prints it: one random generator per step
        dict(DECODE, name="decode_planar_site_d9", layout="planar", noise="paper", d="9", p="0.10,0.15", eta="1,5,10",
             n=2048, reps=10, sweeps=100, schedule="paper_log", b0=0.9, b1=1.0, order="site", via="graph"),
        # the paper's N_SA = 10 and N_beta = 100 on the rotated lattice, per-chain results kept: 40 chains a syndrome
        dict(DECODE, name="decode_rotated_nsa10_d13", d="13", p="0.15", eta="5", n=4099, reps=10, sweeps=100,
             schedule="paper_log", b0=0.9, b1=1.0, chains=True),
        # replica exchange
        dict(DECODE, name="decode_ladder_d11", d="11", p="0.10,0.15,0.20,0.25", eta="100", n=512, reps=32, sweeps=1000,
             ladder=4, via="kept"),
        # the serving loop with a burst of requests of mixed distances
        dict(name="serve_burst_d7_25", kind="serve", d="7,11,15,19,25", p="0.12", eta="1,10,1000", n=48, reps=16,
             sweeps=1000),
    ]


def _log_int(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return int(round(lo * (hi / lo) ** rng.random()))


# attempts of a drawn case: a small part of the largest listed one's, since a small batch runs far below the full rate
MOST_ATTEMPTS = 4e9


def draw(rng):
    kind = rng.choice(["syndrome", "greedy", "decode", "decode", "decode", "decode", "decode", "anneal", "serve"])
    layout = rng.choice(["rotated", "rotated", "planar"])
    p, eta = round(rng.uniform(0.02, 0.25), 3), rng.choice([1, 5, 10, 100, 1000])
    noise = "paper" if layout == "planar" else "ratio"
    if kind == "syndrome":
        d = rng.randrange(3, 32, 2)
        n = min(_log_int(rng, 1000, 1_000_000), 250_000_000 // (2 * _qubits(layout, d)))
        return dict(kind=kind, layout=layout, d=str(d), p=str(p), eta=str(eta), noise=noise, n=n)
    if kind == "greedy":
        d, reps = rng.randrange(3, 32, 2), _log_int(rng, 1, 100)
        n = min(_log_int(rng, 1, 8192), max(1, 60_000 // reps))
        return dict(kind=kind, layout=layout, d=str(d), p=str(p), eta=str(eta), noise=noise, n=n, reps=reps,
                    mode=rng.choice(["random", "random", "same", "boundary"]))
    if kind == "serve":
        ds = sorted(rng.sample([7, 11, 15, 19, 25], rng.randint(1, 4)))
        return dict(kind=kind, d=",".join(map(str, ds)), p=str(p), eta=str(eta), n=_log_int(rng, 1, 200), reps=16,
                    sweeps=_log_int(rng, 100, 1000))
    order, ladder = "colour", 0
    top = 31 if layout == "rotated" else 21
    if kind == "decode":
        special = rng.choice(["", "", "", "site", "ladder"])
        if special == "site":
            order, top = "site", 15
        elif special == "ladder":
            ladder, top = rng.choice([2, 4, 8]), 15
    ds = [rng.randrange(3, top + 1, 2) for _ in range(rng.choice([1, 1, 1, 2, 4]))]
    reps = rng.choice([1, 2, 5, 10, 16, 20, 32, 50, 64])
    if ladder:
        reps = ladder * max(1, reps // ladder)
    sweeps = _log_int(rng, 50, 5000)
    per = sum(4.0 * reps * sweeps * _stabs(layout, d) for d in ds)
    n = int(max(1, min(_log_int(rng, 1, 8192), MOST_ATTEMPTS / per)))
    schedule, b0, b1 = rng.choice([("geometric", 0.05, 10.0), ("paper_log", 0.9, 1.0), ("linear", 0.1, 5.0)])
    return dict(DECODE, kind=kind, layout=layout, noise=noise, d=",".join(map(str, ds)), p=str(p), eta=str(eta), n=n,
                reps=reps, sweeps=sweeps, schedule=schedule, b0=b0, b1=b1, order=order, ladder=ladder,
                via="kept" if kind == "anneal" or len(ds) > 1 else rng.choice(["call", "kept", "graph"]),
                chains=rng.random() < 0.3)


def _qubits(layout, d):
    return d * d if layout == "rotated" else d * d + (d - 1) * (d - 1)


def _stabs(layout, d):
    return d * d - 1 if layout == "rotated" else 2 * d * (d - 1)


def _settings(case):
    """One (d, p, eta) per group of syndromes: every combination the case names."""
    return [(int(d), float(p), float(e)) for d in case["d"].split(",") for p in case["p"].split(",")
            for e in case["eta"].split(",")]


def _plan(case, d, p, eta):
    pxyz = D.noise(p, eta, NOISE[case.get("noise", "ratio")])
    w, wg = D.weights(p, pxyz)
    if "schedule" in case:
        beta = D.schedule(SCHEDULE[case["schedule"]], case["b0"], case["b1"], case["sweeps"])
    else:
        beta = D.schedule(X.SCHED_GEOMETRIC, 0.05, 10.0, case.get("sweeps", 0))
    plan = D.Plan(D.Lattice(LAYOUT[case.get("layout", "rotated")], d), w, wg, beta)
    if case.get("order") == "site":
        plan.set_order(X.ORDER_RANDOM_SITE)
    if case.get("ladder"):
        plan.set_ladder(case["ladder"], case["ladder_lo"], case["ladder_hi"])
    return plan, pxyz


def _errors(n, nq, pxyz, seed):
    """n i.i.d. error configurations on the GPU (Pauli codes I=0, Z=1, X=2, Y=3)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.rand((n, nq), generator=gen, device="cuda")
    px, py, pz = (float(v) for v in pxyz)
    cfg = torch.zeros((n, nq), dtype=torch.uint8, device="cuda")
    cfg[u < px + py + pz] = 1
    cfg[u < px + py] = 3
    cfg[u < px] = 2
    return cfg


def prepare(case, seed):
    kind = case["kind"]
    groups = []
    for k, (d, p, eta) in enumerate(_settings(case)):
        plan, pxyz = _plan(case, d, p, eta)
        n = case["n"] if kind != "serve" else -(-case["n"] // len(_settings(case)))
        cfg = _errors(n, plan.nq, pxyz, 1000 * seed + k)
        groups.append((plan, cfg, torch.arange(k * n, k * n + n, dtype=torch.int32, device="cuda")))
    state = dict(case=case)
    if kind == "syndrome":
        state.update(plan=groups[0][0], cfg=groups[0][1])
        return state
    state["in"] = [(plan, D.syndrome(plan, cfg), uid) for plan, cfg, uid in groups]
    if kind == "serve":
        # requests of the settings in turn, as their host programs hand them in
        host = [(plan, syn.cpu().numpy(), uid.cpu().numpy()) for plan, syn, uid in state["in"]]
        reqs = [(host[i % len(host)], i // len(host)) for i in range(case["n"])]
        state["plans"] = [h[0] for h, _ in reqs]
        state["syndromes"] = [np.ascontiguousarray(h[1][j]) for h, j in reqs]
        state["uids"] = [int(h[2][j]) for h, j in reqs]
        state["server"] = D.Server(max_slots=256, max_rep=16, max_qubits=625, sweeps_per_slice=250,
                                   greedy_seed=GREEDY_SEED, anneal_seed=ANNEAL_SEED)
    elif kind == "anneal":
        made = []
        for plan, syn, uid in state["in"]:
            refs, qcls = D.greedy_init(plan, syn, uid, case["reps"], GREEDY_SEED, MODE[case["mode"]])
            made.append(D.make_group(plan, case["reps"], uid, refs=refs, qcls=qcls, want_chains=case["chains"]))
        state["groups"], state["outs"] = [g for g, _ in made], [o for _, o in made]
        state["ws"] = D.workspace(state["groups"])
    elif kind == "decode" and case["via"] != "call":
        made = [D.make_group(plan, case["reps"], uid, syn=syn, want_chains=case["chains"])
                for plan, syn, uid in state["in"]]
        state["groups"], state["outs"] = [g for g, _ in made], [o for _, o in made]
        if case["via"] == "graph":
            torch.cuda.synchronize()
            state["graph"] = D.Graph(state["groups"], GREEDY_SEED, ANNEAL_SEED, MODE[case["mode"]])
        else:
            state["ws"] = D.workspace(state["groups"])
    return state


def _results(o):
    names = ["e_best", "cls", "recovery", "paper_recovery", "e_cls", "best_chain", "refs", "qcls", "chain_emin",
             "chain_stop", "chain_e"]
    return {n: getattr(o, n) for n in names if getattr(o, n) is not None}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "syndrome":
        return D.syndrome(state["plan"], state["cfg"])
    if kind == "greedy":
        plan, syn, uid = state["in"][0]
        return D.greedy_init(plan, syn, uid, case["reps"], GREEDY_SEED, MODE[case["mode"]])
    if kind == "serve":
        srv = state["server"]
        tickets = srv.submit_many(state["plans"], state["syndromes"], state["uids"], case["reps"])
        srv.drain()
        done = [srv.poll(t) for t in tickets]
        return dict(e_best=np.array([r["e_best"] for r in done]), cls=np.array([r["cls"] for r in done]),
                    e_cls=np.array([r["e_cls"] for r in done]), recovery=np.concatenate([r["recovery"] for r in done]))
    if kind == "anneal":
        D.anneal_groups(state["groups"], ANNEAL_SEED, ws=state["ws"])
    elif case["via"] == "call":
        plan, syn, uid = state["in"][0]
        return _results(D.decode(plan, syn, uid, case["reps"], GREEDY_SEED, ANNEAL_SEED, MODE[case["mode"]],
                                 want_chains=case["chains"]))
    elif case["via"] == "graph":
        state["graph"].launch(torch.cuda.current_stream())
    else:
        D.decode_groups(state["groups"], GREEDY_SEED, ANNEAL_SEED, MODE[case["mode"]], ws=state["ws"])
    outs = [_results(o) for o in state["outs"]]
    if len(outs) <= 5:
        return outs
    # many groups: one tensor per result, the groups' one after another
    return {name: torch.cat([o[name].reshape(-1) for o in outs]) for name in outs[0]}


def work(case):
    """Bytes: syndromes and ids in, results out, each once.  Operations: 19
    int32 operations per flip attempt (a quarter of a Philox4x32-10 block, 10;
    pattern, table index, acceptance, energy and flips of the move, 9)."""
    kind, layout = case["kind"], case.get("layout", "rotated")
    settings = _settings(case)
    nbytes = attempts = 0
    for d, _, _ in settings:
        nq, ns = _qubits(layout, d), _stabs(layout, d)
        n = case["n"] / (len(settings) if kind == "serve" else 1)
        if kind == "syndrome":
            nbytes += n * (nq + ns)
            continue
        reps = case["reps"]
        nbytes += n * (ns + 4)
        if kind == "greedy":
            nbytes += n * reps * (nq + 1)
            continue
        attempts += n * 4 * reps * case["sweeps"] * ns
        nbytes += n * (nq + 21)
        if kind != "serve":
            nbytes += n * (nq + 4 + reps * (nq + 1)) + (n * 48 * reps if case["chains"] else 0)
    return {"bytes": nbytes, "flops": 19 * attempts}


def _syndrome_slots(layout, d):
    """Qubits of every generator's X_left, Z_up, Z_down, X_right slots (the
    last index is an absent qubit), generators numbered row by row."""
    rows = []
    if layout == "rotated":
        def at(x, y):
            return y * d + x if 0 <= x < d and 0 <= y < d else d * d
        for j in range(-1, d):
            for i in range(-1, d):
                inside_i, inside_j = 0 <= i <= d - 2, 0 <= j <= d - 2
                keep = (inside_i and inside_j) or (inside_i and j == -1 and i % 2 == 1) \
                    or (inside_i and j == d - 1 and i % 2 == 0) or (inside_j and i == -1 and j % 2 == 0) \
                    or (inside_j and i == d - 1 and j % 2 == 1)
                if keep:
                    rows.append([at(i, j), at(i + 1, j), at(i, j + 1), at(i + 1, j + 1)])
        return rows, d * d
    index = {}
    for y in range(2, 2 * d - 1, 2):
        for x in range(3, 2 * d, 2):
            index[x, y] = len(index)
    for y in range(1, 2 * d, 2):
        for x in range(2, 2 * d + 1, 2):
            index[x, y] = len(index)
    nq = len(index)
    faces = [(2 * j, 2 * i) for i in range(1, d + 1) for j in range(1, d)]
    faces += [(2 * j - 1, 2 * i + 1) for i in range(1, d) for j in range(1, d + 1)]
    for y, x in sorted(faces):
        rows.append([index.get(q, nq) for q in ((x - 1, y), (x, y + 1), (x, y - 1), (x + 1, y))])
    return rows, nq


def exact(case, seed):
    """Syndromes are parities of the sampled errors (Eq. (2)).  The other
    kinds return whole numbers that a random walk defines."""
    if case["kind"] != "syndrome":
        return None
    d, p, eta = _settings(case)[0]
    if case["noise"] == "ratio":
        pxyz = (p / (2 * (eta + 1)), p * eta / (eta + 1), p / (2 * (eta + 1)))
    else:
        pxyz = (p / (eta + 2), p * eta / (eta + 2), p / (eta + 2))
    rows, nq = _syndrome_slots(case["layout"], d)
    cfg = _errors(case["n"], nq, pxyz, 1000 * seed)
    q = torch.tensor(rows, device="cuda")
    out = torch.empty((case["n"], len(rows)), dtype=torch.uint8, device="cuda")
    for a in range(0, case["n"], 1 << 16):
        c = torch.nn.functional.pad(cfg[a:a + (1 << 16)], (0, 1))
        out[a:a + (1 << 16)] = ((c[:, q[:, 0]] & 1) ^ (c[:, q[:, 1]] >> 1) ^ (c[:, q[:, 2]] >> 1) ^ (c[:, q[:, 3]] & 1))
    return out
