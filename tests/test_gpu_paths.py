"""Kernel paths chosen by size, at the sizes where the choice or the kernel's
tiles end, against the oracle (whole numbers: exact equality)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2509_17837_amd import _lib as X
from paper_2509_17837_amd import decoder as D
from tests._parity import Problem, compare_decode, gpu_plan, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no ROCm GPU visible")
    X.lib()
    torch.cuda.synchronize()


@pytest.mark.parametrize("layout,d,n,offset", [
    (0, 3, 1, 0), (0, 3, 17, 1), (0, 11, 15, 3), (0, 31, 16, 0), (1, 31, 33, 2), (1, 9, 65, 1),
    (0, 5, 65535, 0), (0, 5, 65536 + 7, 1), (1, 3, 65536 + 63, 0), (1, 15, 65536, 3)])
def test_syndrome_tiles(layout, d, n, offset):
    """Tiles of 16 and of 64 configurations, with whole and ragged last tiles,
    from buffers of every byte alignment; bits above a code are ignored."""
    print(f"[paths] syndrome layout={layout} d={d} n={n} offset={offset}", flush=True)
    olat = O.Lattice(layout, d)
    rng = np.random.default_rng(100 * d + n)
    cfg = rng.integers(0, 256, (n, olat.nq), dtype=np.uint8)
    plan = gpu_plan(Problem(layout, d, 0.1, 10.0, 0, 1, 0))
    buf = torch.zeros(n * olat.nq + offset, dtype=torch.uint8, device="cuda")
    buf[offset:] = to_dev(cfg.reshape(-1))
    got = D.syndrome(plan, buf[offset:].reshape(n, olat.nq)).cpu().numpy()
    fq, fm = olat.fq, olat.fm
    pad = np.concatenate([cfg & 3, np.zeros((n, 1), np.uint8)], axis=1)
    want = np.zeros((n, olat.nstab), np.uint8)
    for s in range(4):
        c = pad[:, np.where(fq[:, s] < 0, olat.nq, fq[:, s])]
        want ^= np.where(fm[:, s] == 2, c & 1, np.where(fm[:, s] == 1, c >> 1, 0)).astype(np.uint8)
    for i in {0, n // 2, n - 1}:
        assert np.array_equal(want[i], olat.syndrome(cfg[i] & 3))
    assert np.array_equal(got, want)


# every (lanes, moves per lane) of the grid core: one, two, four and eight
# moves, classes that fill the lanes and classes that leave some idle
GRID_CASES = [
    (0, 3, 4), (0, 3, 64), (0, 5, 4), (0, 5, 8), (0, 7, 4), (0, 7, 8), (0, 7, 16), (0, 9, 8), (0, 9, 16),
    (0, 9, 32), (0, 11, 4), (0, 11, 8), (0, 11, 16), (0, 11, 32), (0, 11, 64), (0, 13, 16), (0, 13, 32), (0, 13, 64),
    (0, 15, 8), (0, 15, 16), (0, 15, 32), (0, 15, 64), (0, 17, 32), (0, 17, 64), (0, 21, 16), (0, 21, 32), (0, 21, 64),
    (0, 25, 64), (0, 29, 32), (0, 31, 32), (0, 31, 64), (1, 3, 4), (1, 5, 16), (1, 7, 8), (1, 7, 32), (1, 9, 16),
    (1, 9, 64), (1, 13, 32), (1, 15, 64), (1, 17, 64), (1, 21, 64), (1, 23, 64), (1, 25, 64), (1, 31, 64)]


@pytest.mark.parametrize("layout,d,lanes", GRID_CASES)
def test_grid_core(layout, d, lanes):
    """Chains over several lanes: every chain, its final state, and the
    recoveries taken from the states kept at E_min."""
    print(f"[paths] grid layout={layout} d={d} lanes={lanes}", flush=True)
    prob = Problem(layout, d, 0.15, 5.0, 3, 3, 25 if d < 20 else 9, seed=40 + d, conv=layout)
    plan = gpu_plan(prob, lanes=lanes)
    out = D.decode(plan, to_dev(prob.syn), to_dev(prob.uid.view(np.int32)), prob.n_rep, prob.greedy_seed,
                   prob.anneal_seed, want_chains=True, want_final=True)
    torch.cuda.synchronize()
    compare_decode(prob, out, prob.oracle_decode())


@pytest.mark.parametrize("d", range(3, 32, 2))
def test_tasks_spanning_syndromes(d):
    """The packed-row kernels specialised to d where 4 n_rep is no multiple of
    64: tasks of 64 chains span syndromes (12 chains each, the last task
    ragged).  Annealing with checkpoints and with a workspace too short for
    them, in the plain form, and ladders (24 chains each)."""
    print(f"[paths] spanning tasks d={d}", flush=True)
    prob = Problem(0, d, 0.15, 10.0, 11, 3, 70, seed=60 + d)
    plan = gpu_plan(prob)
    plan.set_kernel(X.KERNEL_ROWS)
    ref = prob.oracle_decode()
    syn, uid = to_dev(prob.syn), to_dev(prob.uid.view(np.int32))
    for flags, short in ((0, 0), (0, 1), (X.FLAG_PLAIN, 0)):
        g, out = D.make_group(plan, prob.n_rep, uid, syn=syn, want_chains=True, want_final=True)
        ws = D.workspace([g])
        D.decode_groups([g], prob.greedy_seed, prob.anneal_seed, flags=flags, ws=ws[:ws.numel() - short])
        torch.cuda.synchronize()
        compare_decode(prob, out, ref)
    prob = Problem(0, d, 0.15, 10.0, 5, 6, 12, seed=90 + d)
    plan = gpu_plan(prob)
    plan.set_ladder(2, 0.5, 4.0)
    ref = prob.oracle_decode(order=O.ORDER_LADDER, ladder=(2, 0.5, 4.0))
    syn, uid = to_dev(prob.syn), to_dev(prob.uid.view(np.int32))
    for short in (0, 1):
        g, out = D.make_group(plan, prob.n_rep, uid, syn=syn, want_chains=True, want_final=True)
        ws = D.workspace([g])
        D.decode_groups([g], prob.greedy_seed, prob.anneal_seed, ws=ws[:ws.numel() - short])
        torch.cuda.synchronize()
        compare_decode(prob, out, ref)


def test_short_workspace_leaves_the_grid_core():
    """A small call whose workspace holds no grid states runs one chain per
    lane: the same results."""
    prob = Problem(0, 11, 0.15, 10.0, 3, 16, 20, seed=77)
    plan = gpu_plan(prob)
    ref = prob.oracle_decode()
    syn, uid = to_dev(prob.syn), to_dev(prob.uid.view(np.int32))
    for short in (0, 1):
        g, out = D.make_group(plan, prob.n_rep, uid, syn=syn, want_chains=True)
        ws = D.workspace([g])
        D.decode_groups([g], prob.greedy_seed, prob.anneal_seed, ws=ws[:ws.numel() - short])
        torch.cuda.synchronize()
        compare_decode(prob, out, ref)


@pytest.mark.parametrize("layout,d,how", [(0, 7, "rows"), (0, 7, 16), (0, 17, "rows"), (0, 17, 64), (1, 5, "rows"),
                                          (1, 5, 32), (0, 5, "site"), (1, 9, "site"), (0, 7, "ladder"),
                                          (1, 5, "ladder")])
def test_extreme_temperatures(layout, d, how):
    """Thresholds at the ends of their range (beta 0 and 1e-12: 2^32 - 1; about
    2^31; 1; 0 where the exponential underflows), which the energy tables fold
    into the word that also marks the moves that always accept."""
    print(f"[paths] extreme temperatures layout={layout} d={d} {how}", flush=True)
    beta = [0.0, 1e-12, 1e-5, 0.1, 0.3, 5.0, 40.0, 3e2, 1e4, 1e8, 0.0]
    prob = Problem(layout, d, 0.2, 10.0, 3, 4, len(beta), seed=30 + d, conv=layout, beta=beta)
    plan = gpu_plan(prob)
    kw = {}
    if how == "rows":
        plan.set_kernel(X.KERNEL_ROWS)
    elif how == "site":
        plan.set_order(X.ORDER_RANDOM_SITE)
        kw = dict(order=O.ORDER_RANDOM_SITE)
    elif how == "ladder":
        plan.set_ladder(4, 0.0, 400.0)
        kw = dict(order=O.ORDER_LADDER, ladder=(4, 0.0, 400.0))
    else:
        plan.set_lanes(how)
    out = D.decode(plan, to_dev(prob.syn), to_dev(prob.uid.view(np.int32)), prob.n_rep, prob.greedy_seed,
                   prob.anneal_seed, want_chains=True, want_final=True)
    torch.cuda.synchronize()
    compare_decode(prob, out, prob.oracle_decode(**kw))


@pytest.mark.parametrize("layout,d,n_syn", [(0, 3, 1001), (1, 9, 1001), (0, 13, 37), (0, 17, 5), (1, 31, 3)])
def test_random_site_workgroups(layout, d, n_syn):
    """The random-site kernel: rows that share words and rows of several words,
    one wavefront a workgroup and (from 8 wavefronts per CU) eight, the last
    workgroup mostly empty; all outputs and, without a final state, the replay."""
    print(f"[paths] site layout={layout} d={d} n_syn={n_syn}", flush=True)
    prob = Problem(layout, d, 0.15, 10.0, n_syn, 33, 3, seed=40 + d, conv=layout)
    plan = gpu_plan(prob)
    plan.set_order(X.ORDER_RANDOM_SITE)
    ref = prob.oracle_decode(order=O.ORDER_RANDOM_SITE)
    syn, uid = to_dev(prob.syn), to_dev(prob.uid.view(np.int32))
    for short in (0, 1):
        g, out = D.make_group(plan, prob.n_rep, uid, syn=syn, want_chains=True, want_final=not short)
        ws = D.workspace([g])
        D.decode_groups([g], prob.greedy_seed, prob.anneal_seed, ws=ws[:ws.numel() - short])
        torch.cuda.synchronize()
        compare_decode(prob, out, ref)


@pytest.mark.parametrize("layout,d,n_syn,R", [(0, 5, 3001, 23), (1, 9, 2200, 30), (0, 3, 66001, 2), (0, 15, 40, 17),
                                              (0, 21, 7, 33), (0, 31, 5, 12), (1, 31, 2, 5), (0, 17, 1, 1)])
@pytest.mark.parametrize("mode", [X.GREEDY_RANDOM, X.GREEDY_SAME, X.GREEDY_BOUNDARY])
def test_greedy_workgroups(layout, d, n_syn, R, mode):
    """Greedy references where wavefronts share a syndrome: one or several
    references a wavefront, one or several workgroups a syndrome, weights in LDS
    and not; every node a defect (more ties than the list of the first round
    holds, and weights beyond the cache), every second one, one and none."""
    print(f"[paths] greedy layout={layout} d={d} n_syn={n_syn} R={R} mode={mode}", flush=True)
    prob = Problem(layout, d, 0.18, 0.5, n_syn, R, 1, seed=70 + d, conv=layout)
    k = min(5, n_syn)
    prob.syn[0] = 1
    for i, step in ((1, 2), (2, 0), (3, prob.olat.nstab)):
        if i < k:
            prob.syn[i] = 0
            if step:
                prob.syn[i, ::step] = 1
    plan = gpu_plan(prob)
    refs, qcls = D.greedy_init(plan, to_dev(prob.syn), to_dev(prob.uid.view(np.int32)), R, prob.greedy_seed, mode)
    refs, qcls = refs.cpu().numpy(), qcls.cpu().numpy()
    for i in sorted({*range(k), n_syn // 2, n_syn - 1}):
        for r in range(R):
            want = prob.oracle_greedy(i, r, mode)
            assert np.array_equal(refs[i, r], want), (i, r)
            assert qcls[i, r] == prob.olat.cls(want, refs[i, 0]), (i, r)


@pytest.mark.parametrize("layout,d,R", [(0, 5, 16), (1, 5, 4), (0, 9, 20), (0, 17, 4)])
@pytest.mark.parametrize("lo,hi", [(0.7, 0.7), (0.5, 0.5 + 1e-9), (0.5, 0.51), (0.2, 2.0), (0.0, 3e3), (0.0, 1e9)])
def test_exchange_rule(layout, d, R, lo, hi):
    """Exchanges are decided by a bound and, between its two sides, by the
    fixed-point product: equal levels (every exchange nearly certain), spacings
    from the least to one whose first power underflows."""
    print(f"[paths] exchange layout={layout} d={d} R={R} beta={lo}..{hi}", flush=True)
    prob = Problem(layout, d, 0.2, 5.0, 4, R, 40, seed=50 + d, conv=layout)
    plan = gpu_plan(prob)
    plan.set_ladder(4, lo, hi)
    out = D.decode(plan, to_dev(prob.syn), to_dev(prob.uid.view(np.int32)), prob.n_rep, prob.greedy_seed,
                   prob.anneal_seed, want_chains=True, want_final=True)
    torch.cuda.synchronize()
    compare_decode(prob, out, prob.oracle_decode(order=O.ORDER_LADDER, ladder=(4, lo, hi)))


def test_finish_of_mixed_groups():
    """One call over groups of every kind of recovery (states kept by the grid
    core, the planar and ladder kernels and the random-site kernel, and replays),
    with one to more than 64 chains a syndrome."""
    kinds = [("auto", 0, 5, 3, 1), ("auto", 1, 7, 2, 5), ("rows", 0, 7, 5, 3), ("rows", 0, 5, 9, 17),
             ("rows", 1, 5, 4, 2), ("rows", 1, 9, 1, 33), ("site", 0, 5, 6, 3), ("site", 1, 9, 2, 5),
             ("ladder", 0, 5, 3, 4), ("ladder", 0, 17, 2, 20), ("ladder", 1, 7, 3, 6), ("ladder", 1, 17, 2, 4),
             ("bytes", 0, 9, 3, 2), ("bytes", 1, 3, 7, 1), ("rows", 0, 31, 1, 2), ("auto", 1, 17, 1, 1)]
    made = []
    for kind, layout, d, n, R in kinds:
        prob = Problem(layout, d, 0.15, 5.0, n, R, 6, seed=123, conv=layout)
        plan = gpu_plan(prob)
        kw = {}
        if kind == "rows":
            plan.set_kernel(X.KERNEL_ROWS)
        elif kind == "bytes":
            plan.set_lanes(2)
        elif kind == "site":
            plan.set_order(X.ORDER_RANDOM_SITE)
            kw = dict(order=O.ORDER_RANDOM_SITE)
        elif kind == "ladder":
            plan.set_ladder(2, 0.5, 2.0)
            kw = dict(order=O.ORDER_LADDER, ladder=(2, 0.5, 2.0))
        g, out = D.make_group(plan, R, to_dev(prob.uid.view(np.int32)), syn=to_dev(prob.syn), want_chains=True,
                              want_final=True)
        made.append((prob, g, out, kw))
    seeds = made[0][0]
    D.decode_groups([g for _, g, _, _ in made], seeds.greedy_seed, seeds.anneal_seed)
    torch.cuda.synchronize()
    for (prob, _, out, kw), what in zip(made, kinds):
        print(f"[paths] finish {what}", flush=True)
        compare_decode(prob, out, prob.oracle_decode(**kw))


@pytest.mark.parametrize("sweeps", [16, 17, 18, 100, 129, 513])
def test_checkpoint_intervals(sweeps):
    """Checkpoints of short schedules (none at 16 sweeps; one, at the start of
    the last sweep, at 17; at most eight) and, with a workspace short of the
    full size, the sparser ones (at 16 and 513 sweeps the two are the same, and
    the full size is the least)."""
    prob = Problem(0, 9, 0.2, 10.0, 5, 16, sweeps, seed=500 + sweeps)
    plan = gpu_plan(prob)
    plan.set_kernel(X.KERNEL_ROWS)
    ref = prob.oracle_decode()
    syn, uid = to_dev(prob.syn), to_dev(prob.uid.view(np.int32))
    for short in (0, 1) if 16 < sweeps < 513 else (0,):
        g, out = D.make_group(plan, prob.n_rep, uid, syn=syn, want_chains=True, want_final=True)
        ws = D.workspace([g])
        D.decode_groups([g], prob.greedy_seed, prob.anneal_seed, ws=ws[:ws.numel() - short])
        torch.cuda.synchronize()
        compare_decode(prob, out, ref)
