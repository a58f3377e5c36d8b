"""The kernel a call runs on: what selects it, by the library's own account
(xzzx_decode_routes) or by its time, and the results of kernels that the
default leaves to other sizes, against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2509_17837_amd import _lib as X
from paper_2509_17837_amd import decoder as D
from tests._parity import Problem, compare_decode, gpu_plan, to_dev

pytestmark = pytest.mark.gpu

GRID = 16   # xzzx_decode_routes: one chain over several lanes, the states a grid of bytes


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no ROCm GPU visible")
    X.lib()
    torch.cuda.synchronize()


def routes(groups, ws_bytes):
    """[(kernel, lanes per chain)] of the groups of a call with such a workspace."""
    n = len(groups)
    kernel, lanes = (C.c_int32 * n)(), (C.c_int32 * n)()
    X.check("xzzx_decode_routes", X.lib().xzzx_decode_routes(
        (X.Group * n)(*groups), n, C.c_size_t(ws_bytes), kernel, lanes))
    return list(zip(kernel, lanes))


def group_of(plan, n, n_rep):
    uid = torch.arange(n, dtype=torch.int32, device="cuda")
    return D.make_group(plan, n_rep, uid, syn=torch.zeros((n, plan.nstab), dtype=torch.uint8, device="cuda"))


def anneal_ms(g):
    """Least time of the annealing stage over three runs after a first one."""
    ws = D.decode_groups([g], 1, 2, flags=X.STAGE_GREEDY)
    times = []
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        D.decode_groups([g], 1, 2, flags=X.STAGE_ANNEAL, ws=ws)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times[1:])


def test_autotuner_small_call():
    """One syndrome: the packed-row candidate is the packed-row kernel (a chain
    a lane, a tenth of the speed of 32 lanes), and the plan keeps both the
    grid core for such calls and the packed rows for large ones."""
    plan = gpu_plan(Problem(0, 11, 0.12, 10.0, 0, 1, 200, seed=3))
    tuned = plan.autotune(16, n_syn=1, probe_sweeps=200)
    print(f"[routes] tuned {tuned}", flush=True)
    assert tuned["times_ms"]["rows"] > 3.0 * tuned["times_ms"]["bytes32"]
    assert tuned["kernel"] == "bytes" and tuned["lanes_per_chain"] >= 16
    small, large = group_of(plan, 1, 16)[0], group_of(plan, 2000, 16)[0]
    assert routes([small], D.workspace([small]).numel())[0][0] == GRID
    assert routes([large], D.workspace([large]).numel())[0][0] == X.KERNEL_ROWS


def test_autotuner_large_call():
    """Chosen lanes are timed on the kernel that a plan with those lanes runs on,
    also where the default's workspace holds no states of it."""
    n, R = 4096, 16
    prob = Problem(0, 11, 0.12, 10.0, 0, 1, 64, seed=4)
    plan = gpu_plan(prob)
    tuned = plan.autotune(R, n_syn=n, probe_sweeps=64)
    print(f"[routes] tuned {tuned}", flush=True)
    assert tuned["kernel"] == "rows"
    rng = np.random.default_rng(5)
    for lanes in (16, 32):
        plan.set_lanes(lanes)
        g, o = group_of(plan, n, R)
        o.keep[2].copy_(torch.from_numpy(rng.integers(0, 2, (n, plan.nstab), dtype=np.uint8)))
        assert routes([g], D.workspace([g]).numel()) == [(GRID, lanes)]
        alone = anneal_ms(g)
        print(f"[routes] {lanes} lanes {alone:.3f} ms", flush=True)
        assert tuned["times_ms"][f"bytes{lanes}"] < 1.4 * alone


def serve_routes(srv, plans, n_rep):
    """[(kernel, lanes per chain)] in a slice that holds one request of each plan."""
    n = len(plans)
    reqs = (X.Request * n)(*[X.Request(p.h, None, 0, n_rep) for p in plans])
    kernel, lanes = (C.c_int32 * n)(), (C.c_int32 * n)()
    X.check("xzzx_server_routes", X.lib().xzzx_server_routes(srv.h, reqs, n, kernel, lanes))
    return list(zip(kernel, lanes))


def test_serving_forms():
    """Which requests of a slice run one chain per lane: those with a specialised
    packed-row kernel, where their work fills the device in that form (more than
    32768 chains of the largest lattice among them); planar lattices and plans
    with another kernel chosen do not."""
    def plan(layout, d, **kw):
        return gpu_plan(Problem(layout, d, 0.15, 10.0, 0, 1, 10, seed=d, conv=layout), **kw)

    srv = D.Server(max_slots=8, max_rep=16, max_qubits=1861)
    limited = D.Server(max_slots=8, max_rep=16, max_qubits=1861, max_lanes_per_chain=1)
    try:
        r11 = plan(0, 11)
        assert set(serve_routes(srv, [r11] * 100, 16)) == {(GRID, 32)}
        assert set(serve_routes(srv, [r11] * 600, 16)) == {(X.KERNEL_ROWS, 1)}
        assert set(serve_routes(limited, [r11] * 100, 16)) == {(X.KERNEL_ROWS, 1)}
        for d in (17, 21, 31):
            p = plan(1, d)
            assert set(serve_routes(srv, [p] * 1024, 16)) == {(GRID, 64)}
            assert {k for k, _ in serve_routes(limited, [p] * 1024, 16)} == {X.KERNEL_BYTES}
        for p in (plan(1, 5), plan(1, 9), plan(1, 15), plan(0, 15, lanes=1)):
            got = serve_routes(srv, [p] * 400, 16)
            assert {k for k, _ in got} <= {GRID, X.KERNEL_BYTES} and min(l for _, l in got) >= 8
        # a third of the chains cannot fill the device with one of d = 25 on each lane
        wide = [plan(0, d) for d in (7, 13, 25)]
        assert X.KERNEL_ROWS not in {k for k, _ in serve_routes(srv, [wide[i % 3] for i in range(400)], 16)}
        assert serve_routes(srv, [wide[i % 3] for i in range(400)], 16)[2] == (GRID, 32)
        assert serve_routes(srv, [wide[i % 3] for i in range(330)], 16)[2] == (GRID, 32)
        both = serve_routes(srv, [plan(1, 21), r11] * 600, 16)
        assert both[0] == (GRID, 64) and both[1] == (X.KERNEL_ROWS, 1)
    finally:
        srv.close()
        limited.close()


@pytest.mark.parametrize("kinds", [[(1, 21), (0, 11)], [(1, 9), (0, 25), (0, 5)]])
def test_serving_under_load_matches_decode(kinds):
    """Requests past the grid core's range in mixed forms: the results of a batch
    decode (which the parity tests compare with the oracle)."""
    probs = [Problem(l, d, 0.15, 10.0, -(-450 // len(kinds)), 16, 12, seed=7, conv=l) for l, d in kinds]
    plans = [gpu_plan(p) for p in probs]
    srv = D.Server(max_slots=512, max_rep=16, max_qubits=841, sweeps_per_slice=5, greedy_seed=21, anneal_seed=22)
    try:
        reqs = [(k, i) for i in range(probs[0].n_syn) for k in range(len(kinds))]
        tickets = srv.submit_many([plans[k] for k, _ in reqs], [probs[k].syn[i] for k, i in reqs],
                                  [int(probs[k].uid[i]) for k, i in reqs], 16)
        srv.drain()
        got = [srv.poll(t) for t in tickets]
    finally:
        srv.close()
    for k, (prob, plan) in enumerate(zip(probs, plans)):
        out = D.decode(plan, to_dev(prob.syn), to_dev(prob.uid.view(np.int32)), 16, 21, 22)
        torch.cuda.synchronize()
        mine = [g for g, (kk, _) in zip(got, reqs) if kk == k]
        assert np.array_equal([g["e_best"] for g in mine], out.e_best.cpu().numpy())
        assert np.array_equal([g["cls"] for g in mine], out.cls.cpu().numpy())
        assert np.array_equal(np.stack([g["recovery"] for g in mine]), out.recovery.cpu().numpy())


def test_random_site_states_in_a_short_workspace():
    """Random-site calls keep each chain's best state also with the least
    workspace: the finish reads it, where a replay would run whole schedules."""
    prob = Problem(1, 9, 0.15, 5.0, 0, 1, 100, seed=9, conv=1)
    plan = gpu_plan(prob)
    plan.set_order(X.ORDER_RANDOM_SITE)
    g, o = group_of(plan, 2048, 10)
    rng = np.random.default_rng(6)
    o.keep[2].copy_(torch.from_numpy(rng.integers(0, 2, (2048, plan.nstab), dtype=np.uint8)))
    full = D.workspace([g])
    ws = full[:full.numel() - 1]
    times = {}
    for stage in (X.STAGE_GREEDY, X.STAGE_ANNEAL, X.STAGE_FINISH, X.STAGE_ANNEAL, X.STAGE_FINISH):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        D.decode_groups([g], 1, 2, flags=stage, ws=ws)
        b.record()
        torch.cuda.synchronize()
        times[stage] = a.elapsed_time(b)
    print(f"[routes] stages {times}", flush=True)
    assert times[X.STAGE_FINISH] < 0.2 * times[X.STAGE_ANNEAL]
    short = [t.clone() for t in (o.e_best, o.cls, o.recovery)]
    D.decode_groups([g], 1, 2, ws=full)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(short, (o.e_best, o.cls, o.recovery)))


@pytest.mark.parametrize("layout,d,n", [(1, 31, 1), (1, 31, 17), (1, 25, 100), (1, 31, 4100), (1, 23, 16)])
def test_syndrome_large_lattices(layout, d, n):
    """Syndromes of large lattices: a few workgroups with more threads, many with
    fewer; a small batch costs about what one of a small lattice does."""
    olat = O.Lattice(layout, d)
    rng = np.random.default_rng(d + n)
    cfg = rng.integers(0, 4, (n, olat.nq), dtype=np.uint8)
    plan = gpu_plan(Problem(layout, d, 0.1, 10.0, 0, 1, 0))
    got = D.syndrome(plan, to_dev(cfg)).cpu().numpy()
    for i in {0, n // 2, n - 1}:
        assert np.array_equal(got[i], olat.syndrome(cfg[i]))
    if n > 1000:
        return

    def us(plan, nq):
        x = torch.zeros((n, nq), dtype=torch.uint8, device="cuda")
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(50):
                D.syndrome(plan, x)
            b.record()
            torch.cuda.synchronize()
            best = min(best, 20.0 * a.elapsed_time(b))
        return best

    small = us(gpu_plan(Problem(1, 3, 0.1, 10.0, 0, 1, 0)), 13)
    large = us(plan, olat.nq)
    print(f"[routes] syndrome d={d} n={n}: {large:.1f} us, d=3 {small:.1f}", flush=True)
    assert large < 1.3 * small


@pytest.mark.parametrize("layout,d,n_syn,R", [
    (0, 17, 2500, 7), (0, 31, 150, 24), (1, 17, 6000, 2), (0, 21, 9001, 1), (1, 31, 1, 9), (0, 27, 3, 1), (1, 13, 60, 3),
    (0, 11, 4001, 1), (0, 9, 1, 16), (0, 15, 3000, 4), (0, 7, 12001, 5), (0, 3, 6001, 10), (1, 3, 90, 3), (0, 5, 2, 300)])
def test_greedy_forms(layout, d, n_syn, R):
    """Greedy references in wide and narrow workgroups: several workgroups a
    syndrome, one wavefront for both colours, wavefronts that only help in the
    scan, shorter lists of first ties; every node a defect (more ties than any
    list), every second and third one, one and none among the syndromes."""
    print(f"[routes] greedy layout={layout} d={d} n_syn={n_syn} R={R}", flush=True)
    prob = Problem(layout, d, 0.18, 0.5, n_syn, R, 1, seed=170 + d, conv=layout)
    for i, step in enumerate((1, 2, 3, 0, prob.olat.nstab)):
        if i < n_syn:
            prob.syn[i] = 0
            if step:
                prob.syn[i, ::step] = 1
    plan = gpu_plan(prob)
    refs, qcls = D.greedy_init(plan, to_dev(prob.syn), to_dev(prob.uid.view(np.int32)), R, prob.greedy_seed,
                               X.GREEDY_RANDOM)
    refs, qcls = refs.cpu().numpy(), qcls.cpu().numpy()
    for i in sorted({*range(min(5, n_syn)), n_syn // 2, n_syn - 1}):
        for r in {*range(min(R, 8)), R - 1}:
            want = prob.oracle_greedy(i, r, X.GREEDY_RANDOM)
            assert np.array_equal(refs[i, r], want), (i, r)
            assert qcls[i, r] == prob.olat.cls(want, refs[i, 0]), (i, r)


@pytest.mark.parametrize("layout,d,n_syn,R", [
    (0, 21, 1500, 12), (0, 21, 250, 32), (0, 31, 1000, 10), (1, 25, 300, 16), (0, 15, 1250, 32), (0, 7, 30000, 10)])
def test_greedy_forms_by_size(layout, d, n_syn, R):
    """Launches past the smallest that take wide workgroups: by their wavefronts,
    by turns over the device, where LDS bounds the narrow ones, in the split form;
    and references nine in turn."""
    test_greedy_forms(layout, d, n_syn, R)


@pytest.mark.parametrize("layout,d,n,R", [(0, 21, 8192, 4), (0, 25, 8192, 4), (0, 15, 26000, 5), (1, 17, 12000, 5)])
def test_greedy_sharing_pays(layout, d, n, R):
    """R replicas that share their syndrome's scan take no longer than R calls of
    one replica, also where weights kept in LDS would leave a CU few wavefronts."""
    plan = gpu_plan(Problem(layout, d, 0.1, 10.0, 0, 1, 1, seed=d, conv=layout))
    rng = np.random.default_rng(d)
    syn = to_dev((rng.random((n, plan.nstab)) < 0.06).astype(np.uint8))
    uid = torch.arange(n, dtype=torch.int32, device="cuda")

    def us(reps):
        best = 1e9
        for k in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            D.greedy_init(plan, syn, uid, reps, 3)
            b.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b)) if k else best
        return best

    one, many = us(1), us(R)
    print(f"[routes] greedy d={d} n={n}: 1 x {one:.0f} us, {R} x {many:.0f} us", flush=True)
    assert many < R * one


def least_bytes(groups):
    n = C.c_size_t()
    X.check("xzzx_decode_workspace_least", X.lib().xzzx_decode_workspace_least(
        (X.Group * len(groups))(*groups), len(groups), C.byref(n)))
    return n.value


def made(probs, plans, **kw):
    out = [D.make_group(plan, p.n_rep, to_dev(p.uid.view(np.int32)), syn=to_dev(p.syn), want_chains=True, **kw)
           for p, plan in zip(probs, plans)]
    return [g for g, _ in out], [o for _, o in out]


def test_workspace_is_shared_out_by_group():
    """A workspace short by a byte costs only the group whose better form takes
    most its form: the small group stays on the grid core."""
    probs = [Problem(0, 11, 0.15, 10.0, 2, 8, 40, seed=5), Problem(0, 21, 0.15, 10.0, 9, 5, 40, seed=5),
             Problem(1, 7, 0.15, 5.0, 3, 6, 40, seed=5, conv=1)]
    plans = [gpu_plan(p) for p in probs]
    plans[1].set_kernel(X.KERNEL_ROWS)
    plans[2].set_order(X.ORDER_RANDOM_SITE)
    groups, outs = made(probs, plans)
    full, least = D.workspace(groups).numel(), least_bytes(groups)
    assert least < full
    refs = [probs[0].oracle_decode(), probs[1].oracle_decode(), probs[2].oracle_decode(order=O.ORDER_RANDOM_SITE)]
    for size, first in ((full, GRID), (full - 1, GRID), (least, X.KERNEL_ROWS)):
        assert routes(groups, size)[0][0] == first
        D.decode_groups(groups, probs[0].greedy_seed, probs[0].anneal_seed,
                        ws=torch.empty(size, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        for prob, o, ref in zip(probs, outs, refs):
            compare_decode(prob, o, ref)
    with pytest.raises(X.XzzxError) as e:
        D.decode_groups(groups, 1, 2, ws=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.rc == X.XZZX_ENOMEM


def test_stages_agree_on_the_references():
    """A greedy stage with one workspace size and the other stages with another
    find the references in the same place."""
    probs = [Problem(0, 11, 0.15, 10.0, 2, 8, 30, seed=6), Problem(0, 13, 0.15, 10.0, 3, 5, 30, seed=6)]
    plans = [gpu_plan(p) for p in probs]
    for p in plans:
        p.set_kernel(X.KERNEL_ROWS)
    groups, outs = made(probs, plans, want_extra=False)
    ws = torch.empty(D.workspace(groups).numel(), dtype=torch.uint8, device="cuda")
    seeds = probs[0].greedy_seed, probs[0].anneal_seed
    D.decode_groups(groups, *seeds, flags=X.STAGE_GREEDY, ws=ws)
    D.decode_groups(groups, *seeds, flags=X.STAGE_ANNEAL | X.STAGE_FINISH, ws=ws[:least_bytes(groups)])
    torch.cuda.synchronize()
    for prob, o in zip(probs, outs):
        compare_decode(prob, o, prob.oracle_decode())


@pytest.mark.parametrize("layout,d,R,n", [(1, 31, 16, 1 << 20), (0, 31, 5, 1 << 22), (1, 17, 16, 1 << 22)])
def test_workspace_stays_near_the_least(layout, d, R, n):
    """What a call asks for beyond the least is bounded."""
    plan = gpu_plan(Problem(layout, d, 0.15, 10.0, 0, 1, 2000, seed=d, conv=layout))
    plan.set_kernel(X.KERNEL_ROWS if layout == 0 else X.KERNEL_AUTO)
    g = X.Group()
    g.plan, g.n_syn, g.n_rep = plan.h, n, R
    full = C.c_size_t()
    X.check("xzzx_decode_workspace", X.lib().xzzx_decode_workspace((X.Group * 1)(g), 1, C.byref(full)))
    assert least_bytes([g]) <= full.value <= least_bytes([g]) + (18 << 30)


def test_workspace_falls_back_when_memory_is_short(monkeypatch):
    """Where the whole size cannot be allocated, the Python face takes the least."""
    prob = Problem(0, 11, 0.15, 10.0, 2, 8, 30, seed=7)
    groups, outs = made([prob], [gpu_plan(prob)])
    full, empty = D.workspace(groups).numel(), torch.empty

    def short(size, *a, **kw):
        if size == full:
            raise torch.OutOfMemoryError("no room")
        return empty(size, *a, **kw)

    monkeypatch.setattr(torch, "empty", short)
    ws = D.workspace(groups)
    monkeypatch.undo()
    assert ws.numel() == least_bytes(groups) < full
    D.decode_groups(groups, prob.greedy_seed, prob.anneal_seed, ws=ws)
    torch.cuda.synchronize()
    compare_decode(prob, outs[0], prob.oracle_decode())


def test_recoveries_past_four_gigabytes():
    """A call with more than 2^32 bytes of recoveries on a lattice without a
    packed-row kernel is accepted, and the ends of the batch are right."""
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of device memory")
    prob = Problem(1, 17, 0.15, 5.0, 2, 1, 1, seed=8, conv=1)
    plan = gpu_plan(prob)
    n = (1 << 32) // plan.nq + 1000
    syn = torch.zeros((n, plan.nstab), dtype=torch.uint8, device="cuda")
    uid = torch.zeros(n, dtype=torch.int32, device="cuda")
    ends = [0, n - 1]
    for k, i in enumerate(ends):
        syn[i] = to_dev(prob.syn[k])
        uid[i] = int(prob.uid[k])
    g, o = D.make_group(plan, 1, uid, syn=syn, want_extra=False)
    D.decode_groups([g], prob.greedy_seed, prob.anneal_seed, ws=D.workspace([g]))
    torch.cuda.synchronize()
    for (i, ref) in zip(ends, prob.oracle_decode()):
        assert o.e_best[i].item() == ref["e_best"] and o.cls[i].item() == ref["cls"]
        assert np.array_equal(o.recovery[i].cpu().numpy(), ref["recovery"])


def check_decodes(prob, plan, want, ref, sizes=("full",), flags=(0,), final=True):
    """Decodes of a problem whose only group must run on the kernel `want`."""
    for size in sizes:
        for flag in flags:
            g, o = D.make_group(plan, prob.n_rep, to_dev(prob.uid.view(np.int32)), syn=to_dev(prob.syn),
                                want_chains=True, want_final=final)
            ws = D.workspace([g])
            if size == "least":
                ws = ws[:least_bytes([g])]
            assert routes([g], ws.numel())[0] == want
            D.decode_groups([g], prob.greedy_seed, prob.anneal_seed, flags=flag, ws=ws)
            torch.cuda.synchronize()
            compare_decode(prob, o, ref)


@pytest.mark.parametrize("d", range(3, 32, 2))
def test_rows_of_one_syndrome(d):
    """The packed-row kernel specialised to d with tasks inside one syndrome, which
    the default leaves to calls larger than these: both forms."""
    prob = Problem(0, d, 0.2, 10.0, 3 if d <= 21 else 2, 32 if d <= 9 else 16, 24 if d <= 21 else 12, seed=900 + d)
    plan = gpu_plan(prob)
    plan.set_kernel(X.KERNEL_ROWS)
    check_decodes(prob, plan, (X.KERNEL_ROWS, 1), prob.oracle_decode(), flags=(0, X.FLAG_PLAIN))


@pytest.mark.parametrize("d,R,sweeps", [(7, 16, 64), (7, 16, 65), (7, 16, 300), (7, 5, 300), (7, 16, 2100), (15, 16, 300),
                                        (19, 16, 300), (31, 16, 300), (31, 5, 600)])
def test_rows_replayed_from_checkpoints(d, R, sweeps):
    """Recoveries of the packed-row kernels, replayed from dense and sparse
    checkpoints (one and two words a row) and, spanning with the least
    workspace, from the references."""
    prob = Problem(0, d, 0.2, 10.0, 4 if d < 15 else 2, R, sweeps, seed=950 + sweeps + d)
    plan = gpu_plan(prob)
    plan.set_kernel(X.KERNEL_ROWS)
    check_decodes(prob, plan, (X.KERNEL_ROWS, 1), prob.oracle_decode(), sizes=("full", "least"), final=False)


@pytest.mark.parametrize("layout,d", [(0, 5), (0, 11), (0, 17), (1, 7), (1, 17)])
def test_byte_states_on_every_lane_count(layout, d):
    """The byte-state kernels with 1 to 64 lanes: chosen lanes from four up run
    there only with the least workspace."""
    prob = Problem(layout, d, 0.15, 8.0, 3, 5, 20, seed=970 + d, conv=layout)
    ref = prob.oracle_decode()
    for lanes in (1, 2, 4, 8, 16, 32, 64):
        plan = gpu_plan(prob)
        try:
            plan.set_lanes(lanes)
        except X.XzzxError as e:   # 64 / lanes chains of a large lattice pass the LDS of a workgroup
            assert e.rc == X.XZZX_ERANGE and lanes < 4
            continue
        check_decodes(prob, plan, (X.KERNEL_BYTES, lanes), ref, sizes=("least",), flags=(0, X.FLAG_PLAIN))


@pytest.mark.parametrize("d", [17, 25, 31])
def test_large_planar_default_without_room(d):
    """Planar lattices beyond d = 15: the grid core, or byte states with the least workspace."""
    prob = Problem(1, d, 0.15, 8.0, 2, 3, 8, seed=980 + d, conv=1)
    plan, ref = gpu_plan(prob), prob.oracle_decode()
    check_decodes(prob, plan, (GRID, 64), ref)
    check_decodes(prob, plan, (X.KERNEL_BYTES, plan.info()["lanes_per_chain"]), ref, sizes=("least",))


@pytest.mark.parametrize("R", [4, 16])
def test_mixed_distances_on_packed_rows(R):
    """Uneven distances in one call on the packed-row kernels, tasks inside and
    across syndromes."""
    probs = [Problem(0, d, 0.18, 10.0, n, R, 30, seed=990 + d) for d, n in [(5, 7), (9, 5), (13, 3), (17, 2), (21, 2)]]
    plans = [gpu_plan(p) for p in probs]
    for p in plans:
        p.set_kernel(X.KERNEL_ROWS)
    for p in probs:
        p.greedy_seed, p.anneal_seed = probs[0].greedy_seed, probs[0].anneal_seed
    groups, outs = made(probs, plans, want_final=True)
    ws = D.workspace(groups)
    assert set(routes(groups, ws.numel())) == {(X.KERNEL_ROWS, 1)}
    D.decode_groups(groups, probs[0].greedy_seed, probs[0].anneal_seed, ws=ws)
    torch.cuda.synchronize()
    for prob, o in zip(probs, outs):
        compare_decode(prob, o, prob.oracle_decode())
