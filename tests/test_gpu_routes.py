"""The kernel a call runs on: what selects it, by the library's own account
(xzzx_decode_routes) or by its time, and the results of kernels that the
default leaves to other sizes, against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

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
