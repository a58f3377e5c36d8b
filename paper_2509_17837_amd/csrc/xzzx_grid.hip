// Annealing and serving kernels of the grid core (one chain over several lanes).
#include "xzzx_grid.h"

namespace xzzx {

template <int LOGG, int MV>
__global__ __launch_bounds__(kWave) void k_anneal_grid(AnnealArgs A)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const PlanDev *loaded = nullptr;
    for (uint32_t task = blockIdx.x; task < A.n_tasks; task = later_task(A)) {
        int gi = 0;
        while (gi + 1 < A.n_groups && (int64_t)task >= A.g[gi + 1].task_begin) ++gi;
        const GroupArgs &G = A.g[gi];
        const int64_t unit0 = ((int64_t)task - G.task_begin) << (6 - LOGG);
        if (G.plan != loaded) {
            wave_lds_fence();
            load_grid_tables(G.plan, smem);
            loaded = G.plan;
        }
        const ChainJob J = batch_job(G, unit0 + (threadIdx.x >> LOGG), false);
        grid_core<LOGG, MV>(G.plan, J, 0, G.plan->n_sweeps, A.seed_lo, A.seed_hi, smem, G.min_snap);
    }
}

template <int LOGG>
static AnnealKernel pick(int mv)
{
    switch (mv) {
    case 1: return k_anneal_grid<LOGG, 1>;
    case 2: return k_anneal_grid<LOGG, 2>;
    case 4: return k_anneal_grid<LOGG, 4>;
    case 8: return k_anneal_grid<LOGG, 8>;
    default: return nullptr;
    }
}

AnnealKernel grid_kernel(int lanes, int mv)
{
    switch (lanes) {
    case 4: return pick<2>(mv);
    case 8: return pick<3>(mv);
    case 16: return pick<4>(mv);
    case 32: return pick<5>(mv);
    case 64: return pick<6>(mv);
    default: return nullptr;
    }
}

// Serving slices: one workgroup per task, the tasks of every lane count with
// MV moves per lane in one launch (a launch per lane count as well would not
// fit the device's few queues, and the slice would wait for one after the
// other).  Bound by the latency of a sweep (see the grid core): 250 sweeps of
// d = 25 take 0.43 ms, where the byte-state kernel took 1.0; a burst of 48
// requests of d = 7..25 6.2 -> 3.6 ms, p50 at 10^3 and 10^4 requests/s 3.7 ->
// 1.4 and 8.6 -> 3.4 ms.
template <int MV>
__global__ __launch_bounds__(kWave) void k_serve_grid(const ServeTask *tasks, uint32_t slo, uint32_t shi)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const ServeTask &T = tasks[blockIdx.x];
    const PlanDev *pl = T.plan;
    load_grid_tables(pl, smem);
    const int lg = (int)uni((uint32_t)T.log_lanes);
    const ChainJob J = serve_job(T, threadIdx.x >> lg, false);
    switch (lg) {
    case 2: grid_core<2, MV>(pl, J, T.t_begin, T.t_end, slo, shi, smem, T.gs); break;
    case 3: grid_core<3, MV>(pl, J, T.t_begin, T.t_end, slo, shi, smem, T.gs); break;
    case 4: grid_core<4, MV>(pl, J, T.t_begin, T.t_end, slo, shi, smem, T.gs); break;
    case 5: grid_core<5, MV>(pl, J, T.t_begin, T.t_end, slo, shi, smem, T.gs); break;
    default: grid_core<6, MV>(pl, J, T.t_begin, T.t_end, slo, shi, smem, T.gs); break;
    }
}

ServeKernel serve_grid_kernel(int mv)
{
    switch (mv) {
    case 1: return k_serve_grid<1>;
    case 2: return k_serve_grid<2>;
    case 4: return k_serve_grid<4>;
    case 8: return k_serve_grid<8>;
    default: return nullptr;
    }
}

}  // namespace xzzx
