// Random-site annealing (Algs. 2-3 as printed): every step picks one generator
// uniformly at random, so the steps of a chain are sequential and the
// parallelism is across chains: one chain per lane.
//
// Bound by VALU issue (half of it Philox: a block serves two steps), LDS
// cycles and the latency of the LDS round trips a step needs one after
// another, about evenly.  So a step makes few of each:
// - the state is packed 2 bits per qubit, row by row of the lattice's grid (as
//   turned for the packed-row kernels), so that a generator's 2 x 2 block is
//   two runs of four bits: two reads and two writes a step.  Word w of lane l
//   sits at LDS word 64 w + l of its wavefront, so whatever generators the
//   lanes pick, an access falls in distinct banks;
// - a block's pattern, masked by the generator's own cells, addresses its
//   (threshold, dE) entry directly, as in the grid core (two dependent reads a
//   step: the rows, the entry);
// - the generators' descriptors follow from the draws alone and are read a
//   Philox block ahead of the state;
// - acceptance is branch-free: both rows are written back in every step;
// - the wavefronts of a workgroup share the descriptors and entries (the
//   thresholds change every sweep, so they meet at a barrier before and after
//   the change), which leaves room for eight wavefronts per SIMD.
// Measured (planar d = 9, 20 480 to 491 520 chains): 1.4x to 1.9x of one
// wavefront a workgroup with two 16-bit reads a row, branches on acceptance and
// descriptors read in the step itself; at 491 520 chains the launch went from
// 15.8 to 11.3 ms, vector issue three quarters busy, LDS one half.
//
// Step m of sweep t uses Philox(uid, chain, 2^31 + t, m div 2): words 2 (m mod
// 2) and 2 (m mod 2) + 1 are the site draw (site = floor(u N_stab / 2^32),
// face-id order) and the acceptance draw.  E_min is tracked after every step;
// stop = t N_stab + m + 1 (0 = the start), and the state at the first E_min is
// kept in `snap` for the recovery: word w of chain ci at snap[w * snap_stride +
// ci].  With a full workspace the words are the state's own; COMPACT (a short
// workspace) closes the packing's gaps, so that nq / 16 + 1 words hold them.
#include "xzzx_grid.h"

namespace xzzx {

// LDS: entries, descriptors, then the wavefronts' states (site_words of 64
// words each, see PlanDev)
__device__ __forceinline__ uint32_t site_desc_off(const PlanDev *pl) { return (8u * ((uint32_t)pl->grid_slots + 1u) + 15u) & ~15u; }
__device__ __forceinline__ uint32_t site_state_off(const PlanDev *pl)
{
    return site_desc_off(pl) + ((8u * (uint32_t)pl->nstab + 255u) & ~255u);
}

__device__ __forceinline__ uint2 lds_read_pair(uint32_t a)   // words a and a + 256 bytes
{
    typedef const __attribute__((address_space(3))) uint32_t *P;
    return make_uint2(*(P)(uintptr_t)a, *(P)(uintptr_t)(a + 256u));
}

template <bool WIDE, bool COMPACT>
__device__ __forceinline__ void site_core(const PlanDev *pl, const ChainJob &J, uint32_t seed_lo, uint32_t seed_hi,
                                          uint8_t *smem, uint32_t *snap, int64_t snap_stride)
{
    const int nq = (int)uni(pl->nq), nranks = (int)uni(pl->nranks), n_sweeps = (int)uni(pl->n_sweeps);
    const uint32_t nstab = uni(pl->nstab);
    const int words = (int)uni(pl->site_words);
    const uint32_t k0 = uni(seed_lo), k1 = uni(seed_hi);
    const uint32_t cc = J.cc;
    const int lane = threadIdx.x & (kWave - 1), wave = (int)uni(threadIdx.x / kWave);
    const uint32_t base = lds_addr(smem), desc0 = base + site_desc_off(pl);
    uint32_t *st = reinterpret_cast<uint32_t *>(smem + site_state_off(pl)) + wave * words * kWave + lane;
    const uint32_t st0 = base + site_state_off(pl) + 4u * (uint32_t)(wave * words * kWave + lane);
    const LaneKey lk = lane_key(J.uid, k1);

    int32_t E = 0;
    {
        int32_t W[4];
        W[0] = 0; W[1] = (int32_t)uni(pl->W[1]); W[2] = (int32_t)uni(pl->W[2]); W[3] = (int32_t)uni(pl->W[3]);
        const bool use_x = (J.lp == 1 || J.lp == 2), use_z = (J.lp == 2 || J.lp == 3);
        for (int w = 0; w < words; ++w) st[w * kWave] = 0u;
        for (int q = 0; q < nq; ++q) {
            const uint32_t p = uni(pl->site_pos[q]);
            uint32_t v = J.active ? (J.src[q] & 3u) : 0u;
            if (use_x) v ^= pl->lx[q];
            if (use_z) v ^= pl->lz[q];
            st[(p >> 5) * kWave] |= v << (p & 31u);
            E += weight_of(W, v);
        }
    }
    int32_t Emin = E, stop = 0;
    auto save_state = [&](uint8_t *dst) {
        for (int q = 0; q < nq; ++q) {
            const uint32_t p = uni(pl->site_pos[q]);
            dst[q] = (uint8_t)((st[(p >> 5) * kWave] >> (p & 31u)) & 3u);
        }
    };
    uint32_t *const keep = J.active ? snap + J.ci : nullptr;
    auto keep_min = [&]() {
        if constexpr (COMPACT) {
            uint64_t acc = 0;
            uint32_t fill = 0;   // bits of acc in use, uniform
            uint32_t *dst = keep;
            auto piece = [&](uint32_t r, uint32_t v) {
                const uint32_t n = r >> 16;
                v >>= (r >> 8) & 31u;
                acc |= (uint64_t)(n < 32u ? v & ((1u << n) - 1u) : v) << fill;
                fill += n;
                if (fill >= 32u) {
                    *dst = (uint32_t)acc;
                    dst += snap_stride;
                    acc >>= 32;
                    fill -= 32u;
                }
            };
            // eight pieces' words are read before any is placed, and the next
            // eight pieces fetched meanwhile
            const int n8 = (int)uni(pl->site_runs) / 8;
            uint4 nx = pl->site_run[0], ny = pl->site_run[1];
            for (int i = 0; i < n8; ++i) {
                const uint32_t r[8] = {uni(nx.x), uni(nx.y), uni(nx.z), uni(nx.w), uni(ny.x), uni(ny.y), uni(ny.z), uni(ny.w)};
                const int next = min(i + 1, n8 - 1);
                nx = pl->site_run[2 * next];
                ny = pl->site_run[2 * next + 1];
                uint32_t v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = st[(r[k] & 0xFFu) * kWave];
#pragma unroll
                for (int k = 0; k < 8; ++k) piece(r[k], v[k]);
            }
            if (fill) *dst = (uint32_t)acc;
        } else {
#pragma unroll 4
            for (int w = 0; w < words; ++w) keep[w * snap_stride] = st[w * kWave];
        }
    };
    if (keep) keep_min();

    auto site_desc = [&](uint32_t u) -> uint2 {
        return lds_read64(desc0 + (__umulhi(u, 8u * nstab) & ~7u));   // 8 floor(u N / 2^32)
    };
    auto step = [&](const uint2 &d, uint32_t u, int32_t s) {
        const uint32_t a = st0 + (d.x & 0xFFFFu), b = st0 + (d.x >> 16);
        uint2 ra, rb;
        if (WIDE) {
            ra = lds_read_pair(a);
            rb = lds_read_pair(b);
        } else {
            ra = make_uint2(st[(d.x & 0xFFFFu) >> 2], 0u);
            rb = make_uint2(st[d.x >> 18], 0u);
        }
        const uint32_t bo_b = d.y >> 6, cells = d.y >> 12;
        const uint32_t xa = (WIDE ? __builtin_amdgcn_alignbit(ra.y, ra.x, d.y) : ra.x >> (d.y & 31u)) & 0xFu;
        const uint32_t xb = WIDE ? __builtin_amdgcn_alignbit(rb.y, rb.x, bo_b) : rb.x >> (bo_b & 31u);
        const uint32_t pat = ((xb << 4) | xa) & cells;   // cells: 8 bits, the entry table above them
        const uint2 e = lds_read64(base + 8u * ((d.y >> 20) + (pat & 0xFFu)));
        const uint32_t sel = accept_mask(u, e);
        const uint32_t fa = __builtin_amdgcn_bitop3_b32(sel, 6u, cells, 0x80);        // X left | Z right of the upper row
        const uint32_t fb = __builtin_amdgcn_bitop3_b32(sel, 9u, cells >> 4, 0x80);   // Z left | X right of the lower one
        typedef __attribute__((address_space(3))) uint32_t *P;
        // in this order: the second word of a pair is the row's own only where a
        // row takes several words, else it is written back as it was read, and
        // may be the lower row's first
        *(P)(uintptr_t)a = ra.x ^ (fa << (d.y & 31u));
        if (WIDE) *(P)(uintptr_t)(a + 256u) = ra.y ^ ((fa >> 1) >> (~d.y & 31u));
        *(P)(uintptr_t)b = rb.x ^ (fb << (bo_b & 31u));
        if (WIDE) *(P)(uintptr_t)(b + 256u) = rb.y ^ ((fb >> 1) >> (~bo_b & 31u));
        E = add_energy(E, e.y & sel);
        if (E < Emin) {
            Emin = E;
            stop = s + 1;
            if (keep) keep_min();
        }
    };

    const int n_rising = (int)uni(pl->grid_rising);
    const uint32_t *thr = pl->thr;
    for (int t = 0; t < n_sweeps; ++t) {
        // this sweep's thresholds, in the entries all wavefronts read
        __syncthreads();
        for (int i = threadIdx.x; i < n_rising; i += blockDim.x) {
            const uint32_t g = pl->grid_entry[i];
            uint2 *et = reinterpret_cast<uint2 *>(smem) + (g & 0xFFFFu);
            const uint32_t v = thr[(size_t)t * nranks + (g >> 16)];
            *et = make_uint2(v, (et->y & 0x7FFFFFFFu) | (v & 0x80000000u));
        }
        __syncthreads();
        const LaneHead h = lane_head(lk, cc, 0x80000000u + (uint32_t)t, k0, k1);
        const int32_t s0 = t * (int32_t)nstab;
        uint4 r = lane_philox_block_at(lk, h, 0u, k0, k1);
        uint2 d0 = site_desc(r.x), d1 = site_desc(r.z);
        for (uint32_t m = 0; m < nstab; m += 2) {
            const uint32_t u0 = r.y, u1 = r.w;
            const uint2 c0 = d0, c1 = d1;
            r = lane_philox_block_at(lk, h, (m >> 1) + 1u, k0, k1);
            d0 = site_desc(r.x);
            d1 = site_desc(r.z);
            step(c0, u0, s0 + (int32_t)m);
            step(c1, u1, s0 + (int32_t)m + 1);   // N_stab is even
        }
    }
    if (J.active) {
        J.emin[J.ci] = Emin;
        J.stop[J.ci] = stop;
        J.efin[J.ci] = E;
        if (J.states) save_state(J.states + (size_t)J.ci * nq);
    }
}

template <bool WIDE, bool COMPACT>
__device__ __forceinline__ void site_body(const AnnealArgs &A)
{
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint32_t next;
    const PlanDev *loaded = nullptr;
    // every wavefront of the workgroup on one task of blockDim.x chains
    for (uint32_t task = blockIdx.x; task < A.n_tasks;) {
        int gi = 0;
        while (gi + 1 < A.n_groups && (int64_t)task >= A.g[gi + 1].task_begin) ++gi;
        const GroupArgs &G = A.g[gi];
        const int64_t unit0 = ((int64_t)task - G.task_begin) * blockDim.x;
        __syncthreads();
        if (G.plan != loaded) {
            const PlanDev *pl = G.plan;
            uint2 *et = reinterpret_cast<uint2 *>(smem);
            for (int i = threadIdx.x; i < pl->grid_entries; i += blockDim.x) {
                const uint32_t g = pl->grid_entry[i];
                et[g & 0xFFFFu] = move_entry(pl->dE[g >> 16], 0u);
            }
            uint2 *desc = reinterpret_cast<uint2 *>(smem + site_desc_off(pl));
            for (int i = threadIdx.x; i < pl->nstab; i += blockDim.x) desc[i] = pl->site_desc[i];
            loaded = pl;
        }
        const ChainJob J = batch_job(G, unit0 + threadIdx.x, false);
        site_core<WIDE, COMPACT>(G.plan, J, A.seed_lo, A.seed_hi, smem, G.min_snap, G.n_chains);
        if (!A.counter) break;
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t t = atomicAdd(A.counter, 1u);
            next = t < A.n_tasks - A.grid ? A.grid + t : 0xFFFFFFFFu;
        }
        __syncthreads();
        task = uni(next);
    }
}

template <bool WIDE, bool COMPACT>
__global__ __launch_bounds__(8 * kWave) void k_anneal_site(AnnealArgs A) { site_body<WIDE, COMPACT>(A); }

AnnealKernel site_kernel(bool wide, bool compact)
{
    if (compact) return wide ? k_anneal_site<true, true> : k_anneal_site<false, true>;
    return wide ? k_anneal_site<true, false> : k_anneal_site<false, false>;
}

}  // namespace xzzx
