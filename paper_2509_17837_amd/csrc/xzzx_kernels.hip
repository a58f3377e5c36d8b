// gfx950 kernels of the XZZX simulated-annealing decoder (those not
// specialised to a distance) and the device-side entry points of the C ABI.
//
//   k_syndrome     Eq. (2): syndrome of a batch of configurations.
//   k_greedy       Algs. 5-6: greedy matching per (syndrome, replica), both
//                  decoding-graph colours, paths XOR-ed into an LDS configuration.
//   k_qcls         Alg. 7: class Q_r of each reference relative to replica 0.
//   k_anneal<L>    Algs. 2-3 on byte-per-qubit states, 2^L lanes per chain
//                  (any lattice); k_anneal_rows: the generic packed-row kernel
//                  (rotated lattices, d <= 29).  Both are persistent: wavefronts
//                  pull tasks from an atomic queue spanning every syndrome group
//                  of the launch.  The packed-row kernels specialised to one
//                  distance (every odd d <= 31) are in xzzx_device.h /
//                  xzzx_static_*.hip.
//   k_replay<L>    re-runs each syndrome's best chain up to the phase of its
//                  minimum (from a checkpoint where the specialised kernel left
//                  one) and stores that state: the recovery.
//   k_finish       Eqs. (18)-(21): per-coset minima, P*, best chain; the
//                  recovery, where the kernels kept each chain's best state.
//   k_serve_*      the serving loop's slices, finish and result gather.
//
// The host half turns xzzx_group descriptions into launches: one persistent
// launch per kernel family and distance, run concurrently on side streams.
#include <hip/hip_runtime.h>

#include <utility>

#include <algorithm>
#include <functional>
#include <mutex>
#include <cstring>
#include <vector>

#include "xzzx_device.h"

namespace xzzx {

// ---------------------------------------------------------------------------
// Syndrome, Eq. (2): s_f = 1 iff the configuration anticommutes with G_f.
// Slots 0 and 3 carry X (detect a Z component), slots 1 and 2 carry Z (detect
// an X component).
//
// Bound by memory: n_q + n_stab bytes per configuration and five operations
// per generator.  A workgroup takes a tile of 4 << lg4 configurations, moves
// it through registers as dwords (four bytes of four configurations, 4 x 4
// byte transpose) and keeps it in LDS qubit by qubit, so a dword read gives
// one qubit of four configurations and every parity is taken for four at
// once.  The outputs go back through the same transpose as dwords.  One
// thread per output byte, each reading its four qubits and dividing a 64-bit
// index, took 525 us for 10^6 configurations of the planar d = 9 lattice
// (0.55 TB/s); this form takes 98 us (2.96 TB/s; a large copy runs at
// 4.8 TB/s on the same card).
// Lanes: four dword columns (configurations) by sixteen consecutive dwords
// of a row, so a wavefront's LDS accesses fall in distinct banks (the row
// pitch is odd) and its global ones in 64-byte runs.
// ---------------------------------------------------------------------------
// A workgroup has 256 threads, or 1024 where a few workgroups have large
// lattices to take and their latency counts (planar d = 31, 1 to 1000
// configurations: 10.3 us with 256 threads, 6.8 so).
constexpr int kSynThreads = 256, kSynThreadsMost = 1024;

// bytes (v0.j, v1.j, v2.j, v3.j) of four dwords into dword j
__device__ __forceinline__ void transpose4x4(uint32_t (&v)[4])
{
    const uint32_t a = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), b = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u), d = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
    v[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    v[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    v[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    v[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// LDS rows of a tile: the qubits and the all-zero row of absent slots,
// padded to whole dwords of a configuration
static int syndrome_rows(int nq) { return (nq + 4) / 4 * 4; }

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_syndrome(const PlanDev *__restrict__ pl,
                                                          const uint8_t *__restrict__ cfg, int64_t n, int lg4,
                                                          uint8_t *__restrict__ syn)
{
    extern __shared__ uint32_t tile[];   // [rows][pitch]: qubit, four configurations per dword
    const int nstab = pl->nstab, nq = pl->nq;
    const int n4 = 1 << lg4, pitch = n4 + 1;
    const int64_t s0 = (int64_t)blockIdx.x << (lg4 + 2);
    const int nc = (nq + 4) / 4;
    for (int idx = threadIdx.x; idx < nc << lg4; idx += THREADS) {
        const int hi = (idx >> 2) / nc, c = (idx >> 2) - hi * nc, s4 = 4 * hi + (idx & 3);
        uint32_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t s = s0 + 4 * s4 + i;
            v[i] = 0;
            if (s >= n) continue;
            const uint8_t *p = cfg + s * nq + 4 * c;
            if (4 * c + 4 <= nq) {
                __builtin_memcpy(&v[i], p, 4);
            } else {
                for (int b = 0; 4 * c + b < nq; ++b) v[i] |= (uint32_t)p[b] << (8 * b);
            }
        }
        transpose4x4(v);
#pragma unroll
        for (int j = 0; j < 4; ++j) tile[(4 * c + j) * pitch + s4] = v[j];
    }
    __syncthreads();
    const int nf = nstab / 4;
    for (int idx = threadIdx.x; idx < nf << lg4; idx += THREADS) {
        const int hi = (idx >> 2) / nf, f4 = (idx >> 2) - hi * nf, s4 = 4 * hi + (idx & 3);
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const Desc d = pl->face_desc[4 * f4 + j];
            const uint32_t x = tile[(d.x & 0xFFFFu) * pitch + s4] ^ tile[((d.y >> 16) & 0x7FFu) * pitch + s4];
            const uint32_t z = tile[(d.x >> 16) * pitch + s4] ^ tile[(d.y & 0xFFFFu) * pitch + s4];
            v[j] = (x ^ (z >> 1)) & 0x01010101u;
        }
        transpose4x4(v);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t s = s0 + 4 * s4 + i;
            if (s < n) __builtin_memcpy(syn + s * nstab + 4 * f4, &v[i], 4);
        }
    }
}

// ---------------------------------------------------------------------------
// Greedy matching (Algs. 5-6) -- one workgroup per syndrome (or per share of
// its replicas), one wavefront per replica.
//
// The sequential rule -- take the free pair of least (weight, key, pair id) --
// is evaluated as repeated mutual-best elimination: every free defect finds
// its least free partner, and pairs that are each other's least are matched.
// Under a strict total order the pair taken first by the sequential scan is
// always mutual-best, and removing matched defects never changes the order of
// the rest, so both procedures produce the same matching.  Paths follow the
// canonical tight-edge walk (smallest edge id) and are XOR-ed into the
// configuration with LDS atomics (paths may overlap).
//
// Only the keys differ between replicas.  So the workgroup first finds, all
// wavefronts together, the defects, the pair weights (kept in LDS where they
// fit) and each defect's partners at its least weight; a replica's first round
// draws the keys of those ties alone, spread evenly over the lanes.  Then each
// wavefront goes on by itself (later rounds, paths, output) without barriers.
// The first round's scan was 40-70 % of the time when every replica did it,
// gathering distances through L1 at a line per lane.
// Bound now by latency and instruction issue of the later rounds and the walks.
// References alone, a wavefront to each with a scan of its own -> now (three
// defects in ten generators): d = 21, 1021 syndromes x 10: 466 -> 219 us; d = 11, 8192
// x 32: 1172 -> 671 us; planar d = 9, 12288 x 10: 691 -> 393 us; d = 11, 20000 x 1: 128 ->
// 112 us; d = 31, 512 x 32: 2.85 -> 0.81 ms.
// ---------------------------------------------------------------------------
// partners whose distances a scan loads at once (the table is in HBM or L2:
// the loads of a batch overlap)
constexpr int kGreedyBatch = 4;
// lanes per defect in the shared scan, wavefronts (replicas) per workgroup
constexpr int kGreedyRow = 8;
constexpr int kGreedyWaves = 16;
constexpr int kGreedyCuLds = 163840;   // LDS of a CU

// LDS of a greedy workgroup, byte offsets.  Shared, per colour set: the tied
// pairs of the first round, boundary distances, the weight cache, the defects
// and their first partners; then per wavefront: 8 bytes a defect (see
// GreedyNode), the configuration and the free flags.
struct GreedyLds {
    uint32_t ents, db, weights, defects, first, waves;   // shared arrays, then the wavefronts' parts
    uint32_t cfg, flags, per_wave;                       // within a wavefront's part
};
__host__ __device__ inline GreedyLds greedy_lds_layout(int sets, int stride, int nwords, int cache_entries, int ties)
{
    GreedyLds L;
    const uint32_t n = (uint32_t)(sets * stride);
    L.ents = 0;
    L.db = L.ents + 4 * (uint32_t)(sets * ties);
    L.weights = L.db + 4 * n;
    L.defects = L.weights + 4 * (uint32_t)(sets * cache_entries);
    L.first = L.defects + 2 * n;
    L.waves = (L.first + 2 * n + 7u) & ~7u;
    L.cfg = 8 * n;
    L.flags = L.cfg + 4 * (uint32_t)nwords;
    L.per_wave = (L.flags + n + 7u) & ~7u;
    return L;
}

struct GreedyArgs {
    const PlanDev *plan;
    const uint8_t *syn;
    const uint32_t *uid;
    uint8_t *refs;
    uint8_t *qraw;
    int64_t syn_stride;        // bytes between syndromes
    const int32_t *slot_map;   // optional: syndrome s writes to slot slot_map[s]
    int64_t refs_stride;       // bytes between slots (with slot_map)
    int64_t qraw_stride;
    int n_rep;
    int mode;
    uint32_t seed_lo, seed_hi;
    int stride;                // defects a colour can have, and the virtual node, rounded up
    int rep_div;               // ladders: replicas of equal r / rep_div share a reference (1: each its own)
    int cache_entries;         // LDS words per colour for the pair weights (0: none)
    int n_units;               // references per syndrome: n_rep / rep_div, rounded up
    int shares;                // workgroups per syndrome
    int unit_step;             // wavefronts per syndrome: a wavefront's references are so many apart
    int ties;                  // entries of a colour's list of first ties
    int64_t syn0;              // syndrome and share of this launch's first workgroup
    int share0;
};

__device__ __forceinline__ void xor_edge(uint32_t *cfgw, int eid)
{
    const int q = eid >> 1;
    const uint32_t code = (eid & 1) ? 2u : 1u;
    atomicXor(&cfgw[q >> 2], code << (8 * (q & 3)));
}

// The canonical walk from x along tight edges of `dist` (smallest edge id
// first) to the target node, or, with none (-1), out through the boundary.
// Each step reads the node's four adjacency entries (in edge-id order) and
// their far ends' distances at once, then takes the first tight edge; the
// distance of the next node is known, so a step costs two dependent rounds of
// loads rather than one per entry tried.
__device__ __forceinline__ void walk(const PlanDev *pl, int g, const int32_t *dist, int x, int target, uint32_t *cfgw)
{
    const int n = pl->ncol[g];
    const int4 *adj = pl->adj[g];
    int32_t dx = dist[x];
    for (int step = 0; step <= n && x != target; ++step) {
        int4 e[4];
        int32_t de[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) e[s] = adj[4 * x + s];
#pragma unroll
        for (int s = 0; s < 4; ++s) de[s] = e[s].y >= 0 ? dist[e[s].y] : 0;   // an edge to the boundary: distance 0
        int edge = -1, next = -1;
        int32_t dn = 0;
#pragma unroll
        for (int s = 3; s >= 0; --s)
            if (e[s].x >= 0 && (target < 0 || e[s].y >= 0) && de[s] + e[s].z == dx) {
                edge = e[s].x;
                next = e[s].y;
                dn = de[s];
            }
        if (edge < 0) return;
        xor_edge(cfgw, edge);
        if (next < 0) return;
        x = next;
        dx = dn;
    }
}

// v of lane ^ 1 (0xB1), of lane ^ 2 (0x4E), or of the lane 4 or 8 further
// round its 16 (0x124, 0x128)
template <int CTRL>
__device__ __forceinline__ uint32_t lane_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// A wavefront's 8 bytes per defect.  In the first round the least (key << 32 |
// partner), for a 64-bit LDS minimum; after it `best` stays the partner and the
// rest holds three lists: the defects to search for, the free ones, and the
// matched pairs (pair p in entries 2p and 2p + 1).
struct GreedyNode {
    uint16_t best, need, free_list, pair;
};

// what the shared scan found for a defect: its first partner at the least
// weight, and whether others tie with it (listed, or, past the list's end, not)
constexpr uint32_t kGreedyListed = 0x4000u, kGreedyScan = 0x8000u, kGreedyPartner = 0x3FFFu;

// SPLIT: the two decoding-graph colours are independent matchings, so each
// half of a wavefront (32 lanes) runs one, and both XOR their paths into the
// shared configuration -- twice the lanes at work where a colour has no more
// than a few dozen defects.  Otherwise the whole wavefront runs the colours one
// after the other.
// SEVERAL (with SPLIT): a wavefront takes several references of its syndrome
// in turn.
// The kernel waits on memory and LDS most of the time, so the split form is
// held to eight wavefronts per SIMD (64 VGPRs); with several references the
// loop's state spills at that, and seven were 6-12 % faster.
template <bool SPLIT, bool SEVERAL>
__global__ __launch_bounds__(kGreedyWaves *kWave)
    __attribute__((amdgpu_waves_per_eu(SEVERAL ? 7 : SPLIT ? 8 : 4, 8))) void k_greedy(GreedyArgs A)
{
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ int s_nd[2], s_ents[2], s_scan[2];
    constexpr int kSets = SPLIT ? 2 : 1;
    constexpr int kHalf = SPLIT ? kWave / 2 : kWave;   // lanes per colour
    const PlanDev *pl = A.plan;
    const int lane = threadIdx.x % kWave, wave = (int)uni(threadIdx.x / kWave), n_waves = blockDim.x / kWave;
    const int hl = lane % kHalf;
    const int nq = pl->nq, nwords = (nq + 3) / 4, stride = A.stride;
    const int64_t s = A.syn0 + blockIdx.x;
    const int unit0 = (A.share0 + (int)blockIdx.y) * n_waves + wave;
    const uint32_t uid = A.uid[s];
    const GreedyLds L = greedy_lds_layout(kSets, stride, nwords, A.cache_entries, A.ties);
    uint8_t *mine = smem + L.waves + (uint32_t)wave * L.per_wave;
    uint32_t *cfgw = reinterpret_cast<uint32_t *>(mine + L.cfg);
    const bool randomized = A.mode == XZZX_GREEDY_RANDOM;
    const uint8_t *sy = A.syn + s * A.syn_stride;
    const int ent_cap = A.ties;

    // the reference in cfgw and its symplectic products with L_Z and L_X, for
    // each replica that shares it
    auto write_out = [&](int unit) {
        const uint8_t *cb = reinterpret_cast<const uint8_t *>(cfgw);
        const int r0 = unit * A.rep_div, r1 = min(A.n_rep, r0 + A.rep_div);
        uint8_t *out = A.slot_map ? A.refs + A.slot_map[s] * A.refs_stride : A.refs + (size_t)s * A.n_rep * nq;
        uint8_t *qraw_out = A.slot_map ? A.qraw + A.slot_map[s] * A.qraw_stride : A.qraw + s * A.n_rep;
        uint32_t vz = 0, vx = 0;
        wave_lds_fence();
        for (int q = lane; q < nq; q += kWave) {
            const uint32_t c = cb[q];
            for (int r = r0; r < r1; ++r) out[(size_t)r * nq + q] = (uint8_t)c;
            const uint32_t z = pl->lz[q], x = pl->lx[q];
            vz ^= (((c >> 1) & z) ^ (c & (z >> 1))) & 1;
            vx ^= (((c >> 1) & x) ^ (c & (x >> 1))) & 1;
        }
        const int az = __popcll(__ballot(vz)) & 1;
        const int ax = __popcll(__ballot(vx)) & 1;
        for (int r = r0 + lane; r < r1; r += kWave) qraw_out[r] = (uint8_t)(az | (ax << 1));
        wave_lds_fence();
    };
    for (int gg = 0; gg < (SPLIT ? 1 : 2); ++gg) {
        // a pair (i, j) weighs the interior distance or the two boundary
        // distances, whichever is less; a pair with the virtual node (an
        // odd count) weighs the real defect's boundary distance
        auto pair_weight = [&](const int32_t *dbD, int nd, int i, int j, int32_t dij) -> uint32_t {
            return i == nd ? (uint32_t)dbD[j] : j == nd ? (uint32_t)dbD[i] : (uint32_t)min(dij, dbD[i] + dbD[j]);
        };
        auto ents_of = [&](int set) { return reinterpret_cast<uint32_t *>(smem + L.ents) + set * ent_cap; };
        auto db_of = [&](int set) { return reinterpret_cast<int32_t *>(smem + L.db) + set * stride; };
        auto weights_of = [&](int set) { return reinterpret_cast<uint32_t *>(smem + L.weights) + set * A.cache_entries; };
        auto defects_of = [&](int set) { return reinterpret_cast<uint16_t *>(smem + L.defects) + set * stride; };
        auto first_of = [&](int set) { return reinterpret_cast<uint16_t *>(smem + L.first) + set * stride; };
        // rows of an odd stride: the lanes' reads of one column fall in distinct banks
        auto cached_of = [&](int na) { return (int64_t)na * (na | 1) <= (int64_t)A.cache_entries; };

        // ---- shared: the defects of each colour, ascending node index (a lone
        // wavefront takes the two colours on its halves) ----
        if (gg) __syncthreads();   // the wavefronts have left the other colour
        const bool halves = SPLIT && n_waves == 1;
        const int width = halves ? kHalf : kWave, wl = lane & (width - 1);
        if (const int set = halves ? lane / kHalf : wave; set < kSets) {
            const int g = SPLIT ? set : gg;
            const int n = pl->ncol[g], n_both = halves ? max(pl->ncol[0], pl->ncol[1]) : n;
            const int32_t *cf = pl->col_face[g], *db = pl->db[g];
            int nd = 0;
            for (int base = 0; base < n_both; base += width * kGreedyBatch) {
                bool flag[kGreedyBatch];
                int32_t face[kGreedyBatch], dbv[kGreedyBatch];
#pragma unroll
                for (int k = 0; k < kGreedyBatch; ++k) {
                    const int v = min(base + k * width + wl, n - 1);
                    face[k] = cf[v];
                    dbv[k] = db[v];
                }
#pragma unroll
                for (int k = 0; k < kGreedyBatch; ++k) flag[k] = base + k * width + wl < n && sy[face[k]];
#pragma unroll
                for (int k = 0; k < kGreedyBatch; ++k) {
                    uint64_t mask = __ballot(flag[k]);
                    if (halves) mask = (mask >> (set * kHalf)) & 0xFFFFFFFFull;
                    const int pos = nd + __popcll(mask & ((1ull << wl) - 1ull));
                    if (flag[k]) {
                        defects_of(set)[pos] = (uint16_t)(base + k * width + wl);
                        db_of(set)[pos] = dbv[k];
                    }
                    nd += __popcll(mask);
                }
            }
            if (wl == 0) { s_nd[set] = nd; s_ents[set] = 0; s_scan[set] = 0; }
        }
        __syncthreads();

        // ---- shared: weights, and each defect's partners at the least one ----
        if (A.mode != XZZX_GREEDY_BOUNDARY) {
            const int na0 = s_nd[0] + (s_nd[0] & 1), rows = na0 + (SPLIT ? s_nd[kSets - 1] + (s_nd[kSets - 1] & 1) : 0);
            const int sub = lane % kGreedyRow;
            for (int row = threadIdx.x / kGreedyRow; row < rows; row += blockDim.x / kGreedyRow) {
                const int set = row >= na0 ? 1 : 0;
                const int g = SPLIT ? set : gg, i = row - set * na0;
                const int nd = s_nd[set], na = nd + (nd & 1), rs = na | 1;   // odd count: the boundary joins as node nd
                const int32_t *dbD = db_of(set);
                const uint16_t *D = defects_of(set);
                const int32_t *drow = pl->dint[g] + (size_t)(i == nd ? 0 : D[i]) * pl->ncol[g];
                const bool cached = cached_of(na);
                uint32_t *wrow = weights_of(set) + i * rs;
                uint32_t bw = 0xFFFFFFFFu, bj = kGreedyPartner;
                int nt = 0;   // this lane's partners at weight bw
                for (int j0 = sub; j0 < na; j0 += kGreedyRow * kGreedyBatch) {
                    int32_t dv[kGreedyBatch];
#pragma unroll
                    for (int k = 0; k < kGreedyBatch; ++k) {
                        const int j = j0 + kGreedyRow * k;
                        dv[k] = drow[j < nd ? D[j] : 0];
                    }
#pragma unroll
                    for (int k = 0; k < kGreedyBatch; ++k) {
                        const int j = j0 + kGreedyRow * k;
                        if (j >= na || j == i) continue;
                        const uint32_t w = pair_weight(dbD, nd, i, j, dv[k]);
                        if (cached) wrow[j] = w;
                        if (w > bw) continue;
                        if (w < bw) { bw = w; nt = 0; }
                        if (nt == 0) bj = (uint32_t)j;
                        ++nt;
                    }
                }
                uint32_t least = bw;
#pragma unroll
                for (int m = 1; m < kGreedyRow; m *= 2) least = min(least, (uint32_t)__shfl_xor((int)least, m));
                if (bw != least) { nt = 0; bj = kGreedyPartner; }
                int before = nt;   // ties of the row's lanes up to this one
#pragma unroll
                for (int m = 1; m < kGreedyRow; m *= 2) {
                    bj = min(bj, (uint32_t)__shfl_xor((int)bj, m));
                    const int o = __shfl_up(before, m, kGreedyRow);
                    before += sub >= m ? o : 0;
                }
                const int all = __shfl(before, kGreedyRow - 1, kGreedyRow);
                before -= nt;
                uint32_t mark = 0;
                if (randomized && all > 1) {
                    int at = 0;
                    if (sub == 0) at = atomicAdd(&s_ents[set], all);
                    at = __shfl(at, 0, kGreedyRow);
                    mark = at + all <= ent_cap ? kGreedyListed : kGreedyScan;
                    uint32_t *ents = ents_of(set);
                    if (mark == kGreedyScan) {
                        // no room: the places left stay empty
                        for (int e = at + sub; e < ent_cap; e += kGreedyRow) ents[e] = 0xFFFFFFFFu;
                        if (sub == 0) s_scan[set] = 1;
                    } else if (nt > 0) {
                        at += before;
                        for (int j = sub; j < na; j += kGreedyRow) {
                            if (j == i) continue;
                            const uint32_t w = cached ? wrow[j] : pair_weight(dbD, nd, i, j, drow[j < nd ? D[j] : 0]);
                            if (w == least) ents[at++] = ((uint32_t)i << 16) | (uint32_t)j;
                        }
                    }
                }
                if (sub == 0) first_of(set)[i] = (uint16_t)(bj | mark);
            }
            __syncthreads();
        }
        // ---- this wavefront's replicas (one, where the colours go in turn) ----
        const int set = SPLIT ? lane / kHalf : 0, g = SPLIT ? set : gg;
        const int nd = s_nd[set], na = nd + (nd & 1), rs = na | 1;
        const int n = pl->ncol[g];
        const int32_t *dint = pl->dint[g], *db = pl->db[g];
        const uint16_t *D = defects_of(set);
        const int32_t *dbD = db_of(set);
        const uint32_t *wc = weights_of(set);
        const bool cached = cached_of(na);
        GreedyNode *node = reinterpret_cast<GreedyNode *>(mine) + set * stride;
        uint8_t *freef = mine + L.flags + set * stride;
        // of a colour's defects, the ones flagged (per half wavefront)
        auto half_mask = [&](bool flag) -> uint64_t {
            const uint64_t m = __ballot(flag);
            return SPLIT ? (m >> (set * kHalf)) & 0xFFFFFFFFull : m;
        };
        const uint64_t below = (1ull << hl) - 1ull;
        const int na_all = SPLIT ? max(__shfl(na, 0, kWave), __shfl(na, kHalf, kWave)) : na;
        for (int unit = unit0; unit < A.n_units; unit = SEVERAL ? unit + A.unit_step : A.n_units) {
            if (SPLIT || gg == 0)
                for (int i = lane; i < nwords; i += kWave) cfgw[i] = 0;
            wave_lds_fence();
            if (A.mode == XZZX_GREEDY_BOUNDARY) {
                for (int i = hl; i < nd; i += kHalf) walk(pl, g, db, D[i], -1, cfgw);
                if (SPLIT || gg == 1) write_out(unit);
                continue;
            }
            auto pair_key = [&](int i, int j) {
                const uint32_t id = (uint32_t)(min(i, j) * na + max(i, j));
                return philox4x32_10(make_uint4(uid, (uint32_t)unit, 0x100u + (uint32_t)g, id), A.seed_lo, A.seed_hi).x;
            };
            // the least of each defect's first ties
            for (int i = hl; i < na; i += kHalf) {
                const uint32_t f = first_of(set)[i];
                reinterpret_cast<uint64_t *>(node)[i] = (f & (kGreedyListed | kGreedyScan)) ? ~0ull : (uint64_t)f;
                freef[i] = 1;
            }
            wave_lds_fence();
            for (int e = hl; e < min(s_ents[set], ent_cap); e += kHalf) {
                const uint32_t ij = ents_of(set)[e];
                if (ij == 0xFFFFFFFFu) continue;
                const uint32_t i = ij >> 16, j = ij & 0xFFFFu;
                atomicMin(reinterpret_cast<unsigned long long *>(node) + i, ((uint64_t)pair_key((int)i, (int)j) << 32) | j);
            }
            wave_lds_fence();
            // every round matches at least the least free pair, so na / 2 rounds
            // suffice (rounds continue while either half has work).  Free defects
            // only leave, so a defect whose least partner is still free keeps it;
            // only the others search again.
            int np = 0;
            for (int round = 0; round < na_all / 2; ++round) {
                if (round > 0 || __ballot(s_scan[set]) != 0) {
                    // the free defects, and of those the ones to search for, ascending
                    int nfl = 0, nn = 0;
                    for (int base = 0; base < na_all; base += kHalf) {
                        const int v = base + hl;
                        const bool free_v = v < na && freef[v];
                        const bool need = free_v && (round > 0 ? !freef[node[v].best] : (first_of(set)[v] & kGreedyScan) != 0);
                        const uint64_t mf = half_mask(free_v), mn = half_mask(need);
                        if (free_v) node[nfl + __popcll(mf & below)].free_list = (uint16_t)v;
                        if (need) node[nn + __popcll(mn & below)].need = (uint16_t)v;
                        nfl += __popcll(mf);
                        nn += __popcll(mn);
                    }
                    wave_lds_fence();
                    // each one's least (weight, key, id) over the free partners, four
                    // lanes a defect: the least weight, then keys for the partners at
                    // it only.  Ids ascend with the partner, so equal keys go to the
                    // least.
                    for (int t = hl / 4; t < nn; t += kHalf / 4) {
                        const int i = node[t].need, sub = lane % 4;
                        const int32_t *drow = dint + (size_t)(i == nd ? 0 : D[i]) * n;
                        const uint32_t *wrow = wc + i * rs;
                        uint32_t bw = 0xFFFFFFFFu, bj = 0xFFFFu;
                        uint64_t ties = 0;   // this lane's last four partners at weight bw
                        int nt = 0;
                        for (int t0 = sub; t0 < nfl; t0 += 4 * kGreedyBatch) {
                            int32_t dv[kGreedyBatch];
                            int jj[kGreedyBatch];
    #pragma unroll
                            for (int k = 0; k < kGreedyBatch; ++k) jj[k] = t0 + 4 * k < nfl ? (int)node[t0 + 4 * k].free_list : i;
    #pragma unroll
                            for (int k = 0; k < kGreedyBatch; ++k)
                                dv[k] = cached ? (int32_t)wrow[jj[k]] : drow[jj[k] < nd ? D[jj[k]] : 0];
    #pragma unroll
                            for (int k = 0; k < kGreedyBatch; ++k) {
                                const int j = jj[k];
                                if (j == i) continue;
                                const uint32_t w = cached ? (uint32_t)dv[k] : pair_weight(dbD, nd, i, j, dv[k]);
                                if (w > bw) continue;
                                if (w < bw) { bw = w; nt = 0; }
                                if (nt == 0) bj = (uint32_t)j;
                                ties = (ties << 16) | (uint64_t)j;
                                ++nt;
                            }
                        }
                        uint32_t least = min(bw, lane_move<0xB1>(bw));
                        least = min(least, lane_move<0x4E>(least));
                        if (bw != least) { nt = 0; bj = 0xFFFFu; }
                        int all = nt + (int)lane_move<0xB1>((uint32_t)nt);
                        all += (int)lane_move<0x4E>((uint32_t)all);
                        uint32_t bk = 0;
                        if (randomized && all > 1) {
                            bk = 0xFFFFFFFFu;
                            auto try_partner = [&](uint32_t j) {
                                const uint32_t key = pair_key(i, (int)j);
                                if (key < bk || (key == bk && j < bj)) { bk = key; bj = j; }
                            };
                            bj = 0xFFFFu;
                            if (nt <= 4) {
                                for (int m = 0; m < nt; ++m, ties >>= 16) try_partner((uint32_t)ties & 0xFFFFu);
                            } else {
                                for (int m = sub; m < nfl; m += 4) {
                                    const int j = (int)node[m].free_list;
                                    if (j == i) continue;
                                    const int32_t dj = cached ? 0 : drow[j < nd ? D[j] : 0];
                                    if ((cached ? wrow[j] : pair_weight(dbD, nd, i, j, dj)) == least) try_partner((uint32_t)j);
                                }
                            }
                        }
                        // the quad's least (key, partner)
                        uint32_t ok = lane_move<0xB1>(bk), oj = lane_move<0xB1>(bj);
                        if (ok < bk || (ok == bk && oj < bj)) { bk = ok; bj = oj; }
                        ok = lane_move<0x4E>(bk);
                        oj = lane_move<0x4E>(bj);
                        if (ok < bk || (ok == bk && oj < bj)) { bk = ok; bj = oj; }
                        if (sub == 0) node[i].best = (uint16_t)bj;
                    }
                    wave_lds_fence();
                }
                // pairs that are each other's least
                const int before = np;
                for (int base = 0; base < na_all; base += kHalf) {
                    const int i = base + hl;
                    const int j = i < na && freef[i] ? (int)node[i].best : 0;
                    const bool flag = j > i && (int)node[j].best == i;
                    const uint64_t mask = half_mask(flag);
                    if (flag) {
                        const int p = np + __popcll(mask & below);
                        node[2 * p].pair = (uint16_t)i;
                        node[2 * p + 1].pair = (uint16_t)j;
                    }
                    np += __popcll(mask);
                }
                wave_lds_fence();
                for (int p = before + hl; p < np; p += kHalf) {
                    freef[node[2 * p].pair] = 0;
                    freef[node[2 * p + 1].pair] = 0;
                }
                wave_lds_fence();
                if (__ballot(2 * np < na) == 0) break;
            }
            // the paths, two lanes a pair: the interior one, or one to the boundary
            // from each (real) end
            for (int t = hl; t < 2 * np; t += kHalf) {
                const int i = node[t & ~1].pair, j = node[t | 1].pair;
                const int u = D[i], v = j == nd ? u : D[j];
                const bool inner = j != nd && dint[(size_t)u * n + v] <= db[u] + db[v];
                if ((t & 1) && (inner || j == nd)) continue;
                walk(pl, g, inner ? dint + (size_t)u * n : db, inner || (t & 1) ? v : u, inner ? u : -1, cfgw);
            }
            if (SPLIT || gg == 1) write_out(unit);
        }
    }
}

// Pauli class index (I=0, X=1, Y=2, Z=3) <-> (x, z) bits, and products.
__device__ __forceinline__ int cls_from_bits(int x, int z) { return x ? (z ? 2 : 1) : (z ? 3 : 0); }
__device__ __forceinline__ int cls_x(int c) { return (c == 1) | (c == 2); }
__device__ __forceinline__ int cls_z(int c) { return (c == 2) | (c == 3); }
__device__ __forceinline__ int cls_mul(int a, int b) { return cls_from_bits(cls_x(a) ^ cls_x(b), cls_z(a) ^ cls_z(b)); }

// Class of R_r relative to R_0 from the symplectic products with L_Z (bit 0:
// an X-type logical anticommutes with L_Z) and L_X (bit 1).  One thread per
// syndrome reads replica 0 first, so qcls may alias qraw.
__global__ void k_qcls(const uint8_t *qraw, int64_t n_syn, int n_rep, uint8_t *qcls)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_syn) return;
    const int r0 = qraw[s * n_rep] & 3;
    for (int r = 0; r < n_rep; ++r) {
        const int v = (qraw[s * n_rep + r] & 3) ^ r0;
        qcls[s * n_rep + r] = (uint8_t)cls_from_bits(v & 1, v >> 1);
    }
}

// Caller-supplied references (the anneal-only entry point), one wavefront per
// (syndrome, replica): the raw symplectic products with L_Z and L_X, as the
// greedy kernel writes them, and, when syndromes are given, whether the
// reference has syndrome S (Alg. 7 requires a configuration with boundary S;
// Eq. (2)).  A mismatch sets *bad.
__global__ __launch_bounds__(kWave) void k_ref_check(const PlanDev *__restrict__ pl, const uint8_t *__restrict__ refs,
                                                     const uint8_t *__restrict__ syn, int n_rep, int64_t block0,
                                                     uint8_t *__restrict__ qraw, uint32_t *bad)
{
    const int nq = pl->nq, nstab = pl->nstab, lane = threadIdx.x;
    const int64_t sr = block0 + blockIdx.x;
    const uint8_t *c = refs + sr * nq;
    uint32_t vz = 0, vx = 0;
    for (int q = lane; q < nq; q += kWave) {
        const uint32_t v = c[q], z = pl->lz[q], x = pl->lx[q];
        vz ^= (((v >> 1) & z) ^ (v & (z >> 1))) & 1;
        vx ^= (((v >> 1) & x) ^ (v & (x >> 1))) & 1;
    }
    const int az = __popcll(__ballot(vz)) & 1;
    const int ax = __popcll(__ballot(vx)) & 1;
    if (lane == 0) qraw[sr] = (uint8_t)(az | (ax << 1));
    if (!syn) return;
    const uint8_t *S = syn + (sr / n_rep) * nstab;
    uint32_t diff = 0;
    for (int f = lane; f < nstab; f += kWave) {
        const Desc d = pl->face_desc[f];
        const int q[4] = {(int)(d.x & 0xFFFF), (int)(d.x >> 16), (int)(d.y & 0xFFFF), (int)((d.y >> 16) & 0x7FF)};
        uint32_t bit = 0;
        if (q[0] < nq) bit ^= c[q[0]] & 1;
        if (q[1] < nq) bit ^= (c[q[1]] >> 1) & 1;
        if (q[2] < nq) bit ^= (c[q[2]] >> 1) & 1;
        if (q[3] < nq) bit ^= c[q[3]] & 1;
        diff |= bit ^ (S[f] & 1u);
    }
    if (__ballot(diff) && lane == 0) atomicOr(bad, 1u);
}

template <int LOGG>
__global__ __launch_bounds__(kWave) void k_anneal(AnnealArgs A) { batch_kernel_body<false, LOGG, false>(A); }
template <int LOGG>
__global__ __launch_bounds__(kWave) void k_replay(AnnealArgs A) { batch_kernel_body<false, LOGG, true>(A); }

__global__ __launch_bounds__(kWave) void k_anneal_rows(AnnealArgs A) { batch_kernel_body<true, 0, false>(A); }

static AnnealKernel static_rows_kernel(int d, bool span)
{
#define XZZX_TRY_PART(P) \
    if (AnnealKernel k = static_rows_kernel_##P(d, span)) return k;
    XZZX_STATIC_PARTS(XZZX_TRY_PART)
#undef XZZX_TRY_PART
    return nullptr;
}

// serving kernel of the specialised class holding d (NULL outside [3, 31])
static ServeKernel static_serve_kernel(int d)
{
    if (d < kStaticMinD || d > kStaticMaxD) return nullptr;
    switch (serve_class_max(d)) {
    case 9: return serve_class_kernel_9();
    case 15: return serve_class_kernel_15();
    case 21: return serve_class_kernel_21();
    case 25: return serve_class_kernel_25();
    case 29: return serve_class_kernel_29();
    default: return serve_class_kernel_31();
    }
}

static AnnealKernel bytes_kernel(bool replay, int lg)
{
    static const AnnealKernel tab[2][7] = {
        {k_anneal<0>, k_anneal<1>, k_anneal<2>, k_anneal<3>, k_anneal<4>, k_anneal<5>, k_anneal<6>},
        {k_replay<0>, k_replay<1>, k_replay<2>, k_replay<3>, k_replay<4>, k_replay<5>, k_replay<6>}};
    return tab[replay][lg];
}

__global__ __launch_bounds__(kWave) void k_serve_rows(const ServeTask *tasks, uint32_t slo, uint32_t shi)
{
    serve_kernel_body<true, false>(tasks, slo, shi);
}
__global__ __launch_bounds__(kWave) void k_serve_bytes(const ServeTask *tasks, uint32_t slo, uint32_t shi)
{
    serve_kernel_body<false, false>(tasks, slo, shi);
}
__global__ __launch_bounds__(kWave) void k_serve_replay(const ServeTask *tasks, uint32_t slo, uint32_t shi)
{
    serve_kernel_body<false, true>(tasks, slo, shi);
}

// Before a slice: every task resuming at t_begin > 0 copies the stored state
// of each of its chains into the chain's buffer that its replay entry does
// not name (the range's start state, for a later replay).  One workgroup per
// task, bytes of the task's chains spread over the lanes.
__global__ __launch_bounds__(256) void k_serve_stash(const ServeTask *tasks)
{
    const ServeTask &T = tasks[blockIdx.x];
    if (T.t_begin == 0 || !T.cpm || T.grid_mv) return;   // the grid core keeps the state at E_min itself
    const int nq = T.plan->nq;
    const int64_t nc = 4 * (int64_t)T.n_rep;
    const int64_t total = (int64_t)T.nchains * nq;
    for (int64_t i = threadIdx.x; i < total; i += blockDim.x) {
        const int64_t k = i / nq;
        const int64_t c = T.chain0 + k, q = i - k * nq;
        const int64_t b = kept_scratch(T.cpm[c]);
        T.cp[(b * nc + c) * nq + q] = T.states[c * nq + q];
    }
}



__global__ void k_zero_u32(uint32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Reduction (Alg. 7, Eq. (21)) -- one wavefront per syndrome.  Chain c of
// replica r = c/4 runs in coset Q_r * P' (P' = c mod 4); E_P is the minimum
// E_min over the chains of coset P; P* = argmin with ties to the lowest index;
// the best chain is the lowest chain of coset P* attaining E_P*.
// ---------------------------------------------------------------------------
// How a kernel lays out the states it keeps at each chain's first E_min (ci:
// the chain, n_chains: the group's): packed words [q div 16][ci], qubit q at
// bits 2 (q mod 16) (generic ladder kernel); rows chain-major, `words` words a
// chain, word Y * row_words + c / 16 holding row Y, column c, of the planar
// lattice's qpos or (rotated) of qubit dY + c; the grid core's bytes, code << 3
// per cell, `words` words a chain; the random-site kernel's words [w][ci], or
// (SiteOrder) its rows' bits in sequence, [place div 16][ci].
enum class Kept { None, Packed, PlanarRows, RotatedRows, Grid, Site, SiteOrder };

struct FinishGroup {
    const PlanDev *plan;
    const uint8_t *qcls;
    const uint8_t *refs;
    const int32_t *emin;
    const uint32_t *snap;      // states kept at E_min (kept != None)
    int32_t *e_best;
    uint8_t *cls;
    int32_t *best_chain;
    int32_t *e_cls;
    uint8_t *paper_recovery;
    uint8_t *recovery;
    int64_t n_syn;
    int64_t wave_begin;        // wavefronts of the launch before this group's (one a syndrome)
    int n_rep;
    Kept kept;
    int words, row_words;
    int d;                     // RotatedRows
};
constexpr int kFinishWaves = 4;   // per workgroup
struct FinishArgs {
    FinishGroup g[kMaxGroups];
    int n_groups;
    int64_t n_waves;
};

__device__ __forceinline__ void least_of(uint64_t &best, uint32_t hi, uint32_t lo)
{
    best = min(best, ((uint64_t)hi << 32) | lo);
}

// Eqs. (18)-(21) and, where the kernels kept each chain's state at its E_min,
// the recovery: one wavefront a syndrome, all groups of a call in one launch.
// A reference's four chains start in four different classes, so a lane reads
// the chain of class lane mod 4 and the classes reduce side by side.  It took
// two launches a group, in turn, most of it 24 64-bit shuffles one after the
// other (planar d = 9, six groups of 2048 syndromes with 40 chains: 19 and 6 us
// a group, now 15.5 for all; d = 3, 1000 syndromes with 4 chains: 17 + 5, now 4.8).
__global__ __launch_bounds__(kFinishWaves *kWave) void k_finish(FinishArgs A)
{
    const int lane = threadIdx.x % kWave;
    const int64_t wave = (int64_t)blockIdx.x * kFinishWaves + (int)uni(threadIdx.x / kWave);
    if (wave >= A.n_waves) return;
    int gi = 0;
    while (gi + 1 < A.n_groups && wave >= A.g[gi + 1].wave_begin) ++gi;
    const FinishGroup &G = A.g[gi];
    const int64_t s = wave - G.wave_begin;
    const int nc = 4 * G.n_rep;
    uint64_t best = ~0ull;
    for (int c0 = lane; c0 < nc; c0 += kWave) {
        const int c = (c0 & ~3) | cls_mul(G.qcls[s * G.n_rep + (c0 >> 2)], c0 & 3);
        least_of(best, (uint32_t)G.emin[s * nc + c], (uint32_t)c);
    }
    // over the lanes of one class: rotations within 16 lanes, then across
    least_of(best, lane_move<0x124>((uint32_t)(best >> 32)), lane_move<0x124>((uint32_t)best));
    least_of(best, lane_move<0x128>((uint32_t)(best >> 32)), lane_move<0x128>((uint32_t)best));
    best = min(best, (uint64_t)__shfl_xor((unsigned long long)best, 16, kWave));
    best = min(best, (uint64_t)__shfl_xor((unsigned long long)best, 32, kWave));
    if (G.e_cls && lane < 4) G.e_cls[s * 4 + lane] = best == ~0ull ? INT32_MAX : (int32_t)(best >> 32);
    // the class of least energy, the first of equals
    uint32_t e = (uint32_t)(best >> 32), chain = (uint32_t)best, ps = lane & 3u;
    auto take = [&](uint32_t oe, uint32_t oc, uint32_t op) {
        if (oe < e || (oe == e && op < ps)) { e = oe; chain = oc; ps = op; }
    };
    take(lane_move<0xB1>(e), lane_move<0xB1>(chain), lane_move<0xB1>(ps));
    take(lane_move<0x4E>(e), lane_move<0x4E>(chain), lane_move<0x4E>(ps));
    if (lane == 0) {
        G.e_best[s] = (int32_t)e;
        G.cls[s] = (uint8_t)ps;
        G.best_chain[s] = (int32_t)chain;
    }
    const PlanDev *pl = G.plan;
    const int nq = pl->nq;
    if (G.paper_recovery) {
        const bool ux = (ps == 1 || ps == 2), uz = (ps == 2 || ps == 3);
        const uint8_t *r0 = G.refs + (size_t)s * G.n_rep * nq;
        for (int q = lane; q < nq; q += kWave)
            G.paper_recovery[(size_t)s * nq + q] = r0[q] ^ (ux ? pl->lx[q] : 0) ^ (uz ? pl->lz[q] : 0);
    }
    if (G.kept == Kept::None) return;
    const int64_t n_chains = G.n_syn * nc, ci = s * nc + uni(chain);
    uint8_t *out = G.recovery + (size_t)s * nq;
    const uint32_t *own = G.snap + ci * G.words;
    switch (G.kept) {
    case Kept::Packed:
        for (int q = lane; q < nq; q += kWave) out[q] = (uint8_t)((G.snap[(q >> 4) * n_chains + ci] >> (2 * (q & 15))) & 3u);
        break;
    case Kept::PlanarRows:
        for (int q = lane; q < nq; q += kWave) {
            const uint32_t p = pl->qpos[q];
            out[q] = (uint8_t)((own[(p >> 8) * G.row_words + ((p & 0xFFu) >> 4)] >> (2 * (p & 15u))) & 3u);
        }
        break;
    case Kept::RotatedRows: {
        const uint32_t d = (uint32_t)G.d;
        for (int q = lane; q < nq; q += kWave) {
            const uint32_t y = (uint32_t)q / d, x = (uint32_t)q - y * d;
            out[q] = (uint8_t)((own[y * G.row_words + (x >> 4)] >> (2 * (x & 15))) & 3u);
        }
        break;
    }
    case Kept::Grid:
        for (int q = lane; q < nq; q += kWave) out[q] = reinterpret_cast<const uint8_t *>(own)[pl->grid_cell[q]] >> 3;
        break;
    case Kept::SiteOrder:
        for (int q = lane; q < nq; q += kWave) {
            const uint32_t o = pl->site_order[q];
            out[q] = (uint8_t)((G.snap[(int64_t)(o >> 4) * n_chains + ci] >> (2u * (o & 15u))) & 3u);
        }
        break;
    default:
        for (int q = lane; q < nq; q += kWave) {
            const uint32_t p = pl->site_pos[q];
            out[q] = (uint8_t)((G.snap[(int64_t)(p >> 5) * n_chains + ci] >> (p & 31u)) & 3u);
        }
    }
}

// Serving: per-coset reduction of a finished request (one wavefront each).
// The class of replica r relative to replica 0 comes from the raw symplectic
// bits the greedy kernel stored (bit 0: with L_Z, bit 1: with L_X).
// Results and recoveries of the finished requests, packed for one copy to the host.
__global__ __launch_bounds__(kWave) void k_serve_gather(const ServeFinish *fin)
{
    const ServeFinish &F = fin[blockIdx.x];
    const int lane = threadIdx.x;
    if (lane < 8) reinterpret_cast<int32_t *>(F.out)[lane] = F.result[lane];
    for (int q = lane; q < F.nq; q += kWave) F.out[32 + q] = F.recovery[q];
}

__global__ __launch_bounds__(kWave) void k_serve_reduce(const ServeFinish *fin)
{
    const ServeFinish &F = fin[blockIdx.x];
    const int lane = threadIdx.x;
    const int nc = 4 * F.n_rep;
    const int raw0 = F.qraw[0] & 3;
    uint64_t best[4] = {~0ull, ~0ull, ~0ull, ~0ull};
    for (int c = lane; c < nc; c += kWave) {
        const int v = (F.qraw[c >> 2] & 3) ^ raw0;
        const int cls = cls_mul(cls_from_bits(v & 1, v >> 1), c & 3);
        const uint64_t key = ((uint64_t)(uint32_t)F.e3[nc + c] << 32) | (uint32_t)c;
#pragma unroll
        for (int P = 0; P < 4; ++P)
            if (cls == P) best[P] = min(best[P], key);
    }
#pragma unroll
    for (int P = 0; P < 4; ++P)
#pragma unroll
        for (int sh = 1; sh < kWave; sh <<= 1) best[P] = min(best[P], (uint64_t)__shfl_xor(best[P], sh, kWave));
    int ps = 0;
#pragma unroll
    for (int P = 1; P < 4; ++P)
        if ((best[P] >> 32) < (best[ps] >> 32)) ps = P;
    if (lane == 0) {
        F.result[0] = (int32_t)(best[ps] >> 32);
        F.result[1] = ps;
        F.result[2] = (int32_t)(best[ps] & 0xFFFFFFFFu);
        for (int P = 0; P < 4; ++P) F.result[4 + P] = best[P] == ~0ull ? INT32_MAX : (int32_t)(best[P] >> 32);
    }
}

// ---------------------------------------------------------------------------
// Host-side launch logic.
// ---------------------------------------------------------------------------
// A launch addresses at most 2^32 - 1 work-items (larger grids wrap
// silently), i.e. this many wavefronts of 64.
constexpr int64_t kMaxLaunchItems = 0xFFFFFFFFll;
constexpr int64_t kMaxLaunchWaves = kMaxLaunchItems / kWave;

static int check_hip(hipError_t e, const char *what)
{
    if (e == hipSuccess) return XZZX_OK;
    set_error(std::string(what) + ": " + hipGetErrorString(e));
    return XZZX_EDEVICE;
}

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
static int device_cus();

// One colour per half wavefront where a colour has at most 128 nodes (rotated
// d <= 15: few enough defects that 32 lanes take them in one or two turns);
// the whole wavefront per colour on larger lattices.
static bool greedy_split(const Plan &P) { return std::max(P.hdev.ncol[0], P.hdev.ncol[1]) <= 128; }

// A workgroup of the greedy references: `fit` wavefronts at most, `least` at
// least, for `units` tasks of a syndrome, shared evenly by its workgroups.
struct GreedyForm {
    int shares, waves, cache_entries;
    uint32_t lds;
    int per_cu;                // workgroups that a CU holds at once
};
static GreedyForm greedy_form(int sets, int nodes, int stride, int nwords, int ties, int units, int fit, int least, bool weights)
{
    const GreedyLds base = greedy_lds_layout(sets, stride, nwords, 0, ties);
    GreedyForm f{};
    f.shares = (units + fit - 1) / fit;
    f.waves = std::max(least, (units + f.shares - 1) / f.shares);
    if (weights) {
        const int rows = nodes * 7 / 16 + 8, room = 65536 - 64 - (int)(base.waves + f.waves * base.per_wave);
        f.cache_entries = std::max(0, std::min(rows * (rows | 1), room / (4 * sets)));
    }
    f.lds = greedy_lds_layout(sets, stride, nwords, f.cache_entries, ties).waves + f.waves * base.per_wave;
    f.per_cu = std::max(1, std::min(kGreedyCuLds / (int)f.lds, 32 / f.waves));
    return f;
}

// The greedy references of n syndromes, A's outputs and syndromes set by the
// caller.  A workgroup's wavefronts take replicas of one syndrome and share its
// scan.  Two forms:
// - wide: up to kGreedyWaves wavefronts, and the pair weights of up to about
//   half the nodes as defects (more are rare: each fires with probability below
//   one half) in what a 64 KiB share has left;
// - narrow: up to four wavefronts and no weights in LDS, but for whole workgroups
//   of small lattices, so that many workgroups fit a CU and go through their
//   phases at different times; in the split form a wavefront takes several
//   references in turn, which saves dispatches.
// Small launches go wide, for latency.  Beyond them the lines stand where the
// two forms cross in dense syndromes, three or four defects in ten generators;
// sparse ones cross earlier, as they need few weights.  Wide / narrow, us, at
// three in ten (in brackets one in twelve):
// - d >= 17, by the wavefronts of a wide workgroup: 11 or 12 (two workgroups a CU,
//   with room for weights) wide at any size (4017 syndromes x 12 at d = 21 637 / 827,
//   1774 x 12 at d = 19 261 / 329); 8 to 10 up to 2048 references for each (1021 x 10 at
//   d = 21 220 us, 800 x 10 164 / 215 (93 / 96)); others in one turn of workgroups over the
//   device that leaves no CU far fuller than narrow ones would (250 x 32 at d = 21
//   182 / 223 (100 / 102), but 156 x 32 158 / 144 (93 / 65), 1250 x 32 730 / 722 (409 /
//   327)).  13 to 15 wavefronts leave the weights no room (625 x 64 at d = 27 1577 / 1267
//   (630 / 456)), fewer than eight share too little (2000 x 4 at d = 21 324 / 213 (155 /
//   99)).  Where LDS keeps the narrow form below 32 wavefronts a CU: also where the
//   wide one takes no more turns (4000 x 10 at d = 31 2.02 / 2.46 ms, planar d = 25 1250 x
//   32 2.79 / 3.43 ms (0.80 / 0.85), but 4000 x 10 there 4.82 / 4.01 (1.09 / 0.99));
// - split form: beyond 64 nodes, where weights from L1 cost most, up to 5120
//   references for each wavefront (1250 x 32 at d = 15 232 / 284 (132 / 151), 4096 x 32
//   683 / 690 (376 / 355)); else up to 2048 and only with one or two workgroups a
//   syndrome (625 x 32 at d = 11 80 / 81 (62 / 56), 2048 x 32 214 / 212 (155 / 146)).
constexpr int64_t kGreedyWide = 2048;   // references of a launch that is wide whatever its workgroups
static int launch_greedy(const Plan &P, GreedyArgs A, int64_t n_syn, uint64_t seed, int mode, hipStream_t stream)
{
    const bool split = greedy_split(P), random = mode == XZZX_GREEDY_RANDOM;
    const int sets = split ? 2 : 1, nwords = (P.lat.nq + 3) / 4;
    const int nodes = std::max(P.hdev.ncol[0], P.hdev.ncol[1]);
    A.plan = P.ddev;
    A.mode = mode;
    A.seed_lo = (uint32_t)seed;
    A.seed_hi = (uint32_t)(seed >> 32);
    A.stride = (nodes + 2) & ~1;
    A.n_units = (A.n_rep + A.rep_div - 1) / A.rep_div;
    // the list of first ties: small lattices have about as many as a dense
    // syndrome's; larger ones have fewer each, and LDS that costs occupancy (one
    // replica of planar d = 31, 30000 syndromes: 42.0 ms with three entries a node,
    // 29.8 with half of one)
    A.ties = !random ? 0 : split ? 3 * A.stride : A.n_units == 1 ? A.stride / 2 : A.stride;
    const GreedyLds base = greedy_lds_layout(sets, A.stride, nwords, 0, A.ties);
    // boundary references share no scan: a wavefront each, over as many CUs
    const bool alone = mode == XZZX_GREEDY_BOUNDARY;
    // (tiny lattices have little to share: their dispatches count more)
    const bool tiny = nodes <= 16;
    const int64_t refs = n_syn * A.n_units;
    const int cap = std::min(kGreedyWaves, (int)((65536 - 64 - base.waves) / base.per_wave));
    const int most_waves = std::min(cap, A.n_units);
    auto form = [&](int units, int fit, int least, bool weights) {
        return greedy_form(sets, nodes, A.stride, nwords, A.ties, units, std::min(cap, fit), least, weights);
    };
    bool wide = !alone && refs <= kGreedyWide;
    if (!alone && !wide && most_waves >= 5) {
        const GreedyForm w = form(A.n_units, kGreedyWaves, 1, true), n = form(A.n_units, 4, 1, false);
        if (split) {
            wide = nodes > 64 ? refs <= 5120 * most_waves
                              : w.shares <= 2 && refs <= (tiny ? 1024 * std::min(most_waves, 12) : 2048 * std::max(most_waves, 10));
        } else {
            // turns of workgroups over the device, and the references of the fullest CU by those of a syndrome
            const int64_t cus = device_cus();
            auto turns = [&](const GreedyForm &g) { return (n_syn * g.shares + g.per_cu * cus - 1) / (g.per_cu * cus); };
            auto load = [&](const GreedyForm &g) { return (double)((n_syn * g.shares + cus - 1) / cus) / g.shares; };
            const bool lds_bound = n.per_cu < 32 / n.waves;
            wide = (turns(w) == 1 && load(w) <= 1.4 * load(n)) || w.waves == 11 || w.waves == 12 ||
                   (w.waves >= 8 && w.waves <= 10 && refs <= 2048 * w.waves) ||
                   (lds_bound && w.waves <= 12 && turns(w) <= turns(n));
        }
    }
    if (random && split && !wide && nodes > 48) A.ties = A.stride;
    // a wavefront's references in turn: three, or four where that fills workgroups;
    // more of small lattices where a launch has very many (d = 7, 30000 x 10: 514 us
    // with three, 476 with nine)
    int64_t in_turn = tiny ? std::min<int64_t>(refs / 10000, 3) : A.n_units % 16 ? (refs < 40000 ? 1 : 3) : refs < 49152 ? 1 : 4;
    if (nodes <= 48) in_turn = std::max(in_turn, std::min<int64_t>(refs / 32768, A.n_units));
    const int each = split && !alone && !wide && A.n_units > (tiny ? 2 : 4) ? (int)std::max<int64_t>(1, in_turn) : 1;
    const int fit = alone ? 1 : split && (wide ? refs <= 256 && nodes <= 48 : tiny) ? 2 : wide ? kGreedyWaves : 4;
    const int per_syn = (A.n_units + each - 1) / each;
    GreedyForm f = form(per_syn, fit, 1, wide);
    A.shares = f.shares;
    A.unit_step = f.shares * f.waves;
    // a few references of a large lattice: wavefronts without one help in the scan
    if (!split && !alone && refs <= 256) f = form(per_syn, fit, std::min(cap, 4), wide);
    else if (split && !alone && !wide && nodes <= 84 && f.waves == 4) f = form(per_syn, fit, 1, true);
    A.cache_entries = f.cache_entries;
    const int waves = f.waves;
    void (*kernel)(GreedyArgs) = k_greedy<false, false>;
    if (split) kernel = each > 1 ? k_greedy<true, true> : k_greedy<true, false>;
    // one launch addresses fewer than 2^32 work-items, and 2^16 rows of workgroups
    const int rows = std::min(A.shares, 65535);
    const int64_t most = std::max<int64_t>(1, kMaxLaunchWaves / ((int64_t)waves * rows));
    for (A.syn0 = 0; A.syn0 < n_syn; A.syn0 += most)
        for (A.share0 = 0; A.share0 < A.shares; A.share0 += rows) {
            const dim3 grid((unsigned)std::min<int64_t>(most, n_syn - A.syn0), (unsigned)std::min(rows, A.shares - A.share0));
            hipLaunchKernelGGL(kernel, grid, dim3(waves * kWave), f.lds, stream, A);
            const int rc = check_hip(hipGetLastError(), "k_greedy launch");
            if (rc) return rc;
        }
    return XZZX_OK;
}

static int launch_greedy(const Plan &P, const uint8_t *d_syn, const uint32_t *d_uid, int64_t n_syn,
                         int n_rep, uint64_t seed, int mode, uint8_t *d_refs, uint8_t *d_qraw,
                         hipStream_t stream)
{
    if (n_syn == 0) return XZZX_OK;
    GreedyArgs A{};
    A.syn = d_syn;
    A.uid = d_uid;
    A.refs = d_refs;
    A.qraw = d_qraw;
    A.n_rep = n_rep;
    A.rep_div = std::max(P.ladder_k, 1);
    A.syn_stride = P.lat.nstab;
    return launch_greedy(P, A, n_syn, seed, mode, stream);
}

static int launch_qcls(const uint8_t *d_qraw, int64_t n_syn, int n_rep, uint8_t *d_qcls, hipStream_t stream)
{
    if (n_syn == 0) return XZZX_OK;
    hipLaunchKernelGGL(k_qcls, dim3((unsigned)((n_syn + 255) / 256)), dim3(256), 0, stream, d_qraw, n_syn, n_rep, d_qcls);
    return check_hip(hipGetLastError(), "k_qcls launch");
}

// Per-group workspace layout.
struct GroupWs {
    uint8_t *refs, *qraw, *qcls;
    int32_t *emin, *stop, *efin, *best_chain;
    uint32_t *cp_rows;     // checkpoints of groups on the specialised packed-row kernel
    uint32_t *min_snap;    // random-site, planar specialised, ladder and grid groups: each chain's state at its first E_min
    int grid;              // lanes per chain on the grid core (0: another kernel)
    bool lean;             // short of workspace (see call_form)
};

// Replica exchange on the packed-row kernels specialised to d: the distance
// when the group's ladders run there (rotated: d <= kLadderRowsMaxD; planar:
// d <= 15), else 0.  Depends on the plan, n_rep and the workspace's size, so
// every stage of a decode agrees.  spans: the tasks of 64 chains do not all
// lie inside one syndrome; such ladders keep more words per chain than the
// generic kernel, which runs them where the workspace is short (lean).
static bool spans(const xzzx_group &g) { return (4 * g.n_rep) % kWave != 0; }

static int ladder_rows_d(const xzzx_group &g, bool lean)
{
    const Plan &P = g.plan->P;
    if (!P.ladder_k || !P.use_rows || P.order != XZZX_ORDER_COLOUR) return 0;
    if (P.static_d && P.static_d <= kLadderRowsMaxD && !(lean && spans(g))) return P.static_d;
    return 0;
}

static int ladder_planar_d(const xzzx_group &g)
{
    const Plan &P = g.plan->P;
    if (!P.ladder_k || !P.use_rows || P.order != XZZX_ORDER_COLOUR) return 0;
    return P.planar_d;
}

// Words per chain of the state kept at E_min: random-site chains (their packed
// rows), the generic ladder kernel (packed, the position nq scratch), the
// planar kernels specialised to d and the rotated ladder kernels specialised
// to d (their rows); 0 for other groups.  A plan's kernel must not change between the
// stages of one decode.
static int64_t min_snap_words(const xzzx_group &g, bool lean)
{
    const Plan &P = g.plan->P;
    if (ladder_rows_d(g, lean)) return ladder_rows_state_words(ladder_rows_d(g, lean));
    if (ladder_planar_d(g)) return planar_state_words(ladder_planar_d(g));
    if (P.order == XZZX_ORDER_RANDOM_SITE) return lean ? P.lat.nq / 16 + 1 : P.hdev.site_words;
    if (P.ladder_k) return P.lat.nq / 16 + 1;
    if (P.use_rows && P.planar_d) return planar_state_words(P.planar_d);
    return 0;
}

// A group runs on the packed-row kernel specialised to its distance when the
// plan allows it: in the form whose tasks of 64 chains may span syndromes
// where they do not all lie inside one.  (That form takes two more products
// per Philox block: 2.16 against 2.28 x 10^12 attempts/s at d = 11, 2.37 against
// 2.40 at d = 17, 1.95 against 2.03 at d = 31, 200 sweeps of 524288 chains, half as
// many from d = 21; before, such groups ran on the generic packed-row
// kernel, rows in LDS (a decode of 4099 syndromes of 40 chains at d = 13, 100
// sweeps: 4.03 -> 2.29 ms), or, d = 31, on byte states.)
static bool uses_static(const xzzx_group &g)
{
    const Plan &P = g.plan->P;
    return P.order == XZZX_ORDER_COLOUR && !P.ladder_k && P.use_rows && P.static_d;
}

// Sweeps between the checkpoints of a plan: kCheckpointEvery, or the least
// interval that leaves at most kMaxCheckpoints before the last sweep.  Short
// schedules keep about eight, at least 16 sweeps apart: the replay covers up to
// an interval, and beside 100 sweeps one of 64 showed (d = 13, 4099 syndromes of
// 40 chains: a pass took 2.18 ms, now 2.08); not with a short workspace (lean).
static int checkpoint_interval(const Plan &P, bool lean)
{
    const int last = P.n_sweeps - 1;
    const int dense = std::min(kCheckpointEvery, std::max(kCheckpointEvery / 4, (last + 7) / 8));
    const int every = lean ? kCheckpointEvery : dense;
    return std::max(every, (last + kMaxCheckpoints - 1) / kMaxCheckpoints);
}

// Checkpoints a specialised group keeps: the states at the start of sweeps
// c, 2c, ... before the last sweep, for c = checkpoint_interval.
static int checkpoints_of(const xzzx_group &g, bool lean)
{
    if (!uses_static(g) || g.plan->P.n_sweeps <= 0) return 0;
    return (g.plan->P.n_sweeps - 1) / checkpoint_interval(g.plan->P, lean);
}

static int device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    return cus;
}

// Lanes per chain of each group on the grid core, 0 where another kernel runs
// it.  A plan whose lanes were chosen (the byte-state kernel with L lanes per
// chain) takes the grid core with those lanes; it has the same use and half
// the LDS round trips a phase.  A plan left to the default takes it, with
// the least power of two of lanes that holds a colour class (64 at most),
//   - where no packed-row kernel applies (planar d > 15): at 64 lanes it ran
//     2048 syndromes of 64 chains in 9.5 against 14.4 ms (d = 21, 60 sweeps);
//   - where the call is too small for one chain per lane: up to
//     kGridChainsPerCu chains per CU, when less than two in five SIMDs would
//     get a wavefront of 64 chains, each of which takes the whole latency of
//     a sweep on one lane (7.3 us at d = 11, 0.61 us on 32 or 64 lanes).
//     Rotated d = 11, 500 sweeps: 64 chains 3.62 -> 0.31 ms, 16384 3.69 ->
//     1.23, 32768 3.7 -> 2.3, 65536 3.87 -> 4.5 (the packed-row kernel is
//     the better one from there); the lines of the other lattices cross
//     between 28000 (planar d = 5) and 65000 chains.  The groups of a call
//     share the device, so the smallest ones take it while all of them
//     together stay below the line.
static int grid_lanes(const Plan &P)
{
    int lanes = 4;
    while (lanes < kWave && lanes < P.lat.per_class) lanes *= 2;
    return P.grid_moves(lanes) ? lanes : 0;
}

static std::vector<int> grid_routes(const xzzx_group *groups, int n_groups)
{
    std::vector<int> lanes(n_groups, 0);
    std::vector<std::pair<int64_t, int>> small;   // chains, group
    for (int i = 0; i < n_groups; ++i) {
        const xzzx_group &g = groups[i];
        const Plan &P = g.plan->P;
        if (P.order != XZZX_ORDER_COLOUR || P.ladder_k || g.n_syn <= 0 || g.n_rep <= 0) continue;
        if (!P.use_rows) {
            const int l = P.grid_auto ? grid_lanes(P) : P.lanes;
            if (l >= 4 && P.grid_moves(l)) lanes[i] = l;
        } else if (P.grid_auto) {
            small.push_back({g.n_syn * 4 * (int64_t)g.n_rep, i});
        }
    }
    std::sort(small.begin(), small.end());
    int64_t left = kGridChainsPerCu * device_cus();
    for (const auto &[chains, i] : small) {
        if (chains > left) break;
        left -= chains;
        lanes[i] = grid_lanes(groups[i].plan->P);
    }
    return lanes;
}

// Bytes of the buffers a group has in every form.
static size_t fixed_bytes(const xzzx_group &g, bool decode)
{
    const Plan &P = g.plan->P;
    const size_t nq = P.lat.nq, ns = (size_t)g.n_syn, R = (size_t)g.n_rep, nc = 4 * R * ns;
    size_t b = 0;
    if (decode && !g.d_refs) b += align256(ns * R * nq);
    b += align256(ns * R);                                  // qraw
    if (!g.d_qcls) b += align256(ns * R);
    if (!g.d_chain_emin) b += align256(nc * 4);
    if (!g.d_chain_stop) b += align256(nc * 4);
    if (!g.d_chain_e) b += align256(nc * 4);
    if (!g.d_best_chain) b += align256(ns * 4);
    return b;
}

// Checkpoints and words per chain of the states kept at E_min, by the group's
// form.  grid: on the grid core (lanes per chain); lean: short of workspace.
static size_t form_checkpoints(const xzzx_group &g, int grid, bool lean)
{
    return grid || (lean && spans(g)) ? 0 : (size_t)checkpoints_of(g, lean);
}
static size_t form_words(const xzzx_group &g, int grid, bool lean)
{
    return grid ? (size_t)g.plan->P.hdev.grid_words : (size_t)min_snap_words(g, lean);
}
static size_t form_bytes(const xzzx_group &g, int grid, bool lean)
{
    const Plan &P = g.plan->P;
    const size_t nc = 4 * (size_t)g.n_rep * (size_t)g.n_syn;
    return align256(form_checkpoints(g, grid, lean) * P.lat.d * P.static_words * nc * 4) +
           align256(form_words(g, grid, lean) * nc * 4);
}

// The forms of a call's groups with a workspace of so many bytes.  A call is
// accepted with `least` bytes, in which no group runs on the grid core, groups
// whose tasks span syndromes keep no checkpoints (their recoveries are replayed
// from the references), short schedules keep sparser ones, random-site groups
// keep their states in fewer words and spanning ladders run on the generic
// kernel.  What is left goes to the groups' better forms, those that take fewest
// bytes first: at most kMostForms bytes of a call (a sixteenth of the card's
// memory), so that a large call does not ask for much more than it needs.
constexpr size_t kMostForms = (size_t)18 << 30;

struct CallForm {
    std::vector<int> grid;     // lanes per chain on the grid core (0: another kernel)
    std::vector<char> lean;    // short of workspace
    size_t least = 256;
    size_t bytes = 256;        // what the forms use
};

static CallForm call_form(const xzzx_group *groups, int n_groups, bool decode, size_t workspace_bytes)
{
    CallForm F;
    F.grid = grid_routes(groups, n_groups);
    F.lean.assign(n_groups, 0);
    std::vector<std::pair<size_t, int>> more;   // bytes a better form takes beyond the least, group
    for (int i = 0; i < n_groups; ++i) {
        const size_t lean = form_bytes(groups[i], 0, true), best = form_bytes(groups[i], F.grid[i], false);
        F.least += fixed_bytes(groups[i], decode) + lean;
        more.push_back({best > lean ? best - lean : 0, i});
    }
    std::sort(more.begin(), more.end());
    F.bytes = F.least;
    size_t left = workspace_bytes > F.least ? std::min(workspace_bytes - F.least, kMostForms) : 0;
    for (const auto &[bytes, i] : more) {
        if (bytes > left) {
            F.lean[i] = 1;
            F.grid[i] = 0;
            continue;
        }
        left -= bytes;
        F.bytes += bytes;
    }
    return F;
}

// The buffers of every form come first, so that stages agree on them.
static std::vector<GroupWs> carve(const xzzx_group *groups, int n_groups, bool decode, const CallForm &F, uint8_t *p)
{
    std::vector<GroupWs> ws(n_groups);
    auto take = [&](size_t bytes) { uint8_t *r = p; p += align256(bytes); return r; };
    for (int i = 0; i < n_groups; ++i) {
        const xzzx_group &g = groups[i];
        const size_t nq = g.plan->P.lat.nq, ns = (size_t)g.n_syn, R = (size_t)g.n_rep, nc = 4 * R * ns;
        GroupWs &w = ws[i];
        w.grid = F.grid[i];
        w.lean = F.lean[i];
        w.refs = g.d_refs ? g.d_refs : (decode ? take(ns * R * nq) : nullptr);
        w.qraw = take(ns * R);
        w.qcls = g.d_qcls ? g.d_qcls : take(ns * R);
        w.emin = g.d_chain_emin ? g.d_chain_emin : reinterpret_cast<int32_t *>(take(nc * 4));
        w.stop = g.d_chain_stop ? g.d_chain_stop : reinterpret_cast<int32_t *>(take(nc * 4));
        w.efin = g.d_chain_e ? g.d_chain_e : reinterpret_cast<int32_t *>(take(nc * 4));
        w.best_chain = g.d_best_chain ? g.d_best_chain : reinterpret_cast<int32_t *>(take(ns * 4));
    }
    for (int i = 0; i < n_groups; ++i) {
        const xzzx_group &g = groups[i];
        const Plan &P = g.plan->P;
        const size_t nc = 4 * (size_t)g.n_rep * (size_t)g.n_syn;
        const size_t ncp = form_checkpoints(g, F.grid[i], F.lean[i]), words = form_words(g, F.grid[i], F.lean[i]);
        ws[i].cp_rows = ncp ? reinterpret_cast<uint32_t *>(take(ncp * P.lat.d * P.static_words * nc * 4)) : nullptr;
        ws[i].min_snap = words ? reinterpret_cast<uint32_t *>(take(words * nc * 4)) : nullptr;
    }
    return ws;
}

static int validate_groups(const xzzx_group *groups, int n_groups, bool decode)
{
    if (!groups || n_groups < 1 || n_groups > kMaxGroups) {
        set_error("need 1..16 groups");
        return XZZX_EINVAL;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { set_error("hipGetDevice failed"); return XZZX_EDEVICE; }
    for (int i = 0; i < n_groups; ++i) {
        const xzzx_group &g = groups[i];
        if (!g.plan || g.n_syn < 0 || g.n_rep < 1 || g.n_rep > (1 << 20)) { set_error("bad group (plan, n_syn or n_rep)"); return XZZX_EINVAL; }
        if (g.plan->P.ladder_k && g.n_rep % g.plan->P.ladder_k) { set_error("n_rep must be a multiple of the ladder's levels"); return XZZX_EINVAL; }
        if (g.plan->P.device != dev) { set_error("plan was created on another device"); return XZZX_EINVAL; }
        if (g.n_syn == 0) continue;
        if (!g.d_uid || !g.d_e_best || !g.d_cls || !g.d_recovery) { set_error("missing required group buffer"); return XZZX_EINVAL; }
        if (decode && !g.d_syn) { set_error("decode needs d_syn"); return XZZX_EINVAL; }
        if (!decode && !g.d_refs) { set_error("anneal needs d_refs"); return XZZX_EINVAL; }
        if ((int64_t)g.n_syn * 4 * g.n_rep >= ((int64_t)1 << 31)) { set_error("too many chains in one group"); return XZZX_ERANGE; }
    }
    return XZZX_OK;
}

static int anneal_grid(const void *kernel, int block, size_t lds_bytes, uint32_t n_tasks, unsigned *grid)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, lds_bytes) != hipSuccess || per_cu <= 0)
        per_cu = 1;
    const uint64_t full = (uint64_t)device_cus() * (uint64_t)per_cu;
    *grid = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(full, n_tasks));
    return XZZX_OK;
}

static int log2_int(int v)
{
    int lg = 0;
    while ((1 << lg) < v) ++lg;
    return lg;
}

enum class AnnealMode { Persistent, Replay, Plain };

// Launch one annealing kernel over `units` of the selected groups (chains, or
// syndromes in replay mode).  rows: packed-row kernel (one chain per lane);
// otherwise the byte-state kernel with the plan's lanes per chain.  The replay
// re-runs one chain per syndrome with the byte-state kernel, spreading a chain
// over more lanes when that is needed to give every CU several wavefronts.
static int launch_set(const xzzx_group *groups, const GroupWs *ws, const std::vector<int> &sel, bool rows, int lanes,
                      AnnealMode mode, uint64_t seed, int64_t unit_offset, int64_t units_override,
                      uint32_t *d_counter, hipStream_t stream, int static_d = 0, bool site = false,
                      int planar_d = 0, bool ladder = false, int grid_mv = 0, int priority = 0)
{
    const bool replay = mode == AnnealMode::Replay;
    AnnealArgs A{};
    A.priority = priority;
    A.seed_lo = (uint32_t)seed;
    A.seed_hi = (uint32_t)(seed >> 32);
    A.counter = d_counter;
    auto units_of = [&](int i) -> int64_t {
        return units_override >= 0 ? units_override : (replay ? groups[i].n_syn : groups[i].n_syn * 4 * groups[i].n_rep);
    };
    // order groups by work per task (largest first) so the queue is LPT-like
    std::vector<int> order = sel;
    auto cost = [&](int i) {
        const Plan &P = groups[i].plan->P;
        return (double)P.n_sweeps * P.lat.nstab;
    };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost(a) > cost(b); });
    uint64_t tasks = 0;
    size_t lds = 0;
    int ng = 0;
    const int lg = log2_int(lanes);
    // random-site workgroups: up to eight wavefronts share the descriptors and
    // entries, which fits the device's most wavefronts; one each where there
    // are too few to give every SIMD two, so that they spread over the CUs
    int site_waves = 1;
    bool site_wide = false;
    if (site) {
        int64_t waves = 0;
        size_t most = 0;
        for (int i : order) waves += (units_of(i) + kWave - 1) / kWave;
        site_wide = !order.empty() && groups[order[0]].plan->P.site_wide;   // the same for a set
        for (int w = 2; w <= 8; w *= 2) {
            most = 0;
            for (int i : order) most = std::max(most, groups[i].plan->P.lds_bytes_site(w));
            if (mode == AnnealMode::Persistent && waves >= 8LL * device_cus() && most <= 65536) site_waves = w;
        }
    }
    for (int i : order) {
        const xzzx_group &g = groups[i];
        const Plan &P = g.plan->P;
        GroupArgs &G = A.g[ng++];
        G.plan = P.ddev;
        G.uid = g.d_uid;
        G.refs = ws[i].refs;
        G.emin = ws[i].emin;
        G.stop = ws[i].stop;
        G.efin = ws[i].efin;
        G.final = replay ? nullptr : g.d_chain_final;
        G.best_chain = ws[i].best_chain;
        G.recovery = g.d_recovery;
        G.n_rep = g.n_rep;
        G.log_lanes = lg;
        G.row_words = rows ? P.row_words : 0;
        // checkpoints: written by the specialised kernel, read by the replay
        const bool cp = ws[i].cp_rows && (static_d || replay);
        G.cp_rows = cp ? ws[i].cp_rows : nullptr;
        G.cp_every = cp ? checkpoint_interval(P, ws[i].lean) : 0;
        G.n_chains = g.n_syn * 4 * g.n_rep;
        G.min_snap = (site || planar_d || ladder || grid_mv) ? ws[i].min_snap : nullptr;
        G.unit_offset = unit_offset;
        const int64_t units = units_of(i);
        G.n_units = units;
        G.task_begin = (int64_t)tasks;
        const int C = site ? site_waves * kWave : kWave / lanes;
        tasks += (uint64_t)((units + C - 1) / C);
        lds = std::max(lds, (ladder && (static_d || planar_d))
                                ? 8 * (size_t)P.ladder_k * P.nranks()
                            : (static_d || planar_d) ? (size_t)0
                            : grid_mv ? P.lds_bytes_grid(lanes)
                            : ladder ? P.lds_bytes_ladder()
                            : site   ? P.lds_bytes_site(site_waves)
                            : rows   ? P.lds_bytes_rows()
                                     : P.lds_bytes_anneal(lanes));
    }
    if (ng == 0 || tasks == 0) return XZZX_OK;
    if (tasks >= 0xFFFFFFF0ull) { set_error("too many anneal tasks in one launch"); return XZZX_ERANGE; }
    A.n_groups = ng;
    A.n_tasks = (uint32_t)tasks;
    if (lds > 65536) { set_error("LDS demand above 64 KiB"); return XZZX_ERANGE; }
    const bool span = static_d && spans(groups[order[0]]);
    const AnnealKernel kern = grid_mv ? grid_kernel(lanes, grid_mv)
                              : (ladder && static_d) ? ladder_rows_kernel(static_d, span)
                              : (ladder && planar_d) ? ladder_planar_kernel(planar_d)
                              : ladder     ? ladder_kernel()
                              : site     ? site_kernel(site_wide, ws[order[0]].lean)
                              : planar_d ? planar_rows_kernel(planar_d)
                              : static_d ? static_rows_kernel(static_d, span)
                              : rows     ? k_anneal_rows
                                         : bytes_kernel(replay, lg);
    if (mode == AnnealMode::Plain) {
        A.counter = nullptr;
        A.grid = (uint32_t)tasks;
        hipLaunchKernelGGL(kern, dim3((unsigned)tasks), dim3(kWave * site_waves), lds, stream, A);
        return check_hip(hipGetLastError(), "plain anneal launch");
    }
    unsigned grid = 0;
    int rc = anneal_grid((const void *)kern, kWave * site_waves, lds, A.n_tasks, &grid);
    if (rc) return rc;
    A.grid = grid;
    // The clear takes a workgroup of one wavefront for every SIMD.  After
    // workgroups of several wavefronts (the greedy stage's) the dispatcher puts
    // two of the next single-wavefront ones on some SIMDs and none on others,
    // until a launch of such has passed through the same queue (read from the
    // hardware ids of four launches of 1024: 20 to 80 SIMDs hold two of a
    // launch, most seven wavefronts in all; after this clear all hold one of
    // each).  Chains last long and a SIMD with one more ends last: five
    // distances d = 5..21 of 256 syndromes and 256 chains took 201 ms, now 152;
    // ladders at d = 11, four wavefronts a SIMD, 18.9 ms, now 16.4.
    hipLaunchKernelGGL(k_zero_u32, dim3(4 * (unsigned)device_cus()), dim3(kWave), 0, stream, d_counter, 1);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kWave * site_waves), lds, stream, A);
    return check_hip(hipGetLastError(), "anneal launch");
}

// Side streams (default priority) and reusable events for running the
// independent launches of one call concurrently.  Each (device, caller stream)
// pair has a set of its own, created on first use and kept until the process
// ends, so calls on different streams -- among them a graph capture on one
// stream and a serving loop on another -- never share a side stream; calls on
// one caller stream hold the set's lock while they fork and join.  Past
// kMaxSideSets sets, calls run their launches one after another on the caller
// stream instead (same results).
constexpr int kSideStreams = 3;
constexpr int kMaxSideSets = 256;

struct SideSet {
    std::mutex mu;
    hipStream_t side[kSideStreams] = {};
    hipEvent_t fork = nullptr;
    hipEvent_t join[kSideStreams] = {};
};

// The set of `caller` on the current device, nullptr when the table is full;
// an error status if a stream or event cannot be created.
static int side_set(hipStream_t caller, SideSet **out)
{
    static std::mutex mu;
    static std::vector<std::pair<std::pair<int, hipStream_t>, SideSet *>> sets;   // never freed
    *out = nullptr;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { set_error("hipGetDevice failed"); return XZZX_EDEVICE; }
    const std::pair<int, hipStream_t> key(dev, caller);
    std::lock_guard<std::mutex> lk(mu);
    for (auto &e : sets)
        if (e.first == key) { *out = e.second; return XZZX_OK; }
    if ((int)sets.size() >= kMaxSideSets) return XZZX_OK;
    auto *S = new SideSet();
    bool ok = hipEventCreateWithFlags(&S->fork, hipEventDisableTiming) == hipSuccess;
    for (int i = 0; i < kSideStreams && ok; ++i)
        ok = hipStreamCreateWithFlags(&S->side[i], hipStreamNonBlocking) == hipSuccess &&
             hipEventCreateWithFlags(&S->join[i], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        for (int i = 0; i < kSideStreams; ++i) {
            if (S->side[i]) (void)hipStreamDestroy(S->side[i]);
            if (S->join[i]) (void)hipEventDestroy(S->join[i]);
        }
        if (S->fork) (void)hipEventDestroy(S->fork);
        delete S;
        set_error("side stream or event creation failed");
        return XZZX_EDEVICE;
    }
    sets.emplace_back(key, S);
    *out = S;
    return XZZX_OK;
}

// Runs launch(i, stream_i) for i < n: launch 0 on `stream`, the others on the
// caller's side streams, which wait for `stream`'s prior work; `stream` then
// waits for all.  Works under hipGraph capture (the events become graph
// dependencies).  serial: every launch on `stream`, in order (no side
// streams or events are created or used).
template <typename F>
static int fork_join(hipStream_t stream, int n, F launch, bool serial = false)
{
    if (serial) {
        int rc = XZZX_OK;
        for (int i = 0; i < n && !rc; ++i) rc = launch(i, stream);
        return rc;
    }
    if (n <= 1) return n ? launch(0, stream) : XZZX_OK;
    SideSet *S = nullptr;
    int rc = side_set(stream, &S);
    if (rc) return rc;
    if (!S) {
        for (int i = 0; i < n && !rc; ++i) rc = launch(i, stream);
        return rc;
    }
    std::lock_guard<std::mutex> lk(S->mu);
    rc = check_hip(hipEventRecord(S->fork, stream), "fork record");
    bool used[kSideStreams] = {false, false, false};
    for (int i = 0; i < n && !rc; ++i) {
        hipStream_t s = stream;
        if (i > 0) {
            const int k = (i - 1) % kSideStreams;
            s = S->side[k];
            if (!used[k]) {
                rc = check_hip(hipStreamWaitEvent(s, S->fork, 0), "fork wait");
                used[k] = true;
            }
        }
        if (!rc) rc = launch(i, s);
    }
    // join every side stream that waited, also after a failed launch, so no
    // side stream is left inside a capture of `stream`
    for (int k = 0; k < kSideStreams; ++k) {
        if (!used[k]) continue;
        int r = check_hip(hipEventRecord(S->join[k], S->side[k]), "join record");
        if (!r) r = check_hip(hipStreamWaitEvent(stream, S->join[k], 0), "join wait");
        if (!rc) rc = r;
    }
    return rc;
}

// where the group's annealing left each chain's state at its E_min (None: the
// recovery comes from a replay)
static Kept kept_state(const xzzx_group &g, const GroupWs &w)
{
    const Plan &P = g.plan->P;
    if (!w.min_snap) return Kept::None;
    if (w.grid) return Kept::Grid;
    if (P.order == XZZX_ORDER_RANDOM_SITE) return w.lean ? Kept::SiteOrder : Kept::Site;
    if (ladder_rows_d(g, w.lean)) return Kept::RotatedRows;
    if (P.ladder_k && !ladder_planar_d(g)) return Kept::Packed;
    return min_snap_words(g, w.lean) ? Kept::PlanarRows : Kept::None;
}

// Annealing of every non-empty group.  Packed-row groups share one persistent
// launch; byte-state groups are launched per lanes-per-chain value.  The
// replay re-runs one chain per syndrome with the byte-state kernel, spreading
// a chain over more lanes when that is needed to give every CU several
// wavefronts.  Each launch has its own queue counter: launch i of an annealing
// stage d_counters[i]; a replay (with its own d_counters base) uses [0] and [2].
constexpr int kReplayCounters = 16;   // words before the replay's counters
static int launch_anneal(const xzzx_group *groups, const GroupWs *ws, int n_groups, AnnealMode mode,
                         uint64_t seed, int64_t unit_offset, int64_t units_override, uint32_t *d_counters,
                         hipStream_t stream, bool serial = false)
{
    std::vector<int> rows_sel;
    std::vector<int> bytes_sel[7];
    std::vector<int> static_sel[2][kStaticMaxD + 1];   // [tasks span syndromes][d]
    std::vector<int> replay_cp;   // replays starting from checkpoints: one chain per wavefront
    std::vector<int> site_sel[2][2];   // random-site plans, by site_wide and form: one chain per lane
    std::vector<int> planar_sel[kPlanarStaticMaxD + 1];   // planar kernels specialised to d
    std::vector<int> grid_sel[5][4];   // grid core, by lanes per chain (4..64) and moves per lane (1, 2, 4, 8)
    std::vector<int> ladder_sel;  // replica exchange: one chain per lane
    std::vector<int> ladder_rows_sel[2][kLadderRowsMaxD + 1];   // ... on the rotated kernels specialised to d
    std::vector<int> ladder_planar_sel[kPlanarStaticMaxD + 1];  // ... on the planar kernels specialised to d
    int64_t total_syn = 0;
    for (int i = 0; i < n_groups; ++i) {
        if (groups[i].n_syn <= 0) continue;
        const Plan &P = groups[i].plan->P;
        if (ws[i].grid && mode != AnnealMode::Replay) {
            grid_sel[log2_int(ws[i].grid) - 2][log2_int(P.grid_moves(ws[i].grid))].push_back(i);
            continue;
        }
        if (ws[i].grid || P.order == XZZX_ORDER_RANDOM_SITE || P.ladder_k ||
            (mode == AnnealMode::Replay && min_snap_words(groups[i], ws[i].lean))) {
            if (mode == AnnealMode::Replay) continue;   // these kept their states
            if (const int ld = ladder_rows_d(groups[i], ws[i].lean)) ladder_rows_sel[spans(groups[i])][ld].push_back(i);
            else if (ladder_planar_d(groups[i])) ladder_planar_sel[ladder_planar_d(groups[i])].push_back(i);
            else (P.ladder_k ? ladder_sel : site_sel[P.site_wide][ws[i].lean]).push_back(i);
            continue;
        }
        total_syn += groups[i].n_syn;
        if (mode != AnnealMode::Replay && P.use_rows && P.planar_d) planar_sel[P.planar_d].push_back(i);
        else if (mode != AnnealMode::Replay && uses_static(groups[i])) static_sel[spans(groups[i])][P.static_d].push_back(i);
        else if (mode == AnnealMode::Replay && ws[i].cp_rows) replay_cp.push_back(i);
        else if (mode != AnnealMode::Replay && P.use_rows && P.row_words) rows_sel.push_back(i);
        else bytes_sel[log2_int(P.lanes)].push_back(i);
    }
    if (mode == AnnealMode::Replay) {
        // one chain per syndrome: enough wavefronts for 8 per CU
        std::vector<int> all;
        int C = kWave;
        for (int l = 0; l < 7; ++l)
            for (int i : bytes_sel[l]) {
                all.push_back(i);
                C = std::min(C, kWave / groups[i].plan->P.lanes);
            }
        const int64_t want = 8LL * device_cus();
        while (C > 1 && total_syn / C < want) C >>= 1;
        int rc = launch_set(groups, ws, all, false, kWave / C, mode, seed, unit_offset, units_override, d_counters,
                            stream);
        if (!rc)
            rc = launch_set(groups, ws, replay_cp, false, kWave, mode, seed, unit_offset, units_override,
                            d_counters + 2, stream);
        return rc;
    }
    // the launches of one call (one per kernel family and distance) run
    // concurrently: each alone may not fill the device (a mixed-distance batch
    // with a few hundred syndromes per distance)
    struct Set {
        const std::vector<int> *sel;
        bool rows;
        int lanes;
        int static_d;
        bool site;
        int planar_d;
        bool ladder;
        int grid_mv;
    };
    std::vector<Set> sets;
    if (!rows_sel.empty()) sets.push_back({&rows_sel, true, 1, 0, false, 0, false, 0});
    for (auto &wide : site_sel)
        for (auto &sel : wide)
            if (!sel.empty()) sets.push_back({&sel, false, 1, 0, true, 0, false, 0});
    if (!ladder_sel.empty()) sets.push_back({&ladder_sel, false, 1, 0, false, 0, true, 0});
    for (int d = 3; d <= kPlanarStaticMaxD; d += 2)
        if (!planar_sel[d].empty()) sets.push_back({&planar_sel[d], true, 1, 0, false, d, false, 0});
    for (auto &sel : ladder_rows_sel)
        for (int d = 3; d <= kLadderRowsMaxD; d += 2)
            if (!sel[d].empty()) sets.push_back({&sel[d], true, 1, d, false, 0, true, 0});
    for (int d = 3; d <= kPlanarStaticMaxD; d += 2)
        if (!ladder_planar_sel[d].empty()) sets.push_back({&ladder_planar_sel[d], true, 1, 0, false, d, true, 0});
    for (auto &sel : static_sel)
        for (int d = kStaticMinD; d <= kStaticMaxD; d += 2)
            if (!sel[d].empty()) sets.push_back({&sel[d], true, 1, d, false, 0, false, 0});
    for (int l = 0; l < 7; ++l)
        if (!bytes_sel[l].empty()) sets.push_back({&bytes_sel[l], false, 1 << l, 0, false, 0, false, 0});
    for (int l = 0; l < 5; ++l)
        for (int m = 0; m < 4; ++m)
            if (!grid_sel[l][m].empty()) sets.push_back({&grid_sel[l][m], false, 4 << l, 0, false, 0, false, 1 << m});
    // the sets whose tasks take longest first: with more sets than queues the
    // last ones start when earlier ones have ended, and the longest tasks
    // must not be among them (256 syndromes of 256 chains each at d = 5..21, 1000
    // sweeps: 42.1 ms in ascending order, 31.4 so; d = 19, 25, 31: 29.2 and 27.5)
    auto task_work = [&](const Set &S) {
        double w = 0;
        for (int i : *S.sel) w = std::max(w, (double)groups[i].plan->P.n_sweeps * groups[i].plan->P.lat.nstab / S.lanes);
        return w;
    };
    std::stable_sort(sets.begin(), sets.end(), [&](const Set &a, const Set &b) { return task_work(a) > task_work(b); });
    // Wavefronts of the sets whose tasks take longer go first on their SIMDs (see
    // wave_priority).  Which sets share a SIMD with which is the dispatcher's, and
    // without this one call in three had some of the longest chains wait for
    // others' (d = 5..21, 5000 sweeps: 150 to 165 ms a call, so 150 to 152).  A call of
    // one set, and serving, leave the priority alone: others share the device.
    const int most_priority = std::min<int>((int)sets.size() - 1, 3);
    // each set holds at least one group, so at most kMaxGroups of them
    static_assert(kMaxGroups <= kReplayCounters, "queue counters of the sets");
    auto one = [&](int i, hipStream_t s) {
        const Set &S = sets[i];
        return launch_set(groups, ws, *S.sel, S.rows, S.lanes, mode, seed, unit_offset, units_override, d_counters + i,
                          s, S.static_d, S.site, S.planar_d, S.ladder, S.grid_mv, std::max(0, most_priority - i));
    };
    if (sets.size() <= 1 || mode == AnnealMode::Plain) {
        int rc = XZZX_OK;
        for (int i = 0; i < (int)sets.size() && !rc; ++i) rc = one(i, stream);
        return rc;
    }
    return fork_join(stream, (int)sets.size(), one, serial);
}

// reductions of the groups, and recoveries of those whose kernels kept states
static int launch_finish(const xzzx_group *groups, const GroupWs *ws, int n_groups, hipStream_t stream)
{
    FinishArgs A{};
    auto flush = [&]() -> int {
        if (A.n_waves == 0) return XZZX_OK;
        hipLaunchKernelGGL(k_finish, dim3((unsigned)((A.n_waves + kFinishWaves - 1) / kFinishWaves)),
                           dim3(kFinishWaves * kWave), 0, stream, A);
        A.n_groups = 0;
        A.n_waves = 0;
        return check_hip(hipGetLastError(), "k_finish launch");
    };
    for (int i = 0; i < n_groups; ++i) {
        const xzzx_group &g = groups[i];
        const Plan &P = g.plan->P;
        if (g.n_syn <= 0) continue;
        if (g.n_syn * kWave > kMaxLaunchItems) { set_error("too many syndromes in one group for one launch"); return XZZX_ERANGE; }
        const Kept kept = kept_state(g, ws[i]);
        if (kept != Kept::None && (g.n_syn * (int64_t)P.lat.nq + 255) / 256 * 256 > kMaxLaunchItems) {
            set_error("too many recovery bytes in one group");
            return XZZX_ERANGE;
        }
        if (A.n_waves + g.n_syn > kMaxLaunchWaves - kFinishWaves) {
            const int rc = flush();
            if (rc) return rc;
        }
        FinishGroup &G = A.g[A.n_groups++];
        G.plan = P.ddev;
        G.qcls = ws[i].qcls;
        G.refs = ws[i].refs;
        G.emin = ws[i].emin;
        G.snap = ws[i].min_snap;
        G.e_best = g.d_e_best;
        G.cls = g.d_cls;
        G.best_chain = ws[i].best_chain;
        G.e_cls = g.d_e_cls;
        G.paper_recovery = g.d_paper_recovery;
        G.recovery = g.d_recovery;
        G.n_syn = g.n_syn;
        G.wave_begin = A.n_waves;
        G.n_rep = g.n_rep;
        G.kept = kept;
        G.words = kept == Kept::Grid ? P.hdev.grid_words : (int)min_snap_words(g, ws[i].lean);
        G.d = kept == Kept::RotatedRows ? ladder_rows_d(g, ws[i].lean) : 0;
        G.row_words = G.d ? (2 * (G.d + 1) <= 32 ? 1 : 2) : P.row_words;
        A.n_waves += g.n_syn;
    }
    return flush();
}

// The reference stage of the anneal-only entry point: the class of every
// caller reference relative to replica 0 (Alg. 7, Eqs. (35)-(36)), and, for
// groups that pass their syndromes, the check that every reference has
// syndrome S.  The check reads a flag back, so it synchronizes `stream` and
// is refused while `stream` is being captured.
static int check_references(const xzzx_group *groups, const GroupWs *ws, int n_groups, uint32_t *d_flag,
                            hipStream_t stream)
{
    bool any_syn = false;
    for (int i = 0; i < n_groups; ++i) any_syn |= groups[i].n_syn > 0 && groups[i].d_syn;
    if (any_syn) {
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        int rc = check_hip(hipStreamIsCapturing(stream, &st), "hipStreamIsCapturing");
        if (rc) return rc;
        if (st != hipStreamCaptureStatusNone) {
            set_error("checking references against d_syn synchronizes the stream: not allowed under capture");
            return XZZX_EINVAL;
        }
        hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, d_flag, 1);
        rc = check_hip(hipGetLastError(), "flag clear launch");
        if (rc) return rc;
    }
    for (int i = 0; i < n_groups; ++i) {
        const xzzx_group &g = groups[i];
        if (g.n_syn <= 0) continue;
        const int64_t blocks = g.n_syn * g.n_rep;
        for (int64_t b0 = 0; b0 < blocks; b0 += kMaxLaunchWaves) {
            const int64_t nb = std::min<int64_t>(kMaxLaunchWaves, blocks - b0);
            hipLaunchKernelGGL(k_ref_check, dim3((unsigned)nb), dim3(kWave), 0, stream, g.plan->P.ddev, ws[i].refs,
                               g.d_syn, g.n_rep, b0, ws[i].qraw, d_flag);
            const int rc = check_hip(hipGetLastError(), "k_ref_check launch");
            if (rc) return rc;
        }
        const int rc = launch_qcls(ws[i].qraw, g.n_syn, g.n_rep, ws[i].qcls, stream);
        if (rc) return rc;
    }
    if (!any_syn) return XZZX_OK;
    uint32_t bad = 0;
    int rc = check_hip(hipMemcpyAsync(&bad, d_flag, sizeof(bad), hipMemcpyDeviceToHost, stream), "flag read");
    if (!rc) rc = check_hip(hipStreamSynchronize(stream), "hipStreamSynchronize");
    if (rc) return rc;
    if (bad) { set_error("a reference's syndrome differs from the group's syndrome S"); return XZZX_EINVAL; }
    return XZZX_OK;
}

// serial: every launch on `stream`, in order, with no side streams or events
static int run_decode(const xzzx_group *groups, int n_groups, uint64_t greedy_seed, uint64_t anneal_seed,
                      int greedy_mode, int flags, void *d_workspace, size_t workspace_bytes,
                      hipStream_t stream, bool decode, bool serial = false)
{
    int rc = validate_groups(groups, n_groups, decode);
    if (rc) return rc;
    if (decode && greedy_mode != XZZX_GREEDY_RANDOM && greedy_mode != XZZX_GREEDY_SAME &&
        greedy_mode != XZZX_GREEDY_BOUNDARY) {
        set_error("unknown greedy mode");
        return XZZX_EINVAL;
    }
    const CallForm form = call_form(groups, n_groups, decode, workspace_bytes);
    if (!d_workspace || workspace_bytes < form.least) { set_error("workspace too small"); return XZZX_ENOMEM; }
    uint32_t *counter = static_cast<uint32_t *>(d_workspace);
    const std::vector<GroupWs> ws = carve(groups, n_groups, decode, form, static_cast<uint8_t *>(d_workspace) + 256);
    const int stage_bits = XZZX_FLAG_STAGE_GREEDY | XZZX_FLAG_STAGE_ANNEAL | XZZX_FLAG_STAGE_FINISH;
    const int stages = (flags & stage_bits) ? (flags & stage_bits) : stage_bits;
    // the groups' greedy launches run concurrently (one group's launch alone
    // leaves the device idle in its tail)
    std::vector<int> gsel;
    for (int i = 0; i < n_groups; ++i)
        if (decode && groups[i].n_syn > 0 && (stages & XZZX_FLAG_STAGE_GREEDY)) gsel.push_back(i);
    // (largest lattices first, as the annealing sets)
    std::stable_sort(gsel.begin(), gsel.end(), [&](int a, int b) {
        return groups[a].plan->P.lat.nstab > groups[b].plan->P.lat.nstab;
    });
    rc = fork_join(stream, (int)gsel.size(), [&](int k, hipStream_t s) {
        const int i = gsel[k];
        const xzzx_group &g = groups[i];
        int r = launch_greedy(g.plan->P, g.d_syn, g.d_uid, g.n_syn, g.n_rep, greedy_seed, greedy_mode, ws[i].refs,
                              ws[i].qraw, s);
        if (!r) r = launch_qcls(ws[i].qraw, g.n_syn, g.n_rep, ws[i].qcls, s);
        return r;
    }, serial);
    if (rc) return rc;
    if (!decode && (stages & XZZX_FLAG_STAGE_GREEDY)) {
        rc = check_references(groups, ws.data(), n_groups, counter + 63, stream);
        if (rc) return rc;
    }
    if (!(stages & XZZX_FLAG_STAGE_ANNEAL)) {
        // annealing skipped in this call
    } else if (flags & XZZX_FLAG_PLAIN) {
        // one launch per syndrome, grid = its own tasks, no persistence
        for (int i = 0; i < n_groups; ++i) {
            const xzzx_group &g = groups[i];
            for (int64_t s = 0; s < g.n_syn; ++s) {
                rc = launch_anneal(&g, &ws[i], 1, AnnealMode::Plain, anneal_seed, s * 4 * g.n_rep, 4 * g.n_rep, counter,
                                   stream);
                if (rc) return rc;
            }
        }
    } else {
        rc = launch_anneal(groups, ws.data(), n_groups, AnnealMode::Persistent, anneal_seed, 0, -1, counter, stream,
                           serial);
        if (rc) return rc;
    }
    if (!(stages & XZZX_FLAG_STAGE_FINISH)) return XZZX_OK;
    rc = launch_finish(groups, ws.data(), n_groups, stream);
    if (rc) return rc;
    return launch_anneal(groups, ws.data(), n_groups, AnnealMode::Replay, anneal_seed, 0, -1, counter + kReplayCounters,
                         stream, serial);
}


// ---- serving launches (used by xzzx_server.cpp) ----
int serve_greedy(const Plan &P, const uint8_t *d_syn, int64_t syn_stride, const uint32_t *d_uid,
                 const int32_t *d_slot_map, int n, int n_rep, uint8_t *refs_base, int64_t refs_stride,
                 uint8_t *qraw_base, int64_t qraw_stride, uint64_t seed, int mode, hipStream_t stream)
{
    if (n <= 0) return XZZX_OK;
    GreedyArgs A{};
    A.syn = d_syn;
    A.syn_stride = syn_stride;
    A.uid = d_uid;
    A.refs = refs_base;
    A.qraw = qraw_base;
    A.slot_map = d_slot_map;
    A.refs_stride = refs_stride;
    A.qraw_stride = qraw_stride;
    A.n_rep = n_rep;
    A.rep_div = 1;
    return launch_greedy(P, A, n, seed, mode, stream);
}

int serve_slice(const ServeLaunch *launches, int n_launches, uint64_t seed, hipStream_t stream)
{
    const uint32_t lo = (uint32_t)seed, hi = (uint32_t)(seed >> 32);
    // the launches' tasks are consecutive: stash the start states of them all
    int n_tasks = 0;
    for (int i = 0; i < n_launches; ++i) n_tasks += launches[i].n;
    bool stash = false;
    for (int i = 0; i < n_launches; ++i) stash |= launches[i].n > 0 && launches[i].kind != 3;
    if (stash) {
        hipLaunchKernelGGL(k_serve_stash, dim3((unsigned)n_tasks), dim3(256), 0, stream, launches[0].tasks);
        const int rc = check_hip(hipGetLastError(), "serving stash launch");
        if (rc) return rc;
    }
    auto one = [&](int i, hipStream_t s) -> int {
        const ServeLaunch &L = launches[i];
        if (L.n <= 0) return XZZX_OK;
        if (L.kind == 0) {
            hipLaunchKernelGGL(k_serve_rows, dim3((unsigned)L.n), dim3(kWave), L.lds, s, L.tasks, lo, hi);
        } else if (L.kind == 1) {
            hipLaunchKernelGGL(k_serve_bytes, dim3((unsigned)L.n), dim3(kWave), L.lds, s, L.tasks, lo, hi);
        } else if (L.kind == 3) {
            hipLaunchKernelGGL(serve_grid_kernel(L.d), dim3((unsigned)L.n), dim3(kWave), L.lds, s, L.tasks, lo, hi);
        } else {
            const ServeKernel k = static_serve_kernel(L.d);
            if (!k) { set_error("no specialised serving kernel for this distance"); return XZZX_EINVAL; }
            hipLaunchKernelGGL(k, dim3((unsigned)L.n), dim3(kWave), 0, s, L.tasks, lo, hi);
        }
        return check_hip(hipGetLastError(), "serving slice launch");
    };
    // the kernels of one slice (one per family and distance) run concurrently
    if (n_launches <= 1) return n_launches ? one(0, stream) : XZZX_OK;
    return fork_join(stream, n_launches, one);
}

int run_concurrently(hipStream_t stream, int n, const std::function<int(int, hipStream_t)> &launch)
{
    if (n <= 1) return n ? launch(0, stream) : XZZX_OK;
    return fork_join(stream, n, launch);
}

int serve_finish(const ServeFinish *d_fin, const ServeTask *d_replay, int n, size_t lds_replay, uint64_t seed,
                 hipStream_t stream)
{
    if (n <= 0) return XZZX_OK;
    hipLaunchKernelGGL(k_serve_reduce, dim3((unsigned)n), dim3(kWave), 0, stream, d_fin);
    hipLaunchKernelGGL(k_serve_replay, dim3((unsigned)n), dim3(kWave), lds_replay, stream, d_replay,
                       (uint32_t)seed, (uint32_t)(seed >> 32));
    hipLaunchKernelGGL(k_serve_gather, dim3((unsigned)n), dim3(kWave), 0, stream, d_fin);
    return check_hip(hipGetLastError(), "serving finish launch");
}

}  // namespace xzzx

using namespace xzzx;

extern "C" {

int xzzx_syndrome(const xzzx_plan *plan, const uint8_t *d_cfg, int64_t n, uint8_t *d_syn, void *stream)
{
    if (!plan || n < 0 || (n > 0 && (!d_cfg || !d_syn))) { set_error("bad syndrome arguments"); return XZZX_EINVAL; }
    if (n == 0) return XZZX_OK;
    const int64_t total = n * plan->P.lat.nstab;
    const int64_t items = (total + 255) / 256 * 256;
    if (items > kMaxLaunchItems) { set_error("batch too large for one launch (2^32 work-items)"); return XZZX_ERANGE; }
    // tiles of 64 configurations where they fit a quarter of the LDS and give
    // every CU several workgroups; else of 16 (a small batch spreads over more
    // CUs, a large lattice keeps several workgroups per CU)
    const int rows = syndrome_rows(plan->P.lat.nq);
    const int lg4 = rows * 17 * 4 <= 40960 && n >= 64 * 1024 ? 4 : 2;
    const int64_t per = (int64_t)4 << lg4, blocks = (n + per - 1) / per;
    const bool wide = blocks <= device_cus() && (rows / 4 << lg4) > kSynThreadsMost;
    hipLaunchKernelGGL(wide ? k_syndrome<kSynThreadsMost> : k_syndrome<kSynThreads>, dim3((unsigned)blocks),
                       dim3(wide ? kSynThreadsMost : kSynThreads), rows * ((1 << lg4) + 1) * 4, (hipStream_t)stream,
                       plan->P.ddev, d_cfg, n, lg4, d_syn);
    return check_hip(hipGetLastError(), "k_syndrome launch");
}

int xzzx_greedy_init(const xzzx_plan *plan, const uint8_t *d_syn, const uint32_t *d_uid, int64_t n_syn,
                     int n_rep, uint64_t greedy_seed, int mode, uint8_t *d_refs, uint8_t *d_qcls, void *stream)
{
    if (!plan || n_syn < 0 || n_rep < 1) { set_error("bad greedy arguments"); return XZZX_EINVAL; }
    if (mode != XZZX_GREEDY_RANDOM && mode != XZZX_GREEDY_SAME && mode != XZZX_GREEDY_BOUNDARY) {
        set_error("unknown greedy mode");
        return XZZX_EINVAL;
    }
    if (n_syn == 0) return XZZX_OK;
    if (!d_syn || !d_uid || !d_refs || !d_qcls) { set_error("NULL buffer"); return XZZX_EINVAL; }
    // the raw symplectic bits land in d_qcls and are turned into classes in place
    int rc = launch_greedy(plan->P, d_syn, d_uid, n_syn, n_rep, greedy_seed, mode, d_refs, d_qcls, (hipStream_t)stream);
    if (rc) return rc;
    return launch_qcls(d_qcls, n_syn, n_rep, d_qcls, (hipStream_t)stream);
}

static int workspace_query(const xzzx_group *groups, int n_groups, size_t *bytes, bool least)
{
    if (!groups || !bytes || n_groups < 1 || n_groups > kMaxGroups) { set_error("bad arguments"); return XZZX_EINVAL; }
    for (int i = 0; i < n_groups; ++i)
        if (!groups[i].plan) { set_error("group without plan"); return XZZX_EINVAL; }
    const CallForm F = call_form(groups, n_groups, true, SIZE_MAX);
    *bytes = least ? F.least : F.bytes;
    return XZZX_OK;
}

int xzzx_decode_workspace(const xzzx_group *groups, int n_groups, size_t *bytes)
{
    return workspace_query(groups, n_groups, bytes, false);
}

int xzzx_decode_workspace_least(const xzzx_group *groups, int n_groups, size_t *bytes)
{
    return workspace_query(groups, n_groups, bytes, true);
}

int xzzx_decode_routes(const xzzx_group *groups, int n_groups, size_t workspace_bytes, int32_t *kernel, int32_t *lanes)
{
    const CallForm form = call_form(groups, n_groups, true, workspace_bytes);
    if (workspace_bytes < form.least) { set_error("workspace too small"); return XZZX_ENOMEM; }
    for (int i = 0; i < n_groups; ++i) {
        const Plan &P = groups[i].plan->P;
        const int on_grid = form.grid[i];
        lanes[i] = 1;
        if (P.order == XZZX_ORDER_RANDOM_SITE) kernel[i] = XZZX_KERNEL_SITE;
        else if (P.ladder_k) kernel[i] = XZZX_KERNEL_LADDER;
        else if (on_grid) kernel[i] = kRouteGrid;
        else if (P.use_rows) kernel[i] = P.planar_d || P.static_d ? XZZX_KERNEL_ROWS : XZZX_KERNEL_ROWS_GENERIC;
        else kernel[i] = XZZX_KERNEL_BYTES;
        if (kernel[i] == kRouteGrid) lanes[i] = on_grid;
        if (kernel[i] == XZZX_KERNEL_BYTES) lanes[i] = P.lanes;
    }
    return XZZX_OK;
}

int xzzx_decode(const xzzx_group *groups, int n_groups, uint64_t greedy_seed, uint64_t anneal_seed,
                int greedy_mode, int flags, void *d_workspace, size_t workspace_bytes, void *stream)
{
    return run_decode(groups, n_groups, greedy_seed, anneal_seed, greedy_mode, flags, d_workspace, workspace_bytes,
                      (hipStream_t)stream, true);
}

int xzzx_anneal(const xzzx_group *groups, int n_groups, uint64_t anneal_seed, int flags, void *d_workspace,
                size_t workspace_bytes, void *stream)
{
    return run_decode(groups, n_groups, 0, anneal_seed, XZZX_GREEDY_RANDOM, flags, d_workspace, workspace_bytes,
                      (hipStream_t)stream, false);
}

}  // extern "C"

// ---- decode without allocation ----
// The workspace of xzzx_decode_noalloc: one array per device, resident from
// the library's load on that device until the process ends.  Host code never
// passes the array's name to a kernel (in host code it is only a stand-in for
// the symbol): it uses the device address that hipGetSymbolAddress returns,
// looked up once per device.
static __device__ __align__(256) uint8_t scratch[XZZX_NOALLOC_SCRATCH_BYTES];

static int scratch_address(void **out)
{
    static std::mutex mu;
    static void *addr[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { set_error("hipGetDevice failed"); return XZZX_EDEVICE; }
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        const int rc = check_hip(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress");
        if (rc) return rc;
        if (!p) { set_error("hipGetSymbolAddress returned NULL"); return XZZX_EDEVICE; }
        addr[dev] = p;
    }
    *out = addr[dev];
    return XZZX_OK;
}

extern "C" {

int xzzx_decode_noalloc(const xzzx_group *groups, int n_groups, uint64_t greedy_seed, uint64_t anneal_seed,
                        int greedy_mode, int flags, void *stream)
{
    size_t need = 0;
    int rc = xzzx_decode_workspace_least(groups, n_groups, &need);
    if (rc) return rc;
    if (need > (size_t)XZZX_NOALLOC_SCRATCH_BYTES) {
        set_error("workspace of these groups exceeds XZZX_NOALLOC_SCRATCH_BYTES");
        return XZZX_ERANGE;
    }
    void *ws = nullptr;
    rc = scratch_address(&ws);
    if (rc) return rc;
    return run_decode(groups, n_groups, greedy_seed, anneal_seed, greedy_mode, flags, ws,
                      (size_t)XZZX_NOALLOC_SCRATCH_BYTES, (hipStream_t)stream, true, true);
}

}  // extern "C"

struct xzzx_graph {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

extern "C" {

int xzzx_graph_create(const xzzx_group *groups, int n_groups, uint64_t greedy_seed, uint64_t anneal_seed,
                      int greedy_mode, int flags, void *d_workspace, size_t workspace_bytes, void *stream,
                      xzzx_graph **out)
{
    if (!out) { set_error("out is NULL"); return XZZX_EINVAL; }
    *out = nullptr;
    if (!stream) { set_error("graph capture needs a non-null stream"); return XZZX_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    // the stream's side streams and events exist before the capture begins
    SideSet *side = nullptr;
    int rc = side_set(s, &side);
    if (rc) return rc;
    rc = check_hip(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
    if (rc) return rc;
    const int drc = run_decode(groups, n_groups, greedy_seed, anneal_seed, greedy_mode, flags, d_workspace,
                               workspace_bytes, s, true);
    hipGraph_t g = nullptr;
    rc = check_hip(hipStreamEndCapture(s, &g), "hipStreamEndCapture");
    if (drc) {
        if (g) (void)hipGraphDestroy(g);
        return drc;
    }
    if (rc) return rc;
    auto *h = new xzzx_graph();
    h->graph = g;
    rc = check_hip(hipGraphInstantiate(&h->exec, g, nullptr, nullptr, 0), "hipGraphInstantiate");
    if (rc) {
        (void)hipGraphDestroy(g);
        delete h;
        return rc;
    }
    *out = h;
    return XZZX_OK;
}

int xzzx_graph_launch(xzzx_graph *graph, void *stream)
{
    if (!graph || !graph->exec) { set_error("graph is NULL"); return XZZX_EINVAL; }
    return check_hip(hipGraphLaunch(graph->exec, (hipStream_t)stream), "hipGraphLaunch");
}

void xzzx_graph_destroy(xzzx_graph *graph)
{
    if (!graph) return;
    if (graph->exec) (void)hipGraphExecDestroy(graph->exec);
    if (graph->graph) (void)hipGraphDestroy(graph->graph);
    delete graph;
}

}  // extern "C"
