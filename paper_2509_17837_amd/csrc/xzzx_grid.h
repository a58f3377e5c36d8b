// Grid core: one chain over 2^LOGG lanes of a wavefront, for launches with too
// few chains to give every lane one of its own (one syndrome awaited, a few
// requests being served).  Same chains as the other cores, bit for bit.
//
// What bounds it: a wavefront alone on its SIMD issues an instruction in about
// eight cycles, whatever the others wait for, so a sweep takes as long as its
// instructions are many; then a serial chain of LDS round trips, four per sweep
// and class (read the qubits, look the move up, store).  So the form is chosen for
// the shortest chain rather than the least work:
// - the lattice is a grid of bytes in LDS, code << 3 per qubit, every absent
//   cell 0; a generator is a 2 x 2 block of it, so a move reads two adjacent
//   bytes of two rows into one register, which one dot product turns into
//   the LDS address of its (dE, threshold) entry: two dependent LDS reads a
//   phase instead of four (descriptor, qubits, rank, entry);
// - each lane keeps its moves (block address, entry table, flip mask) of all
//   four classes in registers;
// - a Philox block serves four generators: lanes with one move (MV = 1) draw
//   the block of one class each and exchange words inside the quad, lanes
//   with two (MV = 2) likewise in pairs, so no block is drawn twice;
// - energies are summed over the chain's lanes once a sweep for its four
//   phases together.  In a sweep that finds a new least energy -- few do --
//   the phases after it are undone in LDS, the state is written out as the
//   chain's recovery, and they are redone; so no replay follows.
// Measured (rotated d = 11, 64 chains): 0.61 us a sweep on 32 or 64 lanes, where
// one chain per lane takes 7.3 us; with the device full, 4 x 10^5 chains and
// more, 1.1 x 10^12 attempts/s on 32 lanes, half the packed-row kernel's rate.
// 145 VALU and 34 LDS instructions a wavefront and sweep: 179 x 8 cycles are the
// 0.61 us.
#pragma once

#include "xzzx_device.h"

namespace xzzx {

// Draws of one lane: round 0's and 1's products that do not depend on the
// sweep (uid and the block are fixed) are taken once.
struct GridDraw {
    uint32_t uid_lo;         // low word of M0 * uid
    uint64_t p1;             // M1 * (round-0 output z of the lane's block)
};

__device__ __forceinline__ GridDraw grid_draw(uint32_t uid, uint32_t b, uint32_t k1)
{
    const uint64_t p = (uint64_t)uid * kPhM0;
    return GridDraw{(uint32_t)p, (uint64_t)((uint32_t)(p >> 32) ^ b ^ k1) * kPhM1};
}

// Philox4x32-10 of the counter (uid, cc, c2, block): rounds 0 and 1, then
// rounds 2..9 one by one (the core places them between its LDS accesses).
__device__ __forceinline__ uint4 grid_philox_head(const GridDraw &g, uint32_t cc, uint32_t c2, uint32_t k0, uint32_t k1)
{
    const uint64_t p = (uint64_t)c2 * kPhM1;                                   // round 0
    const uint64_t q = (uint64_t)((uint32_t)(p >> 32) ^ cc ^ k0) * kPhM0;      // round 1
    return make_uint4((uint32_t)(g.p1 >> 32) ^ (uint32_t)p ^ (k0 + kPhW0), (uint32_t)g.p1,
                      (uint32_t)(q >> 32) ^ g.uid_lo ^ (k1 + kPhW1), (uint32_t)q);
}
__device__ __forceinline__ uint4 grid_philox_round(const uint4 &c, int i, uint32_t k0, uint32_t k1)
{
    const uint64_t q0 = (uint64_t)c.x * kPhM0, q1 = (uint64_t)c.z * kPhM1;
    return make_uint4(xor3_key((uint32_t)(q1 >> 32), c.y, k0 + (uint32_t)i * kPhW0), (uint32_t)q1,
                      xor3_key((uint32_t)(q0 >> 32), c.w, k1 + (uint32_t)i * kPhW1), (uint32_t)q0);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;   // quad_perm [1,0,3,2] and [2,3,0,1]
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128; // rotations of a row of 16 lanes

// lanes with `odd` keep b, the others a; each gets its partner's other value
template <int CTRL>
__device__ __forceinline__ void dpp_exchange(uint32_t &a, uint32_t &b, bool odd)
{
    const uint32_t pa = dpp<CTRL>(a), pb = dpp<CTRL>(b);
    a = odd ? pb : a;
    b = odd ? b : pa;
}

// Energies after the four classes of a sweep, in every lane of the chain: E
// plus the running sums of the lanes' changes.  Chains of 16 and more lanes
// sum the four classes side by side, lane j of a quad class j (two folds),
// then over the quads; smaller chains one class after another.
template <int LOGG>
__device__ __forceinline__ void grid_energies(int32_t E, const int32_t (&de)[4], int32_t (&out)[4], int gl)
{
    if constexpr (LOGG >= 4) {
        const bool o1 = gl & 1, o2 = gl & 2;
        const uint32_t a = o1 ? de[1] : de[0], ax = o1 ? de[0] : de[1];
        const uint32_t b = o1 ? de[3] : de[2], bx = o1 ? de[2] : de[3];
        const uint32_t s = a + dpp<kDppXor1>(ax), r = b + dpp<kDppXor1>(bx);
        uint32_t v = (o2 ? r : s) + dpp<kDppXor2>(o2 ? s : r);
        v += dpp<kDppRor4>(v);
        v += dpp<kDppRor8>(v);
        if constexpr (LOGG >= 5) {
            const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
            v = p[0] + p[1];
        }
        if constexpr (LOGG >= 6) {
            const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
            v = p[0] + p[1];
        }
        out[0] = E + (int32_t)dpp<0x00>(v);
        out[1] = out[0] + (int32_t)dpp<0x55>(v);
        out[2] = out[1] + (int32_t)dpp<0xAA>(v);
        out[3] = out[2] + (int32_t)dpp<0xFF>(v);
    } else {
        for (int k = 0; k < 4; ++k) {
            E += chain_sum<LOGG>(de[k]);
            out[k] = E;
        }
    }
}

// LDS by byte address.
typedef __attribute__((address_space(3))) uint8_t lds_u8;
__device__ __forceinline__ uint32_t lds_addr(const uint8_t *p) { return (uint32_t)(uintptr_t)(const lds_u8 *)p; }
__device__ __forceinline__ uint32_t lds_read16(uint32_t a)
{
    return *(const __attribute__((address_space(3))) uint16_t *)(uintptr_t)a;
}
__device__ __forceinline__ uint32_t lds_read8(uint32_t a) { return *(const lds_u8 *)(uintptr_t)a; }
__device__ __forceinline__ void lds_write8(uint32_t a, uint32_t v) { *(lds_u8 *)(uintptr_t)a = (uint8_t)v; }
__device__ __forceinline__ void lds_write16(uint32_t a, uint32_t v)
{
    *(__attribute__((address_space(3))) uint16_t *)(uintptr_t)a = (uint16_t)v;
}
__device__ __forceinline__ uint2 lds_read64(uint32_t a)
{
    const uint64_t v = *(const __attribute__((address_space(3))) uint64_t *)(uintptr_t)a;
    return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ void lds_write32(uint32_t a, uint32_t v)
{
    *(__attribute__((address_space(3))) uint32_t *)(uintptr_t)a = v;
}
// Memory order of this wavefront's LDS accesses only (LDS takes them in the
// order issued); unlike wave_lds_fence it does not hold back the scheduler,
// which has the next draws to place between the accesses.
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// LDS of a workgroup: the (dE, threshold) entries and one spare, then the
// grids of its chains.
__device__ __forceinline__ uint32_t grid_state_off(const PlanDev *pl)
{
    return (8u * ((uint32_t)pl->grid_slots + 1u) + 15u) & ~15u;
}

__device__ inline void load_grid_tables(const PlanDev *pl, uint8_t *smem)
{
    uint2 *et = reinterpret_cast<uint2 *>(smem);
    for (int i = threadIdx.x; i < pl->grid_slots + 1; i += kWave) et[i] = make_uint2(0u, 0u);
    wave_lds_fence();
    for (int i = threadIdx.x; i < pl->grid_entries; i += kWave) {
        const uint32_t e = pl->grid_entry[i];
        et[e & 0xFFFFu].x = (uint32_t)pl->dE[e >> 16];
    }
    wave_lds_fence();
}

// Rank of move m of lane gl, and of its Philox block, among the 2^LOGG lanes.
template <int LOGG, int MV>
__device__ __forceinline__ int grid_rank(int gl, int m)
{
    if constexpr (MV == 8) return 4 * (gl + (m >> 2 << LOGG)) + (m & 3);
    return MV * gl + m;
}

template <int LOGG, int MV>
__device__ __forceinline__ void grid_core(const PlanDev *pl, const ChainJob &J, int t_begin, int t_end,
                                          uint32_t seed_lo, uint32_t seed_hi, uint8_t *smem, uint32_t *snap)
{
    constexpr int G = 1 << LOGG;
    constexpr int kThr = kGridMaxRising / kWave;
    const int lane = threadIdx.x;
    const int c = lane >> LOGG, gl = lane & (G - 1);
    const int nq = (int)uni(pl->nq), nranks = (int)uni(pl->nranks), words = (int)uni(pl->grid_words);
    const uint32_t pitch = uni(pl->grid_pitch);
    const uint32_t k0 = uni(seed_lo), k1 = uni(seed_hi);
    const uint32_t uid = LOGG == 6 ? uni(J.uid) : J.uid, cc = LOGG == 6 ? uni(J.cc) : J.cc;
    const uint32_t coff = grid_state_off(pl) + (uint32_t)c * 4u * (uint32_t)words;
    uint8_t *st = smem + coff;
    uint32_t *st32 = reinterpret_cast<uint32_t *>(st);
    const uint32_t et0 = lds_addr(smem), st0 = et0 + coff;

    // this lane's moves; ranks past the class run on the scratch cells with
    // the null entry (dE 0, no flip)
    uint32_t top[4][MV], eb[4][MV], fl[4][MV];
    const int mpad = 4 * (int)uni(pl->nblk);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int m = 0; m < MV; ++m) {
            const int r = grid_rank<LOGG, MV>(gl, m);
            const uint2 d = pl->grid_move[k * (mpad + 1) + min(r, mpad)];
            top[k][m] = st0 + (d.x & 0xFFFFu);
            eb[k][m] = et0 + (d.x >> 16);
            fl[k][m] = d.y;
        }
    // entries whose threshold changes every sweep (dE > 0): this lane's
    uint32_t tpos[kThr], trank[kThr], thr_next[kThr];
    const int n_rising = (int)uni(pl->grid_rising);
#pragma unroll
    for (int j = 0; j < kThr; ++j) {
        const int i = lane + j * kWave;
        const uint32_t e = i < n_rising ? pl->grid_entry[i] : (uint32_t)pl->grid_slots;   // the spare entry
        tpos[j] = et0 + 8u * (e & 0xFFFFu) + 4u;
        trank[j] = e >> 16;
    }
    const uint32_t *const thr = pl->thr;
    auto fetch_thr = [&](int t) {
        const uint32_t *row = thr + (size_t)min(t, t_end - 1) * nranks;
#pragma unroll
        for (int j = 0; j < kThr; ++j) thr_next[j] = row[trank[j]];
    };

    // starting state and its energy
    int32_t E;
    {
        int32_t W[4];
        W[0] = 0; W[1] = (int32_t)uni(pl->W[1]); W[2] = (int32_t)uni(pl->W[2]); W[3] = (int32_t)uni(pl->W[3]);
        const bool use_x = !J.resume && (J.lp == 1 || J.lp == 2), use_z = !J.resume && (J.lp == 2 || J.lp == 3);
        for (int w = gl; w < words; w += G) st32[w] = 0u;
        wave_lds_fence();
        int32_t part = 0;
        if (J.active)
            for (int q = gl; q < nq; q += G) {
                uint32_t v = J.src[q] & 3u;
                if (use_x) v ^= pl->lx[q];
                if (use_z) v ^= pl->lz[q];
                st[pl->grid_cell[q]] = (uint8_t)(v << 3);
                part += weight_of(W, v);
            }
        E = chain_sum<LOGG>(part);
    }
    int32_t Emin = E, stop = 0;
    wave_lds_fence();
    uint32_t *const snap_c = snap + J.ci * words;
    auto keep_state = [&](bool on) {
        if (on)
            for (int w = gl; w < words; w += G) snap_c[w] = st32[w];
    };
    if (J.resume && J.active) {
        E = J.efin[J.ci];
        Emin = J.emin[J.ci];
        stop = J.stop[J.ci];
    } else {
        keep_state(J.active);
    }

    // draws
    GridDraw gd[MV == 8 ? 2 : 1];
    gd[0] = grid_draw(uid, MV == 1 ? (uint32_t)gl >> 2 : MV == 2 ? (uint32_t)gl >> 1 : (uint32_t)gl, k1);
    if constexpr (MV == 8) gd[1] = grid_draw(uid, (uint32_t)(gl + G), k1);
    // u: the draws of this sweep's four classes (MV <= 2) or of the coming
    // class; the next ones are drawn meanwhile, in eight steps a sweep (MV <=
    // 2) or two a class.  MV = 1: lane j of a quad draws class j, and the 4 x 4
    // words are transposed inside the quad; MV = 2: lane j of a pair draws
    // classes j and 2 + j.
    constexpr int NU = MV <= 2 ? 4 : 1, ND = MV == 1 ? 1 : MV == 8 ? 2 : MV == 2 ? 2 : 1;
    uint32_t u[NU][MV];
    uint4 nd[ND];
    auto draw_head = [&](uint32_t c2) {   // c2: phase 4t (MV <= 2) or 4t + k
#pragma unroll
        for (int h = 0; h < ND; ++h)
            nd[h] = grid_philox_head(gd[MV == 8 ? h : 0], cc,
                                     MV == 1 ? c2 + ((uint32_t)gl & 3u) : MV == 2 ? c2 + 2u * h + ((uint32_t)gl & 1u) : c2,
                                     k0, k1);
    };
    auto draw_rounds = [&](int from, int to) {
#pragma unroll
        for (int i = from; i < to; ++i)
#pragma unroll
            for (int h = 0; h < ND; ++h) nd[h] = grid_philox_round(nd[h], i, k0, k1);
    };
    auto draw_done = [&]() {
        if constexpr (MV == 1) {
            uint4 r = nd[0];
            dpp_exchange<kDppXor1>(r.x, r.y, gl & 1);
            dpp_exchange<kDppXor1>(r.z, r.w, gl & 1);
            dpp_exchange<kDppXor2>(r.x, r.z, gl & 2);
            dpp_exchange<kDppXor2>(r.y, r.w, gl & 2);
            u[0][0] = r.x;
            u[1][0] = r.y;
            u[2][0] = r.z;
            u[3][0] = r.w;
        } else if constexpr (MV == 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint4 r = nd[h];
                dpp_exchange<kDppXor1>(r.x, r.z, gl & 1);
                dpp_exchange<kDppXor1>(r.y, r.w, gl & 1);
                u[2 * h][0] = r.x;
                u[2 * h][1] = r.y;
                u[2 * h + 1][0] = r.z;
                u[2 * h + 1][1] = r.w;
            }
        } else {
#pragma unroll
            for (int h = 0; h < ND; ++h) {
                u[0][4 * h] = nd[h].x;
                u[0][4 * h + 1] = nd[h].y;
                u[0][4 * h + 2] = nd[h].z;
                u[0][4 * h + 3] = nd[h].w;
            }
        }
    };
    // step `half` of class k: the next draws' share that runs while this
    // class's reads are under way
    auto draw_step = [&](uint32_t t, int k, int half) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MV <= 2) {
            if (k == 0 && half == 0) draw_head(4u * t + 4u);
            draw_rounds(2 + 2 * k + half, 3 + 2 * k + half);
        } else {
            if (half == 0) draw_head(4u * t + (uint32_t)k + 1u);
            draw_rounds(half == 0 ? 2 : 6, half == 0 ? 6 : 10);
        }
        // keeps the step here: its results are used only at the sweep's or
        // class's end, and the compiler would move it there
#pragma unroll
        for (int h = 0; h < ND; ++h) asm volatile("" : "+v"(nd[h].x), "+v"(nd[h].y), "+v"(nd[h].z), "+v"(nd[h].w));
        __builtin_amdgcn_sched_barrier(0);
    };
    // A block's four bytes.  Classes 0 and 2 start at even bytes and move two
    // at a time; a 16-bit access at an odd byte takes the LDS about forty
    // cycles, so classes 1 and 3 move single bytes.
    auto read_block = [&](int k, uint32_t a, uint32_t (&p)[4]) {
        if (k & 1) {
            p[0] = lds_read8(a);
            p[1] = lds_read8(a + 1);
            p[2] = lds_read8(a + pitch);
            p[3] = lds_read8(a + pitch + 1);
        } else {
            p[0] = lds_read16(a);
            p[2] = lds_read16(a + pitch);
            p[1] = p[3] = 0;
        }
    };
    auto join_block = [&](int k, const uint32_t (&p)[4]) -> uint32_t {
        return k & 1 ? (p[0] | (p[1] << 8)) | ((p[2] | (p[3] << 8)) << 16) : p[0] | (p[2] << 16);
    };
    auto write_block = [&](int k, uint32_t a, uint32_t v) {
        if (k & 1) {
            lds_write8(a, v);
            lds_write8(a + 1, v >> 8);
            lds_write8(a + pitch, v >> 16);
            lds_write8(a + pitch + 1, v >> 24);
        } else {
            lds_write16(a, v);
            lds_write16(a + pitch, v >> 16);
        }
    };

    if (t_begin < t_end) {
        fetch_thr(t_begin);
        draw_head(4u * (uint32_t)t_begin);
        draw_rounds(2, 10);
        draw_done();
    }
    for (int t = t_begin; t < t_end; ++t) {
        lds_order();
#pragma unroll
        for (int j = 0; j < kThr; ++j) lds_write32(tpos[j], thr_next[j]);
        fetch_thr(t + 1);
        int32_t de[4];
        uint32_t sel[4][MV];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            lds_order();
            uint32_t p[MV][4], v[MV];
            uint2 e[MV];
#pragma unroll
            for (int m = 0; m < MV; ++m) read_block(k, top[k][m], p[m]);
            draw_step((uint32_t)t, k, 0);
#pragma unroll
            for (int m = 0; m < MV; ++m) {
                asm volatile("" : "+v"(p[m][0]), "+v"(p[m][2]));   // joined (and waited for) only here
                v[m] = join_block(k, p[m]);
            }
            // address of the entry: the four codes (<< 3) weighted 1, 4, 16, 64
#pragma unroll
            for (int m = 0; m < MV; ++m)
                e[m] = lds_read64(__builtin_amdgcn_udot4(v[m], 0x40100401u, eb[k][m], false));
            draw_step((uint32_t)t, k, 1);
            de[k] = 0;
#pragma unroll
            for (int m = 0; m < MV; ++m) {
                // u < threshold, or dE <= 0 (whose threshold entry is 0)
                const uint32_t s = accept_sel(u[MV <= 2 ? k : 0][m], e[m].y, (uint32_t)(((int32_t)e[m].x - 1) >> 31));
                write_block(k, top[k][m], xor_and(v[m], fl[k][m], s));
                de[k] += (int32_t)(e[m].x & s);
                sel[k][m] = s;
            }
            if constexpr (MV > 2) draw_done();
        }
        if constexpr (MV <= 2) draw_done();
        int32_t ek[4];
        grid_energies<LOGG>(E, de, ek, gl);
        E = ek[3];
        int last = 0;   // the last phase of this sweep (1..4) with a new least energy
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (ek[k] < Emin) { Emin = ek[k]; last = k + 1; }
        if (__ballot(last != 0)) {
            if (last) stop = 4 * t + last;
#pragma unroll
            for (int back = 0; back < 2; ++back) {
                // undo (then redo) the phases after `last`
#pragma unroll
                for (int k = 1; k < 4; ++k) {
                    wave_lds_fence();
                    const uint32_t on = last != 0 && k >= last ? 0xFFFFFFFFu : 0u;
#pragma unroll
                    for (int m = 0; m < MV; ++m) {
                        uint32_t p[4];
                        read_block(k, top[k][m], p);
                        write_block(k, top[k][m], join_block(k, p) ^ (fl[k][m] & sel[k][m] & on));
                    }
                }
                wave_lds_fence();
                if (back == 0) keep_state(last != 0 && J.active);
            }
        }
    }
    wave_lds_fence();
    if (J.active) {
        if (gl == 0) {
            J.emin[J.ci] = Emin;
            J.stop[J.ci] = stop;
            J.efin[J.ci] = E;
            // serving: the kept state is this range's if E_min is
            if (J.cp_meta && (!J.resume || stop > 4 * t_begin)) J.cp_meta[J.ci] = kKeptExact;
        }
        if (J.states) {
            uint8_t *dst = J.states + (size_t)J.ci * nq;
            for (int q = gl; q < nq; q += G) dst[q] = st[pl->grid_cell[q]] >> 3;
        }
    }
    wave_lds_fence();
}

}  // namespace xzzx
