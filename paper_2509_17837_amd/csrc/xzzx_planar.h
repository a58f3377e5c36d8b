// Building blocks of the packed-row kernels specialised to the planar
// lattice at distance D (odd, 3..15): the lattice turned by 45 degrees (rows
// of 2D + 1 columns, see PlanarSchedule), every row in registers for the
// whole run, the generator schedule in the instruction stream.  One chain per
// lane; a task's 64 chains may span syndromes (the paper's N_SA = 10 gives 40
// chains per syndrome), so the syndrome word of the Philox counter varies
// across the wavefront (lane_head and lane_philox_block).  Used by
// the annealing and the replica-exchange kernels of this lattice.
#pragma once

#include "xzzx_device.h"

namespace xzzx {

template <int D>
struct PlanarRows {
    static constexpr int R = 2 * D - 1;                        // rows
    static constexpr int C = 2 * D + 1;                        // columns (the last two are padding)
    static constexpr int NW = 2 * C <= 32 ? 1 : 2;             // words per row
    static constexpr int N = R * NW;                           // registers per chain
};

template <int D, int K, int B, int W>
struct PlanarGen {
    static constexpr RotGen g = kPlanarSchedule<D>.g[K][4 * B + W];
    static constexpr bool real = g.shp != 5;
    static constexpr int Y = g.Y, BO = g.bo;
};

// The move's energy-table entry from its 8-bit block pattern (top row, then
// bottom row).
template <int D, int K, int B, int W>
__device__ __forceinline__ uint2 planar_lookup(const uint32_t (&r)[PlanarRows<D>::N], const uint16_t *lut_s,
                                               const uint2 *et_s)
{
    using G = PlanarGen<D, K, B, W>;
    constexpr int NW = PlanarRows<D>::NW;
    if constexpr (!G::real) {
        return make_uint2(0u, 0u);
    } else {
        const uint32_t pat2 = join_pattern(row_bits<NW, G::BO, 1>(r + G::Y * NW) & 0x1Eu,
                                           row_bits<NW, G::BO, 5>(r + (G::Y + 1) * NW));
        const uint32_t off = *reinterpret_cast<const uint16_t *>(reinterpret_cast<const uint8_t *>(lut_s) +
                                                                 512u * G::g.shp + pat2);
        return *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint8_t *>(et_s) + off);
    }
}

template <int D, int K, int B, int W>
__device__ __forceinline__ void planar_apply(uint32_t (&r)[PlanarRows<D>::N], uint32_t u, const uint2 &e, uint32_t &acc,
                                             uint32_t zero)
{
    using G = PlanarGen<D, K, B, W>;
    constexpr int NW = PlanarRows<D>::NW;
    if constexpr (G::real) {
        const uint32_t sel = accept_mask(u, e);
        row_flip_static<NW, G::BO, 6u>(r + G::Y * NW, sel, zero);         // X top-left | Z top-right
        row_flip_static<NW, G::BO, 9u>(r + (G::Y + 1) * NW, sel, zero);   // Z bottom-left | X bottom-right
        take_move(acc, e, sel);
    }
}

// The four moves of block B: entries looked up, then acceptance and flips.
template <int D, int K, int B>
__device__ __forceinline__ void planar_lookups(const uint32_t (&r)[PlanarRows<D>::N], const uint16_t *lut_s,
                                               const uint2 *et_s, uint2 (&e)[4])
{
    e[0] = planar_lookup<D, K, B, 0>(r, lut_s, et_s);
    e[1] = planar_lookup<D, K, B, 1>(r, lut_s, et_s);
    e[2] = planar_lookup<D, K, B, 2>(r, lut_s, et_s);
    e[3] = planar_lookup<D, K, B, 3>(r, lut_s, et_s);
}

template <int D, int K, int B>
__device__ __forceinline__ void planar_applies(uint32_t (&r)[PlanarRows<D>::N], const uint4 &u, const uint2 (&e)[4],
                                               uint32_t &acc)
{
    const uint32_t zero = PlanarRows<D>::NW == 1 ? 0u : opaque_zero();
    planar_apply<D, K, B, 0>(r, u.x, e[0], acc, zero);
    planar_apply<D, K, B, 1>(r, u.y, e[1], acc, zero);
    planar_apply<D, K, B, 2>(r, u.z, e[2], acc, zero);
    planar_apply<D, K, B, 3>(r, u.w, e[3], acc, zero);
    asm("" : "+v"(acc));   // sum block by block (see static_block)
}

// Blocks B..NB-1 of a class, software-pipelined: the generators of one
// colour class act on disjoint qubits, so block B + 1's slots read the same
// before and after block B's flips, and its entries are looked up before
// those flips.  Its LDS round trips then overlap block B's acceptance
// instead of waiting for it (the register dependence through the rows would
// otherwise serialise the blocks; d = 9: 3 % faster).  With entries of twelve bytes
// d = 5, 11 and 15, and ladders at d = 7, were faster without; with eight every
// distance runs it (whole decodes of 262144 chains, against then: 0.80, 0.83 and 0.73
// of the time; ladders of four levels 0.56, 0.73 and 0.60, at d = 7 0.66).
template <int D, int K, int B, int NB>
__device__ __forceinline__ void planar_pipe(uint32_t (&r)[PlanarRows<D>::N], const LaneKey &lk,
                                            const LaneHead &h, uint32_t k0, uint32_t k1, const uint16_t *lut_s,
                                            const uint2 *et_s, uint32_t &acc, const uint2 (&e)[4])
{
    const uint4 u = lane_philox_block<B, true>(lk, h, k0, k1);
    if constexpr (B + 1 < NB) {
        uint2 en[4];
        planar_lookups<D, K, B + 1>(r, lut_s, et_s, en);
        planar_applies<D, K, B>(r, u, e, acc);
        planar_pipe<D, K, B + 1, NB>(r, lk, h, k0, k1, lut_s, et_s, acc, en);
    } else {
        planar_applies<D, K, B>(r, u, e, acc);
    }
}

// One colour class of a sweep: c2 = 4t + k names the sweep and class in the
// Philox counter.
template <int D, int K>
__device__ __forceinline__ void planar_class(uint32_t (&r)[PlanarRows<D>::N], const LaneKey &lk, uint32_t cc,
                                             uint32_t c2, uint32_t k0, uint32_t k1, const uint16_t *lut_s,
                                             const uint2 *et_s, uint32_t &acc)
{
    constexpr int NB = PlanarSchedule<D>::MP / 4;
    const LaneHead h = lane_head(lk, cc, c2, k0, k1);
    uint2 e[4];
    planar_lookups<D, K, 0>(r, lut_s, et_s, e);
    planar_pipe<D, K, 0, NB>(r, lk, h, k0, k1, lut_s, et_s, acc, e);
}

// qubit at row Y, column C of the turned lattice, or -1
template <int D>
__device__ __forceinline__ int planar_qubit_at(int Y, int C)
{
    const int u = Y + 1, v = C - (D - 1);
    return PlanarSchedule<D>::qubit(u + v + 1, u - v);
}

// The chain's starting state packed into the turned rows (the logical
// operators of its coset applied as asked), and its energy.
template <int D>
__device__ __forceinline__ int32_t planar_load(const PlanDev *pl, const ChainJob &J, bool use_x, bool use_z,
                                               const int32_t (&W)[4], uint32_t (&r)[PlanarRows<D>::N])
{
    using PR = PlanarRows<D>;
    constexpr int NW = PR::NW;
    int32_t E = 0;
#pragma unroll
    for (int Y = 0; Y < PR::R; ++Y) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            uint32_t word = 0;
            if (J.active) {
#pragma unroll 1
                for (int C = 16 * w; C < min(PR::C, 16 * w + 16); ++C) {
                    const int q = planar_qubit_at<D>(Y, C);
                    if (q < 0) continue;
                    uint32_t v = J.src[q] & 3u;
                    if (use_x) v ^= pl->lx[q];
                    if (use_z) v ^= pl->lz[q];
                    word |= v << (2 * (C - 16 * w));
                    E += weight_of(W, v);
                }
            }
            r[Y * NW + w] = word;
        }
    }
    return E;
}

// One byte per qubit (the lattice's qubit order) from the turned rows.
template <int D>
__device__ __forceinline__ void planar_unpack(const uint32_t (&r)[PlanarRows<D>::N], uint8_t *dst)
{
    using PR = PlanarRows<D>;
    constexpr int NW = PR::NW;
#pragma unroll
    for (int Y = 0; Y < PR::R; ++Y)
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll 1
            for (int C = 16 * w; C < min(PR::C, 16 * w + 16); ++C) {
                const int q = planar_qubit_at<D>(Y, C);
                if (q >= 0) dst[q] = (uint8_t)((r[Y * NW + w] >> (2 * (C - 16 * w))) & 3u);
            }
}

// The rows of a chain, stored with 16-byte stores from one base address
// (NP = the rows padded to a multiple of four words).
template <int N>
__device__ __forceinline__ void store_rows(uint4 *dst, const uint32_t (&r)[N])
{
    constexpr int NP = (N + 3) / 4 * 4;
#pragma unroll
    for (int i = 0; i < NP / 4; ++i)
        dst[i] = make_uint4(r[4 * i], 4 * i + 1 < N ? r[4 * i + 1] : 0u, 4 * i + 2 < N ? r[4 * i + 2] : 0u,
                            4 * i + 3 < N ? r[4 * i + 3] : 0u);
}

// wavefronts per SIMD (VGPR budget 512 / waves): the rows take 2D - 1
// registers (one word per row, d <= 7) or 2(2D - 1), beside the lane-varying
// Philox words and the look-ahead entries; the most waves that compile with at
// most a register or two spilled (d = 9: five, with entries of eight bytes;
// the paper's set-up 3.79 -> 3.6 ms against four with twelve-byte entries)
constexpr int planar_waves(int d) { return d <= 5 ? 8 : d == 7 ? 6 : d == 9 ? 5 : d == 11 ? 4 : 3; }

}  // namespace xzzx
