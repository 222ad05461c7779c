// metro2d.hpp -- the Metropolis update of 32 same-colour sites of a 2D
// ferromagnet (J = 1) as words, and the settling of their ties: shared by the
// band kernel, the double checkerboard and the whole-lattice kernels.
#pragma once

#include "common.hpp"

namespace mcs {

// The thresholds' top bytes as full masks per bit.  An instruction reads at
// most one scalar register, so the masks of dE = 4 stay in vector registers.
struct MetroMasks {
    uint32_t m4[8], m8[8];
};

__device__ __forceinline__ MetroMasks metro_masks(uint32_t top4, uint32_t top8, bool hold)
{
    MetroMasks m;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        m.m4[k] = ((top4 >> k) & 1u) ? ~0u : 0u;
        m.m8[k] = ((top8 >> k) & 1u) ? ~0u : 0u;
        if (hold) asm volatile("" : "+v"(m.m4[k]));
    }
    return m;
}

// A threshold whose top byte fits a mask: 2^32 is 255 with a low part that
// every draw is below.
__host__ __device__ __forceinline__ Thr metro_thr(Thr t) { return t.top >= 256u ? Thr{255u, 1u << 24} : t; }

struct MetroWord {
    uint32_t S;     // the updated word, tied sites unflipped
    uint32_t c8;    // sites of class dE = 8
    uint32_t pend;  // tied sites (byte equal to the top byte of the class's threshold)
};

// S with neighbour words U, D, O, Sh; random bit-planes of the 32 sites from
// the blocks A, B.  Two or more anti-aligned neighbours: dE <= 0, accepted;
// else r32 < T of the site's class, bit-serially from the least significant
// plane with the class's threshold bit (three instructions per plane).
__device__ __forceinline__ MetroWord metro_update(uint32_t S, uint32_t U, uint32_t D, uint32_t O, uint32_t Sh,
                                                  const uint4 &A, const uint4 &B, const MetroMasks &m)
{
    const uint32_t u1 = S ^ U, u2 = S ^ D, u3 = S ^ O, u4 = S ^ Sh;
    const uint32_t t1 = u1 | u2, t2 = u3 | u4;
    const uint32_t ge2 = MCS_BOP3(u1, u2, MCS_BOP3(u3, u4, t1 & t2, (MCS_A & MCS_B) | MCS_C), (MCS_A & MCS_B) | MCS_C);
    MetroWord w;
    w.c8 = ~(t1 | t2);
    uint32_t lt = 0u, eq = ~0u;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t X = plane_pair(A, B, k);
        const uint32_t T = MCS_BOP3(w.c8, m.m8[k], m.m4[k], (MCS_A & MCS_B) | (~MCS_A & MCS_C));
        lt = MCS_BOP3(X, T, lt, (~MCS_A & MCS_B) | (~MCS_A & MCS_C) | (MCS_B & MCS_C));
        eq = MCS_BOP3(eq, X, T, MCS_A & ~(MCS_B ^ MCS_C));
    }
    w.S = MCS_BOP3(S, ge2, lt, MCS_A ^ (MCS_B | MCS_C));
    w.pend = eq & ~ge2;
    return w;
}

// Low 24 bits of the tied sites of one word (first block blk): the mask of
// those accepted.
__device__ __forceinline__ uint32_t metro_settle(uint32_t pend, uint32_t c8, uint32_t blk, uint32_t rep, uint32_t sweep_lo,
                                                 uint32_t w3lo, uint32_t k0, uint32_t k1, uint32_t low4, uint32_t low8)
{
    uint32_t f = 0u;
    while (pend) {
        const int b = __builtin_ctz(pend);
        pend &= pend - 1u;
        const uint4 lo = philox(make_uint4(16u * blk + (uint32_t)b, rep, sweep_lo, w3lo), k0, k1);
        if ((lo.x & 0xFFFFFFu) < (((c8 >> b) & 1u) ? low8 : low4)) f |= 1u << b;
    }
    return f;
}

// Words with ties wait in a queue of their wave's own (64 items {word, first
// block, tied sites, class dE = 8}) until it cannot take another task's or the
// half-sweep ends, and are then settled one per lane: no other wave reads or
// writes them meanwhile, so a half-sweep needs one barrier.
constexpr int kTieQueue = 64;

__device__ __forceinline__ uint32_t wave_rank(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Sum over a wave, in lane 63.
__device__ __forceinline__ int wave_sum_last(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return v;
}

}  // namespace mcs
