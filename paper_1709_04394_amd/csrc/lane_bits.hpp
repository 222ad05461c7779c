// lane_bits.hpp -- bit transposes across a wave for multi-spin-coded lattices,
// where lane and bit exchange the roles of site and replica, and sums of bits
// over lanes.
//
// A 64 x 64 bit transpose exchanges the six bits of the lane number with the
// six of the bit number, one pair per stage.  Distances 32 and 16 are gfx950's
// register swaps between half-waves and rows of 16 lanes (two registers per
// instruction); 8, 4, 2 and 1 take the partner lane's word by a DPP move and
// merge it by one byte permute (8) or a rotate and a select (4, 2, 1).  DPP
// reaches distance 4 only as the mirror image of 8 lanes, lane ^ 7; numbering
// the lanes of each 8 by  label = l ^ (l & 4 ? 3 : 0)  makes that a change of
// label bit 2 alone, so rows and columns are numbered by label throughout.
// 13 issue slots per 32-bit word, against about 36 with ds_swizzle, 64-bit
// shifts and masks, and no LDS traffic.
#pragma once

#include "common.hpp"

namespace mcs {

struct LaneBits {
    int label;                   // this lane's row / column number
    uint32_t sel8;               // byte selector of the distance-8 merge
    uint32_t rot[3], keep[3];    // rotation and kept bits of distances 4, 2, 1
};

__device__ __forceinline__ LaneBits lane_bits(int lane)
{
    LaneBits b;
    b.label = lane ^ ((lane & 4) ? 3 : 0);
    b.sel8 = (b.label & 8) ? 0x03070105u : 0x06020400u;
    const uint32_t low[3] = {0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int d = 4 >> i;
        const bool hi = b.label & d;
        b.rot[i] = hi ? (uint32_t)d : (uint32_t)(32 - d);
        b.keep[i] = hi ? ~low[i] : low[i];
    }
    return b;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}

// Stages 8, 4, 2, 1: label bits 3..0 exchanged with bits 3..0 of the bit number
// (within both 16-bit halves).
__device__ __forceinline__ uint32_t exchange16(uint32_t x, const LaneBits &b)
{
    x = __builtin_amdgcn_perm(dpp<0x128>(x), x, b.sel8);  // row_ror:8
    uint32_t p = dpp<0x141>(x);                           // row_half_mirror
    x = MCS_BOP3(b.keep[0], x, __builtin_amdgcn_alignbit(p, p, b.rot[0]), (MCS_A & MCS_B) | (~MCS_A & MCS_C));
    p = dpp<0x4E>(x);  // quad_perm:[2,3,0,1]
    x = MCS_BOP3(b.keep[1], x, __builtin_amdgcn_alignbit(p, p, b.rot[1]), (MCS_A & MCS_B) | (~MCS_A & MCS_C));
    p = dpp<0xB1>(x);  // quad_perm:[1,0,3,2]
    return MCS_BOP3(b.keep[2], x, __builtin_amdgcn_alignbit(p, p, b.rot[2]), (MCS_A & MCS_B) | (~MCS_A & MCS_C));
}

// Exchange bit 5 (or 4) of the lane number with the choice between a and b.
__device__ __forceinline__ void swap32(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

__device__ __forceinline__ void swap16(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// 64 x 64 bits between sites on the lanes (a lane's site is its label, bit b of
// {lo, hi} replica b) and replicas on the lanes (a lane's replica is its label):
// then bits 0..15 and 16..31 of q0 are the sites 0..15 and 32..47, those of q1
// 16..31 and 48..63, so that plane_pair(B[0], B[2], k) and plane_pair(B[1],
// B[3], k) are the planes of q0 and q1 for the replica's random blocks B of the
// four groups of 16 sites.
__device__ __forceinline__ void to_replicas(uint32_t lo, uint32_t hi, uint32_t &q0, uint32_t &q1, const LaneBits &b)
{
    swap32(lo, hi);
    q0 = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    q1 = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
    swap16(q0, q1);
    q0 = exchange16(q0, b);
    q1 = exchange16(q1, b);
}

__device__ __forceinline__ void to_sites(uint32_t q0, uint32_t q1, uint32_t &lo, uint32_t &hi, const LaneBits &b)
{
    q0 = exchange16(q0, b);
    q1 = exchange16(q1, b);
    swap16(q0, q1);
    lo = __builtin_amdgcn_perm(q1, q0, 0x05040100u);
    hi = __builtin_amdgcn_perm(q1, q0, 0x07060302u);
    swap32(lo, hi);
}

// Site of bit i of q0 (i < 32) or i - 32 of q1.
__device__ __forceinline__ uint32_t site_of_bit(uint32_t i) { return (i & 15u) | ((i & 16u) << 1) | ((i & 32u) >> 1); }

// Set bits of each replica's column over the wave's lanes: lane's result is
// that of replica label.
__device__ __forceinline__ int column_count(uint64_t v, const LaneBits &b)
{
    uint32_t q0, q1;
    to_replicas((uint32_t)v, (uint32_t)(v >> 32), q0, q1, b);
    return __builtin_popcount(q0) + __builtin_popcount(q1);
}

// Bit-sliced count (c0, c1, c2) of the set bits among Z words.
template <int Z>
__device__ __forceinline__ void count_words(const uint32_t (&x)[6], uint32_t &c0, uint32_t &c1, uint32_t &c2)
{
    const uint32_t s1 = xor3(x[0], x[1], x[2]);
    const uint32_t k1 = MCS_BOP3(x[0], x[1], x[2], (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
    if constexpr (Z == 6) {
        const uint32_t s2 = xor3(x[3], x[4], x[5]);
        const uint32_t k2 = MCS_BOP3(x[3], x[4], x[5], (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
        const uint32_t kk = s1 & s2;
        c0 = s1 ^ s2;
        c1 = xor3(k1, k2, kk);
        c2 = MCS_BOP3(k1, k2, kk, (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
    } else {
        const uint32_t kk = s1 & x[3];
        c0 = s1 ^ x[3];
        c1 = k1 ^ kk;
        c2 = k1 & kk;
    }
}

// Bit-sliced counters of 64 replicas in a lane, P planes: v planes added.
template <int P>
struct BitCounter {
    uint64_t n[P];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < P; ++i) n[i] = 0;
    }
    template <int V>
    __device__ __forceinline__ void add(const uint64_t (&v)[V])
    {
        uint32_t cl = 0u, ch = 0u;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const uint32_t nl = (uint32_t)n[i], nh = (uint32_t)(n[i] >> 32);
            if (i < V) {
                const uint32_t vl = (uint32_t)v[i < V ? i : 0], vh = (uint32_t)(v[i < V ? i : 0] >> 32);
                n[i] = ((uint64_t)xor3(nh, vh, ch) << 32) | xor3(nl, vl, cl);
                cl = MCS_BOP3(nl, vl, cl, (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
                ch = MCS_BOP3(nh, vh, ch, (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
            } else {
                n[i] = ((uint64_t)(nh ^ ch) << 32) | (nl ^ cl);
                cl &= nl;
                ch &= nh;
            }
        }
    }
    // sum over the wave's lanes of the lowest `used` planes (the rest are zero),
    // for the replica of this lane's label; cleared
    __device__ __forceinline__ int flush(const LaneBits &b, int used = P)
    {
        int s = 0;
#pragma unroll
        for (int i = 0; i < P; ++i)
            if (i < used) s += column_count(n[i], b) << i;
        clear();
        return s;
    }
};

}  // namespace mcs
