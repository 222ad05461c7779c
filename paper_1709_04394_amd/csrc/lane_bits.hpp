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

// The random blocks of 64 sites in four groups of 16 (a lane's replica is its
// label) to the bit-planes of 64 replicas (a lane's site is its label): on
// return plane k is plane_pair(B[0], B[1], k) for replicas 0..31 and
// plane_pair(B[2], B[3], k) for 32..63.
__device__ __forceinline__ void transpose_blocks(uint4 (&B)[4], const LaneBits &b)
{
    uint32_t r[4][4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        r[g][0] = B[g].x;
        r[g][1] = B[g].y;
        r[g][2] = B[g].z;
        r[g][3] = B[g].w;
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        swap32(r[0][w], r[2][w]);
        swap32(r[1][w], r[3][w]);
        swap16(r[0][w], r[1][w]);
        swap16(r[2][w], r[3][w]);
#pragma unroll
        for (int g = 0; g < 4; ++g) r[g][w] = exchange16(r[g][w], b);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) B[g] = make_uint4(r[g][0], r[g][1], r[g][2], r[g][3]);
}

// Set bits of each replica's column over the wave's lanes: lane's result is
// that of replica label.
__device__ __forceinline__ int column_count(uint64_t v, const LaneBits &b)
{
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    swap32(lo, hi);
    uint32_t p0 = __builtin_amdgcn_perm(hi, lo, 0x05040100u), p1 = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
    swap16(p0, p1);
    return __builtin_popcount(exchange16(p0, b)) + __builtin_popcount(exchange16(p1, b));
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
