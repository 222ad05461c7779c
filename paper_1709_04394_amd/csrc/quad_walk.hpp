// quad_walk.hpp -- sequential single-spin walks with four lanes per walker, for
// the multicanonical and Wang-Landau kernels.
//
// A walker's updates form one serial chain (each decision needs the level and
// the left neighbour the previous one left behind), so a wave is bound by the
// instructions it issues per update, not by bandwidth, and a run of 4096
// walkers with one lane each keeps 64 of the chip's 1024 SIMDs busy.  Here four
// neighbouring lanes carry the same walker: each computes the Philox block and
// the neighbour counts of another four of the next sixteen updates (a quarter
// of that work per lane) and loads and packs a quarter of every row; the chain
// itself runs in all four lanes alike and takes what another lane prepared
// through a quad_perm operand, which costs no instruction of its own in an add
// or a select.  Sixteen walkers per wave also meet fewer LDS bank conflicts
// than sixty-four.
#pragma once

#include "muca_rows.hpp"

namespace mcs {

// Value that lane Q of the quad holds.
__device__ __forceinline__ uint32_t quad_get(uint32_t x, int Q)
{
    switch (Q) {
    case 0: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x00, 0xF, 0xF, true);
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x55, 0xF, 0xF, true);
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xAA, 0xF, 0xF, true);
    default: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xFF, 0xF, 0xF, true);
    }
}

__device__ __forceinline__ float quad_getf(float x, int Q)
{
    return __builtin_bit_cast(float, quad_get(__builtin_bit_cast(uint32_t, x), Q));
}

// LDS by 32-bit byte address, so that an address kept in a register needs no
// base added to it on each access.
typedef __attribute__((address_space(3))) uint32_t LdsWord;

__device__ __forceinline__ int lds_addr(const void *p)
{
    return (int)(uintptr_t)(__attribute__((address_space(3))) char *)(char *)p;
}

__device__ __forceinline__ uint32_t lds_read(int addr) { return *(const LdsWord *)(uintptr_t)(uint32_t)addr; }

__device__ __forceinline__ void lds_add(int addr, uint32_t v)
{
    __hip_atomic_fetch_add((LdsWord *)(uintptr_t)(uint32_t)addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

typedef __attribute__((address_space(3))) uint64_t LdsDword;

__device__ __forceinline__ uint64_t lds_read64(int addr) { return *(const LdsDword *)(uintptr_t)(uint32_t)addr; }

__device__ __forceinline__ void lds_write64(int addr, uint64_t v) { *(LdsDword *)(uintptr_t)(uint32_t)addr = v; }

__device__ __forceinline__ void lds_add64(int addr, uint64_t v)
{
    __hip_atomic_fetch_add((LdsDword *)(uintptr_t)(uint32_t)addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A Philox block computed a round at a time, for the updates of the group
// after the one being walked: its instructions fill the time in which the walk
// waits for LDS.
struct PhiloxRounds {
    uint4 c;
    __device__ __forceinline__ void round(int r, uint32_t k0, uint32_t k1)
    {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c.x;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * c.z;
        c = make_uint4(xor3((uint32_t)(p1 >> 32), c.y, k0 + (uint32_t)r * kPhiloxW0), (uint32_t)p1,
                       xor3((uint32_t)(p0 >> 32), c.w, k1 + (uint32_t)r * kPhiloxW1), (uint32_t)p0);
    }
};

// 2 f + (this lane's bit of m), m a lane mask as a compare leaves it.
__device__ __forceinline__ uint32_t shift_in(uint32_t f, uint64_t m)
{
    uint32_t r;
    asm("v_addc_co_u32 %0, vcc, %1, %1, %2" : "=v"(r) : "v"(f), "s"(m) : "vcc");
    return r;
}

// A row of L sites as NW words of CB bits (bit set <=> s = -1), CB a multiple of
// 16 or, where the row has no such part, at most 12, so that the groups of
// sixteen updates a word is walked in need no end test (24-bit words, whose
// second group is half a group, took 430 ns per update at L = 48 against
// 62 with 16-bit words).
template <int L>
struct QuadRow {
    static constexpr int CB = L % 32 == 0 ? 32 : L % 16 == 0 ? 16 : L % 12 == 0 ? 12 : L;
    static constexpr int NW = L / CB;
    static constexpr bool kSplit = L % 16 == 0;      // each lane a quarter of the row
    static constexpr int RD = kSplit ? L / 16 : L / 4;  // dwords a lane loads
    static_assert(CB * NW == L && CB % 4 == 0 && (CB % 16 == 0 || CB < 16), "whole words");
    // groups of sixteen updates follow each other block by block through the sweep
    static constexpr bool kAhead = CB % 16 == 0;
};

template <int L>
__device__ __forceinline__ void quad_load(const int8_t *sp, int y, int q, uint32_t (&raw)[QuadRow<L>::RD])
{
    constexpr int RD = QuadRow<L>::RD;
    const int8_t *p = sp + y * L + (QuadRow<L>::kSplit ? q * (L / 4) : 0);
    if constexpr (QuadRow<L>::kSplit && RD % 4 == 0) {
#pragma unroll
        for (int i = 0; i < RD / 4; ++i) {
            const uint4 v = ((const uint4 *)p)[i];
            raw[4 * i] = v.x;
            raw[4 * i + 1] = v.y;
            raw[4 * i + 2] = v.z;
            raw[4 * i + 3] = v.w;
        }
    } else if constexpr (QuadRow<L>::kSplit && RD % 2 == 0) {
#pragma unroll
        for (int i = 0; i < RD / 2; ++i) {
            const uint2 v = ((const uint2 *)p)[i];
            raw[2 * i] = v.x;
            raw[2 * i + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < RD; ++i) raw[i] = ((const uint32_t *)p)[i];
    }
}

// Loaded dwords -> the row's words, in every lane of the quad.
template <int L>
__device__ __forceinline__ void quad_pack(const uint32_t (&raw)[QuadRow<L>::RD], uint32_t (&row)[QuadRow<L>::NW])
{
    using R = QuadRow<L>;
#pragma unroll
    for (int i = 0; i < R::NW; ++i) row[i] = 0u;
    if constexpr (R::kSplit) {
        constexpr int PB = L / 4;  // bits of a quarter
        uint32_t part = 0u;
#pragma unroll
        for (int i = 0; i < R::RD; ++i) part |= pack4(raw[i]) << (4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = quad_get(part, j);
#pragma unroll
            for (int i = 0; i < R::NW; ++i) {
                const int sh = j * PB - i * R::CB;  // position of the quarter in word i
                if (sh >= 0 && sh < R::CB) row[i] |= v << sh;
                else if (sh < 0 && sh + PB > 0) row[i] |= v >> -sh;
            }
        }
        if constexpr (R::CB < 32) {
#pragma unroll
            for (int i = 0; i < R::NW; ++i) row[i] &= (1u << R::CB) - 1u;
        }
    } else {
#pragma unroll
        for (int i = 0; i < R::RD; ++i) row[4 * i / R::CB] |= pack4(raw[i]) << (4 * i % R::CB);
    }
}

template <int L>
__device__ __forceinline__ void quad_store(int8_t *sp, int y, int q, bool live, const uint32_t (&row)[QuadRow<L>::NW])
{
    using R = QuadRow<L>;
    if constexpr (R::kSplit) {
        constexpr int PB = L / 4;
        uint32_t part[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = j * PB / R::CB, sh = j * PB % R::CB;
            part[j] = row[i] >> sh;
            if (sh + PB > R::CB) part[j] |= row[i + 1 < R::NW ? i + 1 : i] << (R::CB - sh);
        }
        const uint32_t v = (q & 2) ? ((q & 1) ? part[3] : part[2]) : ((q & 1) ? part[1] : part[0]);
        uint32_t d[R::RD];
#pragma unroll
        for (int i = 0; i < R::RD; ++i) d[i] = unpack4((v >> (4 * i)) & 0xFu);
        int8_t *p = sp + y * L + q * PB;
        if (live) {
            if constexpr (R::RD % 4 == 0) {
#pragma unroll
                for (int i = 0; i < R::RD / 4; ++i)
                    ((uint4 *)p)[i] = make_uint4(d[4 * i], d[4 * i + 1], d[4 * i + 2], d[4 * i + 3]);
            } else if constexpr (R::RD % 2 == 0) {
#pragma unroll
                for (int i = 0; i < R::RD / 2; ++i) ((uint2 *)p)[i] = make_uint2(d[2 * i], d[2 * i + 1]);
            } else {
#pragma unroll
                for (int i = 0; i < R::RD; ++i) ((uint32_t *)p)[i] = d[i];
            }
        }
    } else {
        // every lane stores the row it will load again
        uint32_t *p = (uint32_t *)(sp + y * L);
        if (live) {
#pragma unroll
            for (int i = 0; i < R::RD; ++i) p[i] = unpack4((row[4 * i / R::CB] >> (4 * i % R::CB)) & 0xFu);
        }
    }
}

// Unsatisfied bonds of the CB sites of a word to their up, down and right
// neighbours as two bit planes, and to the left neighbour as a third, all
// neighbours in the state before the word's updates (lb: the site left of bit
// 0; rb: the site right of bit CB - 1).
struct QuadPlanes {
    uint32_t p0, p1, lw, z;
};

template <int CB>
__device__ __forceinline__ QuadPlanes quad_planes(uint32_t c, uint32_t u, uint32_t d, uint32_t lb, uint32_t rb)
{
    QuadPlanes P;
    const uint32_t X = c ^ u, Y = c ^ d;
    P.z = c ^ ((c >> 1) | (rb << (CB - 1)));
    P.p0 = xor3(X, Y, P.z);
    P.p1 = MCS_BOP3(X, Y, P.z, (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
    P.lw = c ^ ((c << 1) | lb);
    return P;
}

// Counts of this lane's four updates of a group of sixteen (shift: the first
// of them in the word): n3 to up, down and right, l to the left neighbour in
// its old state.  The unsatisfied bonds of update i are n3 + l if the previous
// update was rejected, n3 + 1 - l if it was accepted.
struct QuadCounts {
    int n3[4], l[4];
};

__device__ __forceinline__ QuadCounts quad_counts(const QuadPlanes &P, int shift)
{
    QuadCounts c;
    const uint32_t a = P.p0 >> shift, b = P.p1 >> shift, l = P.lw >> shift;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c.n3[i] = (int)((((b >> i) & 1u) << 1) + ((a >> i) & 1u));
        c.l[i] = (int)((l >> i) & 1u);
    }
    return c;
}

}  // namespace mcs
