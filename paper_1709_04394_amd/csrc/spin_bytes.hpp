// spin_bytes.hpp -- int8 spins (or couplings) +-1 to sign bits and back, 32
// columns at a time, and the rows of a running index.
#pragma once

#include "common.hpp"

namespace mcs {

struct Row32 {
    uint32_t d[8];
};

__device__ __forceinline__ Row32 load_row32(const int8_t *p, uint32_t off)
{
    Row32 r;
    __builtin_memcpy(&r, p + off, 32);
    return r;
}

// The 16 bytes of one parity (sel 0x06040200 even, 0x07050301 odd).
__device__ __forceinline__ uint4 pick16(const Row32 &r, uint32_t sel)
{
    return make_uint4(__builtin_amdgcn_perm(r.d[1], r.d[0], sel), __builtin_amdgcn_perm(r.d[3], r.d[2], sel),
                      __builtin_amdgcn_perm(r.d[5], r.d[4], sel), __builtin_amdgcn_perm(r.d[7], r.d[6], sel));
}

// Sign bits of 16 bytes +-1: sum of -2^i s_i over eight of them is 2 B - 255 for
// their bits B.
__device__ __forceinline__ uint32_t sign_bits16(const uint4 &v)
{
    const int w0 = (int)0xF8FCFEFFu, w1 = (int)0x80C0E0F0u;  // -1, -2, -4, -8; -16, -32, -64, -128
    const int lo = __builtin_amdgcn_sdot4((int)v.y, w1, __builtin_amdgcn_sdot4((int)v.x, w0, 255, false), false);
    const int hi = __builtin_amdgcn_sdot4((int)v.w, w1, __builtin_amdgcn_sdot4((int)v.z, w0, 255, false), false);
    return (((uint32_t)hi << 8) | (uint32_t)lo) >> 1;
}

// n / d, n < 2^28: the product with floor((2^32 - 1) / d) is at most one short
__device__ __forceinline__ uint32_t quotient28(uint32_t n, uint32_t d, uint32_t mul)
{
    const uint32_t q = __umulhi(n, mul);
    return n - q * d >= d ? q + 1u : q;
}

// Four bits to the low bits of four bytes.
__device__ __forceinline__ uint32_t spread4(uint32_t b) { return (b * 0x00204081u) & 0x01010101u; }

}  // namespace mcs
