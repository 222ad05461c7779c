// heatbath.hpp -- threshold planes of bit-sliced heat-bath classes.
//
// A site's class is d = 0 .. z (z = 2 DIMS), the number of its neighbours with
// J s_j = -1, bit-sliced in c0, c1, c2; plane k of its threshold is bit k of the
// top byte of T_d (field h = z - 2d).  A multiplexer over all classes takes z
// operations per plane.  p(+h) + p(-h) = 1, so unless a product p 2^32 falls
// within one of a multiple of 2^24 the top bytes of T_d and T_(z-d) are each
// other's complement, T of h = 0 is exactly 2^31 and the others with h > 0 lie
// above it.  Then with s = (d > z/2), e_i = (d = i or d = z - i):
//   plane 7 = ~s,  plane k < 7 = s ^ (e_0 & m_0[k]) ^ (e_1 & m_1[k]) ...
// z/2 operations per plane, one scalar mask in each.  The kernels have both
// forms, and the host takes this one wherever the top bytes allow it
// (mirrored_classes); beta = 0 and tables with a byte on the edge take the other.
// us per sweep, this form and the multiplexer: fused 3D 256^3 x 4 26.1 and 27.7,
// 64 replicas of 256^3 273 and 290, of 4096^2 261 and 273, 4096^2 half by half
// 24.1 and 24.9, 200^3 +-J 29.6 and 32.4, in one workgroup 12^3 1.29 and 1.42,
// 200^2 3.01 and 3.10.  (A tie's low 24 bits are compared with its own class's
// in both.)
#pragma once

#include "common.hpp"

namespace mcs {

// how a kernel gets its thresholds
enum Rule { kMetropolis = 0, kHeatBath = 1, kHeatBathMirrored = 2 };

struct MirroredClasses {
    uint32_t s, e[3];
};

template <int DIMS>
__device__ __forceinline__ MirroredClasses mirror_classes(uint32_t c0, uint32_t c1, uint32_t c2)
{
    MirroredClasses m;
    if constexpr (DIMS == 3) {
        m.s = c2;
        m.e[0] = MCS_BOP3(c0, c1, c2, ~MCS_A & ~(MCS_B ^ MCS_C));
        m.e[1] = c0 & ~c1;
        m.e[2] = MCS_BOP3(c0, c1, c2, ~MCS_A & (MCS_B ^ MCS_C));
    } else {
        m.s = MCS_BOP3(c0, c1, c2, (MCS_A & MCS_B) | MCS_C);
        m.e[0] = ~(c0 | c1);
        m.e[1] = c0;
        m.e[2] = 0u;
    }
    return m;
}

// Plane k < 7; m: bit k of the top bytes of T_0 .. T_(DIMS-1) as full masks.
template <int DIMS>
__device__ __forceinline__ uint32_t mirrored_plane(const MirroredClasses &c, uint32_t m0, uint32_t m1, uint32_t m2)
{
    uint32_t t = MCS_BOP3(c.s, c.e[0], m0, MCS_A ^ (MCS_B & MCS_C));
    t = MCS_BOP3(t, c.e[1], m1, MCS_A ^ (MCS_B & MCS_C));
    if constexpr (DIMS == 3) t = MCS_BOP3(t, c.e[2], m2, MCS_A ^ (MCS_B & MCS_C));
    return t;
}

// Top bytes (2^32 as 255) of the classes 0 .. z.
inline bool mirrored_classes(const uint32_t *top, int z)
{
    if (top[z / 2] != 128u) return false;
    for (int d = 0; d < z / 2; ++d)
        if (top[d] < 128u || top[z - d] != 255u - top[d]) return false;
    return true;
}

}  // namespace mcs
