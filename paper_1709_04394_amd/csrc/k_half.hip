// k_half.hip -- checkerboard half-sweep in global memory of int8 lattices of
// any even extents with rows of 32 sites or more, 2D or 3D, J = 1 or +-J,
// Metropolis or heat-bath (Sec. "Checkerboard scheme"; Sec. "Disordered
// systems"): the path of lattices that no tile or whole-lattice kernel takes.
//
// A thread updates 16 consecutive sites of one colour of a row: the 32 bytes of
// their pairs (2m, 2m + 1).  It loads the same 32 columns of its own and of the
// 2 or 4 adjacent rows as two 16-byte words each (rows may start at any byte),
// packs the sign bits it needs to 16-bit words (a byte permute picks the parity,
// v_dot4 with powers of two collects the bits), counts bonds and compares
// bit-serially as the whole-lattice kernels do, and writes the 32 bytes back.
// The columns of a row's last chunk are those of the row's last 16 pairs, so
// nothing outside the row is read; its bytes overlap the chunk before and are
// written one by one.  Rows need not hold a multiple of 16 sites of a colour: a
// chunk then takes its random bits from two consecutive blocks, shifted.
//
// E and M are counted in the odd half-sweep, after which no site changes:
// every bond has one odd site, and the pairs of the odd half-sweep's chunks hold
// every even site once.
//
// What bounds it: below about 10^6 sites the latency of a launch and of one
// pass through the kernel (heat-bath 1000 x 750: 9 to 10 us per sweep with the
// launches' gaps, against 63 with a thread that walks 16 sites one by one and a
// measurement of its own); above, memory and VALU issue (4096^2: 24.1 us per
// sweep, 24.9 with a multiplexer over all heat-bath classes, 432 site by site;
// 200^3 +-J 29.6 and 32.4).
#include <algorithm>

#include "heatbath.hpp"
#include "internal.hpp"
#include "lane_bits.hpp"
#include "metro2d.hpp"
#include "spin_bytes.hpp"

namespace mcs {

// Few, large workgroups: each ends with an atomic for E and one for M, all on
// the same line (heat-bath 4096^2 with E, M: 27 us per sweep at 512 workgroups
// of 512, 31 at 1024, 34 at 512 of 256, 48 at 4096 of 256, 76 at 4096 of 128).
constexpr int kHalfThreads = 512;
constexpr uint32_t kHalfBlocks = 512;  // per lattice

struct HalfArgs {
    int8_t *spins;
    const int8_t *J;      // [dims][N] or nullptr
    uint32_t Lx, Ly, Lz, hx;
    int64_t N;
    uint32_t chunks, mul_chunks;  // per row; floor((2^32 - 1) / chunks)
    uint32_t mul_ly;              // floor((2^32 - 1) / Ly)
    uint32_t total;               // chunks of a lattice
    uint32_t blocks;              // workgroups of a lattice
    uint32_t c;                   // colour
    uint32_t seed_lo, seed_hi, replica0, sweep_lo, w3, w3lo;
    // class thresholds (top byte, low 24 bits; T = 2^32 as 255 * 2^24 + 2^24):
    // Metropolis class a = unsatisfied bonds, T of dE = 2z - 4a (a < z/2);
    // heat-bath class d = neighbours with J s_j = -1, T of h = z - 2d
    uint32_t mask[8][8];  // [bit of the top byte][class]: all ones iff set
    uint32_t low[8];
    int64_t *EM;          // this sweep's [count][2], or nullptr
};

template <int DIMS, int RULE, bool HASJ, bool MEASURE>
__global__ __launch_bounds__(kHalfThreads) void k_half(HalfArgs a)
{
    constexpr bool HB = RULE != kMetropolis;
    __shared__ uint32_t tlow[8];
    __shared__ int red[2][kHalfThreads / 64];
    constexpr int Z = 2 * DIMS;
    const int tid = threadIdx.x;
    const uint32_t l = blockIdx.y;
    if (tid < 8) tlow[tid] = a.low[tid];
    __syncthreads();
    int8_t *s = a.spins + (int64_t)l * a.N;
    const int8_t *J0 = a.J, *J1 = a.J + (HASJ ? a.N : 0), *J2 = a.J + (HASJ && DIMS == 3 ? 2 * a.N : 0);
    const uint32_t rep = a.replica0 + l;
    // the masks of even classes in vector registers (an instruction reads one
    // scalar)
    uint32_t tv[8][3];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            tv[k][i] = a.mask[k][2 * i];
            if (RULE != kHeatBathMirrored && i < (HB ? DIMS : 1)) asm volatile("" : "+v"(tv[k][i]));
        }
    int e_acc = 0, m_acc = 0;
    // Large lattices by XCD (4096^2 25.6 against 26.7 us per sweep, 200^3 with
    // couplings 33 against 37); where a thread has one chunk it costs 4 % (1000 x
    // 750).
    const uint32_t b = a.blocks == kHalfBlocks ? xcd_order(blockIdx.x, kHalfBlocks) : blockIdx.x;
    for (uint32_t t = b * kHalfThreads + tid; t < a.total; t += a.blocks * kHalfThreads) {
        const uint32_t row = quotient28(t, a.chunks, a.mul_chunks);
        const uint32_t m0 = 16u * (t - row * a.chunks);
        uint32_t y = row, z = 0;
        if (DIMS == 3) {
            z = quotient28(row, a.Ly, a.mul_ly);
            y = row - z * a.Ly;
        }
        const uint32_t par = (a.c + y + z) & 1u;
        const uint32_t n = a.hx - m0 < 16u ? a.hx - m0 : 16u;  // sites of the chunk
        const uint32_t sh = 16u - n;                            // its first in the window of 16 pairs
        const uint32_t w0 = 2u * (m0 - sh);
        const uint32_t rb = row * a.Lx, area = a.Ly * a.Lx;
        const uint32_t ryp = y + 1 == a.Ly ? rb - (area - a.Lx) : rb + a.Lx;
        const uint32_t rym = y == 0 ? rb + (area - a.Lx) : rb - a.Lx;
        const uint32_t rzp = z + 1 == a.Lz ? rb - (uint32_t)(a.N - area) : rb + area;
        const uint32_t rzm = z == 0 ? rb + (uint32_t)(a.N - area) : rb - area;
        // the x neighbour outside the window: of the first site to the left, or
        // of the last to the right
        const uint32_t xl = m0 == 0 ? a.Lx - 1 : 2 * m0 - 1, xr = m0 + n == a.hx ? 0u : 2 * (m0 + n);
        const uint32_t xe = rb + (par ? xr : xl);
        const Row32 own = load_row32(s, rb + w0), up = load_row32(s, ryp + w0), dn = load_row32(s, rym + w0);
        const int se = s[xe];
        Row32 zu, zd, jx, jy, jyd, jz, jzd;
        int je = 0;
        if (DIMS == 3) {
            zu = load_row32(s, rzp + w0);
            zd = load_row32(s, rzm + w0);
        }
        if (HASJ) {
            jx = load_row32(J0, rb + w0);
            jy = load_row32(J1, rb + w0);
            jyd = load_row32(J1, rym + w0);
            je = J0[xe];
            if (DIMS == 3) {
                jz = load_row32(J2, rb + w0);
                jzd = load_row32(J2, rzm + w0);
            }
        }
        // random planes of the 16 sites
        const uint32_t j0 = row * a.hx + m0, off = j0 & 15u;
        const uint4 A = philox(make_uint4(j0 >> 4, rep, a.sweep_lo, a.w3), a.seed_lo, a.seed_hi);
        uint4 B = A;
        if (a.hx & 15u) B = philox(make_uint4((j0 >> 4) + 1u, rep, a.sweep_lo, a.w3), a.seed_lo, a.seed_hi);

        const uint32_t sel = par ? 0x07050301u : 0x06040200u, selo = par ? 0x06040200u : 0x07050301u;
        const uint32_t valid = (1u << n) - 1u;
        const uint4 own16 = pick16(own, sel);
        const uint4 oth16 = pick16(own, selo);
        const uint32_t S = sign_bits16(own16) >> sh, O = sign_bits16(oth16) >> sh;
        const uint32_t eb = (uint32_t)se >> 31;
        uint32_t wk[6];
        wk[0] = O;                                              // the site's partner in the pair
        wk[1] = par ? (O & valid) >> 1 | eb << (n - 1) : (O << 1) | eb;
        wk[2] = sign_bits16(pick16(up, sel)) >> sh;
        wk[3] = sign_bits16(pick16(dn, sel)) >> sh;
        if (DIMS == 3) {
            wk[4] = sign_bits16(pick16(zu, sel)) >> sh;
            wk[5] = sign_bits16(pick16(zd, sel)) >> sh;
        }
        if (HASJ) {
            // right bonds are the sites' own, left bonds their left neighbours'
            const uint32_t jr = sign_bits16(pick16(jx, sel)) >> sh, jo = sign_bits16(pick16(jx, selo)) >> sh;
            wk[0] ^= par ? jo : jr;
            wk[1] ^= par ? jr : (jo << 1) | ((uint32_t)je >> 31);
            wk[2] ^= sign_bits16(pick16(jy, sel)) >> sh;
            wk[3] ^= sign_bits16(pick16(jyd, sel)) >> sh;
            if (DIMS == 3) {
                wk[4] ^= sign_bits16(pick16(jz, sel)) >> sh;
                wk[5] ^= sign_bits16(pick16(jzd, sel)) >> sh;
            }
        }
        uint32_t xk[6];
#pragma unroll
        for (int k = 0; k < Z; ++k) xk[k] = HB ? wk[k] : (wk[k] ^ S);
        uint32_t c0, c1, c2;
        count_words<Z>(xk, c0, c1, c2);
        // Metropolis: a >= z/2 gives dE <= 0
        const uint32_t ge = HB ? 0u : DIMS == 3 ? MCS_BOP3(c2, c1, c0, MCS_A | (MCS_B & MCS_C)) : (c2 | c1);
        uint32_t lt = 0u, eq = valid;
        MirroredClasses mc;
        if constexpr (RULE == kHeatBathMirrored) mc = mirror_classes<DIMS>(c0, c1, c2);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t X = plane_pair(A, B, k) >> off;
            auto mux = [](uint32_t sel, uint32_t hi, uint32_t lo) {
                return MCS_BOP3(sel, hi, lo, (MCS_A & MCS_B) | (~MCS_A & MCS_C));
            };
            const uint32_t *ts = a.mask[k];
            uint32_t T = mux(c0, ts[1], tv[k][0]);  // classes 0, 1
            if constexpr (RULE == kHeatBathMirrored) {
                T = k == 7 ? ~mc.s : mirrored_plane<DIMS>(mc, ts[0], ts[1], ts[2]);
            } else if (HB) {
                T = mux(c1, mux(c0, ts[3], tv[k][1]), T);
                T = DIMS == 3 ? mux(c2, mux(c1, ts[6], mux(c0, ts[5], tv[k][2])), T) : mux(c2, tv[k][2], T);
            } else if (DIMS == 3) {
                T = mux(c1, tv[k][1], T);
            }
            lt = MCS_BOP3(X, T, lt, (~MCS_A & MCS_B) | (~MCS_A & MCS_C) | (MCS_B & MCS_C));
            eq = MCS_BOP3(eq, X, T, MCS_A & ~(MCS_B ^ MCS_C));
        }
        // heat-bath: down unless r < T; Metropolis: flip where accepted
        uint32_t So = HB ? ~lt : MCS_BOP3(S, ge, lt, MCS_A ^ (MCS_B | MCS_C));
        uint32_t pend = HB ? eq : (eq & ~ge);
        while (pend) {
            const int b = __builtin_ctz(pend);
            pend &= pend - 1u;
            const uint32_t cls = ((c0 >> b) & 1u) | (((c1 >> b) & 1u) << 1) | (((c2 >> b) & 1u) << 2);
            const uint4 lo = philox(make_uint4(j0 + (uint32_t)b, rep, a.sweep_lo, a.w3lo), a.seed_lo, a.seed_hi);
            if ((lo.x & 0xFFFFFFu) < tlow[cls]) So ^= 1u << b;
        }
        const uint32_t F = (So ^ S) & valid;
        if (n == 16u) {
            // flipped bytes: +-1 differ in bits 1..7
            uint32_t q[4] = {own16.x, own16.y, own16.z, own16.w}, o[4] = {oth16.x, oth16.y, oth16.z, oth16.w};
            const uint32_t s0 = par ? 0x01050004u : 0x05010400u, s1 = par ? 0x03070206u : 0x07030602u;
            Row32 out;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                q[i] ^= spread4((F >> (4 * i)) & 15u) * 0xFEu;
                out.d[2 * i] = __builtin_amdgcn_perm(o[i], q[i], s0);
                out.d[2 * i + 1] = __builtin_amdgcn_perm(o[i], q[i], s1);
            }
            __builtin_memcpy(s + (rb + w0), &out, 32);
        } else {
            const uint32_t x0 = rb + 2u * m0 + par;
#pragma unroll
            for (int i = 0; i < 15; ++i)
                if ((F >> i) & 1u) s[x0 + 2u * i] = ((So >> i) & 1u) ? (int8_t)-1 : (int8_t)1;
        }
        if (MEASURE) {
            int u = 0;
#pragma unroll
            for (int k = 0; k < Z; ++k) u += __builtin_popcount((So ^ wk[k]) & valid);
            e_acc += 2 * u - Z * (int)n;
            m_acc += 2 * (int)n - 2 * (__builtin_popcount(So & valid) + __builtin_popcount(O & valid));
        }
    }
    if (MEASURE) {
        const int e = wave_sum_last(e_acc), m = wave_sum_last(m_acc);
    
        if ((tid & 63) == 63) {
            red[0][tid >> 6] = e;
            red[1][tid >> 6] = m;
        }
        __syncthreads();
        if (tid < 2) {
            long long v = 0;
            for (int w = 0; w < kHalfThreads / 64; ++w) v += red[tid][w];
            atomicAdd((unsigned long long *)&a.EM[2 * (int64_t)l + tid], (unsigned long long)v);
        }
    }
}

bool half_supported(const Geom &g) { return g.Lx >= 32; }

template <int D, int RULE, bool HJ>
static hipError_t launch_half_t(const HalfArgs &a, int count, hipStream_t s)
{
    const dim3 grid(a.blocks, (unsigned)count);
    if (a.EM) hipLaunchKernelGGL((k_half<D, RULE, HJ, true>), grid, dim3(kHalfThreads), 0, s, a);
    else hipLaunchKernelGGL((k_half<D, RULE, HJ, false>), grid, dim3(kHalfThreads), 0, s, a);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_half_r(const HalfArgs &a, int rule, int count, hipStream_t s)
{
    const bool hj = a.J != nullptr;
    switch (rule) {
    case kMetropolis: return hj ? launch_half_t<D, kMetropolis, true>(a, count, s) : launch_half_t<D, kMetropolis, false>(a, count, s);
    case kHeatBath: return hj ? launch_half_t<D, kHeatBath, true>(a, count, s) : launch_half_t<D, kHeatBath, false>(a, count, s);
    default: return hj ? launch_half_t<D, kHeatBathMirrored, true>(a, count, s) : launch_half_t<D, kHeatBathMirrored, false>(a, count, s);
    }
}

// One half-sweep (colour c) of every lattice; EM: this sweep's (E, M),
// accumulated (cleared by the caller), in the odd half-sweep only.
hipError_t launch_half(const SweepCall &c, int8_t *spins, uint64_t sweep, int phase, int64_t *EM, hipStream_t s)
{
    HalfArgs a;
    const Geom &g = c.g;
    a.spins = spins;
    a.J = c.J;
    a.Lx = (uint32_t)g.Lx;
    a.Ly = (uint32_t)g.Ly;
    a.Lz = g.dims == 3 ? (uint32_t)g.Lz : 1u;
    a.hx = a.Lx >> 1;
    a.N = g.N;
    a.chunks = (a.hx + 15) / 16;
    a.mul_chunks = 0xFFFFFFFFu / a.chunks;
    a.mul_ly = 0xFFFFFFFFu / a.Ly;
    a.total = a.chunks * (uint32_t)(g.N / g.Lx);
    a.blocks = std::min<uint32_t>((a.total + kHalfThreads - 1) / kHalfThreads, kHalfBlocks);
    a.c = (uint32_t)phase;
    a.seed_lo = c.seed_lo;
    a.seed_hi = c.seed_hi;
    a.replica0 = c.replica0;
    a.sweep_lo = (uint32_t)sweep;
    a.w3 = ctr_w3(kTagSweep, (uint32_t)phase, sweep);
    a.w3lo = ctr_w3(kTagSweepLo, (uint32_t)phase, sweep);
    const int z = 2 * g.dims;
    uint32_t top[8];
    for (int cl = 0; cl < 8; ++cl) {
        Thr th{0u, 0u};
        if (c.rule == 0) {
            if (2 * cl < z) th = c.tab.met[z / 2 - cl];  // dE = 2z - 4a
        } else if (cl <= z) {
            th = c.tab.hb[z - 2 * cl + 6];               // h = z - 2d
        }
        th = metro_thr(th);
        for (int k = 0; k < 8; ++k) a.mask[k][cl] = ((th.top >> k) & 1u) ? ~0u : 0u;
        top[cl] = th.top;
        a.low[cl] = th.low;
    }
    a.EM = phase == 1 ? EM : nullptr;
    const int rule = c.rule == 0 ? kMetropolis : mirrored_classes(top, z) ? kHeatBathMirrored : kHeatBath;
    if (g.dims == 2) return launch_half_r<2>(a, rule, g.count, s);
    return launch_half_r<3>(a, rule, g.count, s);
}

}  // namespace mcs
