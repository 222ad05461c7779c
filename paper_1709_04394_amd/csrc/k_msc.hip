// k_msc.hip -- checkerboard half-sweep of 64-lane multi-spin-coded lattices
// (Sec. "Checkerboard scheme": multi-spin coding packs 64 independent
// replicas into the bits of one word) for 2D and 3D lattices with Lx a
// multiple of 128, Ising or +-J couplings, Metropolis or heat-bath.
//
// Design (gfx950):
//  * A wave takes 64 consecutive same-colour sites of one row (one site per
//    lane) and all 64 replicas of each (the bits of the site's word).  The
//    neighbour words give per-replica classes as bit-sliced counters
//    (carry-save adders over the 4 or 6 bond masks), so one lane updates 64
//    replicas with word operations.
//  * Every replica has its own random stream: lane b draws the Philox blocks
//    of replica b for the 4 groups of 16 sites the wave covers, whose
//    half-words are the random bit-planes of those sites (the stream the int8
//    kernels use, so lane b of the word lattice equals the int8 run of that
//    replica bit for bit).  The sites' classes, two to four bits per site and
//    replica, are transposed to lanes that are replicas (64 x 64 bits per class
//    bit, lane_bits.hpp), compared there bit-serially with the class's threshold
//    where the planes already are, and the outcome is transposed back: three to
//    five transposes instead of the eight planes'.
//  * A tie (a replica whose top byte equals its class's threshold's) is drawn by
//    its replica's lane before that: about one in five has one.
//  * Per-sweep E and M per replica are counted in the odd half-sweep: each lane
//    adds the unsatisfied bonds and down spins of its sites to bit-sliced
//    counters of the 64 replicas, which are summed over the lanes once in 32
//    tasks; one atomic per replica and workgroup.
//
// What bounds it: VALU issue.  4096^2, 64 replicas, Metropolis: 116 us per even
// half-sweep and 147 with E, M; 133 and 173 with the planes transposed and ties
// settled from a queue, 238 and 311 with a transpose per plane through
// ds_swizzle (36 instructions per word), a transpose back for every count of
// every task and rows by 64-bit division.
#include <algorithm>

#include "heatbath.hpp"
#include "internal.hpp"
#include "lane_bits.hpp"

namespace mcs {

struct MscArgs {
    uint64_t *w;
    const int8_t *J;  // [dims][N] or nullptr
    int Lx, Ly, Lz;
    int64_t N;
    uint32_t seed_lo, seed_hi, replica0;
    uint32_t sweep_lo, w3, w3lo;
    int c;  // colour of this half-sweep
    // class thresholds (top byte, low 24 bits; T = 2^32 as 255 * 2^24 + 2^24):
    // Metropolis class a = unsatisfied bonds, T of dE = 2z - 4a (a < z/2);
    // heat-bath class d = neighbours with J s_j = -1, T of h = z - 2d
    uint32_t top[8], low[8];
    int64_t *EM;  // this sweep's [count * 64][2], or nullptr
};

constexpr int kMscWaves = 16;  // of a workgroup that measures, at most
constexpr int kMscFlush = 32;  // tasks between sums of the bit-sliced counters

template <int DIMS, bool MEASURE, int RULE, bool HASJ>
__global__ __launch_bounds__(MEASURE ? 64 * kMscWaves : 256) void k_msc(MscArgs a)
{
    constexpr bool HB = RULE != kMetropolis;
    __shared__ uint32_t tlow[8];
    __shared__ long long red[2][64];
    constexpr int Z = 2 * DIMS;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = blockIdx.y;
    if (tid < 8) tlow[tid] = a.low[tid];
    if (MEASURE && tid < 128) red[tid >> 6][tid & 63] = 0;
    __syncthreads();
    const LaneBits lb = lane_bits(tid & 63);
    uint64_t *w = a.w + (int64_t)l * a.N;
    const uint32_t per_row = (uint32_t)a.Lx >> 7;  // tasks per row
    const uint32_t tasks = (uint32_t)(a.N >> 7);
    const uint32_t rep0 = a.replica0 + 64u * (uint32_t)l;
    // the classes' threshold bits as full masks: even classes in vector
    // registers (an instruction reads one scalar)
    uint32_t tv[8][3], ts[8][4];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            tv[k][i] = ((a.top[2 * i] >> k) & 1u) ? ~0u : 0u;
            if (RULE != kHeatBathMirrored && i < (HB ? DIMS : 1)) asm volatile("" : "+v"(tv[k][i]));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) ts[k][i] = ((a.top[i < 3 ? 2 * i + 1 : 6] >> k) & 1u) ? ~0u : 0u;
    }
    BitCounter<8> cu;  // unsatisfied bonds of the odd sites, up to 6 a task
    BitCounter<7> cd;  // down spins of both sites of a pair
    long long u_acc = 0, d_acc = 0;
    int since = 0;
    if (MEASURE) {
        cu.clear();
        cd.clear();
    }
    uint32_t done = 0;
    const uint32_t waves = MEASURE ? blockDim.x >> 6 : 4u;
    for (uint32_t t = xcd_order(blockIdx.x, gridDim.x) * waves + (uint32_t)wave; t < tasks; t += gridDim.x * waves) {
        const uint32_t j0 = t << 6;
        const uint32_t row = t / per_row, m0 = (t - row * per_row) << 6;
        const uint32_t z = row / (uint32_t)a.Ly, y = row - z * (uint32_t)a.Ly;
        const int par = (int)((uint32_t)a.c + y + z) & 1;
        const uint32_t x = 2u * (m0 + (uint32_t)lb.label) + (uint32_t)par;
        const int64_t plane = (int64_t)a.Ly * a.Lx, rbase = (int64_t)row * a.Lx;
        const uint32_t xp = x + 1 == (uint32_t)a.Lx ? 0 : x + 1, xm = x == 0 ? (uint32_t)a.Lx - 1 : x - 1;
        const int64_t ryp = y + 1 == (uint32_t)a.Ly ? rbase - (plane - a.Lx) : rbase + a.Lx;
        const int64_t rym = y == 0 ? rbase + (plane - a.Lx) : rbase - a.Lx;
        const int64_t rzp = z + 1 == (uint32_t)a.Lz ? rbase - (a.N - plane) : rbase + plane;
        const int64_t rzm = z == 0 ? rbase + (a.N - plane) : rbase - plane;
        const uint64_t S = (w + rbase)[x];
        uint64_t n[6] = {(w + rbase)[xp], (w + rbase)[xm], (w + ryp)[x], (w + rym)[x], 0, 0};
        if (DIMS == 3) {
            n[4] = (w + rzp)[x];
            n[5] = (w + rzm)[x];
        }
        // random blocks: lane = replica, 4 groups of 16 sites
        uint4 B[4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
            B[g] = philox(make_uint4((j0 >> 4) + (uint32_t)g, rep0 + (uint32_t)lb.label, a.sweep_lo, a.w3), a.seed_lo,
                          a.seed_hi);
        uint64_t jm[6] = {0, 0, 0, 0, 0, 0};
        if (HASJ) {
            const int8_t *J = a.J;
            jm[0] = (J + rbase)[x] < 0 ? ~0ull : 0ull;
            jm[1] = (J + rbase)[xm] < 0 ? ~0ull : 0ull;
            jm[2] = (J + a.N + rbase)[x] < 0 ? ~0ull : 0ull;
            jm[3] = (J + a.N + rym)[x] < 0 ? ~0ull : 0ull;
            if (DIMS == 3) {
                jm[4] = (J + 2 * a.N + rbase)[x] < 0 ? ~0ull : 0ull;
                jm[5] = (J + 2 * a.N + rzm)[x] < 0 ? ~0ull : 0ull;
            }
        }
        // lane = site: classes of its 64 replicas, halves of 32
        uint32_t C0[2], C1[2], C2[2], GE[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t Sh = (uint32_t)(S >> (32 * h));
            // n ^ jm: bit set <=> J s_j = -1; Metropolis counts unsatisfied bonds,
            // heat-bath those
            uint32_t xk[6];
#pragma unroll
            for (int k = 0; k < Z; ++k) {
                const uint32_t wk = (uint32_t)((n[k] ^ jm[k]) >> (32 * h));
                xk[k] = HB ? wk : (wk ^ Sh);
            }
            count_words<Z>(xk, C0[h], C1[h], C2[h]);
            // Metropolis: a >= z/2 gives dE <= 0
            GE[h] = HB ? 0u : DIMS == 3 ? MCS_BOP3(C2[h], C1[h], C0[h], MCS_A | (MCS_B & MCS_C)) : (C2[h] | C1[h]);
        }
        // lane = replica: its 64 sites
        uint32_t c0[2], c1[2] = {0u, 0u}, c2[2] = {0u, 0u}, ge[2] = {0u, 0u}, acc[2], pq[2];
        to_replicas(C0[0], C0[1], c0[0], c0[1], lb);
        if (HB || DIMS == 3) to_replicas(C1[0], C1[1], c1[0], c1[1], lb);
        if (HB) to_replicas(C2[0], C2[1], c2[0], c2[1], lb);
        else to_replicas(GE[0], GE[1], ge[0], ge[1], lb);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint32_t lt = 0u, eq = ~0u;
            MirroredClasses mc;
            if constexpr (RULE == kHeatBathMirrored) mc = mirror_classes<DIMS>(c0[q], c1[q], c2[q]);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t X = plane_pair(B[q], B[q + 2], k);
                auto mux = [](uint32_t sel, uint32_t hi, uint32_t lo) {
                    return MCS_BOP3(sel, hi, lo, (MCS_A & MCS_B) | (~MCS_A & MCS_C));
                };
                uint32_t T = mux(c0[q], ts[k][0], tv[k][0]);  // classes 0, 1
                if constexpr (RULE == kHeatBathMirrored) {
                    T = k == 7 ? ~mc.s : mirrored_plane<DIMS>(mc, tv[k][0], ts[k][0], tv[k][1]);
                } else if (HB) {
                    T = mux(c1[q], mux(c0[q], ts[k][1], tv[k][1]), T);
                    T = DIMS == 3 ? mux(c2[q], mux(c1[q], ts[k][3], mux(c0[q], ts[k][2], tv[k][2])), T)
                                  : mux(c2[q], tv[k][2], T);
                } else if (DIMS == 3) {
                    T = mux(c1[q], tv[k][1], T);
                }
                lt = MCS_BOP3(X, T, lt, (~MCS_A & MCS_B) | (~MCS_A & MCS_C) | (MCS_B & MCS_C));
                eq = MCS_BOP3(eq, X, T, MCS_A & ~(MCS_B ^ MCS_C));
            }
            acc[q] = lt | ge[q];
            pq[q] = eq & ~ge[q];
        }
        for (uint64_t pend = ((uint64_t)pq[1] << 32) | pq[0]; pend; pend &= pend - 1ull) {
            const uint32_t i = (uint32_t)__builtin_ctzll(pend), b = i & 31u;
            const bool up = i >= 32u;
            const uint32_t cls = (((up ? c0[1] : c0[0]) >> b) & 1u) | ((((up ? c1[1] : c1[0]) >> b) & 1u) << 1) |
                                 ((((up ? c2[1] : c2[0]) >> b) & 1u) << 2);
            const uint4 lo = philox(make_uint4(j0 + site_of_bit(i), rep0 + (uint32_t)lb.label, a.sweep_lo, a.w3lo),
                                    a.seed_lo, a.seed_hi);
            const uint32_t f = (lo.x & 0xFFFFFFu) < tlow[cls] ? 1u << b : 0u;
            acc[0] |= up ? 0u : f;
            acc[1] |= up ? f : 0u;
        }
        // back to lane = site; Metropolis: flip, heat-bath: up where accepted
        uint32_t A[2];
        to_sites(acc[0], acc[1], A[0], A[1], lb);
        const uint64_t So = HB ? ~(((uint64_t)A[1] << 32) | A[0]) : S ^ (((uint64_t)A[1] << 32) | A[0]);
        (w + rbase)[x] = So;
        uint64_t u[3] = {0, 0, 0}, dn[2] = {0, 0};
        if (MEASURE) {
            // odd sites: their bonds after the update; both sites of the pair
            // (this odd site and the even site at the same row position) for M
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t uk[6], v0, v1, v2;
#pragma unroll
                for (int k = 0; k < Z; ++k) uk[k] = (uint32_t)((So ^ n[k] ^ jm[k]) >> (32 * h));
                count_words<Z>(uk, v0, v1, v2);
                u[0] |= (uint64_t)v0 << (32 * h);
                u[1] |= (uint64_t)v1 << (32 * h);
                u[2] |= (uint64_t)v2 << (32 * h);
            }
            const uint64_t pw = par ? n[1] : n[0];  // even site 2m + (1 - par)
            dn[0] = So ^ pw;
            dn[1] = So & pw;
        }
        if (MEASURE) {
            cu.add(u);
            cd.add(dn);
            ++done;
            if (++since == kMscFlush) {
                u_acc += cu.flush(lb);
                d_acc += cd.flush(lb);
                since = 0;
            }
        }
    }
    if (MEASURE) {
        u_acc += cu.flush(lb);
        d_acc += cd.flush(lb);
        // E: 2 (unsatisfied) - z per odd site; M: 2 - 2 (down) per pair
        const long long e = 2 * u_acc - 64ll * Z * done, mg = 128ll * done - 2 * d_acc;
        atomicAdd((unsigned long long *)&red[0][lb.label], (unsigned long long)e);
        atomicAdd((unsigned long long *)&red[1][lb.label], (unsigned long long)mg);
        __syncthreads();
        if (tid < 128) {
            atomicAdd((unsigned long long *)&a.EM[128 * (int64_t)l + tid], (unsigned long long)red[tid & 1][tid >> 1]);
        }
    }
}

bool msc_fast_supported(const SweepCall &c, int layout)
{
    return layout == MC_MSC64 && (c.g.dims == 2 || c.g.dims == 3) && c.g.Lx % 128 == 0 && c.g.Lx <= 65536 &&
           c.g.N <= (int64_t)1 << 32;
}

template <int D, int RULE, bool HJ>
static hipError_t launch_msc_t(const MscArgs &a, int count, hipStream_t s)
{
    const int64_t tasks = (a.N >> 1) >> 6;
    // Without E, M as many waves as fit at once (eight per SIMD), each walking
    // its share of the tasks.  With them one workgroup per CU of up to sixteen
    // waves, as few as give every task one: each workgroup adds 128 numbers to
    // the same eight lines, which takes 1024 workgroups 40 us whatever the
    // lattice (us per sweep at four waves each: 512 x 1024 57.8, then 24.2;
    // 1024^2 66, 35; 128 x 64^2 heat-bath 60, 26; 4096^2 296, 296).
    if (!a.EM) {
        const dim3 grid((unsigned)std::min<int64_t>((tasks + 3) / 4, 2048), (unsigned)count);
        hipLaunchKernelGGL((k_msc<D, false, RULE, HJ>), grid, dim3(256), 0, s, a);
        return hipGetLastError();
    }
    constexpr int64_t kCUs = 256;
    int waves = 4;
    while (waves < kMscWaves && tasks > kCUs * waves) waves *= 2;
    const dim3 grid((unsigned)std::min<int64_t>((tasks + waves - 1) / waves, kCUs), (unsigned)count);
    hipLaunchKernelGGL((k_msc<D, true, RULE, HJ>), grid, dim3(64 * waves), 0, s, a);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_msc_r(const MscArgs &a, int rule, int count, hipStream_t s)
{
    const bool hj = a.J != nullptr;
    switch (rule) {
    case kMetropolis: return hj ? launch_msc_t<D, kMetropolis, true>(a, count, s) : launch_msc_t<D, kMetropolis, false>(a, count, s);
    case kHeatBath: return hj ? launch_msc_t<D, kHeatBath, true>(a, count, s) : launch_msc_t<D, kHeatBath, false>(a, count, s);
    default: return hj ? launch_msc_t<D, kHeatBathMirrored, true>(a, count, s) : launch_msc_t<D, kHeatBathMirrored, false>(a, count, s);
    }
}

// One half-sweep (colour c) of every word lattice; EM: this sweep's per-lane
// (E, M), accumulated (cleared by the caller), in the odd half-sweep only.
hipError_t launch_msc_phase(const SweepCall &c, uint64_t *words, uint64_t sweep, int phase, int64_t *EM,
                            hipStream_t s)
{
    MscArgs a;
    a.w = words;
    a.J = c.J;
    a.Lx = c.g.Lx;
    a.Ly = c.g.Ly;
    a.Lz = c.g.dims == 3 ? c.g.Lz : 1;
    a.N = c.g.N;
    a.seed_lo = c.seed_lo;
    a.seed_hi = c.seed_hi;
    a.replica0 = c.replica0;
    a.sweep_lo = (uint32_t)sweep;
    a.w3 = ctr_w3(kTagSweep, (uint32_t)phase, sweep);
    a.w3lo = ctr_w3(kTagSweepLo, (uint32_t)phase, sweep);
    a.c = phase;
    const int z = 2 * c.g.dims;
    for (int cl = 0; cl < 8; ++cl) {
        Thr th{0u, 0u};
        if (c.rule == 0) {
            if (2 * cl < z) th = c.tab.met[z / 2 - cl];   // dE = 2z - 4a
        } else if (cl <= z) {
            th = c.tab.hb[z - 2 * cl + 6];                // h = z - 2d
        }
        if (th.top >= 256u) th = Thr{255u, 1u << 24};
        a.top[cl] = th.top;
        a.low[cl] = th.low;
    }
    a.EM = phase == 1 ? EM : nullptr;
    const int rule = c.rule == 0 ? kMetropolis : mirrored_classes(a.top, z) ? kHeatBathMirrored : kHeatBath;
    if (c.g.dims == 2) return launch_msc_r<2>(a, rule, c.g.count, s);
    return launch_msc_r<3>(a, rule, c.g.count, s);
}

}  // namespace mcs
