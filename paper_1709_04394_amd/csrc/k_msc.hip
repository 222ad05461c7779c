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
//    replica bit for bit).  A 64 x 64 bit transpose of all eight planes at once
//    (lane_bits.hpp) turns "replica b, 64 sites" into "site s, 64 replicas";
//    then each lane compares its site's 64 replicas against their classes'
//    thresholds bit-serially.
//  * Words with ties (a replica whose top byte equals its class's threshold's,
//    one word in seven at criticality) wait in a queue of their wave, across
//    tasks, and are settled 64 at a time, one word per lane; their spins are
//    stored then.
//  * Per-sweep E and M per replica are counted in the odd half-sweep: each lane
//    adds the unsatisfied bonds and down spins of its sites to bit-sliced
//    counters of the 64 replicas, which are summed over the lanes once in 32
//    tasks; one atomic per replica and workgroup.
//
// What bounds it: VALU issue.  4096^2, 64 replicas, Metropolis: 133 us per
// even half-sweep and 173 with E, M, against 238 and 311 with a transpose per
// plane through ds_swizzle (36 instructions per word), a transpose back for
// every count of every task, rows by 64-bit division, and ties drawn in place.
#include <algorithm>

#include "internal.hpp"
#include "lane_bits.hpp"
#include "metro2d.hpp"

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

template <int DIMS, bool MEASURE, bool HB, bool HASJ>
__global__ __launch_bounds__(MEASURE ? 64 * kMscWaves : 256) void k_msc(MscArgs a)
{
    constexpr int WAVES = MEASURE ? kMscWaves : 4;
    __shared__ uint32_t tlow[8];
    __shared__ long long red[2][64];
    // tied words: {word, same-colour index, tied replicas}, {word with those
    // unsettled, class bit 0}, {class bits 1, 2}
    __shared__ uint4 q_id[WAVES][kTieQueue], q_s[WAVES][kTieQueue], q_c[(HB || DIMS == 3) ? WAVES : 1][kTieQueue];
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
            if (i < (HB ? DIMS : 1)) asm volatile("" : "+v"(tv[k][i]));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) ts[k][i] = ((a.top[i < 3 ? 2 * i + 1 : 6] >> k) & 1u) ? ~0u : 0u;
    }
    uint32_t qn = 0;
    auto settle = [&]() {
        const uint32_t q = tid & 63;
        if (q < qn) {
            const uint4 id = q_id[wave][q], sw = q_s[wave][q];
            uint4 cw = make_uint4(0u, 0u, 0u, 0u);
            if (HB || DIMS == 3) cw = q_c[wave][q];
            uint64_t pend = ((uint64_t)id.w << 32) | id.z, S = ((uint64_t)sw.y << 32) | sw.x;
            const uint64_t c0 = ((uint64_t)sw.w << 32) | sw.z, c1 = ((uint64_t)cw.y << 32) | cw.x,
                           c2 = ((uint64_t)cw.w << 32) | cw.z;
            while (pend) {
                const int b = __builtin_ctzll(pend);
                pend &= pend - 1ull;
                const uint32_t cls = (uint32_t)((c0 >> b) & 1ull) | ((uint32_t)((c1 >> b) & 1ull) << 1) |
                                     ((uint32_t)((c2 >> b) & 1ull) << 2);
                const uint4 lo =
                    philox(make_uint4(id.y, rep0 + (uint32_t)b, a.sweep_lo, a.w3lo), a.seed_lo, a.seed_hi);
                // Metropolis: flip; heat-bath: the provisional -1 becomes +1
                if ((lo.x & 0xFFFFFFu) < tlow[cls]) {
                    if (MEASURE) {
                        // unsatisfied bonds gained: Metropolis z - 2a, heat-bath 2d - z
                        const int du = HB ? 2 * (int)cls - Z : Z - 2 * (int)cls;
                        atomicAdd((unsigned long long *)&red[0][b], (unsigned long long)(long long)(2 * du));
                        atomicAdd((unsigned long long *)&red[1][b],
                                  (unsigned long long)(((S >> b) & 1ull) ? 2ll : -2ll));
                    }
                    S ^= 1ull << b;
                }
            }
            w[id.x] = S;
        }
        qn = 0;
    };
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
        // random planes: lane = replica, 4 groups of 16 sites -> transpose
        uint4 B[4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
            B[g] = philox(make_uint4((j0 >> 4) + (uint32_t)g, rep0 + (uint32_t)lb.label, a.sweep_lo, a.w3), a.seed_lo,
                          a.seed_hi);
        transpose_blocks(B, lb);
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
        uint32_t So[2], pend[2], C0[2], C1[2], C2[2];
        uint64_t u[3] = {0, 0, 0}, dn[2] = {0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // replicas 32 h .. 32 h + 31
            const uint32_t Sh = (uint32_t)(S >> (32 * h));
            // wk: bit set <=> J s_j = -1; Metropolis counts unsatisfied bonds
            // S ^ wk, heat-bath counts wk
            uint32_t wk[6], xk[6];
#pragma unroll
            for (int k = 0; k < Z; ++k) {
                wk[k] = (uint32_t)((n[k] ^ jm[k]) >> (32 * h));
                xk[k] = HB ? wk[k] : (wk[k] ^ Sh);
            }
            uint32_t c0, c1, c2;
            count_words<Z>(xk, c0, c1, c2);
            // Metropolis: a >= z/2 gives dE <= 0
            const uint32_t ge = HB ? 0u : DIMS == 3 ? MCS_BOP3(c2, c1, c0, MCS_A | (MCS_B & MCS_C)) : (c2 | c1);
            uint32_t lt = 0u, eq = ~0u;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t X = plane_pair(B[2 * h], B[2 * h + 1], k);
                auto mux = [](uint32_t sel, uint32_t hi, uint32_t lo) {
                    return MCS_BOP3(sel, hi, lo, (MCS_A & MCS_B) | (~MCS_A & MCS_C));
                };
                uint32_t T = mux(c0, ts[k][0], tv[k][0]);  // classes 0, 1
                if (HB) {
                    T = mux(c1, mux(c0, ts[k][1], tv[k][1]), T);
                    T = DIMS == 3 ? mux(c2, mux(c1, ts[k][3], mux(c0, ts[k][2], tv[k][2])), T) : mux(c2, tv[k][2], T);
                } else if (DIMS == 3) {
                    T = mux(c1, tv[k][1], T);
                }
                lt = MCS_BOP3(X, T, lt, (~MCS_A & MCS_B) | (~MCS_A & MCS_C) | (MCS_B & MCS_C));
                eq = MCS_BOP3(eq, X, T, MCS_A & ~(MCS_B ^ MCS_C));
            }
            So[h] = HB ? ~lt : MCS_BOP3(Sh, ge, lt, MCS_A ^ (MCS_B | MCS_C));
            pend[h] = HB ? eq : (eq & ~ge);
            C0[h] = c0;
            C1[h] = c1;
            C2[h] = c2;
            if (MEASURE) {
                // odd sites: their bonds after the update; both sites of the pair
                // (this odd site and the even site at the same row position) for M
                uint32_t uk[6], v0, v1, v2;
#pragma unroll
                for (int k = 0; k < Z; ++k) uk[k] = So[h] ^ wk[k];
                count_words<Z>(uk, v0, v1, v2);
                const uint32_t pw = (uint32_t)((par ? n[1] : n[0]) >> (32 * h));  // even site 2m + (1 - par)
                u[0] |= (uint64_t)v0 << (32 * h);
                u[1] |= (uint64_t)v1 << (32 * h);
                u[2] |= (uint64_t)v2 << (32 * h);
                dn[0] |= (uint64_t)(So[h] ^ pw) << (32 * h);
                dn[1] |= (uint64_t)(So[h] & pw) << (32 * h);
            }
        }
        const bool tied = (pend[0] | pend[1]) != 0u;
        if (!tied) (w + rbase)[x] = ((uint64_t)So[1] << 32) | So[0];
        const uint64_t m = __ballot(tied);
        const uint32_t cnt = (uint32_t)__popcll(m);
        if (qn + cnt > (uint32_t)kTieQueue) settle();
        if (tied) {
            const uint32_t at = qn + wave_rank(m);
            q_id[wave][at] = make_uint4((uint32_t)(rbase + x), j0 + (uint32_t)lb.label, pend[0], pend[1]);
            q_s[wave][at] = make_uint4(So[0], So[1], C0[0], C0[1]);
            if (HB || DIMS == 3) q_c[wave][at] = make_uint4(C1[0], C1[1], C2[0], C2[1]);
        }
        qn += cnt;
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
    settle();
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

template <int D, bool HB, bool HJ>
static hipError_t launch_msc_t(const MscArgs &a, int count, hipStream_t s)
{
    const int64_t tasks = (a.N >> 1) >> 6;
    // Without E, M as many waves as fit at once (eight per SIMD), each walking
    // its share of the tasks.  With them one workgroup per CU of up to sixteen
    // waves, as few as give every task one: each workgroup adds 128 numbers to
    // the same eight lines, which takes 1024 workgroups 40 us whatever the
    // lattice (us per sweep at four waves each: 512 x 1024 57.8, now 24.2;
    // 1024^2 66, 35; 128 x 64^2 heat-bath 60, 26; 4096^2 296, 296).
    if (!a.EM) {
        const dim3 grid((unsigned)std::min<int64_t>((tasks + 3) / 4, 2048), (unsigned)count);
        hipLaunchKernelGGL((k_msc<D, false, HB, HJ>), grid, dim3(256), 0, s, a);
        return hipGetLastError();
    }
    constexpr int64_t kCUs = 256;
    int waves = 4;
    while (waves < kMscWaves && tasks > kCUs * waves) waves *= 2;
    const dim3 grid((unsigned)std::min<int64_t>((tasks + waves - 1) / waves, kCUs), (unsigned)count);
    hipLaunchKernelGGL((k_msc<D, true, HB, HJ>), grid, dim3(64 * waves), 0, s, a);
    return hipGetLastError();
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
    const bool hb = c.rule == 1, hj = c.J != nullptr;
    if (c.g.dims == 2) {
        if (hb) return hj ? launch_msc_t<2, true, true>(a, c.g.count, s) : launch_msc_t<2, true, false>(a, c.g.count, s);
        return hj ? launch_msc_t<2, false, true>(a, c.g.count, s) : launch_msc_t<2, false, false>(a, c.g.count, s);
    }
    if (hb) return hj ? launch_msc_t<3, true, true>(a, c.g.count, s) : launch_msc_t<3, true, false>(a, c.g.count, s);
    return hj ? launch_msc_t<3, false, true>(a, c.g.count, s) : launch_msc_t<3, false, false>(a, c.g.count, s);
}

}  // namespace mcs
