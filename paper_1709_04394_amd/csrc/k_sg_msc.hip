// k_sg_msc.hip -- checkerboard half-sweep of +-J spin glasses multi-spin
// coded across 64 disorder realisations (Sec. "Disordered systems": the bits
// of a word are 64 realisations, each with its own couplings, and the coded
// copies share one random number per site, the choice the section reports
// for spin-glass codes).
//
// One lane per site, 64 realisations per word: the neighbour words and the
// per-realisation coupling words give every realisation's class (unsatisfied
// bonds for Metropolis, neighbours with J s_j = -1 for heat-bath) as a
// bit-sliced count.  The site's single 32-bit draw (the byte-lazy stream of
// the word lattice's replica id) is compared once with each class threshold;
// the outcomes, all-ones or zero per class, are selected per realisation by
// the bits of its class.  A lane whose top byte equals a threshold's draws the
// low 24 bits once for all realisations.  Per-sweep E and M per realisation
// are bit-sliced counters of the odd half-sweep, summed over the lanes every
// few tasks (lane_bits.hpp).
//
// What bounds it: memory.  A half-sweep reads every coupling word once and
// every spin word, and writes half of those.  32^3, 4096 realisations (75 MB):
// 15.0 us per even half-sweep, 5.0 TB/s, against 25.6 with workgroups dealt
// round the L2 caches (each then read most rows' words and couplings again)
// and rows by 64-bit division; 21.3 with E, M (21.7 with the workgroup's share
// of the tasks and a task's first row divided out in 64 bits), against 33.4 with five 64 x 64
// transposes per task.  Couplings loaded past the caches (non-temporal) cost
// 15 %: a line of them serves two rows.
#include <algorithm>

#include "internal.hpp"
#include "lane_bits.hpp"

namespace mcs {

struct SgMscArgs {
    uint64_t *w;          // [count][N] spin words, bit b = realisation 64 l + b (set <=> s = -1)
    const uint64_t *J;    // [count][dims][N] coupling words of bond (i, i + e_d) (set <=> J < 0)
    int Lx, Ly, Lz;
    int64_t N;
    uint32_t seed_lo, seed_hi, replica0;
    uint32_t sweep_lo, w3, w3lo;
    int c;                // colour of this half-sweep
    // class thresholds (top byte, low 24 bits; T = 2^32 encoded as top 256):
    // Metropolis class a = unsatisfied bonds < z/2, T of dE = 2z - 4a;
    // heat-bath class d = neighbours with J s_j = -1, T of h = z - 2d
    uint32_t top[8], low[8];
    int64_t *EM;          // this sweep's [count * 64][2], or nullptr
    uint32_t parts;       // workgroups per lattice
    uint32_t per, extra;  // tasks of 64 sites of a lattice: parts per + extra
    uint32_t total;       // workgroups with work
    // n / (Lx / 2) and n / Ly as the high word of a product, for n below the
    // divisor + 64 (the divisor < 64; else the quotient is n >= divisor)
    uint32_t mul_hx, mul_ly;
};

// Workgroups of a launch, over all lattices.  Without E, M a wave takes one
// task where there are enough: all its loads are then in flight with those of
// seven others on its SIMD (32^3, 64 words per site: 15.0 us at 4096 or 8192
// workgroups, 17.8 at 2048, 18.7 at 1024).  With E, M four tasks share a sum of
// the counters over the lanes and the registers hold five waves (odd
// half-sweep: 21.7 us at 1024 or 2048, 28 at 4096).
constexpr int kSgBlocks = 4096, kSgBlocksEM = 1024;
// Tasks between sums of the bit-sliced counters: four keep them at 18 registers
// (32 tasks: 30 registers, and 25 us per odd half-sweep).
constexpr int kSgFlush = 4, kSgPlanes = 5;

// n / d for n < d + 64
__device__ __forceinline__ uint32_t small_quotient(uint32_t n, uint32_t d, uint32_t mul)
{
    return d >= 64u ? (n >= d ? 1u : 0u) : __umulhi(n, mul);
}

// I: the type of byte offsets within a lattice
template <int DIMS, bool MEASURE, bool HB, class I>
__global__ __launch_bounds__(256, 5) void k_sg_msc(SgMscArgs a)
{
    __shared__ int red[2][4][64];
    constexpr int Z = 2 * DIMS;
    constexpr int NC = HB ? Z + 1 : DIMS;  // heat-bath d = 0..z; Metropolis a = 0 .. z/2 - 1
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // neighbouring rows' words and couplings are read on the same XCD
    const uint32_t g = xcd_order(blockIdx.x, gridDim.x);
    if (g >= a.total) return;
    const uint32_t l = g / a.parts, part = g - l * a.parts;
    const LaneBits lb = lane_bits(tid & 63);
    char *w = (char *)(a.w + (int64_t)l * a.N);
    const char *J0 = (const char *)(a.J + (int64_t)l * DIMS * a.N);
    const char *J1 = J0 + a.N * 8, *J2 = J1 + (DIMS == 3 ? a.N * 8 : 0);
    auto at = [](const char *p, I off) { return *(const uint64_t *)(p + off); };
    const uint32_t hx = (uint32_t)a.Lx >> 1;
    const uint32_t rep = a.replica0 + l;  // the shared stream of the 64 realisations
    const I row_b = (I)a.Lx * 8, plane_b = (I)a.Ly * row_b;
    BitCounter<kSgPlanes> cu;      // unsatisfied bonds of the odd sites, up to 6 a task
    BitCounter<kSgPlanes - 1> cd;  // down spins of both sites of a pair
    int u_acc = 0, d_acc = 0;
    int since = 0;
    uint32_t done = 0;
    if (MEASURE) {
        cu.clear();
        cd.clear();
    }
    auto flush = [&]() {
        u_acc += cu.flush(lb, 32 - __builtin_clz((unsigned)(Z * since)));
        d_acc += cd.flush(lb, 32 - __builtin_clz((unsigned)(2 * since)));
        since = 0;
    };
    // tasks of this workgroup: the first a.extra have one more
    const uint32_t t0 = part * a.per + min(part, a.extra), t1 = t0 + a.per + (part < a.extra ? 1u : 0u);
    for (uint32_t t = t0 + (uint32_t)wave; t < t1; t += 4u) {
        // lane: same-colour site j = 64 t + lane (at most 2^31 of them)
        const uint32_t j0 = t << 6, row0 = j0 / hx;
        const uint32_t z0 = row0 / (uint32_t)a.Ly, y0 = row0 - z0 * (uint32_t)a.Ly;
        const uint32_t mm = j0 - row0 * hx + (uint32_t)(tid & 63);
        const uint32_t dr = small_quotient(mm, hx, a.mul_hx);
        const uint32_t yy = y0 + dr, dz = small_quotient(yy, (uint32_t)a.Ly, a.mul_ly);
        const uint32_t m = mm - dr * hx, y = yy - dz * (uint32_t)a.Ly, z = z0 + dz;
        const uint32_t par = ((uint32_t)a.c + y + z) & 1u;
        const I xb = (I)(2u * m + par) * 8, rb = (I)(row0 + dr) * row_b;
        const I xpb = xb + 8 == row_b ? 0 : xb + 8, xmb = xb == 0 ? row_b - 8 : xb - 8;
        const I ryp = y + 1 == (uint32_t)a.Ly ? rb - (plane_b - row_b) : rb + row_b;
        const I rym = y == 0 ? rb + (plane_b - row_b) : rb - row_b;
        const uint64_t S = at(w, rb + xb);
        uint64_t n[6] = {0, 0, 0, 0, 0, 0}, jw[6] = {0, 0, 0, 0, 0, 0};
        n[0] = at(w, rb + xpb), jw[0] = at(J0, rb + xb);
        n[1] = at(w, rb + xmb), jw[1] = at(J0, rb + xmb);
        n[2] = at(w, ryp + xb), jw[2] = at(J1, rb + xb);
        n[3] = at(w, rym + xb), jw[3] = at(J1, rym + xb);
        if (DIMS == 3) {
            const I vol_b = (I)a.Lz * plane_b;
            const I rzp = z + 1 == (uint32_t)a.Lz ? rb - (vol_b - plane_b) : rb + plane_b;
            const I rzm = z == 0 ? rb + (vol_b - plane_b) : rb - plane_b;
            n[4] = at(w, rzp + xb), jw[4] = at(J2, rb + xb);
            n[5] = at(w, rzm + xb), jw[5] = at(J2, rzm + xb);
        }
        // the site's one draw: top byte from block j / 16 (bit k = bit j mod 16
        // of half-word k), compared once with each class threshold
        const uint32_t jl = j0 + (uint32_t)(tid & 63);
        const uint4 B = philox(make_uint4(jl >> 4, rep, a.sweep_lo, a.w3), a.seed_lo, a.seed_hi);
        const uint32_t top = byte_of(B, jl & 15u);
        uint32_t acc[NC];
        bool tie = false;
#pragma unroll
        for (int d = 0; d < NC; ++d) {
            acc[d] = top < a.top[d] ? ~0u : 0u;
            tie |= top == a.top[d];
        }
        if (tie) {
            const uint4 lo = philox(make_uint4(jl, rep, a.sweep_lo, a.w3lo), a.seed_lo, a.seed_hi);
#pragma unroll
            for (int d = 0; d < NC; ++d)
                if (top == a.top[d] && (lo.x & 0xFFFFFFu) < a.low[d]) acc[d] = ~0u;
        }
        uint64_t Sn = 0, u[3] = {0, 0, 0}, dn[2] = {0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // realisations 32 h .. 32 h + 31
            const uint32_t Sh = (uint32_t)(S >> (32 * h));
            // wk: bit set <=> J s_j = -1; Metropolis counts unsatisfied bonds
            // S ^ wk, heat-bath counts wk
            uint32_t wk[6], xk[6];
#pragma unroll
            for (int k = 0; k < Z; ++k) {
                const uint32_t nk = (uint32_t)(n[k] >> (32 * h)), jk = (uint32_t)(jw[k] >> (32 * h));
                wk[k] = nk ^ jk;
                xk[k] = HB ? wk[k] : xor3(nk, jk, Sh);
            }
            uint32_t c0, c1, c2;
            count_words<Z>(xk, c0, c1, c2);
            auto mux = [](uint32_t sel, uint32_t hi, uint32_t lo) {
                return MCS_BOP3(sel, hi, lo, (MCS_A & MCS_B) | (~MCS_A & MCS_C));
            };
            uint32_t t = mux(c0, acc[1], acc[0]), so;
            if constexpr (HB) {
                t = mux(c1, mux(c0, acc[3], acc[2]), t);
                if constexpr (DIMS == 3) t = mux(c2, mux(c1, acc[6], mux(c0, acc[5], acc[4])), t);
                else t = mux(c2, acc[4], t);
                so = ~t;  // s' = +1 (bit clear) where r < T
            } else {
                // a >= z/2 gives dE <= 0: flipped in any case
                uint32_t ge = c1 | c2;
                if constexpr (DIMS == 3) {
                    t = mux(c1, acc[2], t);
                    ge = MCS_BOP3(c2, c1, c0, MCS_A | (MCS_B & MCS_C));
                }
                so = MCS_BOP3(Sh, ge, t, MCS_A ^ (MCS_B | MCS_C));
            }
            Sn |= (uint64_t)so << (32 * h);
            if (MEASURE) {
                // odd sites: the realisations' bond counts after the update; both
                // sites of the pair (this odd site and its even partner of the
                // same row position) for M
                uint32_t uk[6], v0, v1, v2;
#pragma unroll
                for (int k = 0; k < Z; ++k) uk[k] = so ^ wk[k];
                count_words<Z>(uk, v0, v1, v2);
                const uint32_t pw = (uint32_t)((par ? n[1] : n[0]) >> (32 * h));
                u[0] |= (uint64_t)v0 << (32 * h);
                u[1] |= (uint64_t)v1 << (32 * h);
                u[2] |= (uint64_t)v2 << (32 * h);
                dn[0] |= (uint64_t)(so ^ pw) << (32 * h);
                dn[1] |= (uint64_t)(so & pw) << (32 * h);
            }
        }
        *(uint64_t *)(w + (rb + xb)) = Sn;
        if (MEASURE) {
            cu.add(u);
            cd.add(dn);
            ++done;
            if (++since == kSgFlush) flush();
        }
    }
    if (MEASURE) {
        if (since) flush();
        // E: 2 (unsatisfied) - z per odd site; M: 2 - 2 (down) per pair
        red[0][wave][lb.label] = 2 * u_acc - 64 * Z * (int)done;
        red[1][wave][lb.label] = 128 * (int)done - 2 * d_acc;
        __syncthreads();
        if (tid < 128) {
            const int q = tid & 1, b = tid >> 1;
            const long long v = (long long)red[q][0][b] + red[q][1][b] + red[q][2][b] + red[q][3][b];
            atomicAdd((unsigned long long *)&a.EM[128 * (int64_t)l + tid], (unsigned long long)v);
        }
    }
}

// Couplings of realisations realisation0 + 64 l + b, bit b of word (l, d, i):
// set iff byte (b' mod 16) of Philox(ctr = (b' / 16, realisation, 0,
// TAG_COUPLING << 24)) is >= 128, b' = d N + i (the int8 couplings' stream
// with counter word 1 = the realisation).  One thread per (bond group of 16,
// lattice), 64 realisations in a loop.
__global__ void k_couplings_msc64(uint64_t *J, int64_t bonds, uint32_t realisation0, uint32_t k0, uint32_t k1)
{
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int l = blockIdx.y;
    if (g * 16 >= bonds) return;
    uint64_t out[16] = {};
    for (int b = 0; b < 64; ++b) {
        const uint32_t rz = realisation0 + 64u * (uint32_t)l + (uint32_t)b;
        const uint4 blk = philox(make_uint4((uint32_t)g, rz, 0u, ctr_w3(kTagCoupling, 0, 0)), k0, k1);
#pragma unroll
        for (int k = 0; k < 16; ++k) out[k] |= (uint64_t)(top_bit_of(blk, (uint32_t)k)) << b;
    }
    uint64_t *Jl = J + (int64_t)l * bonds;
    for (int k = 0; k < 16 && g * 16 + k < bonds; ++k) Jl[g * 16 + k] = out[k];
}

hipError_t launch_couplings_msc64(const Geom &g, uint64_t *J, uint64_t seed, uint32_t realisation0, hipStream_t s)
{
    const int64_t bonds = (int64_t)g.dims * g.N;
    const int64_t groups = (bonds + 15) / 16;
    dim3 grid((unsigned)((groups + 255) / 256), (unsigned)g.count);
    hipLaunchKernelGGL(k_couplings_msc64, grid, dim3(256), 0, s, J, bonds, realisation0, (uint32_t)seed,
                       (uint32_t)(seed >> 32));
    return hipGetLastError();
}

bool sg_msc_supported(const Geom &g) { return (g.dims == 2 || g.dims == 3) && ((g.N >> 1) % 64) == 0; }

template <int D, bool HB, class I>
static hipError_t launch_sg_t(const SgMscArgs &a, hipStream_t s)
{
    const dim3 grid((a.total + 7u) & ~7u);
    if (a.EM) hipLaunchKernelGGL((k_sg_msc<D, true, HB, I>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_sg_msc<D, false, HB, I>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int D, bool HB>
static hipError_t launch_sg_i(const SgMscArgs &a, hipStream_t s)
{
    return a.N < (int64_t)1 << 29 ? launch_sg_t<D, HB, uint32_t>(a, s) : launch_sg_t<D, HB, uint64_t>(a, s);
}

hipError_t launch_sg_msc_phase(const Geom &g, int rule, const SweepTables &tab, uint64_t *words, const uint64_t *J,
                               uint32_t seed_lo, uint32_t seed_hi, uint32_t replica0, uint64_t sweep, int phase,
                               int64_t *EM, hipStream_t s)
{
    SgMscArgs a;
    a.w = words;
    a.J = J;
    a.Lx = g.Lx;
    a.Ly = g.Ly;
    a.Lz = g.dims == 3 ? g.Lz : 1;
    a.N = g.N;
    a.seed_lo = seed_lo;
    a.seed_hi = seed_hi;
    a.replica0 = replica0;
    a.sweep_lo = (uint32_t)sweep;
    a.w3 = ctr_w3(kTagSweep, (uint32_t)phase, sweep);
    a.w3lo = ctr_w3(kTagSweepLo, (uint32_t)phase, sweep);
    a.c = phase;
    const int z = 2 * g.dims;
    for (int cl = 0; cl < 8; ++cl) {
        Thr th{0u, 0u};
        if (rule == 0) {
            if (2 * cl < z) th = tab.met[z / 2 - cl];  // dE = 2z - 4a
        } else if (cl <= z) {
            th = tab.hb[z - 2 * cl + 6];               // h = z - 2d
        }
        a.top[cl] = th.top;
        a.low[cl] = th.low;
    }
    a.EM = phase == 1 ? EM : nullptr;
    // as many workgroups as are resident at once, in equal parts of a lattice
    const uint32_t tasks = (uint32_t)(a.N >> 7);
    const int64_t resident = a.EM ? kSgBlocksEM : kSgBlocks;
    a.parts = (uint32_t)std::min<int64_t>((tasks + 3) / 4, std::max<int64_t>(1, (resident + g.count - 1) / g.count));
    a.total = a.parts * (uint32_t)g.count;
    a.per = tasks / a.parts;
    a.extra = tasks % a.parts;
    const uint32_t hx = (uint32_t)g.Lx >> 1;
    a.mul_hx = (uint32_t)((((uint64_t)1 << 32) + hx - 1) / hx);
    a.mul_ly = (uint32_t)((((uint64_t)1 << 32) + (uint32_t)g.Ly - 1) / (uint32_t)g.Ly);
    if (g.dims == 2) return rule ? launch_sg_i<2, true>(a, s) : launch_sg_i<2, false>(a, s);
    return rule ? launch_sg_i<3, true>(a, s) : launch_sg_i<3, false>(a, s);
}

}  // namespace mcs
