// k_whole.hip -- checkerboard sweeps of small int8 lattices held whole, as
// bits, in one workgroup's LDS: any even extents, 2D or 3D, J = 1 or +-J,
// Metropolis or heat-bath (Sec. "Checkerboard scheme"; Sec. "Disordered
// systems").  One workgroup per lattice runs every sweep of a call in a single
// launch with one barrier per half-sweep.
//
// Layout: the sites of a colour in the order of their index j = m + (Lx / 2)
// (y + Ly z), 32 to a word, set bit = spin -1, rows following one another
// without gaps.  A thread updates whole words, or halves of them: two Philox
// blocks (one) give the bit-planes of their sites whatever the row length.  The neighbours of
// the sites j are bits of the other colour's words at fixed distances: j (the
// partner in the pair of columns), j - 1 or j + 1 by the row's parity, j +- Lx/2
// (y), j +- Lx Ly / 2 (z).  Those are windows of 32 bits that start at any bit
// and run round the end of the array, which is the periodic boundary of the
// last dimension; the other boundaries are bits that masks take from another
// window (a row's first site has its left neighbour at j - 1 + Lx/2).
// The bonds' couplings are stored per neighbour, at their site's bit.
// Only colour-c words are written and only colour-(1-c) words are read in a
// half-sweep.
//
// Sites 2m and 2m + 1 of a row are bytes 2j and 2j + 1 of the lattice, so a
// word pair is packed from 64 consecutive bytes.
//
// Randomness is that of every half-sweep: site j draws byte j mod 16 of
// Philox(j / 16, replica, sweep, SWEEP | c) and, on a tie with the threshold's
// top byte, the low 24 bits from Philox(j, .., SWEEP_LO | c).  E and M are
// popcounts of the odd half-sweep (every bond has one odd site).
//
// What bounds it: up to about 10^4 sites the issue of single waves (a half-sweep
// is 0.5 to 0.7 us: windows, bit-serial comparison, ties, barrier), above it the
// VALU of the one CU.  us per sweep of long calls with E, M, against a byte per
// site in LDS (rows of 32 sites: a 16-bit word per row and parity): 64^2 1.14
// (3.8), 128^2 1.6 (11.5), 200^2 heat-bath 3.0 (25), 300^2 5.0 (58), 30^3 +-J 2.9
// (23), 32^3 +-J 2.6 (5.7), 32 x 64^2 +-J 8.0 (18).  A half that is a multiple of
// 32 repeats word 0 after the last and needs no test for the end (64^2 1.43
// against 1.59).  One wave that settles the ties of all between two barriers
// made 128^2 2.5 and 32^3 3.0: its latency is longer than the passes it saves.
#include <algorithm>

#include "heatbath.hpp"
#include "internal.hpp"
#include "lane_bits.hpp"
#include "metro2d.hpp"
#include "spin_bytes.hpp"

namespace mcs {

struct WholeArgs {
    int8_t *spins;
    const int8_t *J;      // [dims][N] or nullptr
    uint32_t Ly, hx;
    uint32_t half;        // sites of a colour
    uint32_t area;        // of them in a plane (3D)
    uint32_t words;       // ceil(half / 32)
    uint32_t mul_hx, mul_ly;  // floor((2^32 - 1) / hx), the same of Ly
    uint32_t seed_lo, seed_hi, replica0;
    uint64_t sweep0;
    int nsweeps;
    uint32_t mask[8][8];  // [bit of the top byte][class]: all ones iff set (classes as in k_half.hip)
    uint32_t low[8];
    int64_t *EM;          // [nsweeps][count][2] or nullptr
    int64_t em_stride;
};

// A thread's sites: 32, or 16 for lattices of few words.
template <int BITS>
struct WholeItem;
template <>
struct WholeItem<32> {
    using type = uint32_t;
};
template <>
struct WholeItem<16> {
    using type = uint16_t;
};

constexpr int kWholePad = 2;  // words read past the last one (their bits are not used)

// 33 or more bits of an array of `half` bits from bit pos (0 <= pos < half),
// round its end.  ALIGNED: half is a multiple of 32 and word 0 is repeated after
// the last.
template <bool ALIGNED>
__device__ __forceinline__ uint64_t bit_window(const uint32_t *v, uint32_t pos, uint32_t half)
{
    const uint32_t q = pos >> 5;
    uint64_t r = (((uint64_t)v[q + 1] << 32) | v[q]) >> (pos & 31u);
    if (ALIGNED) return r;
    const uint32_t rem = half - pos;
    if (rem < 33u) r = (r & ((1ull << rem) - 1ull)) | ((((uint64_t)v[1] << 32) | v[0]) << rem);
    return r;
}

// What an item's sites share in every half-sweep.
struct WordGeo {
    uint32_t w;                 // item number
    uint32_t odd;               // sites in rows with y + z odd
    uint32_t first, last;       // first and last sites of their rows
    uint32_t top, bottom;       // 3D: sites with y = Ly - 1, y = 0
    uint32_t valid;
};

// j0 + d round the end of the array, d < half.
__device__ __forceinline__ uint32_t wrap_add(uint32_t j0, uint32_t d, uint32_t half)
{
    const uint32_t p = j0 + d;
    return p < p - half ? p : p - half;
}

template <int DIMS, int BITS>
__device__ __forceinline__ WordGeo word_geo(const WholeArgs &a, uint32_t w)
{
    constexpr uint32_t ALL = BITS == 32 ? ~0u : 0xFFFFu;
    WordGeo g;
    const uint32_t j0 = BITS * w;
    g.w = w;
    g.odd = g.first = g.last = g.top = g.bottom = 0u;
    const uint32_t row = quotient28(j0, a.hx, a.mul_hx);
    uint32_t m = j0 - row * a.hx, z = quotient28(row, a.Ly, a.mul_ly), y = row - z * a.Ly;
    for (uint32_t s = 0; s < BITS;) {
        const uint32_t e = s + (a.hx - m), end = e < BITS ? e : BITS;
        const uint32_t seg = (end < BITS ? (1u << end) - 1u : ALL) & ~((1u << s) - 1u);
        if (m == 0) g.first |= 1u << s;
        if (e <= BITS) g.last |= 1u << (e - 1u);
        if ((y + z) & 1u) g.odd |= seg;
        if (y == 0) g.bottom |= seg;
        if (y + 1 == a.Ly) g.top |= seg;
        s = end;
        m = 0;
        if (++y == a.Ly) {
            y = 0;
            ++z;
        }
    }
    g.valid = a.half - j0 < BITS ? (1u << (a.half - j0)) - 1u : ALL;
    return g;
}

// Rows of 32 sites, BITS = 32: an item is rows 2w and 2w + 1, of one plane.
__device__ __forceinline__ WordGeo word_geo_rows32(const WholeArgs &a, uint32_t w)
{
    WordGeo g;
    const uint32_t row = 2u * w, z = quotient28(row, a.Ly, a.mul_ly), y = row - z * a.Ly;
    g.w = w;
    g.odd = (z & 1u) ? 0x0000FFFFu : 0xFFFF0000u;
    g.first = 0x00010001u;
    g.last = 0x80008000u;
    g.top = y + 2u == a.Ly ? 0xFFFF0000u : 0u;
    g.bottom = y == 0u ? 0x0000FFFFu : 0u;
    g.valid = ~0u;
    return g;
}

// A thread's items in that case: any number of them, nothing kept.
struct Rows32Items {
    const WholeArgs &a;
    uint32_t tid, nt;
    __device__ __forceinline__ WordGeo operator[](int k) const { return word_geo_rows32(a, tid + k * nt); }
};

struct Rows32Mine {
    uint32_t tid, nt, items;
    __device__ __forceinline__ bool operator[](int k) const { return tid + k * nt < items; }
};

__device__ __forceinline__ uint32_t bit_mux(uint32_t sel, uint32_t hi, uint32_t lo)
{
    return MCS_BOP3(sel, hi, lo, (MCS_A & MCS_B) | (~MCS_A & MCS_C));
}

// Bits of the sites' neighbours in the other colour's array v: n[0] at j, n[1]
// the other x neighbour (par: right, else left), n[2], n[3] at y + 1, y - 1,
// n[4], n[5] at z + 1, z - 1.
template <int DIMS, bool ALIGNED, int BITS>
__device__ __forceinline__ void neighbour_words(const uint32_t *v, const WordGeo &g, uint32_t par, const WholeArgs &a,
                                                uint32_t (&n)[6])
{
    const uint32_t half = a.half, j0 = BITS * g.w;
    const auto *vi = (const typename WholeItem<BITS>::type *)v;
    const uint32_t o = vi[g.w], before = vi[(int)g.w - (g.w ? 1 : 0)], after = vi[g.w + 1];
    const uint64_t U = bit_window<ALIGNED>(v, wrap_add(j0, a.hx - 1u, half), half);
    const uint64_t D = bit_window<ALIGNED>(v, wrap_add(j0, half - a.hx, half), half);
    const uint32_t left = bit_mux(g.first, (uint32_t)U, (o << 1) | (before >> (BITS - 1)));
    const uint32_t right = bit_mux(g.last, (uint32_t)(D >> 1), BITS == 32 ? __builtin_amdgcn_alignbit(after, o, 1) : (o | after << 16) >> 1);
    n[0] = o;
    n[1] = bit_mux(par, right, left);
    n[2] = (uint32_t)(U >> 1);
    n[3] = (uint32_t)D;
    if (DIMS == 3) {
        if (g.top)
            n[2] = bit_mux(g.top, (uint32_t)bit_window<ALIGNED>(v, wrap_add(j0, half - a.area + a.hx, half), half), n[2]);
        if (g.bottom)
            n[3] = bit_mux(g.bottom, (uint32_t)bit_window<ALIGNED>(v, wrap_add(j0, a.area - a.hx, half), half), n[3]);
        n[4] = (uint32_t)bit_window<ALIGNED>(v, wrap_add(j0, a.area, half), half);
        n[5] = (uint32_t)bit_window<ALIGNED>(v, wrap_add(j0, half - a.area, half), half);
    }
}

// Sign bits of the pairs j of item w, from the lattice's bytes: even and odd
// bytes.  The last item's are the end of the last BITS pairs.
template <int BITS>
__device__ __forceinline__ void pack_pairs(const int8_t *p, uint32_t w, uint32_t half, uint32_t &ev, uint32_t &od)
{
    const uint32_t cnt = half - BITS * w;
    if (cnt >= BITS || half >= BITS) {
        const uint32_t sh = cnt >= BITS ? 0u : BITS - cnt, off = 2u * (BITS * w - sh);
        const Row32 a = load_row32(p, off);
        ev = sign_bits16(pick16(a, 0x06040200u));
        od = sign_bits16(pick16(a, 0x07050301u));
        if (BITS == 32) {
            const Row32 b = load_row32(p, off + 32u);
            ev |= sign_bits16(pick16(b, 0x06040200u)) << 16;
            od |= sign_bits16(pick16(b, 0x07050301u)) << 16;
        }
        ev >>= sh;
        od >>= sh;
    } else {
        ev = od = 0u;
        for (uint32_t i = 0; i < cnt; ++i) {
            ev |= (p[2 * i] < 0 ? 1u : 0u) << i;
            od |= (p[2 * i + 1] < 0 ? 1u : 0u) << i;
        }
    }
}

template <int BITS>
__device__ __forceinline__ void store_pairs(int8_t *p, uint32_t ev, uint32_t od)
{
#pragma unroll
    for (int h = 0; h < BITS / 16; ++h) {
        Row32 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t e = 0x01010101u ^ (spread4((ev >> (16 * h + 4 * i)) & 15u) * 0xFEu);
            const uint32_t o = 0x01010101u ^ (spread4((od >> (16 * h + 4 * i)) & 15u) * 0xFEu);
            r.d[2 * i] = __builtin_amdgcn_perm(o, e, 0x05010400u);
            r.d[2 * i + 1] = __builtin_amdgcn_perm(o, e, 0x07030602u);
        }
        __builtin_memcpy(p + 32 * h, &r, 32);
    }
}

// K: items of BITS sites of a colour per thread, what their sites share kept in
// registers; 0: as many as there are, of rows of 32 sites without couplings, what
// they share found again in every half-sweep
template <int DIMS, int RULE, bool HASJ, int K, bool ALIGNED, int BITS>
__global__ __launch_bounds__(1024) void k_whole(WholeArgs a)
{
    constexpr bool HB = RULE != kMetropolis;
    constexpr int Z = 2 * DIMS;
    constexpr bool LOOP = K == 0;
    static_assert(!LOOP || (!HASJ && ALIGNED && BITS == 32), "rows of 32 sites");
    constexpr int KA = LOOP ? 1 : K;
    using item_t = typename WholeItem<BITS>::type;
    extern __shared__ uint32_t sm[];  // spins [2][stride], then couplings [2][Z][stride]
    __shared__ uint32_t tlow[8];
    __shared__ unsigned long long sums[2];  // of a sweep: down spins << 32 | unsatisfied bonds
    const uint32_t tid = threadIdx.x, nt = blockDim.x, l = blockIdx.x;
    const uint32_t stride = a.words + kWholePad, items = (a.half + (BITS - 1)) / BITS;
    uint32_t *S = sm, *Jb = sm + 2 * stride;
    auto item = [](uint32_t *v) { return (item_t *)v; };
    // item w of array v, and its copy after the last word
    auto put = [&](uint32_t *v, uint32_t w, uint32_t x) {
        item(v)[w] = (item_t)x;
        if (ALIGNED && w < 32u / BITS) item(v + a.words)[w] = (item_t)x;
    };
    const int64_t N = 2 * (int64_t)a.half;
    if (tid < 8) tlow[tid] = a.low[tid];
    if (tid < 2) sums[tid] = 0ull;
    int8_t *src = a.spins + (int64_t)l * N;
    struct Kept {
        WordGeo g[KA];
        bool mine[KA];
    } kept;
    auto &&g = [&]() -> decltype(auto) {
        if constexpr (LOOP) return Rows32Items{a, tid, nt};
        else return (kept.g);
    }();
    auto &&mine = [&]() -> decltype(auto) {
        if constexpr (LOOP) return Rows32Mine{tid, nt, items};
        else return (kept.mine);
    }();
    const int nk = LOOP ? (int)((items + nt - 1) / nt) : K;
#pragma unroll KA
    for (int k = 0; k < nk; ++k) {
        const uint32_t w = tid + k * nt;
        if constexpr (!LOOP) mine[k] = w < items;
        if (!mine[k]) continue;
        if constexpr (!LOOP) g[k] = word_geo<DIMS, BITS>(a, w);
        uint32_t ev, od;
        pack_pairs<BITS>(src, w, a.half, ev, od);
        put(S, w, bit_mux(g[k].odd, od, ev));
        put(S + stride, w, bit_mux(g[k].odd, ev, od));
        if (HASJ)
#pragma unroll
            for (int d = 0; d < DIMS; ++d) {
                // own couplings: right (for now in n[0]'s place), up, z + 1
                pack_pairs<BITS>(a.J + d * N, w, a.half, ev, od);
                put(Jb + (2 * d) * stride, w, bit_mux(g[k].odd, od, ev));
                put(Jb + (Z + 2 * d) * stride, w, bit_mux(g[k].odd, ev, od));
            }
    }
    __syncthreads();
    if (HASJ) {
        uint32_t j0[2][KA];
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (mine[k])
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    // the bond to a left, lower or z - 1 neighbour is that neighbour's own
                    const uint32_t par = c ? ~g[k].odd : g[k].odd, w = g[k].w;
                    uint32_t *own = Jb + c * Z * stride, *oth = Jb + (1 - c) * Z * stride;
                    uint32_t n[6], nx[6];
                    neighbour_words<DIMS, ALIGNED, BITS>(oth, g[k], 0u, a, nx);  // x, at the left neighbour
                    j0[c][k] = bit_mux(par, item(oth)[w], item(own)[w]);
                    item(own + stride)[w] = (item_t)bit_mux(par, item(own)[w], nx[1]);
                    neighbour_words<DIMS, ALIGNED, BITS>(oth + 2 * stride, g[k], 0u, a, n);
                    item(own + 3 * stride)[w] = (item_t)n[3];
                    if (DIMS == 3) {
                        neighbour_words<DIMS, ALIGNED, BITS>(oth + 4 * stride, g[k], 0u, a, n);
                        item(own + 5 * stride)[w] = (item_t)n[5];
                    }
                }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (mine[k]) {
                item(Jb)[g[k].w] = (item_t)j0[0][k];
                item(Jb + Z * stride)[g[k].w] = (item_t)j0[1][k];
            }
        __syncthreads();
    }
    const uint32_t rep = a.replica0 + l;
    // the masks of even classes in vector registers (an instruction reads one
    // scalar)
    uint32_t tv[8][3];
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            tv[b][i] = a.mask[b][2 * i];
            if (RULE != kHeatBathMirrored && i < (HB ? DIMS : 1)) asm volatile("" : "+v"(tv[b][i]));
        }
    const int64_t sites = N;
    auto publish = [&](int t) {
        // E = 2 (unsatisfied bonds) - DIMS N, M = N - 2 (down spins)
        if (tid == 0) {
            const unsigned long long v = sums[t & 1];
            sums[t & 1] = 0ull;
            a.EM[t * a.em_stride + 2 * (int64_t)l] = 2 * (long long)(uint32_t)v - DIMS * sites;
            a.EM[t * a.em_stride + 2 * (int64_t)l + 1] = sites - 2 * (long long)(v >> 32);
        }
    };
    for (int t = 0; t < a.nsweeps; ++t) {
        const uint64_t sweep = a.sweep0 + (uint64_t)t;
        for (int c = 0; c < 2; ++c) {
            const uint32_t w3 = ctr_w3(kTagSweep, (uint32_t)c, sweep), w3lo = ctr_w3(kTagSweepLo, (uint32_t)c, sweep);
            uint32_t *own = S + c * stride;
            uint32_t *oth = S + (1 - c) * stride;
            uint32_t count = 0;  // down spins << 16 | unsatisfied bonds, of this thread's words
#pragma unroll KA
            for (int k = 0; k < nk; ++k) {
                if (!mine[k]) continue;
                const uint32_t w = g[k].w;
                uint32_t n[6];
                neighbour_words<DIMS, ALIGNED, BITS>(oth, g[k], c ? ~g[k].odd : g[k].odd, a, n);
                const uint32_t s = item(own)[w], blk = BITS / 16 * w;
                const uint4 A = philox(make_uint4(blk, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                uint4 B = A;
                if (BITS == 32) B = philox(make_uint4(blk + 1u, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                uint32_t xk[6];
#pragma unroll
                for (int i = 0; i < Z; ++i) {
                    if (HASJ) n[i] ^= item(Jb + (c * Z + i) * stride)[w];
                    xk[i] = HB ? n[i] : (n[i] ^ s);
                }
                uint32_t c0, c1, c2;
                count_words<Z>(xk, c0, c1, c2);
                // Metropolis: a >= z/2 gives dE <= 0
                const uint32_t ge = HB ? 0u : DIMS == 3 ? MCS_BOP3(c2, c1, c0, MCS_A | (MCS_B & MCS_C)) : (c2 | c1);
                uint32_t lt = 0u, eq = g[k].valid;
                MirroredClasses mc;
                if constexpr (RULE == kHeatBathMirrored) mc = mirror_classes<DIMS>(c0, c1, c2);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    uint32_t X;
                    if (BITS == 32) {
                        X = plane_pair(A, B, b);
                    } else {
                        X = b < 2 ? A.x : b < 4 ? A.y : b < 6 ? A.z : A.w;
                        if (b & 1) X >>= 16;
                    }
                    const uint32_t *ts = a.mask[b];
                    uint32_t T = bit_mux(c0, ts[1], tv[b][0]);  // classes 0, 1
                    if constexpr (RULE == kHeatBathMirrored) {
                        T = b == 7 ? ~mc.s : mirrored_plane<DIMS>(mc, ts[0], ts[1], ts[2]);
                    } else if (HB) {
                        T = bit_mux(c1, bit_mux(c0, ts[3], tv[b][1]), T);
                        T = DIMS == 3 ? bit_mux(c2, bit_mux(c1, ts[6], bit_mux(c0, ts[5], tv[b][2])), T)
                                      : bit_mux(c2, tv[b][2], T);
                    } else if (DIMS == 3) {
                        T = bit_mux(c1, tv[b][1], T);
                    }
                    lt = MCS_BOP3(X, T, lt, (~MCS_A & MCS_B) | (~MCS_A & MCS_C) | (MCS_B & MCS_C));
                    eq = MCS_BOP3(eq, X, T, MCS_A & ~(MCS_B ^ MCS_C));
                }
                // heat-bath: down unless r < T; Metropolis: flip where accepted
                uint32_t so = HB ? ~lt : MCS_BOP3(s, ge, lt, MCS_A ^ (MCS_B | MCS_C));
                uint32_t pend = HB ? eq : (eq & ~ge);
                while (pend) {
                    const int b = __builtin_ctz(pend);
                    pend &= pend - 1u;
                    const uint32_t cls = ((c0 >> b) & 1u) | (((c1 >> b) & 1u) << 1) | (((c2 >> b) & 1u) << 2);
                    const uint4 lo = philox(make_uint4(BITS * w + (uint32_t)b, rep, (uint32_t)sweep, w3lo), a.seed_lo,
                                            a.seed_hi);
                    if ((lo.x & 0xFFFFFFu) < tlow[cls]) so ^= 1u << b;
                }
                put(own, w, so);
                if (c == 1 && a.EM) {
                    uint32_t u = 0;
#pragma unroll
                    for (int i = 0; i < Z; ++i) u += (uint32_t)__builtin_popcount((so ^ n[i]) & g[k].valid);
                    const uint32_t o = HASJ ? item(oth)[w] : n[0];
                    const uint32_t dn = (uint32_t)(__builtin_popcount(so & g[k].valid) + __builtin_popcount(o & g[k].valid));
                    count += u | dn << 16;
                }
            }
            if (c == 1 && a.EM) {
                uint32_t u, dn;
                if constexpr (LOOP) {  // up to eight items a thread: more than 16 bits in a wave
                    u = (uint32_t)__builtin_amdgcn_readlane(wave_sum_last((int)(count & 0xFFFFu)), 63);
                    dn = (uint32_t)__builtin_amdgcn_readlane(wave_sum_last((int)(count >> 16)), 63);
                } else {
                    const uint32_t v = (uint32_t)__builtin_amdgcn_readlane(wave_sum_last((int)count), 63);
                    u = v & 0xFFFFu;
                    dn = v >> 16;
                }
                if ((tid & 63u) == 0u) atomicAdd(&sums[t & 1], (unsigned long long)u | (unsigned long long)dn << 32);
            }
            // the sums of the sweep before: complete at its end, and next added
            // to after this half-sweep's barrier
            if (c == 0 && t > 0 && a.EM) publish(t - 1);
            __syncthreads();
        }
    }
    if (a.EM) publish(a.nsweeps - 1);
    // back to columns: even in S[0], odd in S[1]
#pragma unroll KA
    for (int k = 0; k < nk; ++k) {
        if (!mine[k]) continue;
        const uint32_t w = g[k].w, s0 = item(S)[w], s1 = item(S + stride)[w];
        const uint32_t ev = bit_mux(g[k].odd, s1, s0), od = bit_mux(g[k].odd, s0, s1);
        if (a.half - BITS * w >= BITS) store_pairs<BITS>(src + 2 * BITS * (int64_t)w, ev, od);
        item(S)[w] = (item_t)ev;
        item(S + stride)[w] = (item_t)od;
    }
    if (ALIGNED) return;
    __syncthreads();
    if (a.half >= BITS) {  // the last BITS pairs
        if (tid == 0)
            store_pairs<BITS>(src + 2 * (int64_t)(a.half - BITS), (uint32_t)bit_window<true>(S, a.half - BITS, a.half),
                              (uint32_t)bit_window<true>(S + stride, a.half - BITS, a.half));
    } else if (tid < a.half) {
        src[2 * tid] = ((S[0] >> tid) & 1u) ? (int8_t)-1 : (int8_t)1;
        src[2 * tid + 1] = ((S[stride] >> tid) & 1u) ? (int8_t)-1 : (int8_t)1;
    }
}

static size_t whole_lds_bytes(const Geom &g, bool hasJ)
{
    const size_t words = (size_t)((g.N / 2 + 31) / 32) + kWholePad;
    return 4 * words * (2 + (hasJ ? 4 * (size_t)g.dims : 0));
}

// Two words per thread: the sums of a wave fit their 16 bits, and above 2^17
// sites one workgroup takes longer than two launches over the whole chip, unless
// there are lattices for many of its CUs (rows of 32 sites, up to 2^19 of them;
// the couplings of more than 3 x 2^16 don't fit LDS).  us of a call, modelled: a
// workgroup's lattice 46 per 10^6 sites to load and store (couplings as much
// again) and 1.5 + 59 per sweep, on each of 256 CUs at once; half-sweeps 8.5 +
// 0.95 per sweep over all lattices' sites.  Measured, whole (half-sweeps), per
// sweep of 20 at 16, 64 and 256 lattices: 32^2 x 160 11.7, 12.2, 13.5 (11.0, 18.8,
// 49), 32 x 64 x 256 34, 35, 39 (16.5, 43, 130), 32 x 16384 heat-bath 31, 32, 36
// (14.5, 33, 103), 32 x 5440 +-J 10.3, 10.6, 12.0 (11.6, 21, 61); one sweep of 64
// and 256 of 32 x 64 x 256 78, 109 with the call (53, 134).
bool whole_supported(const Geom &g, bool hasJ, int nsweeps)
{
    if (g.N <= (1 << 17)) return true;
    if (g.Lx != 32 || (hasJ ? g.dims != 2 || g.N > 3 * (1 << 16) : g.N > (1 << 19))) return false;
    constexpr int kCUs = 256;
    const double M = 1e-6 * (double)g.N, n = nsweeps;
    const double whole = (g.count + kCUs - 1) / kCUs * (46.0 * M * (hasJ ? 2.0 : 1.0) + n * (1.5 + 59.0 * M));
    return whole < n * (8.5 + 0.95 * M * g.count);
}

template <int DIMS, int RULE, bool HASJ, int K, bool ALIGNED, int BITS>
static hipError_t launch_whole_a(const WholeArgs &a, int count, size_t lds, hipStream_t s)
{
    static LdsLimit lim;
    const auto f = k_whole<DIMS, RULE, HASJ, K, ALIGNED, BITS>;
    const hipError_t e = lim.ensure((const void *)f, 128 * 1024);
    if (e != hipSuccess) return e;
    const uint32_t items = (a.half + BITS - 1) / BITS;
    hipLaunchKernelGGL(f, dim3((unsigned)count), dim3(std::min(1024u, (items + 63u) & ~63u)), lds, s, a);
    return hipGetLastError();
}

template <int DIMS, int RULE, bool HASJ, int K, int BITS>
static hipError_t launch_whole_t(const WholeArgs &a, int count, size_t lds, hipStream_t s)
{
    return a.half % 32u ? launch_whole_a<DIMS, RULE, HASJ, K, false, BITS>(a, count, lds, s)
                        : launch_whole_a<DIMS, RULE, HASJ, K, true, BITS>(a, count, lds, s);
}

// 16 sites per thread, a Philox block instead of two, where the waves are then
// at most two per SIMD and each issues by itself, or where 32 sites per thread
// leave half a wave idle.  us per sweep (32 sites per thread): 64^2 1.14 (1.43),
// 80^2 1.24 (1.62), 128^2 1.59 (1.74), 12^3 heat-bath 1.29 (1.75), 16^3 +-J 1.50
// (1.80), 4096 of 32^2 2.41 (3.24); beyond, 30^3 +-J 3.24 (2.92), 32^3 3.08
// (2.61), 4096 of 64^2 4.5 (3.4), 2048 of 128^2 8.4 (6.7).
static bool whole_halves(uint32_t words, int count)
{
    constexpr uint32_t kCUs = 256;
    return words <= 32 || words * (((uint32_t)count + kCUs - 1) / kCUs) <= 256;
}

template <int DIMS, int RULE, bool HASJ>
static hipError_t launch_whole_k(const WholeArgs &a, int count, size_t lds, hipStream_t s)
{
    if (whole_halves(a.words, count)) return launch_whole_t<DIMS, RULE, HASJ, 1, 16>(a, count, lds, s);
    if (a.words <= 1024u) return launch_whole_t<DIMS, RULE, HASJ, 1, 32>(a, count, lds, s);
    if (a.words <= 2048u) return launch_whole_t<DIMS, RULE, HASJ, 2, 32>(a, count, lds, s);
    if constexpr (!HASJ) return launch_whole_a<DIMS, RULE, false, 0, true, 32>(a, count, lds, s);
    else if constexpr (DIMS == 2) return launch_whole_a<2, RULE, true, 3, true, 32>(a, count, lds, s);
    else return hipErrorInvalidValue;
}

template <int D>
static hipError_t launch_whole_r(const WholeArgs &a, int rule, int count, size_t lds, hipStream_t s)
{
    const bool hj = a.J != nullptr;
    switch (rule) {
    case kMetropolis: return hj ? launch_whole_k<D, kMetropolis, true>(a, count, lds, s) : launch_whole_k<D, kMetropolis, false>(a, count, lds, s);
    case kHeatBath: return hj ? launch_whole_k<D, kHeatBath, true>(a, count, lds, s) : launch_whole_k<D, kHeatBath, false>(a, count, lds, s);
    default: return hj ? launch_whole_k<D, kHeatBathMirrored, true>(a, count, lds, s) : launch_whole_k<D, kHeatBathMirrored, false>(a, count, lds, s);
    }
}

// Every sweep of a call, one workgroup per lattice.
hipError_t launch_whole(const SweepCall &c, int8_t *spins, uint64_t sweep0, int nsweeps, int64_t *EM,
                        int64_t em_stride, hipStream_t s)
{
    if (nsweeps <= 0) return hipSuccess;
    WholeArgs a;
    const Geom &g = c.g;
    a.spins = spins;
    a.J = c.J;
    a.Ly = (uint32_t)g.Ly;
    a.hx = (uint32_t)g.Lx / 2;
    a.half = (uint32_t)(g.N / 2);
    a.area = a.hx * a.Ly;
    a.words = (a.half + 31) / 32;
    a.mul_hx = 0xFFFFFFFFu / a.hx;
    a.mul_ly = 0xFFFFFFFFu / a.Ly;
    a.seed_lo = c.seed_lo;
    a.seed_hi = c.seed_hi;
    a.replica0 = c.replica0;
    a.sweep0 = sweep0;
    a.nsweeps = nsweeps;
    a.EM = EM;
    a.em_stride = em_stride;
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
    const size_t lds = whole_lds_bytes(g, c.J != nullptr);
    const int rule = c.rule == 0 ? kMetropolis : mirrored_classes(top, z) ? kHeatBathMirrored : kHeatBath;
    if (g.dims == 2) return launch_whole_r<2>(a, rule, g.count, lds, s);
    return launch_whole_r<3>(a, rule, g.count, lds, s);
}

}  // namespace mcs
