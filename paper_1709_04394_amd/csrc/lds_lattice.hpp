// lds_lattice.hpp -- whole 2D L x L ferromagnets (J = 1) held bit-packed in
// one workgroup's LDS, swept there for several checkerboard Metropolis sweeps
// (Sec. "Checkerboard scheme", Eq. metropolis-canonical).  Shared by the
// population-annealing step (every lattice at the step's temperature) and by
// parallel tempering (each lattice at the temperature it currently holds).
//
// LDS image: two arrays of P = max(1, N / 64) words per lattice, one for each
// colour c = (x + y) mod 2, bit set <=> s = -1, so that a half-sweep reads the
// four neighbours from the other colour's array only and every word is 32 of
// the sites that share random bit-planes:
//   L >= 64: word p = w L + r holds the colour's sites 32 w .. 32 w + 31 of
//     row r; the neighbours above and below are words p -+ 1 and the sideways
//     pair is the same word and that word shifted by one site towards the
//     row's parity;
//   L < 64: word p holds the sites j = 32 p .. 32 p + 31 of the colour in row
//     order (64 / L whole rows): the rows above and below are the words around
//     p shifted by L / 2, the sideways pair a rotation inside each row.  L = 4
//     has 8 sites of a colour: its word holds them four times over, which
//     makes the shifts periodic.
// The lattice is periodic inside the image, so no halo is needed.
//
// What bounds it: VALU issue (the image stays in LDS for theta sweeps).  A wave
// spends about 170 VALU instructions on 64 words of 32 sites, 74 of them in two
// Philox blocks.  The earlier form spent 302, with integer divisions per word,
// a site at a time in the tie queue, two barriers per half-sweep and, for
// L < 64, one row per word: 9.46 ms for eight annealing steps of four
// populations of 16384 replicas, 6.46 so, and 5.84 with bytes packed by v_dot4,
// starting lattices written as 16-byte words and the first measurement in place.
// Where a wave has one task a half-sweep, a queue gathers nothing: there each lane
// settles its own word's ties (32 temperatures of 128 sets of L = 64, ten rounds
// of ten sweeps: 764 us with the queue, 715 without; 1000 annealed replicas of
// L = 64, six steps: 402 and 370).
#pragma once

#include "common.hpp"
#include "spin_bytes.hpp"

namespace mcs {

// Tied words per wave: settled 64 at a time as they accumulate.
constexpr int kLdsTieQueue = 128;

struct LdsLattices {
    int L, P, hx, nwr;      // extent, words per lattice and colour, L / 2, words per row (L >= 64)
    int ng, ng_max;         // lattices in this workgroup (at most 64), room for
    uint32_t rep0;          // replica id of lattice g is rep0 + g
    uint64_t sweep0;        // global number of the first sweep
    int theta;              // sweeps
    uint32_t seed_lo, seed_hi;
    // x / P and x / L as high words of a product: exact for the word numbers
    // of a workgroup (below 2^18, times a divisor of at most 2^12)
    uint32_t inv_p, inv_l;
};

__device__ __forceinline__ uint32_t lds_inverse(int n) { return n == 1 ? 0u : 0xFFFFFFFFu / (uint32_t)n + 1u; }

__device__ __forceinline__ int lds_div(int x, int n, uint32_t inv) { return n == 1 ? x : (int)__umulhi((uint32_t)x, inv); }

__device__ __forceinline__ LdsLattices lds_lattices(int L)
{
    LdsLattices a;
    a.L = L;
    a.P = L < 8 ? 1 : L * L / 64;
    a.hx = L / 2;
    a.nwr = L >= 64 ? L / 64 : 1;
    a.inv_p = lds_inverse(a.P);
    a.inv_l = lds_inverse(L);
    return a;
}

// Words of G lattices, both colours.
__host__ __device__ __forceinline__ int lds_lattice_words(int L, int G) { return G * 2 * (L < 8 ? 1 : L * L / 64); }

// Words with ties, {LDS word | lattice << 16, first of its two blocks, tied
// sites, those of class dE = 8}: kLdsTieQueue items per wave, used by that
// wave's lanes only, in the dynamic LDS behind the lattices.
__host__ __device__ __forceinline__ size_t lds_lattice_bytes(int L, int G, int threads)
{
    return ((size_t)lds_lattice_words(L, G) * 4 + 15) / 16 * 16 + (size_t)(threads / 64) * kLdsTieQueue * 16;
}

// Threads per workgroup, for `words` of its lattices (both colours): one wave
// where that fills the chip, since its tied words then gather over all the
// workgroup's words and no wave waits at a barrier; four, with a word a lane
// where the lattices have no more, where the workgroups are few or LDS would
// hold too few single waves per SIMD.  Annealing steps, us at 64, 128 and 256
// threads: five steps of 2338 of L = 128 1000, 970 and 892, of 4096 1187, 1177
// and 1130, of 6000 1460, 1433 and 1443; three of 8192 1107, 1155 and 1121, of
// 16384 1819, 1925 and 1933; three of 4200 of L = 256 (8 KB each) 3080, 2676 and
// 2420, of 8000 4700, 3922 and 3700.
inline int lds_lattice_threads(int blocks, int words) { return blocks >= 6000 && words <= 1024 ? 64 : 256; }

// Bits of the rows of odd y among the rows of one word (L < 64).
__device__ __forceinline__ uint32_t odd_rows(int hx)
{
    return hx == 16 ? 0xFFFF0000u : hx == 8 ? 0xFF00FF00u : hx == 4 ? 0xF0F0F0F0u : 0xCCCCCCCCu;
}

// int8 sites of words p of both colours <-> the LDS image (64 sites: 64 w ..
// of row r for L >= 64, 64 p .. in row order for smaller lattices).
__device__ __forceinline__ void pack_lattice_words(uint32_t *lds, const LdsLattices &a, int g, const int8_t *src, int p)
{
    uint32_t ev = 0, od = 0, odd;
    if (a.L == 4) {
        const uint4 v = *(const uint4 *)src;
        const uint32_t dw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t m = dw[i] & 0x80808080u, Pm = m + (m << 15);
            ev |= ((Pm >> 22) & 3u) << (2 * i);
            od |= (Pm >> 30) << (2 * i);
        }
        ev *= 0x01010101u;
        od *= 0x01010101u;
        odd = odd_rows(2);
    } else {
        int at = 64 * p;
        odd = 0u;
        if (a.L >= 64) {
            const int w = lds_div(p, a.L, a.inv_l), r = p - w * a.L;
            at = r * a.L + 64 * w;
            odd = (r & 1) ? ~0u : 0u;
        } else {
            odd = odd_rows(a.hx);
        }
        Row32 h[2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 v = ((const uint4 *)(src + at))[q];
            h[q >> 1].d[4 * (q & 1)] = v.x;
            h[q >> 1].d[4 * (q & 1) + 1] = v.y;
            h[q >> 1].d[4 * (q & 1) + 2] = v.z;
            h[q >> 1].d[4 * (q & 1) + 3] = v.w;
        }
        ev = sign_bits16(pick16(h[0], 0x06040200u)) | sign_bits16(pick16(h[1], 0x06040200u)) << 16;
        od = sign_bits16(pick16(h[0], 0x07050301u)) | sign_bits16(pick16(h[1], 0x07050301u)) << 16;
    }
    // colour 0: even x in even rows, odd x in odd rows
    uint32_t *c0 = lds + 2 * g * a.P + p;
    c0[0] = (ev & ~odd) | (od & odd);
    c0[a.P] = (od & ~odd) | (ev & odd);
}

__device__ __forceinline__ void unpack_lattice_words(const uint32_t *lds, const LdsLattices &a, int g, int8_t *dst, int p)
{
    const uint32_t *c0 = lds + 2 * g * a.P + p;
    const uint32_t s0 = c0[0], s1 = c0[a.P];
    int at = 64 * p;
    uint32_t odd;
    if (a.L >= 64) {
        const int w = lds_div(p, a.L, a.inv_l), r = p - w * a.L;
        at = r * a.L + 64 * w;
        odd = (r & 1) ? ~0u : 0u;
    } else {
        odd = odd_rows(a.hx);
    }
    const uint32_t ev = (s0 & ~odd) | (s1 & odd), od = (s1 & ~odd) | (s0 & odd);
    uint4 *q4 = (uint4 *)(dst + at);
    const int nq = a.L == 4 ? 1 : 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t dw[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            // four even and four odd columns, bit 0 -> byte 0x01 (+1), 1 -> 0xFF (-1)
            const int sh = 8 * q + 4 * i;
            const uint32_t e = 0x01010101u ^ (spread4((ev >> sh) & 15u) * 0xFEu);
            const uint32_t o = 0x01010101u ^ (spread4((od >> sh) & 15u) * 0xFEu);
            dw[2 * i] = __builtin_amdgcn_perm(o, e, 0x05010400u);
            dw[2 * i + 1] = __builtin_amdgcn_perm(o, e, 0x07030602u);
        }
        if (q < nq) q4[q] = make_uint4(dw[0], dw[1], dw[2], dw[3]);
    }
}

// The word of colour c at place p of a lattice (lat: its LDS words), and its
// neighbours: S, the words above and below, the same place and the shifted one.
struct LdsStencil {
    uint32_t S, U, D, O, Sh;
};

template <bool SMALL>
__device__ __forceinline__ LdsStencil lds_stencil(const uint32_t *lat, const LdsLattices &a, int c, int p, int w, int r)
{
    const uint32_t *own = lat + (c ? a.P : 0), *opp = lat + (c ? 0 : a.P);
    LdsStencil s;
    s.S = own[p];
    s.O = opp[p];
    if constexpr (SMALL) {
        const uint32_t Ou = opp[p == 0 ? a.P - 1 : p - 1], Od = opp[p + 1 == a.P ? 0 : p + 1];
        s.U = __builtin_amdgcn_alignbit(s.O, Ou, 32 - a.hx);
        s.D = __builtin_amdgcn_alignbit(Od, s.O, a.hx);
        // rows whose sites of colour c have even x take the site to the left
        const uint32_t odd = odd_rows(a.hx), par = c ? ~odd : odd;
        const uint32_t lo = a.hx == 16 ? 0x00010001u : a.hx == 8 ? 0x01010101u : a.hx == 4 ? 0x11111111u : 0x55555555u;
        const uint32_t hi = lo << (a.hx - 1);
        const uint32_t rl = ((s.O << 1) & ~lo) | ((s.O >> (a.hx - 1)) & lo);
        const uint32_t rr = ((s.O >> 1) & ~hi) | ((s.O << (a.hx - 1)) & hi);
        s.Sh = (rr & par) | (rl & ~par);
    } else {
        s.U = opp[r == 0 ? p + a.L - 1 : p - 1];
        s.D = opp[r + 1 == a.L ? p + 1 - a.L : p + 1];
        const bool par = (c + r) & 1;  // x parity of the row's sites of colour c
        uint32_t hi = s.O, lo = s.O;
        if (a.nwr > 1) {
            const int side = par ? (w + 1 == a.nwr ? p - (a.nwr - 1) * a.L : p + a.L)
                                 : (w == 0 ? p + (a.nwr - 1) * a.L : p - a.L);
            const uint32_t n = opp[side];
            hi = par ? n : s.O;
            lo = par ? s.O : n;
        }
        s.Sh = __builtin_amdgcn_alignbit(hi, lo, par ? 1u : 31u);
    }
    return s;
}

// The accepted of a word's tied sites (pend; of class dE = 8: c8): their low 24
// bits drawn one after the other.
__device__ __forceinline__ uint32_t accept_lds_ties(const LdsLattices &a, uint32_t blk, uint32_t rep, uint32_t pend,
                                                    uint32_t c8, uint32_t sweep_lo, uint32_t w3lo, uint32_t l4,
                                                    uint32_t l8)
{
    uint32_t f = 0u;
    while (pend) {
        const int b = __builtin_ctz(pend);
        pend &= pend - 1u;
        const uint4 lo = philox(make_uint4(16u * blk + (uint32_t)b, rep, sweep_lo, w3lo), a.seed_lo, a.seed_hi);
        if ((lo.x & 0xFFFFFFu) < (((c8 >> b) & 1u) ? l8 : l4)) f |= 1u << b;
    }
    return f;
}

// Settles the tied sites of the wave's queued words, one word per lane.
template <bool PER_LAT>
__device__ __forceinline__ void settle_lds_ties(uint32_t *lds, const LdsLattices &a, const uint4 *tq, uint32_t n,
                                                uint32_t sweep_lo, uint32_t w3lo, uint32_t low4, uint32_t low8,
                                                const Thr *t4, const Thr *t8)
{
    for (uint32_t i = threadIdx.x & 63; i < n; i += 64) {
        const uint4 it = tq[i];
        const uint32_t g = it.x >> 16;
        uint32_t f = accept_lds_ties(a, it.y, a.rep0 + g, it.z, it.w, sweep_lo, w3lo, PER_LAT ? t4[g].low : low4,
                                     PER_LAT ? t8[g].low : low8);
        if (a.L == 4) f *= 0x01010101u;
        if (f) lds[it.x & 0xFFFFu] ^= f;
    }
}

// A threshold's top byte as select masks; 2^32 is 255 with a low part no draw
// reaches.
__device__ __forceinline__ Thr lds_thr(Thr t) { return t.top >= 256u ? Thr{255u, 1u << 24} : t; }

// ONE: a wave has at most one task, and each lane settles its own word's ties at
// once; else tied words gather over the wave's tasks.
template <bool PER_LAT, bool SMALL, bool ONE>
__device__ void sweep_lds_words(uint32_t *lds, const LdsLattices &a, Thr u4, Thr u8, const Thr *t4, const Thr *t8,
                                uint4 *tq)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    const int tasks = a.ng * a.P;
    // masks of the thresholds' top bytes: those of dE = 4 in vector registers
    // (an instruction reads one scalar register)
    uint32_t m4[8], m8[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        m4[k] = PER_LAT ? 0u : ((u4.top >> k) & 1u) ? ~0u : 0u;
        m8[k] = PER_LAT ? 0u : ((u8.top >> k) & 1u) ? ~0u : 0u;
        if (!PER_LAT) asm volatile("" : "+v"(m4[k]));
    }
    for (int sw = 0; sw < a.theta; ++sw) {
        const uint64_t sweep = a.sweep0 + (uint64_t)sw;
        for (int c = 0; c < 2; ++c) {
            const uint32_t w3 = ctr_w3(kTagSweep, (uint32_t)c, sweep);
            const uint32_t w3lo = ctr_w3(kTagSweepLo, (uint32_t)c, sweep);
            uint32_t qn = 0;
            for (int t0 = tid & ~63; t0 < tasks; t0 += nt) {
                const int t = t0 + (tid & 63);
                uint32_t pend = 0u, c8 = 0u, blk = 0u, wsg = 0u;
                if (SMALL ? t < tasks : true) {  // P is a multiple of 64 for L >= 64
                    int g = lds_div(SMALL ? t : t0, a.P, a.inv_p);
                    if (!SMALL) g = __builtin_amdgcn_readfirstlane(g);
                    const int p = t - g * a.P;
                    int w = 0, r = p;
                    if (!SMALL && a.nwr > 1) {
                        w = lds_div(p, a.L, a.inv_l);
                        r = p - w * a.L;
                    }
                    uint32_t *lat = lds + 2 * g * a.P;
                    const LdsStencil s = lds_stencil<SMALL>(lat, a, c, p, w, r);
                    const uint32_t u1 = s.S ^ s.U, u2 = s.S ^ s.D, u3 = s.S ^ s.O, u4b = s.S ^ s.Sh;
                    const uint32_t t1 = u1 | u2, t2 = u3 | u4b;
                    const uint32_t ge2 = MCS_BOP3(u1, u2, MCS_BOP3(u3, u4b, t1 & t2, (MCS_A & MCS_B) | MCS_C),
                                                  (MCS_A & MCS_B) | MCS_C);
                    c8 = ~(t1 | t2);
                    blk = SMALL ? 2u * (uint32_t)p : 2u * (uint32_t)w + 2u * (uint32_t)(a.nwr * r);
                    const uint32_t rep = a.rep0 + (uint32_t)g;
                    const uint4 A = philox(make_uint4(blk, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                    const uint4 B = philox(make_uint4(blk + 1u, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                    uint32_t top4 = 0u, top8 = 0u;
                    if (PER_LAT) {
                        top4 = t4[g].top;
                        top8 = t8[g].top;
                        if (!SMALL) {
                            top4 = __builtin_amdgcn_readfirstlane(top4);
                            top8 = __builtin_amdgcn_readfirstlane(top8);
                        }
                    }
                    // bit-serial r < T; a site's threshold bit is that of its class
                    // (sites with two or more unsatisfied bonds accept in any case)
                    uint32_t lt = 0u, eq = ~0u;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        uint32_t X = plane_pair(A, B, k);
                        if (SMALL && a.L == 4) X = (X & 0xFFu) * 0x01010101u;
                        const uint32_t b4 = PER_LAT ? (((top4 >> k) & 1u) ? ~0u : 0u) : m4[k];
                        const uint32_t b8 = PER_LAT ? (((top8 >> k) & 1u) ? ~0u : 0u) : m8[k];
                        const uint32_t T = MCS_BOP3(c8, b8, b4, (MCS_A & MCS_B) | (~MCS_A & MCS_C));
                        lt = MCS_BOP3(X, T, lt, (~MCS_A & MCS_B) | (~MCS_A & MCS_C) | (MCS_B & MCS_C));
                        eq = MCS_BOP3(eq, X, T, MCS_A & ~(MCS_B ^ MCS_C));
                    }
                    uint32_t Sn = MCS_BOP3(s.S, ge2, lt, MCS_A ^ (MCS_B | MCS_C));
                    pend = eq & ~ge2;
                    if (SMALL && a.L == 4) pend &= 0xFFu;
                    if (ONE) {
                        uint32_t f = accept_lds_ties(a, blk, rep, pend, c8, (uint32_t)sweep, w3lo,
                                                     PER_LAT ? t4[g].low : u4.low, PER_LAT ? t8[g].low : u8.low);
                        if (SMALL && a.L == 4) f *= 0x01010101u;
                        Sn ^= f;
                    }
                    lat[(c ? a.P : 0) + p] = Sn;
                    wsg = (uint32_t)(2 * g * a.P + (c ? a.P : 0) + p) | ((uint32_t)g << 16);
                }
                if (ONE) continue;
                const uint64_t m = __ballot(pend != 0u);
                if (pend) {
                    const uint32_t at = qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    tq[at] = make_uint4(wsg, blk, pend, c8);
                }
                qn += (uint32_t)__popcll(m);
                // more than 64 words wait: settle all (the queue holds 128, a task adds up to 64)
                if (qn > 64u || t0 + nt >= tasks) {
                    settle_lds_ties<PER_LAT>(lds, a, tq, qn, (uint32_t)sweep, w3lo, u4.low, u8.low, t4, t8);
                    qn = 0;
                }
            }
            // a lattice of at most 64 words per colour is one wave's alone
            if (a.P > 64) {
                __syncthreads();
            } else {
                __builtin_amdgcn_wave_barrier();
                asm volatile("" ::: "memory");
            }
        }
    }
    __syncthreads();
}

// theta checkerboard Metropolis sweeps of the ng lattices in LDS; the
// thresholds of lattice g are t4[g], t8[g] (dE = 4, 8) when PER_LAT, else
// u4, u8 for every lattice (all with tops below 256, lds_thr).  Then the energy
// of each lattice into e_lat[g] (cleared by the caller).  Every thread of the
// workgroup must call this (barriers inside).
template <bool PER_LAT>
__device__ void sweep_lds_lattices(uint32_t *lds, const LdsLattices &a, Thr u4, Thr u8, const Thr *t4,
                                   const Thr *t8, int *e_lat)
{
    const bool small = a.L < 64;
    uint4 *tq = (uint4 *)(lds + (((size_t)a.ng_max * 2 * a.P + 3) & ~(size_t)3)) + (threadIdx.x >> 6) * kLdsTieQueue;
    const bool one = a.ng * a.P <= (int)blockDim.x;
    if (small && one) sweep_lds_words<PER_LAT, true, true>(lds, a, u4, u8, t4, t8, tq);
    else if (small) sweep_lds_words<PER_LAT, true, false>(lds, a, u4, u8, t4, t8, tq);
    else if (one) sweep_lds_words<PER_LAT, false, true>(lds, a, u4, u8, t4, t8, tq);
    else sweep_lds_words<PER_LAT, false, false>(lds, a, u4, u8, t4, t8, tq);
    // ---- energy over the odd sites' words (every bond has one odd end)
    const int tasks = a.ng * a.P;
    for (int t = threadIdx.x; t < tasks; t += blockDim.x) {
        const int g = lds_div(t, a.P, a.inv_p), p = t - g * a.P;
        const uint32_t *lat = lds + 2 * g * a.P;
        LdsStencil s;
        if (small) {
            s = lds_stencil<true>(lat, a, 1, p, 0, 0);
        } else {
            const int w = lds_div(p, a.L, a.inv_l);
            s = lds_stencil<false>(lat, a, 1, p, w, p - w * a.L);
        }
        const int n = __builtin_popcount(s.S ^ s.U) + __builtin_popcount(s.S ^ s.D) + __builtin_popcount(s.S ^ s.O) +
                      __builtin_popcount(s.S ^ s.Sh);
        atomicAdd(&e_lat[g], a.L == 4 ? n / 2 - 32 : 2 * n - 128);
    }
    __syncthreads();
}

}  // namespace mcs
