// k_muca.hip -- parallel-walker multicanonical sweeps (Sec. "Multicanonical
// simulations": p walkers share one weight function, their histograms are
// added; Eq. muca, Eq. weight_modification) for 2D L x L ferromagnets.
//
// Walkers visit the sites of a lattice in the same sequential (typewriter)
// order, each with its own random numbers.  A walker's rows are bit-packed in
// registers while it sweeps them; the rows of the whole lattice stay int8 in
// global memory and stream through once per sweep.  The acceptance table
// T[level][direction] (FP64 host values as 32-bit thresholds) sits in LDS
// (131 KB at L = 128, within gfx950's 160 KB).  Moves that would leave the
// energy window [-2N, 0] are rejected and the current level is counted again.
// k_muca_q (four lanes per walker) does the sweeps; k_muca (one lane per
// walker) those of small lattices without counting where there are walkers
// enough to fill the chip one lane each.
#include <algorithm>

#include "internal.hpp"
#include "muca.hpp"
#include "muca_rows.hpp"
#include "quad_walk.hpp"

namespace mcs {

template <int L>
__global__ __launch_bounds__(64) void k_muca(MucaArgs a)
{
    constexpr int N = L * L, NW = (L + 31) / 32, K = N / 2;
    extern __shared__ uint32_t tab[];  // [(K + 1) * 4] thresholds minus one
    const int lane = threadIdx.x;
    for (int i = lane; i < (K + 1) * 4; i += 64) tab[i] = a.table[i];
    __syncthreads();
    const int w = blockIdx.x * 64 + lane;
    if (w >= a.W) return;
    int8_t *sp = a.spins + (int64_t)w * N;
    int k = (int)((a.E[w] + 2 * N) / 4);
    for (int t = 0; t < a.nsweeps; ++t) {
        const uint64_t sweep = a.sweep0 + (uint64_t)t;
        const uint32_t w3 = ctr_w3(kTagMuca, 0, sweep);
        uint32_t up[NW], cur[NW], dn[NW], row0[NW];
        load_row<L>(sp, L - 1, up);
        load_row<L>(sp, 0, cur);
        load_row<L>(sp, 1 % L, dn);
        for (int y = 0; y < L; ++y) {
            uint4 blk = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int x = 0; x < L; ++x) {
                if (x % 4 == 0)
                    blk = philox(make_uint4((uint32_t)(x + L * y) >> 2, (uint32_t)w, (uint32_t)sweep, w3), a.seed_lo,
                                 a.seed_hi);
                const uint32_t r = (x % 4 == 0) ? blk.x : (x % 4 == 1) ? blk.y : (x % 4 == 2) ? blk.z : blk.w;
                const uint32_t s = bit_at<L>(cur, x);
                const uint32_t nl = bit_at<L>(cur, (x + L - 1) % L), nr = bit_at<L>(cur, (x + 1) % L);
                const uint32_t nu = bit_at<L>(up, x), nd = bit_at<L>(dn, x);
                const int anti = (int)((s ^ nl) + (s ^ nr) + (s ^ nu) + (s ^ nd));
                const int dl = 2 - anti;  // level change if the spin flips (dE = 4 dl)
                const int k2 = k + dl;
                bool acc;
                if (dl == 0) acc = true;
                else acc = k2 <= K && r <= tab[4 * k + (dl < 0 ? dl + 2 : dl + 1)];
                if (acc) {
                    cur[x / 32] ^= 1u << (x % 32);
                    k = k2;
                }
            }
            store_row<L>(sp, y, cur);
            if (y == 0) {
#pragma unroll
                for (int i = 0; i < NW; ++i) row0[i] = cur[i];
            }
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                up[i] = cur[i];
                cur[i] = dn[i];
            }
            if (y + 2 < L) load_row<L>(sp, y + 2, dn);
            else {
#pragma unroll
                for (int i = 0; i < NW; ++i) dn[i] = row0[i];
            }
        }
    }
    a.E[w] = 4 * (int64_t)k - 2 * N;
}

// ---------------------------------------------------------------------------
// k_muca_q<L>: the same walk with four lanes per walker (quad_walk.hpp), the
// visited levels counted.  It draws the same random numbers and takes the same
// decisions as k_muca<L>.
//
// What an update costs is the instructions its wave issues, so little is left
// on the chain:
//  * the level is held as the LDS byte address z of its table row, so an
//    entry's address and the next level are one add of a prepared offset each;
//  * for both outcomes of an update the next one's thresholds are read, and the
//    level it leads to is formed, before that outcome is known; a decision is
//    then a select and one compare r < T, and two selects carry it on;
//  * the next group's Philox block is computed a round per update in the time
//    the reads take;
//  * the row has an entry that always accepts for a = 2 and entries that never
//    accept for moves out of the window (T as a 32-bit word, 2^32 stored as
//    2^32 - 1 and r as min(r, 2^32 - 2); exact unless a threshold is 2^32 - 1
//    itself.  EXACT is the form for such a table: T - 1 stored, r <= T - 1, and
//    the window's end a compare of its own, 16 to 21 % slower: L = 64, 4096
//    walkers 308 us per sweep against 261);
//  * every fourth update the four lanes count the levels of the last four
//    updates with one LDS atomic, each lane one of them.
// Rows are six words (five entries and the count) for L <= 96.  L = 128 has
// room for four-word rows (a = 0, 1, 4, 3; a = 2 accepted by its zero step)
// and 16-bit counts, two levels per word, added to H before they can overflow.
// Counts go straight to H by 64-bit atomics: a workgroup visits few levels.
//
// Measured, 4096 walkers, L = 64, recorded: 153 ns per update with one lane
// per walker (two LDS reads, an LDS atomic and about 57 VALU instructions of
// one wave per update), 65 ns so (about 18 VALU and 2.3 LDS instructions; a
// lone wave issues one in 8 cycles on a chain).  16384 walkers at L = 64: 159 ns
// before, 66 now; 65536 at L = 16: 200 ns before (2.0 ms per 40 sweeps without
// counting, 48 ms with its global atomics), 142 now.
template <int L>
struct MucaRow {
    static constexpr bool kWide = L <= 96;
    static constexpr int S = kWide ? 24 : 16;  // bytes per row
    static constexpr int K = L * L / 2;
    static constexpr int TAB = (K + 4) * S;    // rows K + 1 .. K + 3 are read ahead, never used
    static constexpr int LDS = TAB + (kWide ? 0 : (K / 2 + 1) * 4);
};

constexpr int kMucaMaxWaves = 4;  // 64 walkers per workgroup: at most 64 N counts per sweep

// Adds the LDS counts to H and clears them.  Every wave does so on its own,
// exchanging each word: no wave waits for another.
template <int L>
__device__ __forceinline__ void muca_flush(uint32_t *lds, int64_t *H, int lane)
{
    using M = MucaRow<L>;
    if constexpr (M::kWide) {
        for (int k = lane; k <= M::K; k += 64) {
            const uint32_t v = lds[k * 6 + 5] ? atomicExch(&lds[k * 6 + 5], 0u) : 0u;
            if (v) atomicAdd((unsigned long long *)&H[k], (unsigned long long)v);
        }
    } else {
        uint32_t *h16 = lds + M::TAB / 4;
        for (int i = lane; i <= M::K / 2; i += 64) {
            const uint32_t v = h16[i] ? atomicExch(&h16[i], 0u) : 0u;
            if (v & 0xFFFFu) atomicAdd((unsigned long long *)&H[2 * i], (unsigned long long)(v & 0xFFFFu));
            if (v >> 16) atomicAdd((unsigned long long *)&H[2 * i + 1], (unsigned long long)(v >> 16));
        }
    }
}

template <int L, bool EXACT>
__global__ __launch_bounds__(64 * kMucaMaxWaves) void k_muca_q(MucaArgs a)
{
    using R = QuadRow<L>;
    using M = MucaRow<L>;
    constexpr int N = L * L, K = N / 2, NW = R::NW, CB = R::CB, S = M::S;
    extern __shared__ __align__(16) uint32_t lds[];
    const int tid = threadIdx.x, nt = blockDim.x, q = tid & 3;
    // thresholds: word c of row k (wide: c = a; else c = 0, 1, 2, 3 for
    // a = 0, 1, 4, 3); entries 0..3 of a.table are steps -2, -1, +1, +2
    for (int i = tid; i < (K + 1) * 4; i += nt) {
        const int k = i >> 2, e = i & 3, step = e < 2 ? e - 2 : e - 1;
        const uint32_t v = a.table[i];
        const uint32_t T = EXACT ? v : k + step > K ? 0u : v == ~0u ? ~0u : v + 1u;
        if constexpr (M::kWide) lds[k * 6 + 2 - step] = T;
        else lds[k * 4 + (step == -2 ? 2 : 2 - step)] = T;
    }
    if constexpr (M::kWide) {
        for (int k = tid; k <= K; k += nt) {
            lds[k * 6 + 2] = ~0u;
            lds[k * 6 + 5] = 0u;
        }
    } else {
        for (int i = tid; i <= K / 2; i += nt) lds[M::TAB / 4 + i] = 0u;
    }
    __syncthreads();
    // lanes past the last walker follow walker W - 1 (in the same wave, in step
    // with it) without storing anything; a wave with no walker has nothing to do
    const int wr = blockIdx.x * (nt >> 2) + (tid >> 2);
    if ((int)(blockIdx.x * (nt >> 2) + ((tid & ~63) >> 2)) >= a.W) return;
    const bool live = wr < a.W;
    const int w = live ? wr : a.W - 1;
    int8_t *sp = a.spins + (int64_t)w * N;
    const uint32_t rec = (a.record && live) ? 1u : 0u;
    // 16-bit counts: every wave exchanges the counts it finds after each kFlushRows
    // of its rows, from one sweep to the next as within one, so that between two
    // exchanges of a word, whichever wave makes them, each of the workgroup's
    // waves adds at most kFlushRows rows of 16 walkers, all of them perhaps to
    // one level
    constexpr int kFlushRows = 65535 / (16 * kMucaMaxWaves * L);
    static_assert(M::kWide || (kFlushRows >= 1 && kFlushRows * 16 * kMucaMaxWaves * L < 65536), "16-bit counts");
    int rows_since_flush = 0;
    // z: LDS address of the level's row, plus 8 where the row is indexed by -4 step
    const int zb = lds_addr(lds) + (M::kWide ? 8 : 0), zend = zb + S * K;
    int z = S * (int)((a.E[w] + 2 * N) / 4) + zb;
    for (int t = 0; t < a.nsweeps; ++t) {
        const uint64_t sweep = a.sweep0 + (uint64_t)t;
        const uint32_t w3 = ctr_w3(kTagMuca, 0, sweep);
        uint4 blk = make_uint4(0u, 0u, 0u, 0u);
        if (R::kAhead) blk = philox(make_uint4((uint32_t)q, (uint32_t)w, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
        uint32_t U[NW], C[NW], D[NW], R0[NW], raw[R::RD];
        quad_load<L>(sp, L - 1, q, raw);
        quad_pack<L>(raw, U);
        quad_load<L>(sp, 0, q, raw);
        quad_pack<L>(raw, C);
        quad_load<L>(sp, 1, q, raw);
        quad_pack<L>(raw, D);
        for (int y = 0; y < L; ++y) {
            const bool pre = y + 2 < L;
            if (pre) quad_load<L>(sp, y + 2, q, raw);
            for (int wi = 0; wi < NW; ++wi) {
                const uint32_t c0 = C[0], u = U[0], d = D[0];
                QuadPlanes P = quad_planes<CB>(c0, u, d, C[NW - 1] >> (CB - 1),
                                                     C[NW > 1 ? 1 : 0] & 1u);
                uint32_t F = 0u;
                bool acc = false;  // previous update's outcome (resolved before a word)
                for (int g = 0; g < (CB + 15) / 16; ++g) {  // one group, or two of a 32-bit word
                    // this lane's share of the group: four random words and counts
                    const int sh = 16 * g + 4 * q;
                    const uint32_t ctr0 = (uint32_t)(L * y + CB * wi + sh) >> 2;
                    if (!R::kAhead)
                        blk = philox(make_uint4(ctr0, (uint32_t)w, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                    PhiloxRounds ahead;
                    ahead.c = make_uint4(ctr0 + 4u, (uint32_t)w, (uint32_t)sweep, w3);
                    constexpr uint32_t kTop = EXACT ? ~0u : ~0u - 1u;
                    const uint32_t r4[4] = {min(blk.x, kTop), min(blk.y, kTop), min(blk.z, kTop), min(blk.w, kTop)};
                    const QuadCounts qc = quad_counts(P, sh);
                    // i0, i1: table offset for a rejected / accepted previous
                    // update; s0, s1: the step in bytes
                    int i0[4], i1[4], s0[4], s1[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int a0 = qc.n3[i] + qc.l[i], a1 = qc.n3[i] + 1 - qc.l[i];
                        if constexpr (M::kWide) {
                            i0[i] = 4 * a0 - 8;
                            i1[i] = 4 * a1 - 8;
                        } else {
                            i0[i] = 4 * a0 - ((a0 >> 2) << 3);
                            i1[i] = 4 * a1 - ((a1 >> 2) << 3);
                        }
                        s0[i] = __mul24(a0, -S) + 2 * S;
                        s1[i] = __mul24(a1, -S) + 2 * S;
                    }
                    // zn: the level the update leads to; T0, T1: its threshold for a
                    // rejected / accepted previous update
                    uint32_t T0, T1;
                    const int x0 = z + (int)quad_get((uint32_t)i0[0], 0), x1 = z + (int)quad_get((uint32_t)i1[0], 0);
                    const int v0 = z + (int)quad_get((uint32_t)s0[0], 0), v1 = z + (int)quad_get((uint32_t)s1[0], 0);
                    T0 = T1 = lds_read(acc ? x1 : x0);
                    int zn = acc ? v1 : v0, zc = z;
                    uint32_t Fg = 0u;
                    bool ok0 = false;
#pragma unroll
                    for (int b = 0; b < 16; ++b) {
                        if (b >= CB) break;
                        const int Q = b >> 2, I = b & 3, Qn = (b + 1) >> 2, In = (b + 1) & 3;
                        // next update, for both outcomes of this one: where it leads
                        // and its thresholds
                        uint32_t N0 = 0u, N1 = 0u;
                        int p0 = 0, p1 = 0;
                        if (b < 15) {
                            N0 = lds_read(z + (int)quad_get((uint32_t)i0[In], Qn));
                            N1 = lds_read(zn + (int)quad_get((uint32_t)i1[In], Qn));
                            p0 = z + (int)quad_get((uint32_t)s0[In], Qn);
                            p1 = zn + (int)quad_get((uint32_t)s1[In], Qn);
                        }
                        // the reads go out before the decision waits for the last ones
                        __builtin_amdgcn_sched_barrier(0);
                        if (R::kAhead && b < 10) {
                            ahead.round(b, a.seed_lo, a.seed_hi);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        uint32_t r = quad_get(r4[I], Q);
                        if (!M::kWide) r = zn == z ? 0u : r;  // a = 2: any threshold accepts
                        const uint32_t T = acc ? T1 : T0;
                        const bool ok = EXACT ? r <= T && zn <= zend : r < T;
                        z = ok ? zn : z;
                        zn = ok ? p1 : p0;
                        Fg = shift_in(Fg, __ballot(ok));
                        zc = q == I ? z : zc;
                        if (I == 3 && a.record) {
                            if constexpr (M::kWide) {
                                lds_add(zc + 12, rec);
                            } else {
                                const int kc = zc - zb;  // 16 k: word k / 2, half k mod 2
                                lds_add(zb + M::TAB + ((kc >> 3) & ~3), rec << (kc & 16));
                            }
                        }
                        if (b == 0) ok0 = ok;
                        if (NW == 1 && CB <= 16 && b == 1) {
                            // one-word row: the right neighbour of the last site is
                            // site 0, flipped by now if its update was accepted
                            const int e = (q == (CB - 1) / 4 && ok0) ? (((P.z >> (CB - 1)) & 1u) ? -1 : 1) : 0;
                            i0[(CB - 1) & 3] += 4 * e;
                            i1[(CB - 1) & 3] += 4 * e;
                            s0[(CB - 1) & 3] -= S * e;
                            s1[(CB - 1) & 3] -= S * e;
                        }
                        acc = ok;
                        T0 = N0;
                        T1 = N1;
                    }
                    if (R::kAhead) blk = ahead.c;
                    F |= (__brev(Fg) >> (CB < 16 ? 32 - CB : 16)) << (16 * g);
                    // one-word row: the last site's right neighbour is site 0
                    if (NW == 1 && CB > 16)
                        P = quad_planes<CB>(c0, u, d, c0 >> (CB - 1), (c0 ^ F) & 1u);
                }
                // rotate: the processed word goes last, the next word to index 0
                const uint32_t cn = c0 ^ F;
#pragma unroll
                for (int i = 0; i + 1 < NW; ++i) {
                    C[i] = C[i + 1];
                    U[i] = U[i + 1];
                    D[i] = D[i + 1];
                }
                C[NW - 1] = cn;
                U[NW - 1] = u;
                D[NW - 1] = d;
            }
            quad_store<L>(sp, y, q, live, C);
            if (y == 0) {
#pragma unroll
                for (int i = 0; i < NW; ++i) R0[i] = C[i];
            }
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                U[i] = C[i];
                C[i] = D[i];
            }
            if (pre) quad_pack<L>(raw, D);
            else {
#pragma unroll
                for (int i = 0; i < NW; ++i) D[i] = R0[i];
            }
            if (!M::kWide && a.record && ++rows_since_flush == kFlushRows) {
                muca_flush<L>(lds, a.H, tid & 63);
                rows_since_flush = 0;
            }
        }
    }
    if (a.record) muca_flush<L>(lds, a.H, tid & 63);
    if (live && q == 0) a.E[w] = 4 * (int64_t)((z - zb) / S) - 2 * N;
}

// Walker start: hot start keyed by the walker index (already written by the
// init kernel), energy, and a flip of the odd sub-lattice when E > 0 (E -> -E).
__global__ void k_muca_start(int8_t *spins, int64_t *E, int L, int W)
{
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= W) return;
    const int N = L * L;
    int8_t *s = spins + (int64_t)w * N;
    int64_t e = 0;
    for (int y = 0; y < L; ++y)
        for (int x = 0; x < L; ++x) {
            const int si = s[x + L * y];
            e -= si * (s[(x + 1) % L + L * y] + s[x + L * ((y + 1) % L)]);
        }
    if (e > 0) {
        for (int y = 0; y < L; ++y)
            for (int x = 0; x < L; ++x)
                if ((x + y) & 1) s[x + L * y] = (int8_t)-s[x + L * y];
        e = -e;
    }
    E[w] = e;
}

// Walkers from which, without counting, one lane each is faster than four: four
// lanes take less time per update while SIMDs are idle, and more instructions.
// us per sweep, four lanes (one): L = 4, 32768 walkers 3.6 (3.6), 65536 5.5 (3.7),
// 2^20 61 (15); L = 8, 65536 13.1 (13.5), 98304 17.9 (15.0); L = 12, 65536 24.0
// (28.7), 98304 33.7 (32.5), 262144 84 (82), but 524288 163 (172); L = 16, 98304
// 53 (59), 131072 68 (59), 2^20 500 (469); L = 24, 98304 131 (133), 131072 170
// (135); L = 32, 98304 208 (237), 131072 270 (244), 524288 979 (824); L = 48,
// 131072 596 (803), L = 64 1071 (2057).  With counting the lanes' atomics cost
// more than that at every number.
template <int L>
static bool lane_walkers(int W)  // L <= 32
{
    if (L == 12) return W > 90112 && W <= 294912;
    return W > (L == 4 ? 32768 : L == 8 ? 65536 : 106496);
}

template <int L>
static hipError_t launch_muca_lane(const MucaArgs &a, hipStream_t s)
{
    const size_t lds = (size_t)(L * L / 2 + 1) * 4 * 4;
    hipLaunchKernelGGL(k_muca<L>, dim3((a.W + 63) / 64), dim3(64), lds, s, a);
    return hipGetLastError();
}

template <int L, bool EXACT>
static hipError_t launch_muca_q(const MucaArgs &a, hipStream_t s)
{
    static LdsLimit lim;
    const hipError_t e = lim.ensure((const void *)k_muca_q<L, EXACT>, MucaRow<L>::LDS);
    if (e != hipSuccess) return e;
    // one wave per workgroup until every CU has one, then up to four waves
    // sharing a table (at L = 128 a CU holds one table)
    constexpr int kCUs = 256;
    const int waves = (a.W + 15) / 16;
    const int per = std::min(kMucaMaxWaves, std::max(1, (waves + kCUs - 1) / kCUs));
    hipLaunchKernelGGL((k_muca_q<L, EXACT>), dim3((waves + per - 1) / per), dim3(64 * per), MucaRow<L>::LDS, s, a);
    return hipGetLastError();
}

template <int L>
static hipError_t launch_muca_L(const MucaArgs &a, hipStream_t s)
{
    if constexpr (L <= 32)
        if (!a.record && lane_walkers<L>(a.W)) return launch_muca_lane<L>(a, s);
    return a.edge ? launch_muca_q<L, true>(a, s) : launch_muca_q<L, false>(a, s);
}

bool muca_L_supported(int L)
{
    switch (L) {
    case 4: case 8: case 12: case 16: case 24: case 32: case 48: case 64: case 96: case 128: return true;
    default: return false;
    }
}

hipError_t launch_muca_sweeps(const MucaArgs &a, int L, hipStream_t s)
{
    switch (L) {
    case 4: return launch_muca_L<4>(a, s);
    case 8: return launch_muca_L<8>(a, s);
    case 12: return launch_muca_L<12>(a, s);
    case 16: return launch_muca_L<16>(a, s);
    case 24: return launch_muca_L<24>(a, s);
    case 32: return launch_muca_L<32>(a, s);
    case 48: return launch_muca_L<48>(a, s);
    case 64: return launch_muca_L<64>(a, s);
    case 96: return launch_muca_L<96>(a, s);
    case 128: return launch_muca_L<128>(a, s);
    default: return hipErrorInvalidValue;
    }
}

// Level of disorder of walker w of W in the stratified start: the largest c
// in 0..128 with (257 - 2c)^2 * 2W > 65536 (2W - 2w - 1), i.e. 128 (1 -
// sqrt(1 - (w + 1/2)/W)) rounded, found by bisection in integer arithmetic
// (the condition is monotone in c).
__device__ __forceinline__ uint32_t strat_level(int64_t w, int64_t W)
{
    int lo = 0, hi = 128;
    const int64_t b = 65536ll * (2 * W - 2 * w - 1);
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        const int64_t a = (int64_t)(257 - 2 * mid) * (257 - 2 * mid) * 2 * W;
        if (a > b) lo = mid;
        else hi = mid - 1;
    }
    return (uint32_t)lo;
}

// Walker lattices: site i of walker w is -1 iff byte (i mod 16) of
// Philox(i/16, w, 0, TAG_INIT) >= 256 - c_w, c_w = 128 (hot start) or the
// stratified level.  Threads: x = group of 16 sites, y strides over walkers.
__global__ void k_muca_init(int8_t *spins, int L, int W, int stratified, uint32_t k0, uint32_t k1)
{
    const int N = L * L, groups = (N + 15) / 16;
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= groups) return;
    for (int w = blockIdx.y; w < W; w += gridDim.y) {
        const uint32_t c = stratified ? strat_level(w, W) : 128u;
        const uint4 b = philox(make_uint4((uint32_t)g, (uint32_t)w, 0u, ctr_w3(kTagInit, 0, 0)), k0, k1);
        int8_t *s = spins + (int64_t)w * N;
        for (int k = 0; k < 16 && 16 * g + k < N; ++k) s[16 * g + k] = byte_of(b, (uint32_t)k) >= 256u - c ? -1 : 1;
    }
}

hipError_t launch_muca_settle(int8_t *spins, int64_t *E, int L, int W, hipStream_t s)
{
    hipLaunchKernelGGL(k_muca_start, dim3((W + 63) / 64), dim3(64), 0, s, spins, E, L, W);
    return hipGetLastError();
}

hipError_t launch_muca_start(int8_t *spins, int64_t *E, int L, int W, uint64_t seed, int start, hipStream_t s)
{
    const int groups = (L * L + 15) / 16;
    dim3 grid((unsigned)((groups + 255) / 256), (unsigned)std::min(W, 65535));
    hipLaunchKernelGGL(k_muca_init, grid, dim3(256), 0, s, spins, L, W, start, (uint32_t)seed, (uint32_t)(seed >> 32));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_muca_start, dim3((W + 63) / 64), dim3(64), 0, s, spins, E, L, W);
    return hipGetLastError();
}

}  // namespace mcs
