// k_tile3d.hip -- fused multi-sweep kernel for 3D simple-cubic lattices:
// Ising (J = 1) or +-J couplings, checkerboard Metropolis or heat-bath, int8
// lattices with Lx a multiple of 64 (Sec. "Checkerboard scheme": the
// checkerboard decomposition holds for any bipartite lattice).
//
// Design (gfx950):
//  * One workgroup owns a tile of hy x hz full-width rows (y, z) of one
//    lattice and runs K sweeps on it per launch, redoing a halo of 2K rows on
//    each side in y and z (each half-sweep shrinks the valid region by one row
//    per side), so no workgroup waits for another.
//  * Rows are bit-packed in LDS and split by x parity exactly as in the 2D
//    kernel: the six neighbours of 32 same-colour sites are six words, and
//    with couplings (bit set <=> J < 0, packed the same way) a bond is
//    unsatisfied where spin ^ neighbour ^ coupling is set.
//  * A site's class is a 3-bit count kept bit-sliced (carry-save adders over
//    the six bond words): Metropolis counts unsatisfied bonds a (dE = 12 - 4a,
//    a >= 3 always accepts); heat-bath counts neighbours with J s_j = -1, d
//    (h = 6 - 2d).  Each class has its own threshold; per random bit-plane the
//    threshold bit of every site comes from a multiplexer over the class bits
//    (its inputs alternate between scalar and vector registers), in heat-bath
//    from half the classes and their mirror images (heatbath.hpp), and r32 < T
//    is one bit-serial comparison.  Ties (top byte equal) wait in a queue of their
//    wave (metro2d.hpp).
//  * Per-sweep E and M are summed from the odd half-sweep, as in 2D, and
//    stored per tile in slots that the next launch adds up (em_slots.hpp).
//  * Between the launches of one call the lattice stays packed in global
//    scratch.
//
// What bounds it: VALU issue (heat-bath about 200 instructions of a wave per 64
// words of 32 sites, Metropolis 200) with the redone halo (1.4 times at H = 16,
// K = 2), then the half-sweeps' latency where a CU has one tile.  256^3 x 4
// heat-bath, H = 16, K = 1, 256 threads: 26.1 us per sweep; 27.7 with a
// multiplexer over all seven classes, 29.7 with a tile's rows loaded one after
// the other besides, each by its own division, and a serial sum over the waves
// each sweep; at K = 2 with the thresholds read from LDS for every plane and
// ties settled between two barriers besides 38.7.
// 256^3 alone, 768 threads: 12.0, 12.3, 13.1 and 17.2.
#include "heatbath.hpp"
#include "internal.hpp"
#include "metro2d.hpp"
#include "spin_bytes.hpp"

namespace mcs {

struct Tile3DArgs {
    const void *src;
    void *dst;
    int in_packed, out_packed;
    const uint32_t *Jp;  // packed couplings [3][Lz][Ly][2 Wd] (bit set <=> J < 0), or nullptr
    int Lx, Ly, Lz, nty, ntz;
    int64_t N;
    uint32_t seed_lo, seed_hi, replica0;
    uint64_t sweep0;
    int per_lattice;
    // class thresholds (top byte 0..255 and low 24 bits, low = 2^24 encodes
    // T = 2^32 as 255 * 2^24 + 2^24); Metropolis: class a, T of dE = 12 - 4a
    // (a <= 2); heat-bath: class d, T of h = 6 - 2d
    uint32_t top[kMaxTableLattices][8];
    uint32_t low[kMaxTableLattices][8];
    EmSlots em;  // tile sums of this launch and the previous one
};

// floor(t / n) and t mod n for small non-negative t (below 2^20) through a
// float reciprocal with one correction step
__device__ __forceinline__ void divmod_small(int t, int n, float inv, int &q, int &r)
{
    q = (int)((float)t * inv);
    r = t - q * n;
    if (r < 0) {
        --q;
        r += n;
    } else if (r >= n) {
        ++q;
        r -= n;
    }
}

// First row of tile t of n over L rows: floor(t L / n) (a 64-bit division is a
// hundred scalar instructions, four of them a tile's work of a few words).
__device__ __forceinline__ int tile_cut(int t, int n, int L)
{
    if (L < 65536) return (int)((uint32_t)t * (uint32_t)L / (uint32_t)n);
    return (int)((int64_t)t * L / n);
}

template <int K, bool MEASURE, int RULE, bool HASJ>
__global__ __launch_bounds__(1024) void k_tile3d(Tile3DArgs a)
{
    constexpr bool HB = RULE != kMetropolis;
    extern __shared__ uint32_t lds[];
    __shared__ int sums[2][K > 0 ? K : 1];  // anti-aligned bonds and down spins of each sweep
    __shared__ long long red64[2][16];
    __shared__ uint32_t tlow[8];
    const int l = blockIdx.y;
    const int tz = blockIdx.x / a.nty, ty = blockIdx.x - tz * a.nty;
    const int y0 = tile_cut(ty, a.nty, a.Ly), y1 = tile_cut(ty + 1, a.nty, a.Ly);
    const int z0 = tile_cut(tz, a.ntz, a.Lz), z1 = tile_cut(tz + 1, a.ntz, a.Lz);
    const int hy = y1 - y0, hz = z1 - z0;
    constexpr int R = 2 * K;
    const int Ry = hy + 2 * R, Rz = hz + 2 * R, rows = Ry * Rz;
    const int Wd = a.Lx >> 6;
    const int nt = blockDim.x, tid = threadIdx.x;
    const uint32_t rep = a.replica0 + (uint32_t)l;
    const int li = a.per_lattice ? l : 0;
    if (tid < 8) tlow[tid] = a.low[li][tid];
    uint32_t *Jl = lds + (size_t)rows * 2 * Wd;  // 3 coupling planes of rows
    // behind them: per LDS row its first random block (even), bit 0 the parity
    // of y + z; then each wave's tie queue
    uint32_t *rinfo = lds + (size_t)rows * 2 * Wd * (HASJ ? 4 : 1);
    // per random plane and class the threshold bit as a full mask, those of
    // classes 0, 2, 4 in vector registers (an instruction reads one scalar);
    // mirrored classes 0, 1, 2 in scalar ones
    uint32_t tv[8][3], ts[8][4];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
#pragma unroll
        for (int i = 0; i < (HB ? 3 : 1); ++i) {
            tv[k][i] = ((a.top[li][2 * i] >> k) & 1u) ? ~0u : 0u;
            if (RULE != kHeatBathMirrored) asm volatile("" : "+v"(tv[k][i]));
        }
        ts[k][0] = ((a.top[li][1] >> k) & 1u) ? ~0u : 0u;
        ts[k][1] = ((a.top[li][HB ? 3 : 2] >> k) & 1u) ? ~0u : 0u;
        ts[k][2] = ((a.top[li][5] >> k) & 1u) ? ~0u : 0u;
        ts[k][3] = ((a.top[li][6] >> k) & 1u) ? ~0u : 0u;
    }
    // thread -> (word column, first row, row stride); a row's words are at most
    // the threads
    const int Q = nt / Wd, w0 = tid % Wd, r0 = tid / Wd;
    const bool own = r0 < Q;  // surplus threads idle
    auto widx = [&](int row, int par, int w) { return (row * 2 + par) * Wd + w; };
    auto wrap = [](int v, int n) {
        if (n >= R) return v < 0 ? v + n : v >= n ? v - n : v;
        while (v < 0) v += n;
        while (v >= n) v -= n;
        return v;
    };
    const int wave = tid >> 6;
    if (MEASURE && tid < 2 * K) sums[tid & 1][tid >> 1] = 0;
    uint4 *const tq = (uint4 *)(lds + (((size_t)rows * (2 * Wd * (HASJ ? 4 : 1) + 1) + 3) & ~(size_t)3)) +
                      wave * (kTieQueue * 3 / 2);
    uint2 *const tq2 = (uint2 *)(tq + kTieQueue);
    const int64_t plane_rows = (int64_t)a.Ly * a.Lz;
    const int ntile = gridDim.x, nlat = gridDim.y;
    long long pre_e, pre_m;
    em_prefetch(a.em, blockIdx.x, ntile, l, nlat, tid, pre_e, pre_m);

    // ---- load rows (z0-R .. z1+R-1) x (y0-R .. y1+R-1), row id = rz Ry + ry
    {
        const float invRy = 1.0f / (float)Ry;
        const int sz = Q / Ry, sy = Q - sz * Ry;  // a step of Q rows
        int rz, ry;
        divmod_small(own ? r0 : 0, Ry, invRy, rz, ry);
        constexpr int kBatch = 4;  // rows of a thread in flight at once
        for (int base = 0; base < rows; base += kBatch * Q) {
            const int rb = own ? base + r0 : rows;
            uint32_t at[kBatch];  // word in the lattice
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (base + j * Q >= rows) break;
                const int y = wrap(y0 - R + ry, a.Ly), z = wrap(z0 - R + rz, a.Lz);
                const uint32_t grow = (uint32_t)z * (uint32_t)a.Ly + (uint32_t)y;
                at[j] = grow * (uint32_t)Wd + (uint32_t)w0;
                if (w0 == 0 && rb + j * Q < rows)
                    rinfo[rb + j * Q] = (uint32_t)(a.Lx >> 5) * grow | ((uint32_t)(y + z) & 1u);
                rz += sz;
                ry += sy;
                if (ry >= Ry) {
                    ry -= Ry;
                    ++rz;
                }
            }
            auto copy = [&](const uint2 *src, uint2 *dst) {
                uint2 v[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    if (base + j * Q >= rows) break;
                    if (rb + j * Q < rows) v[j] = src[at[j]];
                }
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    if (base + j * Q >= rows) break;
                    if (rb + j * Q < rows) dst[(rb + j * Q) * Wd + w0] = v[j];
                }
            };
            if (a.in_packed) {
                copy((const uint2 *)a.src + (int64_t)l * plane_rows * Wd, (uint2 *)lds);
            } else {
                const int8_t *src = (const int8_t *)a.src + (int64_t)l * a.N;
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    if (base + j * Q >= rows) break;
                    if (rb + j * Q < rows) {
                        const int8_t *p = src + 64 * (int64_t)at[j];
                        const Row32 h0 = load_row32(p, 0u), h1 = load_row32(p, 32u);
                        lds[widx(rb + j * Q, 0, w0)] =
                            sign_bits16(pick16(h0, 0x06040200u)) | sign_bits16(pick16(h1, 0x06040200u)) << 16;
                        lds[widx(rb + j * Q, 1, w0)] =
                            sign_bits16(pick16(h0, 0x07050301u)) | sign_bits16(pick16(h1, 0x07050301u)) << 16;
                    }
                }
            }
            if (HASJ)
                for (int d = 0; d < 3; ++d)
                    copy((const uint2 *)a.Jp + (int64_t)d * plane_rows * Wd, (uint2 *)Jl + (size_t)d * rows * Wd);
        }
    }
    __syncthreads();
    em_reduce(a.em, blockIdx.x, ntile, l, nlat, tid, nt, pre_e, pre_m, red64);

    for (int s = 0; s < K; ++s) {
        const uint64_t sweep = a.sweep0 + (uint64_t)s;
        int n_acc = 0, d_acc = 0;  // anti-aligned bonds and down spins of this thread's own words
        for (int c = 0; c < 2; ++c) {
            const int p = 2 * s + c;
            const int ny = Ry - 2 * p - 2, nz = Rz - 2 * p - 2;
            const int nrow = ny * nz;
            const float invny = 1.0f / (float)ny;
            const uint32_t w3 = ctr_w3(kTagSweep, (uint32_t)c, sweep);
            const uint32_t w3lo = ctr_w3(kTagSweepLo, (uint32_t)c, sweep);
            uint32_t qn = 0;
            auto draw = [&](uint32_t pend, uint32_t blk, uint32_t c0, uint32_t c1, uint32_t c2, int &dn) {
                uint32_t f = 0u;
                while (pend) {
                    const int b = __builtin_ctz(pend);
                    pend &= pend - 1u;
                    const uint32_t cls = ((c0 >> b) & 1u) | (((c1 >> b) & 1u) << 1) | (((c2 >> b) & 1u) << 2);
                    const uint4 lo = philox(make_uint4(16u * blk + (uint32_t)b, rep, (uint32_t)sweep, w3lo), a.seed_lo,
                                            a.seed_hi);
                    if ((lo.x & 0xFFFFFFu) < tlow[cls]) {
                        f |= 1u << b;
                        // anti-aligned bonds gained: Metropolis 6 - 2a, heat-bath
                        // (-1 -> +1) 2d - 6
                        dn += HB ? 2 * (int)cls - 6 : 6 - 2 * (int)cls;
                    }
                }
                return f;
            };
            // a queued word: {LDS word | own-row flag, first block, tied sites, and
            // their class bits}
            auto settle = [&]() {
                const uint32_t i = tid & 63;
                if (i < qn) {
                    const uint4 it = tq[i];
                    const uint2 cb = tq2[i];
                    int dn = 0;
                    const uint32_t f = draw(it.z, it.y, it.w, cb.x, cb.y, dn);
                    if (f) {
                        const uint32_t ws = it.x & 0x7FFFFFFFu, old = lds[ws];
                        lds[ws] = old ^ f;
                        if (MEASURE && (it.x >> 31)) {
                            n_acc += dn;
                            d_acc += (int)__builtin_popcount(f) - 2 * (int)__builtin_popcount(old & f);
                        }
                    }
                }
                qn = 0;
            };
            // row r0 of the half-sweep's rectangle, advanced by Q rows a step
            const int Qz = Q / ny, Qy = Q - Qz * ny;
            int iz = 0, iy = 0;
            if (own) divmod_small(r0, ny, invny, iz, iy);
            int row = (p + 1 + iz) * Ry + p + 1 + iy;
            for (int rr = 0; rr < nrow; rr += Q) {
                uint32_t pend = 0u, ws = 0u, blk = 0u, c0 = 0u, c1 = 0u, c2 = 0u;
                const bool interior = MEASURE && c == 1 && (uint32_t)(p + 1 + iy - R) < (uint32_t)hy &&
                                      (uint32_t)(p + 1 + iz - R) < (uint32_t)hz;
                if (own && rr + r0 < nrow) {
                    const uint32_t info = rinfo[row];
                    const bool q = (c ^ (int)info) & 1;
                    const int ev = row * 2 * Wd + w0, od = ev + Wd;  // even- and odd-x words
                    const int is = q ? od : ev, io = q ? ev : od;
                    const uint32_t S = lds[is], O = lds[io];
                    // x neighbours: even sites (q = 0) have +x in O, -x one odd
                    // site to the left; odd sites the mirror image
                    const int side = q ? (w0 + 1 == Wd ? 1 - Wd : 1) : (w0 == 0 ? Wd - 1 : -1);
                    const uint32_t Nb = lds[io + side];
                    const uint32_t Sh = __builtin_amdgcn_alignbit(q ? Nb : O, q ? O : Nb, q ? 1u : 31u);
                    uint32_t w1 = O, w2 = Sh;  // the same place, the shifted one
                    uint32_t w3b = lds[is + 2 * Wd], w4 = lds[is - 2 * Wd];
                    uint32_t w5 = lds[is + 2 * Wd * Ry], w6 = lds[is - 2 * Wd * Ry];
                    if (HASJ) {
                        // coupling word of direction d at the place of LDS word i
                        auto J = [&](int d, int i) { return Jl[d * rows * 2 * Wd + i]; };
                        // bonds to + x belong to the left end: the even site's to
                        // its own word, the odd site's (+x) to its own word too
                        const uint32_t Js = J(0, is), Jo = J(0, io);
                        const uint32_t Jl_ = q ? 0u : J(0, io + side);
                        w1 ^= q ? Jo : Js;
                        w2 ^= q ? Js : __builtin_amdgcn_alignbit(Jo, Jl_, 31);
                        w3b ^= J(1, is);
                        w4 ^= J(1, is - 2 * Wd);
                        w5 ^= J(2, is);
                        w6 ^= J(2, is - 2 * Wd * Ry);
                    }
                    // bit set in wk <=> J s_j = -1 for that bond; Metropolis
                    // counts unsatisfied bonds S ^ wk, heat-bath counts wk
                    uint32_t x1 = w1, x2 = w2, x3 = w3b, x4 = w4, x5 = w5, x6 = w6;
                    if (!HB) {
                        x1 ^= S;
                        x2 ^= S;
                        x3 ^= S;
                        x4 ^= S;
                        x5 ^= S;
                        x6 ^= S;
                    }
                    const uint32_t s1 = MCS_BOP3(x1, x2, x3, MCS_A ^ MCS_B ^ MCS_C);
                    const uint32_t k1 = MCS_BOP3(x1, x2, x3, (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
                    const uint32_t s2 = MCS_BOP3(x4, x5, x6, MCS_A ^ MCS_B ^ MCS_C);
                    const uint32_t k2 = MCS_BOP3(x4, x5, x6, (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
                    const uint32_t kk = s1 & s2;
                    c0 = s1 ^ s2;
                    c1 = MCS_BOP3(k1, k2, kk, MCS_A ^ MCS_B ^ MCS_C);
                    c2 = MCS_BOP3(k1, k2, kk, (MCS_A & MCS_B) | (MCS_A & MCS_C) | (MCS_B & MCS_C));
                    // Metropolis: a >= 3 accepts without a random number
                    const uint32_t ge3 = HB ? 0u : MCS_BOP3(c2, c1, c0, MCS_A | (MCS_B & MCS_C));
                    // random planes of the 32 sites
                    blk = 2u * (uint32_t)w0 + (info & ~1u);
                    const uint4 A = philox(make_uint4(blk, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                    const uint4 B = philox(make_uint4(blk + 1u, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                    // bit-serial r < T(class) from the least significant plane;
                    // the threshold bit of each site is chosen by its class
                    uint32_t lt = 0u, eq = ~0u;
                    MirroredClasses mc;
                    if constexpr (RULE == kHeatBathMirrored) mc = mirror_classes<3>(c0, c1, c2);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const uint32_t X = plane_pair(A, B, k);
                        // mux(s, hi, lo): hi where s is set
                        auto mux = [](uint32_t sel, uint32_t hi, uint32_t lo) {
                            return MCS_BOP3(sel, hi, lo, (MCS_A & MCS_B) | (~MCS_A & MCS_C));
                        };
                        const uint32_t m01 = mux(c0, ts[k][0], tv[k][0]);
                        uint32_t T;
                        if constexpr (RULE == kHeatBathMirrored) {
                            T = k == 7 ? ~mc.s : mirrored_plane<3>(mc, tv[k][0], ts[k][0], tv[k][1]);
                        } else if (HB) {
                            const uint32_t lo4 = mux(c1, mux(c0, ts[k][1], tv[k][1]), m01);
                            const uint32_t hi4 = mux(c1, ts[k][3], mux(c0, ts[k][2], tv[k][2]));
                            T = mux(c2, hi4, lo4);
                        } else {
                            T = mux(c1, ts[k][1], m01);
                        }
                        lt = MCS_BOP3(X, T, lt, (~MCS_A & MCS_B) | (~MCS_A & MCS_C) | (MCS_B & MCS_C));
                        eq = MCS_BOP3(eq, X, T, MCS_A & ~(MCS_B ^ MCS_C));
                    }
                    // Metropolis: flip where accepted; heat-bath: new spin
                    // word, +1 (bit 0) where r < T; ties provisionally -1
                    const uint32_t Sn = HB ? ~lt : MCS_BOP3(S, ge3, lt, MCS_A ^ (MCS_B | MCS_C));
                    pend = HB ? eq : (eq & ~ge3);
                    lds[is] = Sn;
                    ws = (uint32_t)is;
                    if (interior) {
                        // bonds of the odd sites after their update
                        n_acc += (int)(__builtin_popcount(Sn ^ w1) + __builtin_popcount(Sn ^ w2) +
                                       __builtin_popcount(Sn ^ w3b) + __builtin_popcount(Sn ^ w4) +
                                       __builtin_popcount(Sn ^ w5) + __builtin_popcount(Sn ^ w6));
                        d_acc += (int)(__builtin_popcount(Sn) + __builtin_popcount(O));
                    }
                }
                const uint64_t m = __ballot(pend != 0u);
                if (m) {
                    const uint32_t cnt = (uint32_t)__popcll(m);
                    if (qn + cnt > (uint32_t)kTieQueue) settle();
                    if (pend) {
                        const uint32_t at = qn + wave_rank(m);
                        tq[at] = make_uint4(ws | ((uint32_t)interior << 31), blk, pend, c0);
                        tq2[at] = make_uint2(c1, c2);
                    }
                    qn += cnt;
                }
                iz += Qz;
                iy += Qy;
                row += Qz * Ry + Qy;
                if (iy >= ny) {
                    iy -= ny;
                    ++iz;
                    row += Ry - ny;
                }
            }
            settle();
            if (MEASURE && c == 1) {
                n_acc = __builtin_amdgcn_readlane(wave_sum_last(n_acc), 63);
                d_acc = __builtin_amdgcn_readlane(wave_sum_last(d_acc), 63);
                if ((tid & 63) < 2) atomicAdd(&sums[tid & 1][s], (tid & 1) ? d_acc : n_acc);
            }
            __syncthreads();
        }
    }
    if (MEASURE && tid < K) {
        // every bond once: 2 (anti-aligned) - 6 per odd site; M from both parities
        const long long words = (long long)hy * hz * Wd;
        *em_slot(a.em.slots, tid, l, nlat, blockIdx.x, ntile) =
            make_longlong2(2ll * sums[0][tid] - 192 * words, 64 * words - 2ll * sums[1][tid]);
    }

    // ---- store the tile's own rows
    if (!own) return;
    const int own_rows = hy * hz, sz = Q / hy, sy = Q - sz * hy;
    int iz, iy;
    divmod_small(r0, hy, 1.0f / (float)hy, iz, iy);
    for (int rr = r0; rr < own_rows; rr += Q) {
        const int row = (R + iz) * Ry + (R + iy);
        const int64_t grow = (int64_t)(z0 + iz) * a.Ly + (y0 + iy);
        if (a.out_packed) {
            uint2 *dst = (uint2 *)a.dst + ((int64_t)l * plane_rows + grow) * Wd;
            dst[w0] = ((const uint2 *)lds)[row * Wd + w0];
        } else {
            const uint32_t ev = lds[widx(row, 0, w0)], od = lds[widx(row, 1, w0)];
            uint4 *pp = (uint4 *)((int8_t *)a.dst + (int64_t)l * a.N + grow * a.Lx + 64 * w0);
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                uint32_t dw[4];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    // four even and four odd columns, bit 0 -> byte 0x01 (+1), 1 -> 0xFF (-1)
                    const int sh = 8 * qq + 4 * i;
                    const uint32_t ee = 0x01010101u ^ (spread4((ev >> sh) & 15u) * 0xFEu);
                    const uint32_t oo = 0x01010101u ^ (spread4((od >> sh) & 15u) * 0xFEu);
                    dw[2 * i] = __builtin_amdgcn_perm(oo, ee, 0x05010400u);
                    dw[2 * i + 1] = __builtin_amdgcn_perm(oo, ee, 0x07030602u);
                }
                pp[qq] = make_uint4(dw[0], dw[1], dw[2], dw[3]);
            }
        }
        iz += sz;
        iy += sy;
        if (iy >= hy) {
            iy -= hy;
            ++iz;
        }
    }
}

// Couplings to the packed row layout: bit b of word w of the even (odd) array
// of row (y, z) of direction d is set iff J[d][z][y][64 w + 2 b (+1)] < 0.
__global__ void k_pack_couplings(const int8_t *J, uint32_t *Jp, int Lx, int64_t rows3)
{
    const int Wd = Lx >> 6;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= rows3 * Wd) return;
    const int64_t r = t / Wd;
    const int w = (int)(t % Wd);
    const int8_t *row = J + r * Lx + 64 * w;
    uint32_t ev = 0, od = 0;
    for (int b = 0; b < 32; ++b) {
        ev |= (uint32_t)(row[2 * b] < 0) << b;
        od |= (uint32_t)(row[2 * b + 1] < 0) << b;
    }
    Jp[(r * 2 + 0) * Wd + w] = ev;
    Jp[(r * 2 + 1) * Wd + w] = od;
}

// ---------------------------------------------------------------------------
bool tile3d_supported(const SweepCall &c, int layout)
{
    return layout == MC_INT8 && c.g.dims == 3 && (c.g.Lx % 64) == 0 && c.g.Lx <= 4096 && c.g.Ly >= 4 &&
           c.g.Lz >= 4 && (!c.per_lattice || c.g.count <= kMaxTableLattices);
}

// Of the tile's rows (with couplings), the size a plan is checked by.
size_t tile3d_lds_bytes(int Lx, int H, int K, bool hasJ)
{
    const size_t side = (size_t)H + 4 * (size_t)K;
    const size_t words = (side * side * 2 * (size_t)(Lx / 64) * (hasJ ? 4 : 1) + 3) & ~(size_t)3;
    return (words + 64) * 4;
}

// The rows, a word per row, each wave's tie queue.
static size_t tile3d_dynamic_lds(int Lx, int H, int K, bool hasJ, int threads)
{
    const size_t side = (size_t)H + 4 * (size_t)K, rows = side * side;
    const size_t words = (rows * (2 * (size_t)(Lx / 64) * (hasJ ? 4 : 1) + 1) + 3) & ~(size_t)3;
    return words * 4 + (K ? (size_t)(threads / 64) * kTieQueue * 24 : 0);
}
// a plan's rows take at most 96 KB, with couplings 4 x 8 bytes and up each
constexpr int kTile3DMaxLds = 98304 + 98304 / 32 * 4 + 16 * kTieQueue * 24;
static_assert(kTile3DMaxLds <= 155 * 1024, "next to the static arrays in 160 KB");

template <int K, int RULE, bool HASJ>
static hipError_t launch3(const Tile3DArgs &a, int H, int count, int threads, hipStream_t s)
{
    const size_t lds = tile3d_dynamic_lds(a.Lx, H, K, HASJ, threads);
    dim3 grid((unsigned)(a.nty * a.ntz), (unsigned)count);
    static LdsLimit lim[2];
    {
        const void *f =
            a.em.slots ? (const void *)k_tile3d<K, true, RULE, HASJ> : (const void *)k_tile3d<K, false, RULE, HASJ>;
        const hipError_t e = lim[a.em.slots ? 1 : 0].ensure(f, kTile3DMaxLds);
        if (e != hipSuccess) return e;
    }
    if (a.em.slots) hipLaunchKernelGGL((k_tile3d<K, true, RULE, HASJ>), grid, dim3(threads), lds, s, a);
    else hipLaunchKernelGGL((k_tile3d<K, false, RULE, HASJ>), grid, dim3(threads), lds, s, a);
    return hipGetLastError();
}

template <int RULE, bool HASJ>
static hipError_t launch3k(const Tile3DArgs &a, int k, int H, int count, int threads, hipStream_t s)
{
    switch (k) {
    case 0: return launch3<0, RULE, HASJ>(a, H, count, threads, s);
    case 1: return launch3<1, RULE, HASJ>(a, H, count, threads, s);
    case 2: return launch3<2, RULE, HASJ>(a, H, count, threads, s);
    case 3: return launch3<3, RULE, HASJ>(a, H, count, threads, s);
    case 4: return launch3<4, RULE, HASJ>(a, H, count, threads, s);
    default: return hipErrorInvalidValue;
    }
}

static void class_thresholds(const SweepTables &t, int rule, uint32_t *top, uint32_t *low)
{
    for (int cl = 0; cl < 8; ++cl) {
        Thr th{0u, 0u};
        if (rule == 0) {
            if (cl <= 2) th = t.met[3 - cl];       // dE = 12 - 4a
        } else if (cl <= 6) {
            th = t.hb[12 - 2 * cl];                // h = 6 - 2d, index h + 6
        }
        if (th.top >= 256u) th = Thr{255u, 1u << 24};  // T = 2^32
        top[cl] = th.top;
        low[cl] = th.low;
    }
}

hipError_t launch_tile3d(const SweepCall &c, const void *src, int in_packed, void *dst, int out_packed,
                         const uint32_t *Jp, uint64_t sweep0, int k, int H, int threads, const EmSlots &em,
                         hipStream_t s)
{
    Tile3DArgs a;
    a.src = src;
    a.dst = dst;
    a.in_packed = in_packed;
    a.out_packed = out_packed;
    a.Jp = Jp;
    a.Lx = c.g.Lx;
    a.Ly = c.g.Ly;
    a.Lz = c.g.Lz;
    a.nty = (c.g.Ly + H - 1) / H;
    a.ntz = (c.g.Lz + H - 1) / H;
    a.N = c.g.N;
    a.seed_lo = c.seed_lo;
    a.seed_hi = c.seed_hi;
    a.replica0 = c.replica0;
    a.sweep0 = sweep0;
    a.per_lattice = c.per_lattice;
    bool mirrored = c.rule == 1;
    for (int i = 0; i < kMaxTableLattices; ++i) {
        const SweepTables &t = (c.per_lattice && i < c.g.count) ? c.tabs[i] : c.tab;
        class_thresholds(t, c.rule, a.top[i], a.low[i]);
        if (i == 0 || (c.per_lattice && i < c.g.count)) mirrored = mirrored && mirrored_classes(a.top[i], 6);
    }
    a.em = em;
    if (k == 0) a.em.slots = nullptr;
    if (!em.red_in) a.em.red_K = 0;
    const bool hj = Jp != nullptr;
    if (mirrored) return hj ? launch3k<kHeatBathMirrored, true>(a, k, H, c.g.count, threads, s)
                            : launch3k<kHeatBathMirrored, false>(a, k, H, c.g.count, threads, s);
    if (c.rule == 1) return hj ? launch3k<kHeatBath, true>(a, k, H, c.g.count, threads, s)
                               : launch3k<kHeatBath, false>(a, k, H, c.g.count, threads, s);
    return hj ? launch3k<kMetropolis, true>(a, k, H, c.g.count, threads, s)
              : launch3k<kMetropolis, false>(a, k, H, c.g.count, threads, s);
}

// Per-tile (E, M) slots of one launch: K <= 4 sweeps x count lattices x
// ceil(Ly / 2) ceil(Lz / 2) tiles (a plan's tile side is at least 2, the
// smallest that fits LDS at Lx = 4096) x 16 bytes.
size_t tile3d_slot_bytes(const Geom &g)
{
    const size_t b = (size_t)4 * (size_t)g.count * (size_t)((g.Ly + 1) / 2) * (size_t)((g.Lz + 1) / 2) * 16;
    return (b + 255) / 256 * 256;
}

hipError_t launch_pack_couplings(const Geom &g, const int8_t *J, uint32_t *Jp, hipStream_t s)
{
    const int64_t rows3 = 3 * (int64_t)g.Ly * g.Lz;
    const int64_t n = rows3 * (g.Lx / 64);
    hipLaunchKernelGGL(k_pack_couplings, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, J, Jp, g.Lx, rows3);
    return hipGetLastError();
}

}  // namespace mcs
