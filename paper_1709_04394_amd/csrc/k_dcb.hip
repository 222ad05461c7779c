// k_dcb.hip -- double-checkerboard Metropolis sweeps with k hits per tile
// (Sec. "Checkerboard scheme": tiles in a coarse checkerboard, each tile
// loaded once and updated k times; multi-hit updates) of the 2D ferromagnet
// (J = 1), on lattices kept bit-packed in global scratch between launches.
//
// One launch updates every tile of one coarse colour: a workgroup loads its
// T x T tile with a one-site halo (one row above and below, one 64-site word
// column left and right, of which only the edge sites are read) from the
// packed lattice into LDS, runs k rounds of the tile's own checkerboard (even
// sites, then odd), and writes the tile back in place.  The halo belongs to
// tiles of the other coarse colour, which no workgroup of this launch writes,
// so the launch has no race and no redone halo: every update is done once.
// A sweep is two launches (coarse colour 0, then 1).  The per-word update
// (four neighbour words, Metropolis classes from 3-input bit operations, the
// random top bytes as eight bit-planes from two Philox blocks, a bit-serial
// compare, ties settled by the word's own lane or from a queue of the wave) is
// the 2D band kernel's (metro2d.hpp).
//
// What bounds it: VALU issue from ten hits on, with one hit the launch, the
// tile's load and the sums.  Attempted updates per ns, 4096^2 x 3, tiles of 128,
// at one, ten and a hundred hits: 2050, 4370 and 5060; 2000, 4320 and 5040 with
// one wave at a time settling the ties of all between two barriers; 1330, 3880
// and 4980 with tiles side by side on different XCDs besides (each then loads
// whole lines for 8 bytes of a row); 1180, 3050 and 3700 with a comparison per
// class besides.  One lattice of 2048^2, ten hits: 400 us for ten sweeps, 490
// with each wave's ties through its queue in LDS although a lane has one word;
// tiles of 64 (4096^2 x 3) 1122 and 1224.
//
// Energy and magnetisation of a sweep: every bond lies inside one tile or
// joins a tile of colour 0 to one of colour 1.  Colour-0 tiles are final
// after their launch and record their internal bonds and spins; colour-1
// tiles record theirs plus all bonds across their edges (the other ends are
// final).  Each tile writes its share to a slot of its own; the first
// workgroup of each lattice in the next sweep's colour-0 launch adds up the
// previous sweep's slots while it loads its tile (em_slots.hpp), and a small
// kernel adds up those of a call's last sweep.
#include <algorithm>

#include "internal.hpp"
#include "metro2d.hpp"

namespace mcs {

constexpr int kDcbMaxWaves = 16;

struct DcbArgs {
    uint32_t *lat;              // packed lattices, rows of 2 L/64 words (even-x array first)
    int L, T;                   // extent, tile side (multiples of 64)
    int coarse;                 // colour of the tiles of this launch
    int hits;
    uint32_t replica0;
    uint64_t sweep;             // global sweep number; hit h draws as plain sweep sweep * hits + h
    uint32_t seed_lo, seed_hi;
    Thr t4, t8;                 // Metropolis thresholds dE = 4, 8
    int64_t *part;              // [count][tiles][2] (E, M) shares of the tiles, or nullptr
    EmSlots prev;               // the previous sweep's slots (red_K = 1) to add up, or none
};

// Workgroup -> tile: tiles of one coarse colour, (L/T)^2 / 2 of them, row by
// row of tiles (on one XCD: tiles side by side share the lines of their rows).
__device__ __forceinline__ void dcb_tile(const DcbArgs &a, int b, int &tx, int &ty)
{
    const int nt = a.L / a.T, half = nt / 2;
    b = (int)xcd_order((uint32_t)b, gridDim.x);
    ty = b / half;
    tx = 2 * (b - ty * half) + ((ty + a.coarse) & 1);
}

// ONE: a lane has one word and settles its ties at once; else a wave's tied words
// gather over its lanes' words.
template <bool ONE>
__global__ __launch_bounds__(64 * kDcbMaxWaves) void k_dcb(DcbArgs a)
{
    extern __shared__ uint32_t lds[];
    __shared__ int red[2][kDcbMaxWaves];
    __shared__ long long red_prev[2][16];
    const int l = blockIdx.y;
    int tx, ty;
    dcb_tile(a, blockIdx.x, tx, ty);
    const int Wl = a.L >> 6;             // words per row and parity in the lattice
    const int Wt = a.T >> 6;             // words per row and parity in the tile
    const int Ww = Wt + 2;               // with the halo columns
    const int rows = a.T + 2;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int wave = tid >> 6, nwaves = nt >> 6;
    const uint32_t rep = a.replica0 + (uint32_t)l;
    const int y0 = ty * a.T, wc0 = tx * Wt, tsh = 31 - __builtin_clz(a.T), wsh = tsh - 6;
    uint32_t *lat = a.lat + (size_t)l * a.L * 2 * Wl;
    // LDS word (r, par, c): tile row r - 1 (r = 0 and T + 1 are halo rows),
    // word column c - 1 of the tile (c = 0 and Wt + 1 are halo columns)
    auto widx = [&](int r, int par, int c) { return (r * 2 + par) * Ww + c; };
    const MetroMasks mm = metro_masks(a.t4.top, a.t8.top, true);
    uint4 *const queue = (uint4 *)(lds + ((rows * 2 * Ww + 3) & ~3));  // behind the tile
    const int slots_per_lattice = (a.L / a.T) * (a.L / a.T);
    long long pre_e, pre_m;
    em_prefetch(a.prev, blockIdx.x, slots_per_lattice, l, gridDim.y, tid, pre_e, pre_m);

    // ---- load the tile and its halo: a row's words of one parity, of the column
    // to the left (odd) or right (even) that word, and the rows above and below
    const int left = wc0 == 0 ? Wl - 1 : wc0 - 1, right = wc0 + Wt == Wl ? 0 : wc0 + Wt;
    for (int i = tid; i < 2 * a.T; i += nt) {
        const uint32_t *src = lat + (size_t)(2 * y0 + i) * Wl;
        uint32_t *dst = lds + (i + 2) * Ww;
        const uint32_t edge = src[(i & 1) ? left : right];
        if (Wt == 1) {
            dst[1] = src[wc0];
        } else {
            for (int c = 0; c < Wt; c += 2) {
                uint2 v;
                __builtin_memcpy(&v, src + wc0 + c, 8);
                dst[1 + c] = v.x;
                dst[2 + c] = v.y;
            }
        }
        dst[(i & 1) ? 0 : Wt + 1] = edge;
    }
    for (int i = tid; i < 4 * Wt; i += nt) {
        const int rp = i >> wsh, c = i & (Wt - 1);
        const int y = rp < 2 ? (y0 == 0 ? a.L - 1 : y0 - 1) : (y0 + a.T == a.L ? 0 : y0 + a.T);
        lds[(rp < 2 ? rp : 2 * a.T + rp) * Ww + 1 + c] = lat[((size_t)y * 2 + (rp & 1)) * Wl + wc0 + c];
    }
    __syncthreads();
    em_reduce(a.prev, blockIdx.x, slots_per_lattice, l, gridDim.y, tid, nt, pre_e, pre_m, red_prev);

    const int tasks = a.T * Wt;  // words of one colour: one per (row, column), a multiple of the threads
    uint4 *const tq = queue + wave * kTieQueue;
    for (int h = 0; h < a.hits; ++h) {
        const uint64_t dsweep = a.sweep * (uint64_t)a.hits + (uint64_t)h;
        for (int col = 0; col < 2; ++col) {
            const uint32_t w3 = ctr_w3(kTagSweep, (uint32_t)col, dsweep);
            const uint32_t w3lo = ctr_w3(kTagSweepLo, (uint32_t)col, dsweep);
            uint32_t qn = 0;
            auto settle = [&](const uint4 &it) {
                const uint32_t f = metro_settle(it.z, it.w, it.y, rep, (uint32_t)dsweep, w3lo, a.seed_lo, a.seed_hi,
                                                a.t4.low, a.t8.low);
                if (f) lds[it.x] ^= f;
            };
            for (int t = tid; t < tasks; t += nt) {
                // words column by column: T is a power of two
                const int c = 1 + (t >> tsh), r = 1 + (t & (a.T - 1));
                const int y = y0 + r - 1;
                const int q = (col + y) & 1;
                const int e = r * 2 * Ww + c, o = e + Ww;  // even- and odd-x words
                const int is = q ? o : e, io = q ? e : o;
                // even-x sites: left neighbours are the odd sites one to the
                // left; odd-x sites: right neighbours are the even sites one
                // to the right (halo columns at the tile's edges)
                const uint32_t S = lds[is], U = lds[is - 2 * Ww], D = lds[is + 2 * Ww], O = lds[io];
                const uint32_t Nb = lds[io + (q ? 1 : -1)];
                const uint32_t Sh = __builtin_amdgcn_alignbit(q ? Nb : O, q ? O : Nb, q ? 1u : 31u);
                // random planes of the 32 same-colour sites j0 .. j0+31,
                // j0 = 32 w + (L/2) y, w the lattice word column
                const uint32_t blk = 2u * (uint32_t)(wc0 + c - 1) + (uint32_t)(a.L >> 5) * (uint32_t)y;
                const uint4 A = philox(make_uint4(blk, rep, (uint32_t)dsweep, w3), a.seed_lo, a.seed_hi);
                const uint4 B = philox(make_uint4(blk + 1u, rep, (uint32_t)dsweep, w3), a.seed_lo, a.seed_hi);
                const MetroWord mw = metro_update(S, U, D, O, Sh, A, B, mm);
                if constexpr (ONE) {
                    lds[is] = mw.S ^ metro_settle(mw.pend, mw.c8, blk, rep, (uint32_t)dsweep, w3lo, a.seed_lo,
                                                  a.seed_hi, a.t4.low, a.t8.low);
                    continue;
                }
                lds[is] = mw.S;
                const uint64_t m = __ballot(mw.pend != 0u);
                const uint32_t cnt = (uint32_t)__popcll(m);
                if (qn + cnt > (uint32_t)kTieQueue) {
                    if ((uint32_t)(tid & 63) < qn) settle(tq[tid & 63]);
                    qn = 0;
                }
                if (mw.pend) tq[qn + wave_rank(m)] = make_uint4((uint32_t)is, blk, mw.pend, mw.c8);
                qn += cnt;
            }
            if (!ONE && (uint32_t)(tid & 63) < qn) settle(tq[tid & 63]);
            __syncthreads();
        }
    }

    // ---- store the tile in place
    for (int i = tid; i < 2 * a.T; i += nt) {
        uint32_t *dst = lat + (size_t)(2 * y0 + i) * Wl + wc0;
        const uint32_t *src = lds + (i + 2) * Ww + 1;
        if (Wt == 1) {
            dst[0] = src[0];
        } else {
            for (int c = 0; c < Wt; c += 2) {
                const uint2 v = make_uint2(src[c], src[c + 1]);
                __builtin_memcpy(dst + c, &v, 8);
            }
        }
    }

    // ---- energy and magnetisation of this tile's share
    if (!a.part) return;
    int e_acc = 0, m_acc = 0;
    const bool edges = a.coarse == 1;
    for (int t = tid; t < tasks; t += nt) {
        const int c = 1 + (t >> tsh), r = 1 + (t & (a.T - 1));
        const int y = y0 + r - 1;
        // the odd-colour word of row r (x parity q) and its four neighbours
        const int q = (1 + y) & 1;
        const int e = r * 2 * Ww + c, o = e + Ww, is = q ? o : e, io = q ? e : o;
        const uint32_t S = lds[is], U = lds[is - 2 * Ww], D = lds[is + 2 * Ww], O = lds[io];
        const uint32_t Nb = lds[io + (q ? 1 : -1)];
        const uint32_t Sh = __builtin_amdgcn_alignbit(q ? Nb : O, q ? O : Nb, q ? 1u : 31u);
        // bonds inside the tile seen from their odd end: up and down unless
        // the neighbour row is a halo row, the same-column partner always,
        // the shifted partner but for the one bit across the tile's edge
        uint32_t shm = ~0u;
        if (q == 0 && c == 1) shm = ~1u;          // x - 1 of the tile's first site
        if (q == 1 && c == Wt) shm = 0x7FFFFFFFu; // x + 1 of the tile's last site
        int anti = __builtin_popcount(S ^ O) + __builtin_popcount((S ^ Sh) & shm);
        int nb = 32 + __builtin_popcount(shm);
        if (r > 1) anti += __builtin_popcount(S ^ U), nb += 32;
        if (r < a.T) anti += __builtin_popcount(S ^ D), nb += 32;
        e_acc += 2 * anti - nb;
        m_acc += 64 - 2 * (int)(__builtin_popcount(S) + __builtin_popcount(O));
    }
    if (edges) {
        // every bond across the tile's edges: top and bottom rows against the
        // halo rows (both parity arrays), first and last column against the
        // halo columns
        for (int t = tid; t < 2 * 2 * Wt; t += nt) {
            const int side = t >> (wsh + 1), par = (t >> wsh) & 1, c = 1 + (t & (Wt - 1));
            const int r = side == 0 ? 1 : a.T, rh = side == 0 ? 0 : a.T + 1;
            e_acc += 2 * __builtin_popcount(lds[widx(r, par, c)] ^ lds[widx(rh, par, c)]) - 32;
        }
        for (int r = 1 + tid; r <= a.T; r += nt) {
            // x0 (even, bit 0 of the first even word) and x0 - 1 (bit 31 of the
            // left halo's odd word); x0 + T - 1 (odd, bit 31 of the last odd
            // word) and x0 + T (bit 0 of the right halo's even word)
            const uint32_t l0 = lds[widx(r, 0, 1)] & 1u, l1 = lds[widx(r, 1, 0)] >> 31;
            const uint32_t r1 = lds[widx(r, 1, Wt)] >> 31, r0 = lds[widx(r, 0, Wt + 1)] & 1u;
            e_acc += 2 * (int)((l0 ^ l1) + (r1 ^ r0)) - 2;
        }
    }
    e_acc = wave_sum_last(e_acc);
    m_acc = wave_sum_last(m_acc);
    if ((tid & 63) == 63) {
        red[0][wave] = e_acc;
        red[1][wave] = m_acc;
    }
    __syncthreads();
    if (tid == 0) {
        // one slot per tile (a plain store: thousands of workgroups adding
        // into the same two words would queue behind each other)
        long long te = 0, tm = 0;
        for (int i = 0; i < nwaves; ++i) te += red[0][i], tm += red[1][i];
        const int nt2 = a.L / a.T;
        int64_t *slot = a.part + 2 * ((int64_t)l * nt2 * nt2 + (int64_t)ty * nt2 + tx);
        slot[0] = te;
        slot[1] = tm;
    }
}

// The tile with its halo, then each wave's tie queue.
static size_t dcb_lds_bytes(int T, int threads)
{
    return (((size_t)(T + 2) * 2 * (size_t)(T / 64 + 2) * 4 + 15) & ~(size_t)15) + (size_t)(threads / 64) * kTieQueue * 16;
}

hipError_t launch_dcb_phase(uint32_t *packed, int L, int T, int count, int coarse, int hits, uint32_t replica0,
                            uint64_t sweep, uint32_t seed_lo, uint32_t seed_hi, const SweepTables &tab, int64_t *part,
                            const EmSlots &prev, hipStream_t s)
{
    DcbArgs a;
    a.lat = packed;
    a.L = L;
    a.T = T;
    a.coarse = coarse;
    a.hits = hits;
    a.replica0 = replica0;
    a.sweep = sweep;
    a.seed_lo = seed_lo;
    a.seed_hi = seed_hi;
    a.t4 = metro_thr(tab.met[1]);
    a.t8 = metro_thr(tab.met[2]);
    a.part = part;
    a.prev = prev;
    if (!prev.red_in) a.prev.red_K = 0;
    const int tiles = (L / T) * (L / T) / 2;
    // one thread per word of a colour (T^2 / 64 of them), at most 256 while that
    // gives three waves per SIMD, up to 1024 with fewer tiles.  4096^2 x 3, ten
    // hits, attempted updates per ns at 256, 512 and 1024 threads: tile 256 3160,
    // 3250 and 2690; tile 512 1500, 1930 and 2030
    int threads = std::min(256, T * T / 64);
    while (threads < std::min(64 * kDcbMaxWaves, T * T / 64) && (int64_t)tiles * count * (threads / 64) < 3072)
        threads *= 2;
    const auto f = threads == T * T / 64 ? k_dcb<true> : k_dcb<false>;
    hipLaunchKernelGGL(f, dim3((unsigned)tiles, (unsigned)count), dim3(threads), dcb_lds_bytes(T, threads), s, a);
    return hipGetLastError();
}

}  // namespace mcs
