// k_tile2d.hip -- fused multi-sweep kernel for the 2D ferromagnet (J = 1),
// checkerboard Metropolis, int8 lattices with Lx a multiple of 64.
//
// Design (gfx950):
//  * One workgroup owns a band of H full-width rows of one lattice and runs K
//    complete sweeps on it per launch.  Counter-based randomness lets it redo
//    the updates of a halo of 2K rows above and below itself exactly as their
//    owners do (each half-sweep shrinks the valid region by one row), so no
//    workgroup ever waits for another; bands read one buffer and write the
//    other.
//  * In LDS the band is bit-packed and split by x parity: word w of the even
//    (odd) array of a row holds sites x = 64 w + 2 b (+1), b = 0..31, bit set
//    <=> s = -1.  In a half-sweep one parity array per row is active and all 32
//    sites of a word share one colour, so the four neighbours of 32 sites are
//    four words (up, down, other parity, other parity shifted by one site) and
//    the Metropolis classes (dE = 8, 4, <= 0) are a few 3-input bit operations
//    (v_bitop3_b32).
//  * Between the launches of one call the lattice stays in exactly that packed
//    form in global scratch (one bit per spin, rows of 2 Lx/64 words), so only
//    the first launch reads int8 and only the last writes int8: the traffic of
//    the intermediate launches is an eighth of the int8 lattice's.
//  * The random top bytes of those 32 sites are eight bit-planes taken straight
//    from two Philox blocks; r32 < T becomes a bit-serial comparison of the
//    planes with the threshold's top byte.  Words with ties (a site whose top
//    byte equals its class's threshold's, probability 1/256 per site) go to a
//    queue of their wave in LDS, one item per word, and are settled up to 64 at
//    a time with one low-24-bit draw per tied site, so a tie in one lane does
//    not stall the other 63 and no wave waits for another's (metro2d.hpp).
//  * Energy and magnetisation of each sweep come from the odd half-sweep:
//    every bond has exactly one odd end, and when the odd sites of a row are
//    updated its even sites are already final, so the band's own rows give E
//    from the odd sites' four bonds and M from both parity words, with no
//    extra pass.  Each band stores its (E, M) share of every sweep in a slot
//    of its own; the first workgroups of the next launch add them up
//    (em_slots.hpp).
//  * Several lattices (each with its own inverse temperature) can share one
//    launch, which gives taller bands and so less redone halo.
//
// What bounds it: VALU issue, about 170 instructions of a wave per 64 words of
// 32 sites (74 of them Philox) and 55 per settled batch of ties, then the
// barriers' and the launch's latency.  Three 4096^2 lattices, (E, M) every
// sweep, us per sweep: bands of 16 rows, 2 sweeps per launch, 512 threads 14.6,
// 15.1 with one word in flight per thread while the band loads and a serial sum
// over the waves each sweep, 17.8 with a comparison per class, both sideways
// words read, and ties settled by the whole workgroup between two barriers
// besides; bands of 49 rows, 4 per launch, 1024 threads 13.4.
#include "em_slots.hpp"
#include "internal.hpp"
#include "metro2d.hpp"
#include "spin_bytes.hpp"

namespace mcs {

struct Tile2DArgs {
    const void *src;                // int8 lattices, or packed rows if in_packed
    void *dst;                      // int8 lattices, or packed rows if out_packed
    int in_packed, out_packed;
    int Lx, Ly, H;
    int64_t N;
    uint32_t seed_lo, seed_hi, replica0;
    uint64_t sweep0;
    int per_lattice;                // thresholds indexed by lattice (else entry 0)
    Thr t4[kMaxTableLattices];      // dE = 4
    Thr t8[kMaxTableLattices];      // dE = 8
    EmSlots em;                     // band sums of this launch and the previous one
};

template <int K, bool MEASURE>
__global__ __launch_bounds__(1024) void k_tile2d(Tile2DArgs a)
{
    extern __shared__ uint32_t lds[];
    __shared__ int sums[2][K > 0 ? K : 1];  // anti-aligned bonds and down spins of each sweep
    __shared__ long long red64[2][16];
    const int l = blockIdx.y;
    const int y0 = blockIdx.x * a.H;
    const int Hh = min(a.H, a.Ly - y0);
    constexpr int R = 2 * K;
    const int rows = Hh + 2 * R;
    const int Wd = a.Lx >> 6;
    const int nt = blockDim.x;
    const int tid = threadIdx.x;
    const uint32_t rep = a.replica0 + (uint32_t)l;
    const Thr t4 = a.t4[a.per_lattice ? l : 0];
    const Thr t8 = a.t8[a.per_lattice ? l : 0];
    const MetroMasks mm = metro_masks(t4.top, t8.top, true);
    // thread -> (word column, first row, row stride); no division in the loops
    int P, Q, w0, r0;
    if (Wd <= nt) {
        P = Wd;
        Q = nt / Wd;
        w0 = tid % Wd;
        r0 = tid / Wd;
        if (r0 >= Q) r0 = 1 << 28;  // surplus threads idle
    } else {
        P = nt;
        Q = 1;
        w0 = tid;
        r0 = 0;
    }
    auto widx = [&](int r, int par, int w) { return (r * 2 + par) * Wd + w; };
    auto lat_row = [&](int r) {
        int y = y0 - R + r;
        while (y < 0) y += a.Ly;
        while (y >= a.Ly) y -= a.Ly;
        return y;
    };
    const int wave = tid >> 6;
    if (MEASURE && tid < 2 * K) sums[tid & 1][tid >> 1] = 0;
    uint4 *const tq = (uint4 *)(lds + ((rows * 2 * Wd + 3) & ~3)) + wave * kTieQueue;
    const int ntile = gridDim.x, nlat = gridDim.y;
    long long pre_e, pre_m;
    em_prefetch(a.em, blockIdx.x, ntile, l, nlat, tid, pre_e, pre_m);

    // ---- load rows y0-R .. y0+Hh+R-1
    if (a.in_packed) {
        // packed row y of lattice l: 2 Wd words at (l Ly + y) 2 Wd, even array first
        const uint2 *src = (const uint2 *)a.src + (int64_t)l * a.Ly * Wd;
        constexpr int kBatch = 8;  // words of a thread in flight at once
        for (int w = w0; w < Wd; w += P)
            for (int rb = r0; rb < rows; rb += kBatch * Q) {
                uint2 v[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (rb + j * Q < rows) v[j] = src[(int64_t)lat_row(rb + j * Q) * Wd + w];
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (rb + j * Q < rows) ((uint2 *)lds)[(rb + j * Q) * Wd + w] = v[j];
            }
    } else {
        // int8: sign bit of each byte, even-x sites to array 0, odd-x to array 1
        const int8_t *src = (const int8_t *)a.src + (int64_t)l * a.N;
        for (int r = r0; r < rows; r += Q) {
            const int8_t *row = src + (int64_t)lat_row(r) * a.Lx;
            for (int w = w0; w < Wd; w += P) {
                const Row32 h0 = load_row32(row, 64u * w), h1 = load_row32(row, 64u * w + 32u);
                lds[widx(r, 0, w)] = sign_bits16(pick16(h0, 0x06040200u)) | sign_bits16(pick16(h1, 0x06040200u)) << 16;
                lds[widx(r, 1, w)] = sign_bits16(pick16(h0, 0x07050301u)) | sign_bits16(pick16(h1, 0x07050301u)) << 16;
            }
        }
    }
    __syncthreads();
    em_reduce(a.em, blockIdx.x, ntile, l, nlat, tid, nt, pre_e, pre_m, red64);

    const int Qm = Q % a.Ly, iters_w = (Wd + P - 1) / P;
    int yn = lat_row(r0 < rows ? r0 : 0);  // lattice row of LDS row r0, then of the half-sweep's first row
    const bool own = r0 < rows;
    for (int s = 0; s < K; ++s) {
        const uint64_t sweep = a.sweep0 + (uint64_t)s;
        int n_acc = 0, d_acc = 0;  // anti-aligned bonds and down spins of this thread's own words
        for (int c = 0; c < 2; ++c) {
            const int p = 2 * s + c;
            const int r_lo = p + 1, r_hi = rows - p - 1;
            const uint32_t w3 = ctr_w3(kTagSweep, (uint32_t)c, sweep);
            const uint32_t w3lo = ctr_w3(kTagSweepLo, (uint32_t)c, sweep);
            uint32_t qn = 0;
            auto settle = [&]() {
                const uint32_t i = tid & 63;
                if (i < qn) {
                    const uint4 it = tq[i];
                    const uint32_t f = metro_settle(it.z, it.w, it.y, rep, (uint32_t)sweep, w3lo, a.seed_lo, a.seed_hi,
                                                    t4.low, t8.low);
                    if (f) {
                        const uint32_t ws = it.x & 0x7FFFFFFFu, old = lds[ws];
                        lds[ws] = old ^ f;
                        if (MEASURE && (it.x >> 31)) {
                            // a flip of class dE = 8 (4) gains four (two) anti-aligned bonds
                            n_acc += 2 * (int)(__builtin_popcount(f) + __builtin_popcount(f & it.w));
                            d_acc += (int)__builtin_popcount(f) - 2 * (int)__builtin_popcount(old & f);
                        }
                    }
                }
                qn = 0;
            };
            if (++yn >= a.Ly) yn -= a.Ly;
            int y = yn;
            for (int rr = r_lo; rr < r_hi; rr += Q) {
                const int r = rr + r0;
                const bool active = own && r < r_hi;
                const int q = (c + y) & 1;
                const bool interior = MEASURE && c == 1 && r >= R && r < R + Hh;
                const uint32_t rowblk = (uint32_t)(a.Lx >> 5) * (uint32_t)y;
                const int row = r * 2 * Wd;
                for (int j = 0; j < iters_w; ++j) {
                    const int w = w0 + j * P;
                    MetroWord mw;
                    mw.pend = 0u;
                    uint32_t blk = 0u, ws = 0u;
                    if (active) {
                        const int e = row + w, o = e + Wd;  // even- and odd-x words
                        const int is = q ? o : e, io = q ? e : o;
                        // even sites: left neighbours are the odd sites one to the
                        // left (carry from the previous odd word); odd sites: right
                        // neighbours are the even sites one to the right
                        const int side = q ? (w + 1 == Wd ? 1 - Wd : 1) : (w == 0 ? Wd - 1 : -1);
                        const uint32_t S = lds[is], U = lds[is - 2 * Wd], D = lds[is + 2 * Wd], O = lds[io];
                        const uint32_t Nb = lds[io + side];
                        const uint32_t Sh = __builtin_amdgcn_alignbit(q ? Nb : O, q ? O : Nb, q ? 1u : 31u);
                        // random planes of the 32 sites j0 .. j0+31, j0 = 32 w + (Lx/2) y
                        blk = 2u * (uint32_t)w + rowblk;
                        const uint4 A = philox(make_uint4(blk, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                        const uint4 B = philox(make_uint4(blk + 1u, rep, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                        mw = metro_update(S, U, D, O, Sh, A, B, mm);
                        lds[is] = mw.S;
                        ws = (uint32_t)is;
                        if (interior) {
                            n_acc += (int)(__builtin_popcount(mw.S ^ U) + __builtin_popcount(mw.S ^ D) +
                                           __builtin_popcount(mw.S ^ O) + __builtin_popcount(mw.S ^ Sh));
                            d_acc += (int)(__builtin_popcount(mw.S) + __builtin_popcount(O));
                        }
                    }
                    const uint64_t m = __ballot(mw.pend != 0u);
                    if (m) {
                        const uint32_t cnt = (uint32_t)__popcll(m);
                        if (qn + cnt > (uint32_t)kTieQueue) settle();
                        if (mw.pend)
                            tq[qn + wave_rank(m)] =
                                make_uint4(ws | ((uint32_t)interior << 31), blk, mw.pend, mw.c8);
                        qn += cnt;
                    }
                }
                y += Qm;
                if (y >= a.Ly) y -= a.Ly;
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
        // every bond once: 2 (anti-aligned) - 4 per odd site; M from both parities
        const long long words = (long long)Hh * Wd;
        *em_slot(a.em.slots, tid, l, nlat, blockIdx.x, ntile) =
            make_longlong2(2ll * sums[0][tid] - 128 * words, 64 * words - 2ll * sums[1][tid]);
    }

    // ---- store the band's own rows
    if (a.out_packed) {
        uint2 *dst = (uint2 *)a.dst + (int64_t)l * a.Ly * Wd;
        for (int r = R + r0; r < R + Hh; r += Q) {
            uint2 *row = dst + (int64_t)(y0 + r - R) * Wd;
            for (int w = w0; w < Wd; w += P) row[w] = ((const uint2 *)lds)[r * Wd + w];
        }
        return;
    }
    int8_t *dst = (int8_t *)a.dst + (int64_t)l * a.N;
    for (int r = R + r0; r < R + Hh; r += Q) {
        int8_t *row = dst + (int64_t)(y0 + r - R) * a.Lx;
        for (int w = w0; w < Wd; w += P) {
            const uint32_t ev = lds[widx(r, 0, w)], od = lds[widx(r, 1, w)];
            uint4 *p = (uint4 *)(row + 64 * w);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t dw[4];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    // four even and four odd columns, bit 0 -> byte 0x01 (+1), 1 -> 0xFF (-1)
                    const int sh = 8 * q + 4 * i;
                    const uint32_t ee = 0x01010101u ^ (spread4((ev >> sh) & 15u) * 0xFEu);
                    const uint32_t oo = 0x01010101u ^ (spread4((od >> sh) & 15u) * 0xFEu);
                    dw[2 * i] = __builtin_amdgcn_perm(oo, ee, 0x05010400u);
                    dw[2 * i + 1] = __builtin_amdgcn_perm(oo, ee, 0x07030602u);
                }
                p[q] = make_uint4(dw[0], dw[1], dw[2], dw[3]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
bool tile2d_supported(const SweepCall &c, int layout)
{
    return layout == MC_INT8 && c.g.dims == 2 && c.J == nullptr && c.rule == 0 && (c.g.Lx % 64) == 0 &&
           c.g.Lx <= 16384 && c.g.Ly >= 4 && (!c.per_lattice || c.g.count <= kMaxTableLattices);
}

size_t tile2d_lds_bytes(int Lx, int H, int K) { return (size_t)(H + 4 * K) * 2 * (size_t)(Lx / 64) * 4; }

// the band's words, then each wave's tie queue
static size_t tile2d_dynamic_lds(int Lx, int H, int K, int threads)
{
    return ((tile2d_lds_bytes(Lx, H, K) + 15) & ~(size_t)15) + (K ? (size_t)(threads / 64) * kTieQueue * 16 : 0);
}

template <int K>
static hipError_t launch_k(const Tile2DArgs &a, int count, int threads, hipStream_t s)
{
    const int tiles = (a.Ly + a.H - 1) / a.H;
    const size_t lds = tile2d_dynamic_lds(a.Lx, a.H, K, threads);
    dim3 grid((unsigned)tiles, (unsigned)count);
    // allow the largest dynamic LDS a plan may ask for (a band of 64 KB and
    // sixteen queues of 1 KB), once per device and kernel instance
    static LdsLimit lim[2];
    const bool measure = a.em.slots != nullptr;
    const void *f = measure ? (const void *)k_tile2d<K, true> : (const void *)k_tile2d<K, false>;
    const hipError_t e = lim[measure ? 1 : 0].ensure(f, 65536 + 16 * kTieQueue * 16);
    if (e != hipSuccess) return e;
    if (measure) hipLaunchKernelGGL((k_tile2d<K, true>), grid, dim3(threads), lds, s, a);
    else hipLaunchKernelGGL((k_tile2d<K, false>), grid, dim3(threads), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_tile2d(const SweepCall &c, const void *src, int in_packed, void *dst, int out_packed,
                         uint64_t sweep0, int k, int H, int threads, const EmSlots &em, hipStream_t s)
{
    Tile2DArgs a;
    a.src = src;
    a.dst = dst;
    a.in_packed = in_packed;
    a.out_packed = out_packed;
    a.Lx = c.g.Lx;
    a.Ly = c.g.Ly;
    a.H = H;
    a.N = c.g.N;
    a.seed_lo = c.seed_lo;
    a.seed_hi = c.seed_hi;
    a.replica0 = c.replica0;
    a.sweep0 = sweep0;
    a.per_lattice = c.per_lattice;
    for (int i = 0; i < kMaxTableLattices; ++i) {
        const SweepTables &t = (c.per_lattice && i < c.g.count) ? c.tabs[i] : c.tab;
        a.t4[i] = metro_thr(t.met[1]);
        a.t8[i] = metro_thr(t.met[2]);
    }
    a.em = em;
    if (k == 0) a.em.slots = nullptr;
    if (!em.red_in) a.em.red_K = 0;
    switch (k) {
    case 0: return launch_k<0>(a, c.g.count, threads, s);
    case 1: return launch_k<1>(a, c.g.count, threads, s);
    case 2: return launch_k<2>(a, c.g.count, threads, s);
    case 3: return launch_k<3>(a, c.g.count, threads, s);
    case 4: return launch_k<4>(a, c.g.count, threads, s);
    case 5: return launch_k<5>(a, c.g.count, threads, s);
    case 6: return launch_k<6>(a, c.g.count, threads, s);
    case 7: return launch_k<7>(a, c.g.count, threads, s);
    case 8: return launch_k<8>(a, c.g.count, threads, s);
    default: return hipErrorInvalidValue;
    }
}

// Adds up the workgroup sums of the last launch of a call: workgroup (j, l)
// writes EM of sweep j of that launch for lattice l.
__global__ __launch_bounds__(256) void k_em_slots(const int64_t *slots, int tiles, int64_t *EM, int64_t em_stride,
                                                  int64_t sweep0)
{
    __shared__ long long part[2][4];
    const int j = blockIdx.x, l = blockIdx.y, count = gridDim.y, tid = threadIdx.x;
    const longlong2 *src = em_slot((int64_t *)slots, j, l, count, 0, tiles);
    long long se = 0, sm = 0;
    for (int t = tid; t < tiles; t += 256) {
        const longlong2 v = src[t];
        se += v.x;
        sm += v.y;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        se += __shfl_xor(se, off, 64);
        sm += __shfl_xor(sm, off, 64);
    }
    if ((tid & 63) == 0) {
        part[0][tid >> 6] = se;
        part[1][tid >> 6] = sm;
    }
    __syncthreads();
    if (tid == 0) {
        int64_t *em = EM + (sweep0 + j) * em_stride + 2 * l;
        em[0] = part[0][0] + part[0][1] + part[0][2] + part[0][3];
        em[1] = part[1][0] + part[1][1] + part[1][2] + part[1][3];
    }
}

hipError_t launch_em_slots(const int64_t *slots, int tiles, int count, int K, int64_t *EM, int64_t em_stride,
                           int64_t sweep0, hipStream_t s)
{
    if (K <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_em_slots, dim3((unsigned)K, (unsigned)count), dim3(256), 0, s, slots, tiles, EM, em_stride,
                       sweep0);
    return hipGetLastError();
}

// Per-band (E, M) slots of one launch: K <= 8 sweeps x count lattices x
// ceil(Ly / 4) bands (a plan's band height is at least 4) x 16 bytes.
size_t tile2d_slot_bytes(const Geom &g)
{
    const size_t b = (size_t)8 * (size_t)g.count * (size_t)((g.Ly + 3) / 4) * 16;
    return (b + 255) / 256 * 256;
}

}  // namespace mcs
