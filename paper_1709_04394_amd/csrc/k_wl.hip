// k_wl.hip -- Wang-Landau sampling of 2D L x L ferromagnets in energy windows
// (Sec. "Wang-Landau update": g(E) multiplied by f at every visit, moves
// accepted with min[1, g(E)/g(E')]; windows sampled by separate walkers, a
// move out of the window rejected and the current level counted again, the
// walkers' estimates averaged before f is reduced).
//
// Walkers visit the sites in the multicanonical walkers' sequential order with
// their random numbers.  Every walker keeps its own estimate G[k] of ln g
// (integers in units of 2^-32, so ln f = 2^-s adds exactly) and its own visit
// counts over the window's levels, both in LDS for the whole call.  The
// acceptance probability exp(-(G[k'] - G[k]) 2^-32) is a fixed-order product of
// five tabulated factors (exp(-n) and one per byte of the fraction), so its
// definition has no transcendental; the integer test r32 < ceil(p 2^32)
// follows.  At the end of a call each walker shifts its estimate to a minimum
// of 0 over the levels with states and reports whether its histogram is flat.
#include <algorithm>

#include "internal.hpp"
#include "muca.hpp"
#include "muca_rows.hpp"
#include "quad_walk.hpp"
#include "wl.hpp"

namespace mcs {

// ceil(exp(-x 2^-32) 2^32), at least 1, for x > 0
__device__ __forceinline__ uint64_t wl_threshold(uint64_t x, const double *xt)
{
    const uint64_t n = x >> 32;
    if (n >= (uint64_t)kWlExpN) return 1;
    const uint32_t f = (uint32_t)x;
    double p = xt[n];
    p = p * xt[kWlExpN + (f >> 24)];
    p = p * xt[kWlExpN + 256 + ((f >> 16) & 255u)];
    p = p * xt[kWlExpN + 512 + ((f >> 8) & 255u)];
    p = p * xt[kWlExpN + 768 + (f & 255u)];
    const uint64_t T = (uint64_t)__builtin_ceil(p * 4294967296.0);
    return T < 1 ? 1 : T;
}

// r32 < ceil(p 2^32) for the integer r32 is r32 < p 2^32, i.e. the difference of
// the estimates is below D(r32) = -ln(r32 2^-32) 2^32, which depends on the
// random number alone and is prepared off the walker's chain in FP32.  Where
// the difference comes within kWlMargin of D, which covers both conversions'
// and the logarithm's rounding twice over (differences that can be near a D are
// below 23 2^32: 2^13.6 from the conversion, 2^14 from the logarithm), the exact
// test decides; that is about one update in 2^15.
constexpr float kWlMargin = 65536.0f;

__device__ __forceinline__ float wl_bound(uint32_t r)
{
    // (32 - log2 r) ln 2 2^32; r = 0 gives infinity: accepted (the threshold is at least 1)
    return (32.0f - __builtin_amdgcn_logf((float)r)) * 2977044471.8f;
}

// Four lanes per walker (quad_walk.hpp), sixteen walkers of one window per
// workgroup of one wave.  The walker's estimates and counts of the window's
// levels sit in LDS as [level][walker], so that two walkers never meet in a
// bank.  The candidate's estimate is read one update ahead for both outcomes
// of the update before (a level's latest increment belongs to the level the
// walker is on, never to the candidate); the walker's own estimate is carried
// in registers and stored after each update; the counts of four updates are
// added by the four lanes at once.
//
// Measured, 64 windows of 256 walkers, L = 64: 352 ns per update with one lane
// per walker (two dependent LDS reads, five more and four FP64 multiplications
// for the acceptance, behind a divergent branch), 103 ns so.
constexpr int kWlGuard = 4;  // levels past either end that a read ahead may touch
constexpr int kWlSG = 16 * 8;  // bytes per level of the estimates; the counts take half

// What the chain carries from update to update.
struct WlChain {
    int z, zn;            // LDS address of the level's estimate; of the level the next update leads to
    uint64_t gk, G0, G1;  // estimate of the level; of the next candidate if this update is rejected / accepted
    bool acc;             // outcome of the last update
    uint32_t F;           // outcomes, newest in bit 0
    int zc;               // level after update q of the last four
    int patch;            // correction of the last site's step in a one-word row
};

// What a lane prepared for the sixteen updates of a group.
struct WlGroup {
    int s0[4], s1[4];  // step in bytes if the previous update was rejected / accepted
    float bd[4];
    uint32_t r[4];
};

struct WlWindow {
    int z0;          // LDS address of the walker's estimate of the window's first level
    uint32_t span;   // bytes of the window's levels
    uint64_t inc;
    const double *xtab;
};

// Updates 4 Q .. 4 Q + 3 of a group.  The decision is one compare: the bound is
// replaced by -inf for a step out of the window (rejected, counted again) and
// by +inf for a step to the same level (accepted) before the estimates arrive.
// Returns whether any update came within the margin of its bound, so that the
// four have to be done again with EXACT.
template <int CB, int NW, int Q, bool EXACT>
__device__ __forceinline__ bool wl_step4(WlChain &c, const WlGroup &g, const WlWindow &wn, int q, uint32_t zlast,
                                         PhiloxRounds &ahead, uint32_t k0, uint32_t k1)
{
    uint64_t near_any = 0;
#pragma unroll
    for (int I = 0; I < 4; ++I) {
        const int b = 4 * Q + I, Qn = (b + 1) >> 2, In = (b + 1) & 3;
        // the next update's candidates for both outcomes of this one
        int p0 = 0, p1 = 0;
        uint64_t N0 = 0, N1 = 0;
        if (b < 15) {
            const int x = NW == 1 && CB <= 16 && b + 2 == CB ? c.patch : 0;
            p0 = c.z + (int)quad_get((uint32_t)(g.s0[In] + x), Qn);
            p1 = c.zn + (int)quad_get((uint32_t)(g.s1[In] + x), Qn);
            N0 = lds_read64(p0);
            N1 = lds_read64(p1);
        }
        // the reads go out before the decision waits for the last ones
        __builtin_amdgcn_sched_barrier(0);
        if (!EXACT && b < 10) {
            ahead.round(b, k0, k1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool still = c.zn == c.z, inw = (uint32_t)(c.zn - wn.z0) < wn.span;
        const uint64_t gc = c.acc ? c.G1 : c.G0;
        const int64_t df = (int64_t)(gc - c.gk);
        bool ok;
        if (EXACT) {
            ok = still || (inw && (df <= 0 || (uint64_t)quad_get(g.r[I], Q) < wl_threshold((uint64_t)df, wn.xtab)));
        } else {
            float bd = quad_getf(g.bd[I], Q);
            bd = inw ? bd : -__builtin_inff();
            bd = still ? __builtin_inff() : bd;
            const float e =
                __builtin_fmaf((float)(int32_t)(df >> 32), 4294967296.0f, (float)(uint32_t)df) - bd;
            ok = e < 0.0f;
            near_any |= __ballot(__builtin_fabsf(e) < kWlMargin);
        }
        // a candidate equal to the level was read before the last increment
        const uint64_t inc = still ? 2 * wn.inc : wn.inc;
        c.gk = (ok ? gc : c.gk) + inc;
        c.z = ok ? c.zn : c.z;
        c.zn = ok ? p1 : p0;
        lds_write64(c.z, c.gk);
        c.F = shift_in(c.F, __ballot(ok));
        c.zc = q == I ? c.z : c.zc;
        if (NW == 1 && CB <= 16 && b == 0) {
            // one-word row: the right neighbour of the last site is site 0,
            // flipped if its update was accepted
            c.patch = (q == (CB - 1) / 4 && ok) ? (((zlast >> (CB - 1)) & 1u) ? kWlSG : -kWlSG) : 0;
        }
        c.acc = ok;
        c.G0 = N0;
        c.G1 = N1;
    }
    return near_any != 0;
}

// The four updates, done again from their start where the margin asks for it
// (their increments taken back first, one by each lane), then their counts.
template <int CB, int NW, int Q>
__device__ __forceinline__ void wl_block(WlChain &c, const WlGroup &g, const WlWindow &wn, int q, int hoff,
                                         uint32_t zlast, PhiloxRounds &ahead, uint32_t k0, uint32_t k1)
{
    const WlChain start = c;
    if (__builtin_expect(wl_step4<CB, NW, Q, false>(c, g, wn, q, zlast, ahead, k0, k1), 0)) {
        lds_add64(c.zc, 0 - wn.inc);
        c = start;
        wl_step4<CB, NW, Q, true>(c, g, wn, q, zlast, ahead, k0, k1);
    }
    lds_add(hoff + ((c.zc - wn.z0) >> 1), 1u);
}

template <int L>
__global__ __launch_bounds__(64) void k_wl(WlArgs a)
{
    using R = QuadRow<L>;
    constexpr int N = L * L, NW = R::NW, CB = R::CB;
    constexpr int SG = kWlSG;
    extern __shared__ __align__(16) unsigned char wl_lds[];
    const int lane = threadIdx.x, q = lane & 3, wi16 = lane >> 2;
    const int w0 = blockIdx.x * 16, win = w0 / a.M;
    if (!a.active[win]) return;
    const int lo = a.lo[win], hi = a.hi[win], n = hi - lo + 1;
    const int w = w0 + wi16;
    int64_t *Gl = (int64_t *)wl_lds;                                         // [guard + n + guard][16]
    uint32_t *Hl = (uint32_t *)(Gl + (size_t)(n + 2 * kWlGuard) * 16);       // likewise
    int64_t *Gg = a.G + (int64_t)w * a.wmax;
    uint32_t *Hg = a.H + (int64_t)w * a.wmax;
    for (int j = q; j < n + 2 * kWlGuard; j += 4) {
        const int jj = j - kWlGuard;
        const bool in = jj >= 0 && jj < n;
        Gl[j * 16 + wi16] = in ? Gg[jj] : 0;
        Hl[j * 16 + wi16] = in ? Hg[jj] : 0u;
    }
    __syncthreads();
    int8_t *sp = a.spins + (int64_t)w * N;
    const int z0 = lds_addr(Gl) + kWlGuard * SG + 8 * wi16;
    const int hoff = lds_addr(Hl) + 4 * wi16 + kWlGuard * (SG / 2);
    const WlWindow wn{z0, (uint32_t)(n * SG), (uint64_t)a.inc[win], a.xtab};
    WlChain c;
    c.z = z0 + SG * ((int)((a.E[w] + 2 * N) / 4) - lo);
    c.gk = lds_read64(c.z);
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
                QuadPlanes P = quad_planes<CB>(c0, u, d, C[NW - 1] >> (CB - 1), C[NW > 1 ? 1 : 0] & 1u);
                uint32_t F = 0u;
                c.acc = false;  // the previous update is part of the word's state
                for (int g = 0; g < (CB + 15) / 16; ++g) {
                    const int sh = 16 * g + 4 * q;
                    const uint32_t ctr0 = (uint32_t)(L * y + CB * wi + sh) >> 2;
                    if (!R::kAhead)
                        blk = philox(make_uint4(ctr0, (uint32_t)w, (uint32_t)sweep, w3), a.seed_lo, a.seed_hi);
                    PhiloxRounds ahead;
                    ahead.c = make_uint4(ctr0 + 4u, (uint32_t)w, (uint32_t)sweep, w3);
                    const QuadCounts qc = quad_counts(P, sh);
                    WlGroup gr{{}, {}, {}, {blk.x, blk.y, blk.z, blk.w}};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        gr.s0[i] = 2 * SG - SG * (qc.n3[i] + qc.l[i]);
                        gr.s1[i] = SG - SG * (qc.n3[i] - qc.l[i]);
                        gr.bd[i] = wl_bound(gr.r[i]);
                    }
                    const int x0 = c.z + (int)quad_get((uint32_t)gr.s0[0], 0);
                    const int x1 = c.z + (int)quad_get((uint32_t)gr.s1[0], 0);
                    c.zn = c.acc ? x1 : x0;
                    c.G0 = c.G1 = lds_read64(c.zn);
                    // a first candidate equal to the level is read after the last increment
                    if (c.zn == c.z) c.G0 = c.G1 = c.gk - wn.inc;
                    c.F = 0u;
                    c.zc = c.z;
                    c.patch = 0;
                    wl_block<CB, NW, 0>(c, gr, wn, q, hoff, P.z, ahead, a.seed_lo, a.seed_hi);
                    if (CB >= 8)
                        wl_block<CB, NW, 1>(c, gr, wn, q, hoff, P.z, ahead, a.seed_lo, a.seed_hi);
                    if (CB >= 12)
                        wl_block<CB, NW, 2>(c, gr, wn, q, hoff, P.z, ahead, a.seed_lo, a.seed_hi);
                    if (CB >= 16)
                        wl_block<CB, NW, 3>(c, gr, wn, q, hoff, P.z, ahead, a.seed_lo, a.seed_hi);
                    const uint32_t Fg = c.F;
                    if (R::kAhead) blk = ahead.c;
                    F |= (__brev(Fg) >> (CB < 16 ? 32 - CB : 16)) << (16 * g);
                    // one-word row: the last site's right neighbour is site 0
                    if (NW == 1 && CB > 16)
                        P = quad_planes<CB>(c0, u, d, c0 >> (CB - 1), (c0 ^ F) & 1u);
                }
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
            quad_store<L>(sp, y, q, true, C);
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
        }
    }
    if (q == 0) a.E[w] = 4 * (int64_t)((c.z - z0) / SG + lo) - 2 * N;
    __syncthreads();
    // the estimate's minimum over the levels with states (all but level 1)
    // to 0; flatness: min H >= flat * mean H over those levels
    int64_t mn = INT64_MAX;
    uint32_t hmin = 0xFFFFFFFFu;
    uint64_t hsum = 0;
    const int64_t *Gw = Gl + kWlGuard * 16 + wi16;
    const uint32_t *Hw = Hl + kWlGuard * 16 + wi16;
    for (int j = q; j < n; j += 4) {
        if (lo + j == 1) continue;
        mn = min(mn, Gw[j * 16]);
        const uint32_t h = Hw[j * 16];
        hmin = min(hmin, h);
        hsum += h;
    }
#pragma unroll
    for (int m = 1; m < 4; m <<= 1) {
        mn = min(mn, __shfl_xor(mn, m, 64));
        hmin = min(hmin, (uint32_t)__shfl_xor((int)hmin, m, 64));
        hsum += __shfl_xor(hsum, m, 64);
    }
    const int cnt = n - (lo <= 1 && hi >= 1 ? 1 : 0);
    for (int j = q; j < n; j += 4) {
        Gg[j] = Gw[j * 16] - mn;
        Hg[j] = Hw[j * 16];
    }
    if (q == 0) a.flat[w] = (double)hmin * (double)cnt >= a.flat_ratio * (double)hsum ? 1 : 0;
}

// Walkers into their windows: from the ground state, typewriter passes taking
// a flip iff the walker is below its window, the flip raises its level and
// the top bit of word (i mod 4) of Philox(WINDOW, i div 4, w, pass) is set,
// until the level reaches lo.  One thread per walker.
__global__ void k_win_drive(int8_t *spins, int64_t *E, int32_t *ok, const int32_t *lo, int L, int W, int M,
                            int max_pass, uint32_t k0, uint32_t k1)
{
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= W) return;
    const int N = L * L;
    int8_t *s = spins + (int64_t)w * N;
    const int klo = lo[w / M];
    int k = 0;
    for (int i = 0; i < N; ++i) s[i] = 1;
    for (int pass = 0; pass < max_pass && k < klo; ++pass)
        for (int y = 0; y < L && k < klo; ++y)
            for (int x = 0; x < L && k < klo; ++x) {
                const int i = x + L * y;
                const int h = s[(x + 1) % L + L * y] + s[(x + L - 1) % L + L * y] + s[x + L * ((y + 1) % L)] +
                              s[x + L * ((y + L - 1) % L)];
                const int dl = s[i] * h / 2;
                if (dl <= 0) continue;
                const uint4 b = philox(make_uint4((uint32_t)i >> 2, (uint32_t)w, (uint32_t)pass,
                                                  ctr_w3(kTagWindow, 0, (uint64_t)pass)), k0, k1);
                const uint32_t r = (i & 3) == 0 ? b.x : (i & 3) == 1 ? b.y : (i & 3) == 2 ? b.z : b.w;
                if (r >> 31) {
                    s[i] = (int8_t)-s[i];
                    k += dl;
                }
            }
    E[w] = 4 * (int64_t)k - 2 * N;
    ok[w] = k >= klo ? 1 : 0;
}

// Average of a window's walker estimates: floor of the integer mean per level,
// shifted to a minimum of 0 over the levels with states, given to every walker
// of the window, whose visit counts are cleared.  One workgroup per window
// with mask[window] set.
__global__ __launch_bounds__(256) void k_wl_average(int64_t *G, uint32_t *H, const int32_t *lo, const int32_t *hi,
                                                    const uint8_t *mask, int M, int wmax)
{
    const int win = blockIdx.x;
    if (!mask[win]) return;
    __shared__ int64_t avg[kWlMaxWidth];
    __shared__ int64_t shift;
    const int klo = lo[win], n = hi[win] - klo + 1;
    const int64_t w0 = (int64_t)win * M;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        int64_t sum = 0;
        for (int m = 0; m < M; ++m) sum += G[(w0 + m) * wmax + j];
        int64_t q = sum / M;
        if (sum % M != 0 && sum < 0) --q;  // floor
        avg[j] = q;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t mn = INT64_MAX;
        for (int j = 0; j < n; ++j)
            if (klo + j != 1) mn = min(mn, avg[j]);
        shift = mn;
    }
    __syncthreads();
    for (int64_t idx = threadIdx.x; idx < (int64_t)M * n; idx += blockDim.x) {
        const int64_t m = idx / n;
        const int j = (int)(idx - m * n);
        G[(w0 + m) * wmax + j] = avg[j] - shift;
        H[(w0 + m) * wmax + j] = 0u;
    }
}

template <int L>
static hipError_t launch_wl_L(const WlArgs &a, int W, hipStream_t s)
{
    const size_t lds = (size_t)(a.wmax + 2 * kWlGuard) * 16 * 12;
    static LdsLimit lim;
    const hipError_t e = lim.ensure((const void *)k_wl<L>, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wl<L>, dim3(W / 16), dim3(64), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_wl_sweeps(const WlArgs &a, int L, int W, hipStream_t s)
{
    switch (L) {
    case 4: return launch_wl_L<4>(a, W, s);
    case 8: return launch_wl_L<8>(a, W, s);
    case 12: return launch_wl_L<12>(a, W, s);
    case 16: return launch_wl_L<16>(a, W, s);
    case 24: return launch_wl_L<24>(a, W, s);
    case 32: return launch_wl_L<32>(a, W, s);
    case 48: return launch_wl_L<48>(a, W, s);
    case 64: return launch_wl_L<64>(a, W, s);
    case 96: return launch_wl_L<96>(a, W, s);
    case 128: return launch_wl_L<128>(a, W, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_win_drive(int8_t *spins, int64_t *E, int32_t *ok, const int32_t *lo, int L, int W, int M,
                            int max_pass, uint64_t seed, hipStream_t s)
{
    hipLaunchKernelGGL(k_win_drive, dim3((W + 63) / 64), dim3(64), 0, s, spins, E, ok, lo, L, W, M, max_pass,
                       (uint32_t)seed, (uint32_t)(seed >> 32));
    return hipGetLastError();
}

hipError_t launch_wl_average(int64_t *G, uint32_t *H, const int32_t *lo, const int32_t *hi, const uint8_t *mask,
                             int nwin, int M, int wmax, hipStream_t s)
{
    hipLaunchKernelGGL(k_wl_average, dim3(nwin), dim3(256), 0, s, G, H, lo, hi, mask, M, wmax);
    return hipGetLastError();
}

}  // namespace mcs
