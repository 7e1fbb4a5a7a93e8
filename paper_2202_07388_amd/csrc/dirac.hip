// dirac.hip -- the Wilson-clover operator D and D^+ on eo-SoA fields.
//
// One lane per output site; a workgroup of 2*ts lanes owns ts consecutive even-odd
// indices of one time slice in BOTH parities (lanes 0..ts-1 even, ts..2ts-1 odd). The even
// site with index i and the odd site with index i are lexicographic neighbours along x3,
// so a workgroup covers a compact run of the lattice: the eight links a site reads are
// mostly the same links its neighbours in the workgroup read (every link joins an even and
// an odd site), and the neighbour spinors are shared through L1/L2. Workgroups are mapped
// XCD-contiguously and walk time-slice-first within a spatial tile (walk_site).
//
// Per hop the neighbour spinor is spin-projected with (1 -+ gamma_mu) to two spin
// components, multiplied by the link (row 2 rebuilt from rows 0, 1 and det U; the U(1)
// phase is stored inside the rows, so no trigonometry), negated when the hop crosses an
// antiperiodic time boundary, and expanded back to four spins; the factor -1/2 of the
// hopping term is applied once at the end. D^+ = gamma_5 D gamma_5 flips the projector
// signs.
//
// The eight hops form a runtime loop; optionally (PIPE) it is software-pipelined over two
// register buffers: the loads of hop k+1 are in flight while hop k is computed. Loop-carried
// site indices pass through an empty asm statement so the optimiser cannot hoist all eight
// hops' address computations out of the loop (that would pin ~80 registers and halve the
// occupancy).
//
// Several right-hand sides on one operator (a table of up to kMaxRhs fields) run in one
// launch with the right-hand side as the fastest-varying workgroup index: the workgroups
// that read a tile's links and clover blocks for different right-hand sides run together,
// so L2 serves those bytes once for all of them.
#include <chrono>
#include <cstdio>
#include <string>
#include <type_traits>
#include <vector>

#include "blas.h"
#include "dirac_core.h"

using namespace qdw;

namespace qdw {
// (the last argument of a kernel, its first field beside the gate: a launch on one field
// reads a few neighbouring words of it)
struct RhsTable {
    const int* gate;  // optional: right-hand side r is skipped when gate[r * gstride] == 0
    int gstride;
    int nrhs;
    struct {
        const void* in;
        void* out;
    } f[kMaxRhs];
};

inline RhsTable one_field(const void* in, void* out)
{
    RhsTable tab{};
    tab.nrhs = 1;
    tab.f[0] = {in, out};
    return tab;
}
}  // namespace qdw

namespace {

// What a kernel does with an output spinor beside storing it. EPI_NORM also sums |out|^2 (as
// stored). EPI_STEP is the second half of a CG step: w = out stays in registers, r -= alpha w
// is stored instead, and |r|^2 (as stored) is summed; alpha comes from the device scalars.
// Either saves passes over whole fields: a separate norm reads q again, and a separate
// residual update writes and reads w.
enum { EPI_NONE = 0, EPI_NORM, EPI_STEP };
struct Epi {
    Sums sums;
    void* r;
    const double* sc;
};

// A value about to be stored, as a rounded FP32 number: left to itself the compiler folds the
// conversion to binary16 into the last FMA of some components, a different choice per kernel,
// and the two ways differ in the last bit for one value in some thousands.
template <int P, typename R>
__device__ __forceinline__ R settled(R v)
{
    if constexpr (P == F16S) asm("" : "+v"(v));
    return v;
}

template <int P, int EPI>
__device__ __forceinline__ void store_out(void* out, const Epi& e, int Vh, int par, int i,
                                          cx<typename Traits<P>::real> acc[12], double& sum)
{
    using R = typename Traits<P>::real;
    if constexpr (EPI == EPI_STEP) {
        const R a = (R)e.sc[S_ALPHA];
        cx<R> r[12];
        load_spinor<P>(e.r, Vh, par, i, r);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = r[c] - scale(acc[c], a);
        out = e.r;
    }
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = {settled<P>(acc[c].re), settled<P>(acc[c].im)};
    store_spinor<P>(out, Vh, par, i, acc);
    if constexpr (EPI != EPI_NONE) {
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const double re = to_real<P>(to_store<P>(acc[c].re)), im = to_real<P>(to_store<P>(acc[c].im));
            sum = __builtin_fma(re, re, __builtin_fma(im, im, sum));
        }
    }
}

template <int P>
struct HopIn {
    cx<typename Traits<P>::real> s[12];  // neighbour spinor
    cx<typename Traits<P>::real> u[6];   // link rows 0, 1
    cx<typename Traits<P>::real> d;      // det of the link
};

// loads of hop k (0: +t, 1: -t, 2: +x1, ... 7: -x3) into site x = (par, i)
template <int P, int MU, bool FWD>
__device__ __forceinline__ void hop_load(const Geom& g, const void* in, const void* links,
                                         const void* dets, int par, int i, const int x[4],
                                         int lex, HopIn<P>& b)
{
    const int j = (FWD ? lex_fwd(g, x, lex, MU) : lex_bwd(g, x, lex, MU)) >> 1;
    load_spinor<P>(in, g.Vh, 1 - par, j, b.s);
    if (FWD) load_link<P>(links, dets, g.Vh, par, i, MU, b.u, b.d);       // U_mu(x)
    else load_link<P>(links, dets, g.Vh, 1 - par, j, MU, b.u, b.d);      // U_mu(x - mu)
}

// w = U (1 -+ gamma) psi(x + mu) or U^+ (1 +- gamma) psi(x - mu), times the boundary sign (and
// -1/2 with HALF), as a half spinor
template <int P, int MU, bool FWD, bool DAG, bool HALF = false>
__device__ __forceinline__ void hop_half(const Geom& g, const int x[4], const HopIn<P>& b,
                                         cx<typename Traits<P>::real> w[6])
{
    using R = typename Traits<P>::real;
    constexpr int SG = (FWD != DAG) ? -1 : +1;  // projector 1 + SG gamma_mu
    cx<R> h[6];
    project<R, MU, SG>(b.s, h);
    const bool flip = MU == 0 && g.bc_t < 0 && x[0] == (FWD ? g.L[0] - 1 : 0);
    if (HALF) {
        const R f = flip ? (R)0.5 : (R)-0.5;
#pragma unroll
        for (int c = 0; c < 6; ++c) h[c] = scale(h[c], f);
    } else if (flip) {
#pragma unroll
        for (int c = 0; c < 6; ++c) h[c] = -h[c];
    }
    su3_mul<R, !FWD, true>(b.u, b.d, h, w);
}

// acc += U (1 -+ gamma) psi(x + mu)  or  U^+ (1 +- gamma) psi(x - mu), times the boundary
// sign; with HALF the term is scaled by -1/2 (the hopping term's factor) before it is added
template <int P, int MU, bool FWD, bool DAG, bool HALF = false>
__device__ __forceinline__ void hop_compute(const Geom& g, const int x[4], const HopIn<P>& b,
                                            cx<typename Traits<P>::real> acc[12])
{
    using R = typename Traits<P>::real;
    constexpr int SG = (FWD != DAG) ? -1 : +1;  // projector 1 + SG gamma_mu
    cx<R> w[6];
    hop_half<P, MU, FWD, DAG, HALF>(g, x, b, w);
    expand_add<R, MU, SG>(w, acc);
}

template <int P>
__device__ __forceinline__ void load_k(int k, const Geom& g, const void* in, const void* links,
                                       const void* dets, int par, int i, const int x[4], int lex,
                                       HopIn<P>& b)
{
    switch (k) {
    case 0: hop_load<P, 0, true>(g, in, links, dets, par, i, x, lex, b); break;
    case 1: hop_load<P, 0, false>(g, in, links, dets, par, i, x, lex, b); break;
    case 2: hop_load<P, 1, true>(g, in, links, dets, par, i, x, lex, b); break;
    case 3: hop_load<P, 1, false>(g, in, links, dets, par, i, x, lex, b); break;
    case 4: hop_load<P, 2, true>(g, in, links, dets, par, i, x, lex, b); break;
    case 5: hop_load<P, 2, false>(g, in, links, dets, par, i, x, lex, b); break;
    case 6: hop_load<P, 3, true>(g, in, links, dets, par, i, x, lex, b); break;
    default: hop_load<P, 3, false>(g, in, links, dets, par, i, x, lex, b); break;
    }
}

template <int P, bool DAG, bool HALF = false>
__device__ __forceinline__ void compute_k(int k, const Geom& g, const int x[4], const HopIn<P>& b,
                                          cx<typename Traits<P>::real> acc[12])
{
    switch (k) {
    case 0: hop_compute<P, 0, true, DAG, HALF>(g, x, b, acc); break;
    case 1: hop_compute<P, 0, false, DAG, HALF>(g, x, b, acc); break;
    case 2: hop_compute<P, 1, true, DAG, HALF>(g, x, b, acc); break;
    case 3: hop_compute<P, 1, false, DAG, HALF>(g, x, b, acc); break;
    case 4: hop_compute<P, 2, true, DAG, HALF>(g, x, b, acc); break;
    case 5: hop_compute<P, 2, false, DAG, HALF>(g, x, b, acc); break;
    case 6: hop_compute<P, 3, true, DAG, HALF>(g, x, b, acc); break;
    default: hop_compute<P, 3, false, DAG, HALF>(g, x, b, acc); break;
    }
}

// One lane per site. With half-precision storage and no software pipelining the kernel
// fits four waves per SIMD without spilling (123 VGPRs instead of 156 at three), which
// hides more of the gather latency.
template <int P, bool DAG, bool PIPE, int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P >= F16S && !PIPE ? 4 : 1)))
void dw_kernel(Geom g, const void* __restrict__ links, const void* __restrict__ dets,
               const void* __restrict__ clover, Epi epi, RhsTable tab)
{
    using R = typename Traits<P>::real;
    const int logical = xcd_tile(blockIdx.x, gridDim.x);
    const int tile = logical / tab.nrhs;
    const int rhs = logical - tile * tab.nrhs;
    if (tab.gate && !tab.gate[(long)rhs * tab.gstride]) return;
    const void* __restrict__ in = tab.f[rhs].in;
    void* __restrict__ out = tab.f[rhs].out;
    int par, i;
    double sum = 0.0;
    if (walk_site(g, tile, threadIdx.x, par, i)) {
        int x[4], lex;
        eo_coords(g, par, i, x, lex);
        cx<R> hop[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) hop[c] = {(R)0, (R)0};
        if constexpr (PIPE) {
            HopIn<P> A, B;
            load_k<P>(0, g, in, links, dets, par, i, x, lex, A);
#pragma unroll 1
            for (int k = 0; k < 8; k += 2) {
                int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
                asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
                load_k<P>(k + 1, g, in, links, dets, par, ii, xx, ll, B);
                compute_k<P, DAG>(k, g, xx, A, hop);
                if (k + 2 < 8) load_k<P>(k + 2, g, in, links, dets, par, ii, xx, ll, A);
                compute_k<P, DAG>(k + 1, g, xx, B, hop);
            }
        } else {
            HopIn<P> A;
#pragma unroll 1
            for (int k = 0; k < 8; ++k) {
                int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
                asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
                load_k<P>(k, g, in, links, dets, par, ii, xx, ll, A);
                compute_k<P, DAG>(k, g, xx, A, hop);
            }
        }
        cx<R> s[12], acc[12];
        load_spinor<P>(in, g.Vh, par, i, s);
        clover54_apply<P>(clover, g.Vh, par, i, (R)g.cdiag, s, acc);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = acc[c] - scale(hop[c], (R)0.5);
        store_out<P, EPI>(out, epi, g.Vh, par, i, acc, sum);
    }
    if constexpr (EPI != EPI_NONE) grid_sums<1>(&sum, epi.sums, blockIdx.x, gridDim.x);
}

// Marching form: a workgroup owns one spatial tile (both parities) and walks the nt time
// slices of its chunk in order. The tile's spinors of the newest slice are kept in LDS (each
// lane loads its own site's once), and serve from there
//   * the +t hop of the slice before: the +t neighbour of a site is the partner lane's spinor
//     (the other parity, same even-odd index: the same spatial point one slice on);
//   * the spatial hops that stay inside the tile (most of x3 and x2); only the others read a
//     neighbour from memory;
//   * the -t hop of the slice after: each lane forms U_0^+ (1 -+ gamma_0) psi of its own site
//     with the forward t link that it has in hand and gives it to the partner through LDS.
// A psi and the six spatial hops of a site are done one step early, in the step that loads
// its slice (every lane its own site, all workgroups of an XCD at about the same time), while
// the neighbours outside the tile are still in L2; the time hops are added in the next step.
// Gathering a slice in the step after it was loaded found most of it evicted (an XCD streams
// more than its 4 MB L2 per step) and read it from HBM a second time. Two barriers a step.
// (In LDS a lane's values lie 64 lanes apart, so that one address and constant offsets reach
// them all; with the lane count as the stride every value's address was held in a register.)
// Two waves per SIMD, except FP64 with the pipelined hop loop: its two register buffers need
// 340 registers, and held to 256 it spilled 516 of them (32^3 x 64 on 512 workgroups: 1132 us
// instead of 513, one wave per SIMD).
template <class R>
struct Tile {
    // (typed as LDS: as generic pointers their loads and the global ones beside them are folded
    // into one load of either)
    template <class T> using Lds = __attribute__((address_space(3))) T;
    Lds<u32x4>* p;     // [lane / 64][24 reals as 16-byte pieces][lane % 64]
    Lds<R>* half;      // [lane / 64][12 reals][lane % 64]: transported -t neighbours
    int base, n;  // spatial index of the tile's first site; sites of each parity
    static constexpr int NP = 24 * sizeof(R) / 16;

    __device__ __forceinline__ void put(int who, const cx<R> v[12]) const
    {
        u32x4 w[NP];
        Lds<u32x4>* at = p + (who >> 6) * (NP * 64) + (who & 63);
        __builtin_memcpy(w, v, sizeof(w));
#pragma unroll
        for (int q = 0; q < NP; ++q) at[q * 64] = w[q];
    }
    __device__ __forceinline__ void get(int who, cx<R> v[12]) const
    {
        u32x4 w[NP];
        const Lds<u32x4>* at = p + (who >> 6) * (NP * 64) + (who & 63);
#pragma unroll
        for (int q = 0; q < NP; ++q) w[q] = at[q * 64];
        __builtin_memcpy(v, w, sizeof(w));
    }
    __device__ __forceinline__ void put_half(int who, const cx<R> v[6]) const
    {
        Lds<R>* at = half + (who >> 6) * (12 * 64) + (who & 63);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            at[(2 * q) * 64] = v[q].re;
            at[(2 * q + 1) * 64] = v[q].im;
        }
    }
    __device__ __forceinline__ void get_half(int who, cx<R> v[6]) const
    {
        const Lds<R>* at = half + (who >> 6) * (12 * 64) + (who & 63);
#pragma unroll
        for (int q = 0; q < 6; ++q) v[q] = {at[(2 * q) * 64], at[(2 * q + 1) * 64]};
    }
};

// loads of spatial hop (MU, FWD) into site x of the slice in `tile`
template <int P, int MU, bool FWD>
__device__ __forceinline__ void tile_hop_load(const Geom& g, const Tile<typename Traits<P>::real>& tile,
                                              const void* in, const void* links, const void* dets, int par,
                                              int i, const int x[4], int lex, HopIn<P>& b)
{
    const int j = (FWD ? lex_fwd(g, x, lex, MU) : lex_bwd(g, x, lex, MU)) >> 1;
    const int off = j - x[0] * g.S - tile.base;
    const bool inside = (unsigned)off < (unsigned)tile.n;
    tile.get((1 - par) * g.ts + (inside ? off : 0), b.s);
    if (!inside) load_spinor<P>(in, g.Vh, 1 - par, j, b.s);
    if (FWD) load_link<P>(links, dets, g.Vh, par, i, MU, b.u, b.d);       // U_mu(x)
    else load_link<P>(links, dets, g.Vh, 1 - par, j, MU, b.u, b.d);      // U_mu(x - mu)
}

template <int P>
__device__ __forceinline__ void tile_load_k(int k, const Geom& g, const Tile<typename Traits<P>::real>& tile,
                                            const void* in, const void* links, const void* dets, int par, int i,
                                            const int x[4], int lex, HopIn<P>& b)
{
    switch (k) {
    case 2: tile_hop_load<P, 1, true>(g, tile, in, links, dets, par, i, x, lex, b); break;
    case 3: tile_hop_load<P, 1, false>(g, tile, in, links, dets, par, i, x, lex, b); break;
    case 4: tile_hop_load<P, 2, true>(g, tile, in, links, dets, par, i, x, lex, b); break;
    case 5: tile_hop_load<P, 2, false>(g, tile, in, links, dets, par, i, x, lex, b); break;
    case 6: tile_hop_load<P, 3, true>(g, tile, in, links, dets, par, i, x, lex, b); break;
    default: tile_hop_load<P, 3, false>(g, tile, in, links, dets, par, i, x, lex, b); break;
    }
}

template <int P, bool DAG, bool PIPE>
__device__ __forceinline__ void march_site_hops(const Geom& g, const Tile<typename Traits<P>::real>& tile,
                                                const void* in, const void* links, const void* dets, int par,
                                                int i, const int x[4], int lex,
                                                cx<typename Traits<P>::real> acc[12])
{
    if constexpr (!PIPE) {
        // the six spatial hops (loop steps 2..7 of dw_kernel), one register buffer
        HopIn<P> A;
#pragma unroll 1
        for (int k = 2; k < 8; ++k) {
            int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
            asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
            tile_load_k<P>(k, g, tile, in, links, dets, par, ii, xx, ll, A);
            compute_k<P, DAG, true>(k, g, xx, A, acc);
        }
        return;
    }
    // the six spatial hops (loop steps 2..7 of dw_kernel), two register buffers
    HopIn<P> A, B;
    tile_load_k<P>(2, g, tile, in, links, dets, par, i, x, lex, A);
#pragma unroll 1
    for (int k = 2; k < 8; k += 2) {
        int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
        asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
        tile_load_k<P>(k + 1, g, tile, in, links, dets, par, ii, xx, ll, B);
        compute_k<P, DAG, true>(k, g, xx, A, acc);
        if (k + 2 < 8) tile_load_k<P>(k + 2, g, tile, in, links, dets, par, ii, xx, ll, A);
        compute_k<P, DAG, true>(k + 1, g, xx, B, acc);
    }
}

// bytes of LDS for ts sites per parity: a spinor and a half spinor per lane
template <class R>
constexpr size_t march_lds(int ts)
{
    return (size_t)2 * ts * 36 * sizeof(R);
}
inline size_t march_lds(int prec, int ts) { return prec == F64 ? march_lds<double>(ts) : march_lds<float>(ts); }

template <int P, bool DAG, bool PIPE, int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P == F64 && PIPE ? 1 : 2)))
void dw_march_kernel(Geom g, const void* __restrict__ links, const void* __restrict__ dets,
                     const void* __restrict__ clover, Epi epi, RhsTable tab)
{
    using R = typename Traits<P>::real;
    constexpr int SGF = DAG ? +1 : -1;  // projector of the +t hop: 1 + SGF gamma_0
    constexpr int SGB = -SGF;           // of the -t hop
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int nl = blockDim.x;  // 2 ts lanes
    const int logical = xcd_tile(blockIdx.x, gridDim.x);
    const int wg = logical / tab.nrhs;
    const int rhs = logical - wg * tab.nrhs;
    if (tab.gate && !tab.gate[(long)rhs * tab.gstride]) return;  // the whole workgroup
    const void* __restrict__ in = tab.f[rhs].in;
    void* __restrict__ out = tab.f[rhs].out;
    const int c = wg / g.ntile, s = wg - c * g.ntile;
    const int t0 = c * g.nt;
    const int tid = threadIdx.x;
    const int par = tid >= g.ts ? 1 : 0;
    const int lane = tid - par * g.ts;
    const int partner = tid + (par ? -g.ts : g.ts);
    Tile<R> tile{(typename Tile<R>::template Lds<u32x4>*)smem,
                 (typename Tile<R>::template Lds<R>*)(smem + 24 * sizeof(R) * nl), 0, 0};
    if (g.walk == 0) {
        tile.base = s * g.ts;
        tile.n = min(g.ts, g.S - tile.base);
    } else {
        const int b = s / g.L[1], x1 = s - b * g.L[1];
        tile.base = x1 * g.slab + b * g.ts;
        tile.n = min(g.ts, g.slab - b * g.ts);
    }
    // (a lane past the tile's end does the last site again, without storing it: a branch around
    // each step kept two copies of what lives across it)
    const bool valid = lane < tile.n;
    const int k = tile.base + min(lane, tile.n - 1);
    // U_0(y)^+ (1 + SGB gamma_0) psi(y), y the lane's site at slice t: the -t hop of the
    // partner's site one slice up (sign when the hop wraps from T-1 to 0)
    auto transport = [&](int t, const cx<R> sp[12], const cx<R> u[6], cx<R> d, cx<R> w[6]) {
        cx<R> h[6];
        project<R, 0, SGB>(sp, h);
        if (g.bc_t < 0 && t == g.L[0] - 1) {
#pragma unroll
            for (int q = 0; q < 6; ++q) h[q] = {-h[q].re, -h[q].im};
        }
        su3_mul<R, true, true>(u, d, h, w);
    };
    // A psi plus the six spatial hops (scaled by -1/2) of this lane's site at slice tt, the
    // slice in `tile`
    auto site_part = [&](int tt, cx<R> acc[12]) {
        const int i = tt * g.S + k;
        int x[4], lex;
        eo_coords(g, par, i, x, lex);
        {
            cx<R> sp[12];
            tile.get(tid, sp);
            clover54_apply<P>(clover, g.Vh, par, i, (R)g.cdiag, sp, acc);
        }
        march_site_hops<P, DAG, PIPE>(g, tile, in, links, dets, par, i, x, lex, acc);
    };
    // the accumulator of the current slice, begun in the step before
    cx<R> acc[12];
    double sum = 0.0;
    {
        const int tp = t0 == 0 ? g.L[0] - 1 : t0 - 1;
        cx<R> sp[12], u[6], d, w[6];
        load_spinor<P>(in, g.Vh, par, tp * g.S + k, sp);
        load_link<P>(links, dets, g.Vh, par, tp * g.S + k, 0, u, d);
        transport(tp, sp, u, d, w);
        tile.put_half(partner, w);
        load_spinor<P>(in, g.Vh, par, t0 * g.S + k, sp);
        tile.put(tid, sp);
    }
    __syncthreads();
    site_part(t0, acc);
    for (int step = 0;; ++step) {
        const int t = t0 + step;
        const int tn = t + 1 == g.L[0] ? 0 : t + 1;
        const int i = t * g.S + k;
        // (1) the spinor of the lane's site at t+1; the site's forward t link, which serves
        //     the +t hop and the partner's -t hop at t+1
        cx<R> nxt[12], u0[6], d0, wn[6], wb[6];
        load_spinor<P>(in, g.Vh, par, tn * g.S + k, nxt);
        load_link<P>(links, dets, g.Vh, par, i, 0, u0, d0);
        {
            // (read again: kept from site_part it would take registers through the hops)
            int me = tid;
            asm volatile("" : "+v"(me));
            cx<R> own[12];
            tile.get(me, own);
            transport(t, own, u0, d0, wn);
        }
        __syncthreads();  // slice t in the tile has been read, with its -t hops given
        tile.put(tid, nxt);
        tile.get_half(tid, wb);
        __syncthreads();  // the tile holds slice t+1, and the -t hops have been read
        tile.put_half(partner, wn);
        {
            // +t: U_0(x) times the projected neighbour
            cx<R> sp[12], h[6], w[6];
            tile.get(partner, sp);
            project<R, 0, SGF>(sp, h);
            const R f = (g.bc_t < 0 && t == g.L[0] - 1) ? (R)0.5 : (R)-0.5;
#pragma unroll
            for (int q = 0; q < 6; ++q) h[q] = scale(h[q], f);
            su3_mul<R, false, true>(u0, d0, h, w);
            expand_add<R, 0, SGF>(w, acc);
            // -t: already transported by the partner
#pragma unroll
            for (int q = 0; q < 6; ++q) wb[q] = scale(wb[q], (R)-0.5);
            expand_add<R, 0, SGB>(wb, acc);
        }
        if (valid) store_out<P, EPI>(out, epi, g.Vh, par, i, acc, sum);
        if (step + 1 == g.nt) break;
        // (2) the next slice's clover term and spatial hops
        site_part(tn, acc);
    }
    if constexpr (EPI != EPI_NONE) grid_sums<1>(&sum, epi.sums, blockIdx.x, gridDim.x);
}

// The marching form without the tile (hand_over says where). Nothing of the tile is kept in
// LDS but what partners exchange: the +t neighbour as a projected half spinor, the -t neighbour
// as a transported one, each in two slots, so that a step has one barrier; a lane's own spinor
// stays in registers and the spatial hops read their neighbours from memory. With about one
// wave per SIMD nothing hides a step's chain of loads, LDS accesses and barriers, and this
// chain is the shorter one; it needs a wave's whole register file, which is free there. The
// order of the sums is dw_march_kernel's.
template <int P, bool DAG, bool PIPE>
__device__ __forceinline__ void hand_site_hops(const Geom& g, const void* in, const void* links,
                                               const void* dets, int par, int i, const int x[4],
                                               int lex, cx<typename Traits<P>::real> acc[12])
{
    if constexpr (!PIPE) {
        HopIn<P> A;
#pragma unroll 1
        for (int k = 2; k < 8; ++k) {
            int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
            asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
            load_k<P>(k, g, in, links, dets, par, ii, xx, ll, A);
            compute_k<P, DAG, true>(k, g, xx, A, acc);
        }
        return;
    }
    HopIn<P> A, B;
    load_k<P>(2, g, in, links, dets, par, i, x, lex, A);
#pragma unroll 1
    for (int k = 2; k < 8; k += 2) {
        int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
        asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
        load_k<P>(k + 1, g, in, links, dets, par, ii, xx, ll, B);
        compute_k<P, DAG, true>(k, g, xx, A, acc);
        if (k + 2 < 8) load_k<P>(k + 2, g, in, links, dets, par, ii, xx, ll, A);
        compute_k<P, DAG, true>(k + 1, g, xx, B, acc);
    }
}

// bytes of LDS for ts sites per parity: two slots of both half spinors of every lane
template <class R>
constexpr size_t hand_lds(int ts)
{
    return (size_t)2 * 2 * 12 * (2 * ts) * sizeof(R);
}

template <int P, bool DAG, bool PIPE, int EPI>
__global__ __launch_bounds__(256)
void dw_hand_kernel(Geom g, const void* __restrict__ links, const void* __restrict__ dets,
                    const void* __restrict__ clover, Epi epi, RhsTable tab)
{
    using R = typename Traits<P>::real;
    constexpr int SGF = DAG ? +1 : -1;  // projector of the +t hop: 1 + SGF gamma_0
    constexpr int SGB = -SGF;           // of the -t hop
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int nl = blockDim.x;  // 2 ts lanes
    R* hp = (R*)smem;           // [2 slots][12 reals][nl]: projected +t neighbours
    R* pw = hp + 2 * 12 * nl;   // [2 slots][12 reals][nl]: transported -t neighbours
    const int logical = xcd_tile(blockIdx.x, gridDim.x);
    const int wg = logical / tab.nrhs;
    const int rhs = logical - wg * tab.nrhs;
    if (tab.gate && !tab.gate[(long)rhs * tab.gstride]) return;  // the whole workgroup
    const void* __restrict__ in = tab.f[rhs].in;
    void* __restrict__ out = tab.f[rhs].out;
    const int c = wg / g.ntile, s = wg - c * g.ntile;
    const int t0 = c * g.nt;
    const int tid = threadIdx.x;
    const int par = tid >= g.ts ? 1 : 0;
    const int lane = tid - par * g.ts;
    const int partner = tid + (par ? -g.ts : g.ts);
    int k;
    bool valid;
    if (g.walk == 0) {
        k = s * g.ts + lane;
        valid = k < g.S;
    } else {
        const int b = s / g.L[1], x1 = s - b * g.L[1];
        k = x1 * g.slab + b * g.ts + lane;
        valid = b * g.ts + lane < g.slab;
    }
    auto put6 = [&](R* buf, int slot, int who, const cx<R> v[6]) {
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            buf[(slot * 12 + 2 * q) * nl + who] = v[q].re;
            buf[(slot * 12 + 2 * q + 1) * nl + who] = v[q].im;
        }
    };
    auto get6 = [&](const R* buf, int slot, cx<R> v[6]) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
            v[q] = {buf[(slot * 12 + 2 * q) * nl + tid], buf[(slot * 12 + 2 * q + 1) * nl + tid]};
    };
    // U_0(y)^+ (1 + SGB gamma_0) psi(y) for the partner's site one slice up (sign when the
    // hop wraps from T-1 to 0)
    auto push = [&](int t, int slot, const cx<R> sp[12], const cx<R> u[6], cx<R> d) {
        cx<R> h[6], w[6];
        project<R, 0, SGB>(sp, h);
        if (g.bc_t < 0 && t == g.L[0] - 1) {
#pragma unroll
            for (int q = 0; q < 6; ++q) h[q] = {-h[q].re, -h[q].im};
        }
        su3_mul<R, true, true>(u, d, h, w);
        put6(pw, slot, partner, w);
    };
    // A psi plus the six spatial hops (scaled by -1/2) of this lane's site at slice tt,
    // whose spinor `sp` the lane holds
    auto site_part = [&](int tt, const cx<R> sp[12], cx<R> acc[12]) {
        const int i = tt * g.S + k;
        int x[4], lex;
        eo_coords(g, par, i, x, lex);
        clover54_apply<P>(clover, g.Vh, par, i, (R)g.cdiag, sp, acc);
        hand_site_hops<P, DAG, PIPE>(g, in, links, dets, par, i, x, lex, acc);
    };
    // the accumulator of the current slice was begun in the step before
    cx<R> own[12], acc[12];
    double sum = 0.0;
    if (valid) {
        const int tp = t0 == 0 ? g.L[0] - 1 : t0 - 1;
        cx<R> u[6], d;
        load_spinor<P>(in, g.Vh, par, tp * g.S + k, own);
        load_link<P>(links, dets, g.Vh, par, tp * g.S + k, 0, u, d);
        push(tp, t0 & 1, own, u, d);
        load_spinor<P>(in, g.Vh, par, t0 * g.S + k, own);
        site_part(t0, own, acc);
    }
    for (int step = 0; step < g.nt; ++step) {
        const int t = t0 + step;
        const int tn = t + 1 == g.L[0] ? 0 : t + 1;
        // (1) the spinor this lane owns at t+1, projected for the partner's +t hop; slot
        //     (t+1)&1 was last read two steps ago, before the previous barrier
        cx<R> nxt[12];
        if (valid) {
            cx<R> h[6];
            load_spinor<P>(in, g.Vh, par, tn * g.S + k, nxt);
            project<R, 0, SGF>(nxt, h);
            put6(hp, (t + 1) & 1, partner, h);
        }
        __syncthreads();
        if (valid) {
            const int i = t * g.S + k;
            // the site's forward t link serves the +t hop and the hand-over below
            cx<R> u0[6], d0;
            load_link<P>(links, dets, g.Vh, par, i, 0, u0, d0);
            // (2) the partner's -t hop at t+1; slot (t+1)&1 was read one step ago, before
            //     this step's barrier
            if (step + 1 < g.nt) push(t, (t + 1) & 1, own, u0, d0);
            {
                // +t: U_0(x) times the projected neighbour from the partner
                cx<R> h[6], w[6];
                get6(hp, (t + 1) & 1, h);
                const R f = (g.bc_t < 0 && t == g.L[0] - 1) ? (R)0.5 : (R)-0.5;
#pragma unroll
                for (int q = 0; q < 6; ++q) h[q] = scale(h[q], f);
                su3_mul<R, false, true>(u0, d0, h, w);
                expand_add<R, 0, SGF>(w, acc);
                // -t: already transported by the partner
                get6(pw, t & 1, w);
#pragma unroll
                for (int q = 0; q < 6; ++q) w[q] = scale(w[q], (R)-0.5);
                expand_add<R, 0, SGB>(w, acc);
            }
            store_out<P, EPI>(out, epi, g.Vh, par, i, acc, sum);
            // (3) the next slice's clover term and spatial hops, on the spinors loaded in
            //     this step
            if (step + 1 < g.nt) {
#pragma unroll
                for (int q = 0; q < 12; ++q) own[q] = nxt[q];
                site_part(tn, own, acc);
            }
        }
    }
    if constexpr (EPI != EPI_NONE) grid_sums<1>(&sum, epi.sums, blockIdx.x, gridDim.x);
}

// Even-odd reduced operator D^ = A_ee - D_eo A_oo^-1 D_oe on the even half of a field, in
// two passes over one parity each (one lane per site):
//   stage 1, odd sites:  t = A_oo^-1 (D_oe psi_e) = A_oo^-1 (-1/2 sum of the hops of psi_e)
//   stage 2, even sites: out = A_ee psi_e - D_eo t = A_ee psi_e + 1/2 sum of the hops of t
// t lives in the odd half of the output field. D^+ = gamma_5 D^ gamma_5 flips the
// projector signs as for D (A and A^-1 commute with gamma_5).
template <int P, bool DAG, int STAGE, bool PIPE, int EPI>
__global__ __launch_bounds__(256) void schur_kernel(Geom g, int ntile1, const void* hsrc,
                                                    const void* dsrc, void* out,
                                                    const void* __restrict__ links,
                                                    const void* __restrict__ dets,
                                                    const void* __restrict__ diag, Epi epi)
{
    using R = typename Traits<P>::real;
    constexpr int par = STAGE == 1 ? 1 : 0;
    // one parity: tiles of 256 consecutive even-odd indices of a slice, nt slices of one
    // tile in a row, XCD-contiguous (as the one-workgroup-per-slice D kernel, walk 0)
    const int logical = xcd_tile(blockIdx.x, gridDim.x);
    const int per_chunk = g.nt * ntile1;
    const int c = logical / per_chunk;
    const int r = logical - c * per_chunk;
    const int sidx = r / g.nt;
    const int t = c * g.nt + (r - sidx * g.nt);
    const int k = sidx * 256 + (int)threadIdx.x;
    double sum = 0.0;
    if (k < g.S) {
        const int i = t * g.S + k;
        int x[4], lex;
        eo_coords(g, par, i, x, lex);
        cx<R> hop[12];
#pragma unroll
        for (int q = 0; q < 12; ++q) hop[q] = {(R)0, (R)0};
        if constexpr (PIPE) {
            HopIn<P> A, B;
            load_k<P>(0, g, hsrc, links, dets, par, i, x, lex, A);
#pragma unroll 1
            for (int kk = 0; kk < 8; kk += 2) {
                int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
                asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
                load_k<P>(kk + 1, g, hsrc, links, dets, par, ii, xx, ll, B);
                compute_k<P, DAG>(kk, g, xx, A, hop);
                if (kk + 2 < 8) load_k<P>(kk + 2, g, hsrc, links, dets, par, ii, xx, ll, A);
                compute_k<P, DAG>(kk + 1, g, xx, B, hop);
            }
        } else {
            HopIn<P> A;
#pragma unroll 1
            for (int kk = 0; kk < 8; ++kk) {
                int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
                asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
                load_k<P>(kk, g, hsrc, links, dets, par, ii, xx, ll, A);
                compute_k<P, DAG>(kk, g, xx, A, hop);
            }
        }
        cx<R> acc[12];
        if constexpr (STAGE == 1) {
#pragma unroll
            for (int q = 0; q < 12; ++q) hop[q] = scale(hop[q], (R)-0.5);
            clover_apply<P>(diag, g.Vh, par, i, hop, acc);
        } else {
            cx<R> sp[12];
            load_spinor<P>(dsrc, g.Vh, par, i, sp);
            clover_apply<P>(diag, g.Vh, par, i, sp, acc);
#pragma unroll
            for (int q = 0; q < 12; ++q) acc[q] = acc[q] + scale(hop[q], (R)0.5);
        }
        store_out<P, EPI>(out, epi, g.Vh, par, i, acc, sum);
    }
    if constexpr (EPI != EPI_NONE) grid_sums<1>(&sum, epi.sums, blockIdx.x, gridDim.x);
}

// Small lattices: with one lane per site a lattice of some ten thousand sites leaves most of
// the machine without work, and the launch lasts as long as one lane's chain of eight hops
// (FP64 at 4^4: 10.6 us, whatever the shape). Here a workgroup of eight wavefronts owns 64
// consecutive sites of one parity, one hop direction per wavefront: the hops run side by side
// and meet in LDS as half spinors, and then four wavefronts form one spin of the outputs
// each, adding the diagonal term, whose loads they issue first. Any 64-site block is a
// workgroup, so lattices of any shape split evenly. Every term is added in the order in which
// the default form of larger launches adds it, so a field's D has the same bits however many
// fields share its launch.
//   KIND 0: out = A psi - 1/2 hops(psi), both parities (D)
//   KIND 1: out = A^-1 (-1/2 hops(psi)) on the odd sites, KIND 2: out = A psi + 1/2 hops(t)
//           on the even sites (the stages of the reduced operator)
template <int P, int KIND, int SPIN, bool DAG>
struct SplitRow {
    using T = Traits<P>;
    using R = typename T::real;
    static constexpr int BLK = SPIN / 2, UP = SPIN % 2;  // chirality block, row group in it
    R a[KIND == 0 ? Cl54Chunks<P>::n * T::PER_CHUNK : 36];
    cx<R> s[6];  // the block's half of psi

    // (entries that the row does not use are not loaded)
    __device__ __forceinline__ void load(const Geom& g, const void* psi, const void* diag, int par, int i)
    {
        if constexpr (KIND == 0) {
            const long base = chunk_at(g.Vh, Cl54Chunks<P>::n, par, 0, i);
#pragma unroll
            for (int k = 0; k < Cl54Chunks<P>::n; ++k) {
                const Chunk<P> c = load_chunk<P>(diag, base + (long)k * kSB);
#pragma unroll
                for (int j = 0; j < T::PER_CHUNK; ++j) a[k * T::PER_CHUNK + j] = to_real<P>(c.v[j]);
            }
        } else {
            const long base = chunk_at(g.Vh, T::CLOVER_CHUNKS, par, 0, i);
#pragma unroll
            for (int k = 0; k < T::CLOVER_CHUNKS; ++k) {
                if ((k + 1) * T::PER_CHUNK <= 36 * BLK || k * T::PER_CHUNK >= 36 * BLK + 36) continue;
                const Chunk<P> c = load_chunk<P>(diag, base + (long)k * kSB);
#pragma unroll
                for (int j = 0; j < T::PER_CHUNK; ++j) {
                    const int q = k * T::PER_CHUNK + j - 36 * BLK;
                    if (q >= 0 && q < 36) a[q] = to_real<P>(c.v[j]);
                }
            }
        }
        if constexpr (KIND != 1) {
            cx<R> all[12];
            load_spinor<P>(psi, g.Vh, par, i, all);
#pragma unroll
            for (int k = 0; k < 6; ++k) s[k] = all[6 * BLK + k];
        }
    }

    // this spin's part of hop (MU, SG) from its half spinor in LDS: w0 or w1 times a phase (and
    // -1/2 with HALF)
    template <int MU, int SG, int SP, bool HALF = false>
    __device__ __forceinline__ static void add_hop(const R (*w)[64], int lane, cx<R> o[3])
    {
        constexpr bool second = SP < 2 ? SP == 1 : (MU == 0 || MU == 3) ? SP == 3 : SP == 2;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int q = 2 * (3 * second + c);
            const cx<R> raw = {w[q][lane], w[q + 1][lane]}, v = HALF ? scale(raw, (R)-0.5) : raw;
            if (SP < 2) o[c] = o[c] + v;
            else if (MU == 0) o[c] = SG > 0 ? o[c] - v : o[c] + v;
            else if (MU == 1) o[c] = SG > 0 ? o[c] + times_i(v) : o[c] - times_i(v);
            else if (MU == 2) o[c] = (SG > 0) == (SP == 2) ? o[c] + v : o[c] - v;
            else o[c] = (SG > 0) == (SP == 2) ? o[c] + times_i(v) : o[c] - times_i(v);
        }
    }
    template <int SP>
    __device__ __forceinline__ static void hop_sum(const R (*hw)[12][64], int lane, cx<R> o[3])
    {
        constexpr int F = DAG ? 1 : -1, Bk = -F;
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = {(R)0, (R)0};
        add_hop<0, F, SP>(hw[0], lane, o);
        add_hop<0, Bk, SP>(hw[1], lane, o);
        add_hop<1, F, SP>(hw[2], lane, o);
        add_hop<1, Bk, SP>(hw[3], lane, o);
        add_hop<2, F, SP>(hw[4], lane, o);
        add_hop<2, Bk, SP>(hw[5], lane, o);
        add_hop<3, F, SP>(hw[6], lane, o);
        add_hop<3, Bk, SP>(hw[7], lane, o);
    }

    // the three output components of this spin
    __device__ __forceinline__ void row(const Geom& g, const R (*hw)[12][64], int lane, cx<R> o[3]) const
    {
        cx<R> v[6];
        if constexpr (KIND == 1) {
            cx<R> h[6];
            hop_sum<2 * BLK>(hw, lane, h);
            hop_sum<2 * BLK + 1>(hw, lane, h + 3);
#pragma unroll
            for (int k = 0; k < 6; ++k) h[k] = scale(h[k], (R)-0.5);
            herm6_apply<R>(a, h, v);
#pragma unroll
            for (int c = 0; c < 3; ++c) o[c] = v[3 * UP + c];
        } else if constexpr (KIND == 0 && (P == F64 || P == F32)) {
            // the order of the marching forms: A psi, the spatial hops, the time hops
            constexpr int F = DAG ? 1 : -1, Bk = -F;
            cl54_block<R>((R)g.cdiag, a + 3 * BLK, a + (BLK ? 30 : 6), a + (BLK ? 36 : 12), s, v);
#pragma unroll
            for (int c = 0; c < 3; ++c) o[c] = v[3 * UP + c];
            add_hop<1, F, SPIN, true>(hw[2], lane, o);
            add_hop<1, Bk, SPIN, true>(hw[3], lane, o);
            add_hop<2, F, SPIN, true>(hw[4], lane, o);
            add_hop<2, Bk, SPIN, true>(hw[5], lane, o);
            add_hop<3, F, SPIN, true>(hw[6], lane, o);
            add_hop<3, Bk, SPIN, true>(hw[7], lane, o);
            add_hop<0, F, SPIN, true>(hw[0], lane, o);
            add_hop<0, Bk, SPIN, true>(hw[1], lane, o);
        } else {
            // the order of the one-lane-per-site kernels: the eight hops, then half of their sum
            cx<R> h[3];
            hop_sum<SPIN>(hw, lane, h);
            if constexpr (KIND == 0)
                cl54_block<R>((R)g.cdiag, a + 3 * BLK, a + (BLK ? 30 : 6), a + (BLK ? 36 : 12), s, v);
            else
                herm6_apply<R>(a, s, v);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                o[c] = KIND == 0 ? v[3 * UP + c] - scale(h[c], (R)0.5) : v[3 * UP + c] + scale(h[c], (R)0.5);
        }
    }
};

// place of component k (of 12) of a stored spinor, in storage scalars
template <int P>
__device__ __forceinline__ long component_at(int Vh, int par, int i, int k)
{
    using T = Traits<P>;
    constexpr int CPC = T::PER_CHUNK / 2;
    return chunk_at(Vh, T::SPIN_CHUNKS, par, k / CPC, i) * T::PER_CHUNK + 2 * (k % CPC);
}

template <int P, int KIND, bool DAG, int EPI>
__global__ __launch_bounds__(512)
void dw_split_kernel(Geom g, const void* psi, const void* __restrict__ links,
                     const void* __restrict__ dets, const void* __restrict__ diag, Epi epi, RhsTable tab)
{
    using T = Traits<P>;
    using R = typename T::real;
    using S = typename T::store;
    __shared__ R hw[8][12][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int logical = xcd_tile(blockIdx.x, gridDim.x);
    const int tile = logical / tab.nrhs, rhs = logical - tile * tab.nrhs;
    if (tab.gate && !tab.gate[(long)rhs * tab.gstride]) return;  // the whole workgroup
    const void* in = tab.f[rhs].in;
    void* out = tab.f[rhs].out;
    if (KIND == 0) psi = in;
    // blocks of the two parities of one index range follow each other
    const int par = KIND == 0 ? tile & 1 : KIND == 1 ? 1 : 0;
    const int i = (KIND == 0 ? tile >> 1 : tile) * 64 + lane;
    const bool live = i < g.Vh;
    int x[4] = {0, 0, 0, 0}, lex = 0;
    double sum = 0.0;
    if (live) eo_coords_fast(g, par, i, x, lex);

    auto hop = [&](auto mu_c, auto fwd_c) {
        constexpr int MU = decltype(mu_c)::value;
        constexpr bool FWD = decltype(fwd_c)::value;
        HopIn<P> b;
        cx<R> w[6];
        hop_load<P, MU, FWD>(g, in, links, dets, par, i, x, lex, b);
        hop_half<P, MU, FWD, DAG>(g, x, b, w);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            hw[wave][2 * q][lane] = w[q].re;
            hw[wave][2 * q + 1][lane] = w[q].im;
        }
    };
    auto store = [&](int spin, cx<R> o[3]) {
        const R a = EPI == EPI_STEP ? (R)epi.sc[S_ALPHA] : (R)0;
        S* f = (S*)(EPI == EPI_STEP ? epi.r : out);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            S* at = f + component_at<P>(g.Vh, par, i, 3 * spin + c);
            S v[2];
            if constexpr (EPI == EPI_STEP) {
                __builtin_memcpy(v, at, 2 * sizeof(S));
                o[c] = cx<R>{to_real<P>(v[0]), to_real<P>(v[1])} - scale(o[c], a);
            }
            v[0] = to_store<P>(settled<P>(o[c].re));
            v[1] = to_store<P>(settled<P>(o[c].im));
            __builtin_memcpy(__builtin_assume_aligned(at, 2 * sizeof(S)), v, 2 * sizeof(S));
            if constexpr (EPI != EPI_NONE) {
                const double re = to_real<P>(v[0]), im = to_real<P>(v[1]);
                sum = __builtin_fma(re, re, __builtin_fma(im, im, sum));
            }
        }
    };
    auto run = [&](auto spin_c, auto mu_c, auto fwd_c) {
        constexpr int SPIN = decltype(spin_c)::value;
        if constexpr (SPIN < 4) {
            SplitRow<P, KIND, SPIN, DAG> row;
            if (live) {
                row.load(g, psi, diag, par, i);
                hop(mu_c, fwd_c);
            }
            __syncthreads();
            if (live) {
                cx<R> o[3];
                row.row(g, hw, lane, o);
                store(SPIN, o);
            }
        } else {
            if (live) hop(mu_c, fwd_c);
            __syncthreads();
        }
    };
    using std::integral_constant;
    using Fw = std::true_type;
    using Bw = std::false_type;
    switch (wave) {
    case 0: run(integral_constant<int, 0>{}, integral_constant<int, 0>{}, Fw{}); break;
    case 1: run(integral_constant<int, 1>{}, integral_constant<int, 0>{}, Bw{}); break;
    case 2: run(integral_constant<int, 2>{}, integral_constant<int, 1>{}, Fw{}); break;
    case 3: run(integral_constant<int, 3>{}, integral_constant<int, 1>{}, Bw{}); break;
    case 4: run(integral_constant<int, 4>{}, integral_constant<int, 2>{}, Fw{}); break;
    case 5: run(integral_constant<int, 4>{}, integral_constant<int, 2>{}, Bw{}); break;
    case 6: run(integral_constant<int, 4>{}, integral_constant<int, 3>{}, Fw{}); break;
    default: run(integral_constant<int, 4>{}, integral_constant<int, 3>{}, Bw{}); break;
    }
    if constexpr (EPI != EPI_NONE) grid_sums<1>(&sum, epi.sums, blockIdx.x, gridDim.x);
}

// Where the split form is used: up to the lattice size (times the fields of a launch) at which
// the other forms have enough sites in flight to overtake it. Kernel times on either side, us,
// split against the other form: FP64 D 11.2 / 12.2 at 16 x 12^3, 22.8 / 18.2 at 16^4; FP32 12.3
// / 13.1 at 16^4, 19.0 / 16.4 at 20x14x18x22; FP16 10.1 / 12.0 and 15.1 / 13.5 at the same; both
// stages of the reduced operator: FP64 27.7 / 32.7 at 16^4 (512 workgroups, one round), 34.9 /
// 33.4 at 18 x 16^3, FP32 15.6 / 23.6 at 16^4 and 24.9 / 25.8 at 20x14x18x22, FP16 11.5 / 18.5
// and 17.4 / 19.7; at 4^4 5.1 / 10.6 (FP64 D), 4.2 / 8.4 (FP32), 3.9 / 9.0 (FP16).
inline bool split_form(int P, bool schur, long sites)
{
    constexpr long kD[4] = {40000, 70000, 90000, 90000}, kSchur[4] = {66000, 120000, 200000, 200000};
    return sites <= (schur ? kSchur[P] : kD[P]);
}

// Marching launches that take the form without the tile in LDS, by their 64-site units (two
// waves each). That form needs nearly a wave's whole register file in FP64, so it is for
// launches of one wave per SIMD (512 units; the tile form with the pipelined loop has one wave
// per SIMD too and needs the launch to be nearly full); FP32 fits two waves per SIMD in either,
// and the tile pays from a full round of them on, the pipelined loop on 64-site tiles in just
// that round. FP16 conversions are folded into mixed-precision FMAs at every use of a value,
// and a value read back from LDS is converted again, so FP16 has no tile form; nor has BF16
// with the pipelined loop, where the two are even.
// us, without the tile / with it: FP64 plain 14.7 / 17.7 at 320 units (20 x 12^2 x 14), 18.2 /
// 20.8 at 512 (16^4), 505 / 552 at 512 (32^3 x 64, nt 32), 30 / 23 at 640 (20 x 16^3); FP64
// pipelined 15.7 / 17.3 at 384, 30.5 / 31.8 at 768, even at 1024; FP32 pipelined 13.7 / 14.5 at
// 768 (24 x 16^3), 16.7 / 16.5 at 1024 (32 x 16^3), 276 / 262 at 1024 (32^3 x 64), then 2 to 4 %
// more; FP32 plain 14.7 / 15.5 at 768, 28.1 / 20.7 at 1196; BF16 plain 5 to 10 % more up to
// 1024, 11 to 25 % less beyond; FP16 2 to 7 % more at any size.
template <int P, bool PIPE>
inline bool hand_over(int ts, long units)
{
    if (P == F64) return units <= (PIPE ? 960 : 512);
    if (P == F32) return ts == 64 && (units <= 960 || (PIPE && units > 1024));
    return P == F16S || PIPE || units <= 1024;
}

template <int P, bool DAG, int EPI>
int schur_launch_t(qdw_op* op, const void* in, void* out, const Epi& epi, hipStream_t st)
{
    const Geom& g = op->g;
    if (split_form(P, true, g.V)) {
        const int nblk = padded(g.Vh) / kSB;
        dw_split_kernel<P, 1, DAG, EPI_NONE><<<nblk, 512, 0, st>>>(
            g, nullptr, op->links[P], op->det[P], op->cloverinv[P], Epi{}, one_field(in, out));
        QDW_LAUNCH_CHECK();
        dw_split_kernel<P, 2, DAG, EPI><<<nblk, 512, 0, st>>>(
            g, in, op->links[P], op->det[P], op->clover[P], epi, one_field(out, out));
        QDW_LAUNCH_CHECK();
        return QDW_OK;
    }
    const int ntile1 = (g.S + 255) / 256;
    const int nb = g.L[0] * ntile1;
    // the hop loop is software-pipelined where the registers allow it (FP64, FP32), as for D
    constexpr bool PIPE = P == F64 || P == F32;
    schur_kernel<P, DAG, 1, PIPE, EPI_NONE><<<nb, 256, 0, st>>>(
        g, ntile1, in, nullptr, out, op->links[P], op->det[P], op->cloverinv[P], Epi{});
    QDW_LAUNCH_CHECK();
    schur_kernel<P, DAG, 2, PIPE, EPI><<<nb, 256, 0, st>>>(
        g, ntile1, out, in, out, op->links[P], op->det[P], op->clover[P], epi);
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

// the operator's geometry with the D kernel's own shape for precision P (the default
// marching shape: with the walk chunk and pipelining for this many fields)
inline Geom shaped(const qdw_op* op, int P, int nrhs, bool& pipe)
{
    Geom g = op->g;
    const auto& s = op->dw_shape[P];
    const MarchShape m = op->dw_auto[P] && s.march && nrhs > 1 ? march_shape(g, P, nrhs) : MarchShape{s.nt, s.pipe, s.walk};
    pipe = m.pipe;
    set_walk(g, s.ts, m.nt, m.walk);
    return g;
}

template <int P, bool DAG, int EPI>
int launch(qdw_op* op, const RhsTable& tab, const Epi& epi, hipStream_t st)
{
    const int nrhs = tab.nrhs;
    bool pipe;
    const Geom g = shaped(op, P, nrhs, pipe);
    if (op->dw_auto[P] && split_form(P, false, (long)g.V * nrhs)) {
        const int nblk = 2 * (padded(g.Vh) / kSB) * nrhs;
        dw_split_kernel<P, 0, DAG, EPI><<<nblk, 512, 0, st>>>(g, nullptr, op->links[P], op->det[P],
                                                             op->clover54[P], epi, tab);
        QDW_LAUNCH_CHECK();
        return QDW_OK;
    }
    if (op->dw_shape[P].march) {
        using R = typename Traits<P>::real;
        const int nblk = (g.L[0] / g.nt) * g.ntile * nrhs;
        auto run = [&](auto pipe_c) {
            constexpr bool PIPE = decltype(pipe_c)::value;
            if (hand_over<P, PIPE>(g.ts, (long)nblk * (g.ts / 64)))
                dw_hand_kernel<P, DAG, PIPE, EPI><<<nblk, 2 * g.ts, hand_lds<R>(g.ts), st>>>(
                    g, op->links[P], op->det[P], op->clover54[P], epi, tab);
            else if constexpr (P <= F32 || (P == BF16S && !PIPE))
                dw_march_kernel<P, DAG, PIPE, EPI><<<nblk, 2 * g.ts, march_lds<R>(g.ts), st>>>(
                    g, op->links[P], op->det[P], op->clover54[P], epi, tab);
        };
        if (pipe) run(std::true_type{});
        else run(std::false_type{});
        QDW_LAUNCH_CHECK();
        return QDW_OK;
    }
    const int nblk = walk_blocks(g) * nrhs;
    if (pipe)
        dw_kernel<P, DAG, true, EPI><<<nblk, 2 * g.ts, 0, st>>>(g, op->links[P], op->det[P], op->clover54[P],
                                                                epi, tab);
    else
        dw_kernel<P, DAG, false, EPI><<<nblk, 2 * g.ts, 0, st>>>(g, op->links[P], op->det[P], op->clover54[P],
                                                                 epi, tab);
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

// f(precision as a compile-time constant)
template <class F>
int by_precision(int prec, F f)
{
    switch (prec) {
    case QDW_F64: return f(std::integral_constant<int, F64>{});
    case QDW_F32: return f(std::integral_constant<int, F32>{});
    case QDW_F16S: return f(std::integral_constant<int, F16S>{});
    case QDW_BF16S: return f(std::integral_constant<int, BF16S>{});
    default: QDW_CHECK(false, QDW_EINVAL, "dw_apply: bad precision");
    }
}

int dispatch(qdw_op* op, const RhsTable& tab, int prec, bool dag, hipStream_t st)
{
    return by_precision(prec, [&](auto P) {
        return dag ? launch<P.value, true, EPI_NONE>(op, tab, Epi{}, st)
                   : launch<P.value, false, EPI_NONE>(op, tab, Epi{}, st);
    });
}

// ------------------------------------------------------------------ uncompressed control
//
// The same operator with every FP64 link read as its full 3x3 matrix (18 reals, 9 chunks
// per link, no row rebuilt in the kernel): the control for the two-row storage. Only the
// one-lane-per-site form with a plain hop loop exists for it; it takes the walk of the
// operator's FP64 shape when that is a one-lane-per-site shape, else 128-site tiles in
// chunks of 4 slices, and is compared with the compressed kernel in the same form.

// full links, [par * 4 + mu][site / 64][9][site % 64] chunks of one complex number each:
// rows 0, 1 as stored and row 2 = d conj(row0 x row1), formed as the compressed kernels
// form it
__global__ __launch_bounds__(256) void full_links_kernel(Geom g, const void* links, const void* dets,
                                                         void* full)
{
    const long n = (long)g.Vh * 8;
    for (long q = (long)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (long)gridDim.x * blockDim.x) {
        const int row = (int)(q / g.Vh), i = (int)(q - (long)row * g.Vh);
        cx<double> u[6], d;
        load_link<F64>(links, dets, g.Vh, row >> 2, i, row & 3, u, d);
        const cx<double> m[9] = {u[0], u[1], u[2], u[3], u[4], u[5],
                                 d * conj_(cmadd(u[1] * u[5], -u[2], u[4])),
                                 d * conj_(cmadd(u[2] * u[3], -u[0], u[5])),
                                 d * conj_(cmadd(u[0] * u[4], -u[1], u[3]))};
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            Chunk<F64> c;
            c.v[0] = m[k].re;
            c.v[1] = m[k].im;
            store_chunk<F64>(full, chunk_at(g.Vh, 9, row, k, i), c);
        }
    }
}

template <bool DAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1)))
void dw_full_kernel(Geom g, const void* __restrict__ in, void* __restrict__ out,
                    const void* __restrict__ full, const void* __restrict__ clover)
{
    int par, i;
    if (!walk_site(g, xcd_tile(blockIdx.x, gridDim.x), threadIdx.x, par, i)) return;
    int x[4], lex;
    eo_coords(g, par, i, x, lex);
    cx<double> hop[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) hop[c] = {0.0, 0.0};
    auto one = [&](auto mu_c, auto fwd_c, int ii, int ll, const int xx[4]) {
        constexpr int MU = decltype(mu_c)::value;
        constexpr bool FWD = decltype(fwd_c)::value;
        constexpr int SG = (FWD != DAG) ? -1 : +1;
        const int j = (FWD ? lex_fwd(g, xx, ll, MU) : lex_bwd(g, xx, ll, MU)) >> 1;
        cx<double> sp[12], m[9], h[6], w[6];
        load_spinor<F64>(in, g.Vh, 1 - par, j, sp);
        const int lrow = (FWD ? par : 1 - par) * 4 + MU, li = FWD ? ii : j;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const Chunk<F64> c = load_chunk_cached<F64>(full, chunk_at(g.Vh, 9, lrow, k, li));
            m[k] = {c.v[0], c.v[1]};
        }
        project<double, MU, SG>(sp, h);
        if (MU == 0 && g.bc_t < 0 && xx[0] == (FWD ? g.L[0] - 1 : 0)) {
#pragma unroll
            for (int c = 0; c < 6; ++c) h[c] = -h[c];
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const cx<double> h0 = h[3 * a], h1 = h[3 * a + 1], h2 = h[3 * a + 2];
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                if (FWD)
                    w[3 * a + r] = cmadd(cmadd(m[3 * r] * h0, m[3 * r + 1], h1), m[3 * r + 2], h2);
                else
                    w[3 * a + r] = cmadd_conj(cmadd_conj(cmul_conj(m[r], h0), m[3 + r], h1), m[6 + r], h2);
            }
        }
        expand_add<double, MU, SG>(w, hop);
    };
    // the eight hops as a runtime loop over opaque site indices (as dw_kernel)
#pragma unroll 1
    for (int k = 0; k < 8; ++k) {
        int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
        asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
        using T = std::true_type;
        using F = std::false_type;
        switch (k) {
        case 0: one(std::integral_constant<int, 0>{}, T{}, ii, ll, xx); break;
        case 1: one(std::integral_constant<int, 0>{}, F{}, ii, ll, xx); break;
        case 2: one(std::integral_constant<int, 1>{}, T{}, ii, ll, xx); break;
        case 3: one(std::integral_constant<int, 1>{}, F{}, ii, ll, xx); break;
        case 4: one(std::integral_constant<int, 2>{}, T{}, ii, ll, xx); break;
        case 5: one(std::integral_constant<int, 2>{}, F{}, ii, ll, xx); break;
        case 6: one(std::integral_constant<int, 3>{}, T{}, ii, ll, xx); break;
        default: one(std::integral_constant<int, 3>{}, F{}, ii, ll, xx); break;
        }
    }
    cx<double> sp[12], acc[12];
    load_spinor<F64>(in, g.Vh, par, i, sp);
    clover54_apply<F64>(clover, g.Vh, par, i, g.cdiag, sp, acc);
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = acc[c] - scale(hop[c], 0.5);
    store_spinor<F64>(out, g.Vh, par, i, acc);
}

int apply_checked(qdw_op* op, const void* in, void* out, qdw_prec prec, bool dag, void* stream)
{
    QDW_CHECK(op && in && out, QDW_EINVAL, "dw_apply: null argument");
    QDW_CHECK(in != out, QDW_EINVAL, "dw_apply: in and out must be distinct fields");
    const RhsTable tab = one_field(in, out);
    return dispatch(op, tab, prec, dag, (hipStream_t)stream);
}

}  // namespace

namespace qdw {
// internal entries used by the solvers (same kernels, no argument re-validation)
int dw_launch(qdw_op* op, const void* in, void* out, int prec, bool dag, hipStream_t st)
{
    const RhsTable tab = one_field(in, out);
    return dispatch(op, tab, prec, dag, st);
}

int schur_launch(qdw_op* op, const void* in, void* out, int prec, bool dag, hipStream_t st)
{
    return by_precision(prec, [&](auto P) {
        return dag ? schur_launch_t<P.value, true, EPI_NONE>(op, in, out, Epi{}, st)
                   : schur_launch_t<P.value, false, EPI_NONE>(op, in, out, Epi{}, st);
    });
}

int cg_apply(qdw_op* op, const void* p, void* q, int prec, bool schur, int ring, hipStream_t st)
{
    const Epi e = {{op->partials, op->tickets, op->scalars, FIN_CG_ALPHA, ring, nullptr}, nullptr, nullptr};
    const RhsTable tab = one_field(p, q);
    return by_precision(prec, [&](auto P) {
        return schur ? schur_launch_t<P.value, false, EPI_NORM>(op, p, q, e, st)
                     : launch<P.value, false, EPI_NORM>(op, tab, e, st);
    });
}

int cg_apply_dag(qdw_op* op, const void* q, void* r, void* t, int prec, bool schur, double* host,
                 hipStream_t st)
{
    const Epi e = {{op->partials, op->tickets, op->scalars, FIN_CG_BETA, 0, host}, r, op->scalars};
    const RhsTable tab = one_field(q, r);
    return by_precision(prec, [&](auto P) {
        return schur ? schur_launch_t<P.value, true, EPI_STEP>(op, q, t, e, st)
                     : launch<P.value, true, EPI_STEP>(op, tab, e, st);
    });
}

int dw_launch_multi(qdw_op* op, const void* const* in, void* const* out, int nrhs, int prec,
                    bool dag, const int* gate, int gstride, hipStream_t st)
{
    RhsTable tab{};
    tab.gate = gate;
    tab.gstride = gstride;
    tab.nrhs = nrhs;
    for (int r = 0; r < nrhs; ++r) tab.f[r] = {in[r], out[r]};
    return dispatch(op, tab, prec, dag, st);
}
}  // namespace qdw

extern "C" int dw_apply(qdw_op* op, const void* in, void* out, qdw_prec prec, void* stream)
{
    return apply_checked(op, in, out, prec, false, stream);
}

extern "C" int dw_dag_apply(qdw_op* op, const void* in, void* out, qdw_prec prec, void* stream)
{
    return apply_checked(op, in, out, prec, true, stream);
}

extern "C" size_t qdw_full_links_bytes(const qdw_op* op)
{
    return op ? (size_t)padded(op->g.Vh) * 8 * 9 * 16 : 0;
}

extern "C" int qdw_set_full_links(qdw_op* op, void* dev_mem, size_t bytes, void* stream)
{
    QDW_CHECK(op && dev_mem, QDW_EINVAL, "qdw_set_full_links: null argument");
    QDW_CHECK(bytes >= qdw_full_links_bytes(op), QDW_EWORKSPACE,
              "qdw_set_full_links: block smaller than qdw_full_links_bytes()");
    QDW_CHECK(((uintptr_t)dev_mem & 15) == 0, QDW_EINVAL,
              "qdw_set_full_links: the block must be 16-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    full_links_kernel<<<1024, 256, 0, st>>>(op->g, op->links[F64], op->det[F64], dev_mem);
    QDW_LAUNCH_CHECK();
    op->full_links = dev_mem;
    return QDW_OK;
}

extern "C" int dw_apply_full_links(qdw_op* op, const void* in, void* out, int dagger, void* stream)
{
    QDW_CHECK(op && in && out, QDW_EINVAL, "dw_apply_full_links: null argument");
    QDW_CHECK(in != out, QDW_EINVAL, "dw_apply_full_links: in and out must be distinct fields");
    QDW_CHECK(op->full_links, QDW_EINVAL,
              "dw_apply_full_links: no full links (call qdw_set_full_links first)");
    Geom g = op->g;
    const auto& sh = op->dw_shape[F64];
    if (sh.march) set_walk(g, 128, g.L[0] % 4 == 0 ? 4 : 1, 0);
    else set_walk(g, sh.ts, sh.nt, sh.walk);
    hipStream_t st = (hipStream_t)stream;
    if (dagger)
        dw_full_kernel<true><<<walk_blocks(g), 2 * g.ts, 0, st>>>(g, in, out, op->full_links,
                                                                   op->clover54[F64]);
    else
        dw_full_kernel<false><<<walk_blocks(g), 2 * g.ts, 0, st>>>(g, in, out, op->full_links,
                                                                    op->clover54[F64]);
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

extern "C" int dw_schur_apply(qdw_op* op, const void* in, void* out, qdw_prec prec, void* stream)
{
    QDW_CHECK(op && in && out, QDW_EINVAL, "dw_schur_apply: null argument");
    QDW_CHECK(in != out, QDW_EINVAL, "dw_schur_apply: in and out must be distinct fields");
    return qdw::schur_launch(op, in, out, prec, false, (hipStream_t)stream);
}

extern "C" int dw_schur_dag_apply(qdw_op* op, const void* in, void* out, qdw_prec prec,
                                  void* stream)
{
    QDW_CHECK(op && in && out, QDW_EINVAL, "dw_schur_dag_apply: null argument");
    QDW_CHECK(in != out, QDW_EINVAL, "dw_schur_dag_apply: in and out must be distinct fields");
    return qdw::schur_launch(op, in, out, prec, true, (hipStream_t)stream);
}

extern "C" int dw_apply_multi(qdw_op* op, const void* const* in, void* const* out, int nrhs,
                              qdw_prec prec, void* stream)
{
    QDW_CHECK(op && in && out, QDW_EINVAL, "dw_apply_multi: null argument");
    QDW_CHECK(nrhs >= 1 && nrhs <= kMaxRhs, QDW_EINVAL, "dw_apply_multi: need 1 <= nrhs <= 64");
    for (int r = 0; r < nrhs; ++r) {
        QDW_CHECK(in[r] && out[r], QDW_EINVAL, "dw_apply_multi: null field");
        for (int q = 0; q < nrhs; ++q)
            QDW_CHECK(in[r] != out[q], QDW_EINVAL, "dw_apply_multi: an output aliases an input");
    }
    return qdw::dw_launch_multi(op, in, out, nrhs, prec, false, nullptr, 0, (hipStream_t)stream);
}

// ------------------------------------------------------------------ shapes and autotuner

namespace {
// timing input of the autotuner: every stored value a hashed number in [-0.5, 0.5) (all-zero
// fields would time a faster memory path than real data)
template <int P>
__global__ void fill_pattern_kernel(void* buf, long n)
{
    using S = typename Traits<P>::store;
    for (long j = (long)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (long)gridDim.x * blockDim.x) {
        uint32_t h = (uint32_t)j * 2654435761u;
        h ^= h >> 15;
        h *= 2246822519u;
        h ^= h >> 13;
        const float v = (float)(h & 0xFFFFu) * (1.0f / 65536.0f) - 0.5f;
        ((S*)buf)[j] = to_store<P>((typename Traits<P>::real)v);
    }
}

int fill_pattern(void* buf, size_t bytes, int prec, hipStream_t st)
{
    switch (prec) {
    case F64: fill_pattern_kernel<F64><<<1024, 256, 0, st>>>(buf, (long)(bytes / 8)); break;
    case F32: fill_pattern_kernel<F32><<<1024, 256, 0, st>>>(buf, (long)(bytes / 4)); break;
    case F16S: fill_pattern_kernel<F16S><<<1024, 256, 0, st>>>(buf, (long)(bytes / 2)); break;
    default: fill_pattern_kernel<BF16S><<<1024, 256, 0, st>>>(buf, (long)(bytes / 2)); break;
    }
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

int check_shape(const qdw_op* op, int prec, int ts, int nt, int pipe, int walk, int march)
{
    QDW_CHECK(!march || march_lds(prec, ts) <= 65536, QDW_EINVAL,
              "D kernel shape: a marching FP64 workgroup of 128 sites per parity needs more "
              "than 64 KB of LDS");
    QDW_CHECK(march == 0 || march == 1, QDW_EINVAL, "D kernel shape: march must be 0 or 1");
    QDW_CHECK(ts == 64 || ts == 128, QDW_EINVAL, "D kernel shape: ts must be 64 or 128");
    QDW_CHECK(nt >= 1 && nt <= 64 && op->g.L[0] % nt == 0, QDW_EINVAL,
              "D kernel shape: nt must divide T and lie in 1..64");
    QDW_CHECK(pipe == 0 || pipe == 1, QDW_EINVAL, "D kernel shape: pipe must be 0 or 1");
    QDW_CHECK(walk == 0 || walk == 1, QDW_EINVAL, "D kernel shape: walk must be 0 or 1");
    return QDW_OK;
}
}  // namespace

extern "C" int qdw_set_dw_shape(qdw_op* op, qdw_prec prec, int ts, int nt, int pipe, int walk,
                                int march)
{
    QDW_CHECK(op, QDW_EINVAL, "qdw_set_dw_shape: null operator");
    QDW_CHECK(prec >= QDW_F64 && prec <= QDW_BF16S, QDW_EINVAL, "qdw_set_dw_shape: bad precision");
    const int rc = check_shape(op, prec, ts, nt, pipe, walk, march);
    if (rc) return rc;
    op->dw_shape[prec] = {ts, nt, pipe, walk, march};
    op->dw_auto[prec] = false;
    return QDW_OK;
}

extern "C" int qdw_get_dw_shape(const qdw_op* op, qdw_prec prec, int* shape5)
{
    QDW_CHECK(op && shape5, QDW_EINVAL, "qdw_get_dw_shape: null argument");
    QDW_CHECK(prec >= QDW_F64 && prec <= QDW_BF16S, QDW_EINVAL, "qdw_get_dw_shape: bad precision");
    shape5[0] = op->dw_shape[prec].ts;
    shape5[1] = op->dw_shape[prec].nt;
    shape5[2] = op->dw_shape[prec].pipe;
    shape5[3] = op->dw_shape[prec].walk;
    shape5[4] = op->dw_shape[prec].march;
    return QDW_OK;
}

extern "C" int qdw_default_dw_shape(qdw_op* op, qdw_prec prec)
{
    QDW_CHECK(op, QDW_EINVAL, "qdw_default_dw_shape: null operator");
    QDW_CHECK(prec >= QDW_F64 && prec <= QDW_BF16S, QDW_EINVAL, "qdw_default_dw_shape: bad precision");
    default_dw_shape(op, prec);
    return QDW_OK;
}

extern "C" int qdw_dw_shape_is_default(const qdw_op* op, qdw_prec prec)
{
    QDW_CHECK(op, QDW_EINVAL, "qdw_dw_shape_is_default: null operator");
    QDW_CHECK(prec >= QDW_F64 && prec <= QDW_BF16S, QDW_EINVAL, "qdw_dw_shape_is_default: bad precision");
    return op->dw_auto[prec] ? 1 : 0;
}

extern "C" size_t qdw_autotune_workspace_bytes(const qdw_op* op, qdw_prec prec, int nrhs)
{
    if (!op || prec < QDW_F64 || prec > QDW_BF16S || nrhs < 1 || nrhs > kMaxRhs) return 0;
    return 2 * spinor_bytes(op->g, prec) * nrhs + 256;
}

extern "C" int qdw_autotune(qdw_op* op, qdw_prec prec, int nrhs, void* work, size_t work_bytes,
                            char* report, size_t report_len, void* stream)
{
    QDW_CHECK(op, QDW_EINVAL, "qdw_autotune: null operator");
    QDW_CHECK(prec >= QDW_F64 && prec <= QDW_BF16S, QDW_EINVAL, "qdw_autotune: bad precision");
    QDW_CHECK(nrhs >= 1 && nrhs <= kMaxRhs, QDW_EINVAL, "qdw_autotune: need 1 <= nrhs <= 64");
    QDW_CHECK(work, QDW_EINVAL, "qdw_autotune: null workspace");
    QDW_CHECK(work_bytes >= qdw_autotune_workspace_bytes(op, prec, nrhs), QDW_EWORKSPACE,
              "qdw_autotune: workspace smaller than qdw_autotune_workspace_bytes()");
    hipStream_t st = (hipStream_t)stream;
    const Geom& g = op->g;
    const size_t fb = spinor_bytes(g, prec);
    char* buf = (char*)(((uintptr_t)work + 255) & ~(uintptr_t)255);
    RhsTable tab{};
    tab.nrhs = nrhs;
    for (int r = 0; r < nrhs; ++r) tab.f[r] = {buf + (size_t)r * fb, buf + (size_t)(nrhs + r) * fb};
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const auto keep = op->dw_shape[prec];
    const bool keep_auto = op->dw_auto[prec];
    float default_ms = 0.f;
    struct Cand { int ts, nt, pipe, walk, march; float ms; };
    std::vector<Cand> cands;
    for (int march = 0; march < 2; ++march)
        for (int walk = 0; walk < 2; ++walk)
            for (int ts : {64, 128})
                for (int nt = 1; nt <= 64; nt *= 2) {
                    if (g.L[0] % nt) continue;
                    if (march && march_lds(prec, ts) > 65536) continue;
                    for (int pipe = 0; pipe < 2; ++pipe)
                        cands.push_back({ts, nt, pipe, walk, march, 0.f});
                }
    int rc = QDW_OK;
    auto run = [&]() -> int {
        int r0 = fill_pattern(buf, 2 * fb * nrhs, prec, st);
        if (r0) return r0;
        QDW_HIP(hipEventCreate(&e0));
        QDW_HIP(hipEventCreate(&e1));
        auto time_form = [&](float* out_ms) -> int {
            int r;
            for (int w = 0; w < 2; ++w)
                if ((r = dispatch(op, tab, prec, false, st))) return r;
            const int reps = 8;
            QDW_HIP(hipEventRecord(e0, st));
            for (int w = 0; w < reps; ++w)
                if ((r = dispatch(op, tab, prec, false, st))) return r;
            QDW_HIP(hipEventRecord(e1, st));
            QDW_HIP(hipEventSynchronize(e1));
            float ms = 0.f;
            QDW_HIP(hipEventElapsedTime(&ms, e0, e1));
            *out_ms = ms / reps;
            return QDW_OK;
        };
        int r;
        default_dw_shape(op, prec);
        if ((r = time_form(&default_ms))) return r;
        op->dw_auto[prec] = false;
        for (Cand& c : cands) {
            op->dw_shape[prec] = {c.ts, c.nt, c.pipe, c.walk, c.march};
            if ((r = time_form(&c.ms))) return r;
        }
        return QDW_OK;
    };
    rc = run();
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipStreamSynchronize(st);
    if (rc) {
        op->dw_shape[prec] = keep;
        op->dw_auto[prec] = keep_auto;
        return rc;
    }
    const Cand* best = &cands[0];
    for (const Cand& c : cands)
        if (c.ms < best->ms) best = &c;
    // the default stays where no shape beats it by more than two runs differ: its chunks need not
    // be powers of two, and it goes on choosing for launches of other sizes
    const bool stays = default_ms <= 1.02f * best->ms;
    if (stays) default_dw_shape(op, prec);
    else op->dw_shape[prec] = {best->ts, best->nt, best->pipe, best->walk, best->march};
    if (report && report_len) {
        std::string s;
        char line[200];
        const auto& c0 = op->dw_shape[prec];
        std::snprintf(line, sizeof line,
                      "lattice %dx%dx%dx%d prec %d nrhs %d: best ts=%d nt=%d pipe=%d walk=%d march=%d %.4f ms%s;"
                      " default %.4f;",
                      g.L[0], g.L[1], g.L[2], g.L[3], (int)prec, nrhs, c0.ts, c0.nt, c0.pipe, c0.walk,
                      c0.march, stays ? default_ms : best->ms, stays ? " (default)" : "", default_ms);
        s += line;
        for (const Cand& c : cands) {
            std::snprintf(line, sizeof line, " [%d,%d,%d,%d,%d]=%.4f", c.ts, c.nt, c.pipe, c.walk,
                          c.march, c.ms);
            s += line;
        }
        std::snprintf(report, report_len, "%s", s.c_str());
    }
    return QDW_OK;
}
