// blas.h -- fused BLAS-1 on eo-SoA spinor fields with FP64 reductions.
//
// The paper (Sec. 2.1) keeps every reduction variable in binary64 whatever the working
// type of the vectors; here every lane accumulates its products in FP64 and the partial
// sums are combined across the wavefront (shuffles), the workgroup (LDS) and the grid
// (by the workgroup that finishes last) in a fixed order, so results are bitwise
// reproducible run to run.
//
// Unit of work: 4 complex numbers of one site. Fields of different storage precisions are
// addressed by the same unit, so mixed-precision kernels (FP32 solution, FP16 residual)
// pair the same lattice components.
#pragma once

#include "qdw_host.h"

namespace qdw {

// ---------------------------------------------------------------- unit load / store

// Unit of a map: run w of 64 sites, w = (parity * blocks of 64 sites + block) * 3 + group,
// and the site within it. A field stores the chunks of one such run contiguously, in the
// order of w, so a wavefront walks every field linearly whatever its precision, with no
// division by the lattice size (chunk_at with chunk = group * NCH + k).
struct Unit { unsigned w; int lane; };

template <int P, typename R>
__device__ __forceinline__ void ld4(const void* f, const Unit& u, cx<R> v[4])
{
    using T = Traits<P>;
    constexpr int CPC = T::PER_CHUNK / 2;        // complex per chunk
    constexpr int NCH = 4 / CPC;                 // chunks per unit
    const long at = (long)u.w * (NCH * kSB) + u.lane;
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        Chunk<P> c = load_chunk_cached<P>(f, at + k * kSB);
#pragma unroll
        for (int j = 0; j < CPC; ++j)
            v[k * CPC + j] = {(R)to_real<P>(c.v[2 * j]), (R)to_real<P>(c.v[2 * j + 1])};
    }
}

template <int P, typename R>
__device__ __forceinline__ void st4(void* f, const Unit& u, const cx<R> v[4])
{
    using T = Traits<P>;
    using RT = typename T::real;
    constexpr int CPC = T::PER_CHUNK / 2;
    constexpr int NCH = 4 / CPC;
    const long at = (long)u.w * (NCH * kSB) + u.lane;
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        Chunk<P> c;
#pragma unroll
        for (int j = 0; j < CPC; ++j) {
            c.v[2 * j] = to_store<P>((RT)v[k * CPC + j].re);
            c.v[2 * j + 1] = to_store<P>((RT)v[k * CPC + j].im);
        }
        uint4 raw;
        __builtin_memcpy(&raw, &c, 16);
        ((uint4*)f)[at + k * kSB] = raw;
    }
}

// The runs of a map launch: nw of them (both parities, or the even half), nb blocks of 64
// sites per parity, tail = sites of a parity's last block (64 when it is full). The padding
// positions of a ragged last block are left alone and never summed.
// `back` walks the runs from the last to the first: a map that reads the fields which the
// map before it has just read starts on the ones still in the 256 MB last-level cache.
struct Runs {
    unsigned nw;
    int nb, tail;
    bool back;
    __device__ __forceinline__ Unit unit(unsigned n) const
    {
        return {back ? nw - 1 - n : n, (int)(threadIdx.x & 63)};
    }
    __device__ __forceinline__ bool holds(const Unit& u) const
    {
        return tail == kSB || u.lane < tail || (int)((u.w / 3) % (unsigned)nb) != nb - 1;
    }
};

inline Runs runs_of(const Geom& g, bool even_half, bool back)
{
    const int nb = padded(g.Vh) / kSB;
    return {(unsigned)(3 * nb) * (even_half ? 1u : 2u), nb, g.Vh - (nb - 1) * kSB, back};
}

// scalar programs run by the finalising workgroup after the sums are formed
enum FinOp {
    FIN_STORE = 0,   // out[j] = sum_j
    FIN_CG_ALPHA,    // out = CG scalars: pap = sum_0; alpha = rr / pap (also at S_RING + k)
    FIN_CG_BETA,     // out = CG scalars: rrnew = sum_0; beta = rrnew / rr; rr = rrnew
    FIN_GCR_DOT,     // out = GCR scalars, step k: a_lk = sum_l / b_l for l < k
    FIN_GCR_NORM,    // out = GCR scalars, step k: b_k = sqrt(sum_0), 1/b_k,
                     //   c_k = (sum_1 + i sum_2)/b_k and the update's coefficient c_k/b_k
};

// The basis vectors chi_k of a GCR cycle are stored as they come out of the Gram-Schmidt
// pass, with norm b_k; the coefficients refer to chi_k / b_k. (Normalising them in memory
// took one more pass over a field per step.)
// GCR scalar block (doubles): a[k][l] complex at 2*(16*k + l), b_k at G_B + k, c_k complex
// at G_C + 2k, 1/b_k at G_IB + k, the update coefficient c_k/b_k at G_COEF
constexpr int kMaxKv = 16;
enum { G_A = 0, G_B = 2 * kMaxKv * kMaxKv, G_C = G_B + kMaxKv, G_IB = G_C + 2 * kMaxKv,
       G_COEF = G_IB + kMaxKv, G_NORM = G_COEF + 2, G_SIZE = G_NORM + 2 };

// scalar slots of the CG solver
enum { S_RR = 0, S_PAP = 1, S_ALPHA = 2, S_RRNEW = 3, S_BETA = 4, S_TMP = 8, S_RING = 40 };

// Directions of a CG that the iterate has not moved along yet, with their step lengths at
// S_RING. The iterate (FP32 or FP64) is the widest field of a step: moving it along four
// directions at a time reads and writes it a quarter as often for one more read of each
// direction (FP16 storage: 228 instead of 336 B per site and step on average).
constexpr int kRing = 4;

// the scalar program `op` on the grid's sums (one lane)
__device__ inline void scalar_program(const double* sums, int ns, double* out, int op, int k)
{
    switch (op) {
    case FIN_STORE:
        for (int j = 0; j < ns; ++j) out[j] = sums[j];
        break;
    case FIN_CG_ALPHA:  // a vanishing direction leaves the iterate unchanged
        out[S_PAP] = sums[0];
        out[S_ALPHA] = out[S_RING + k] = sums[0] != 0.0 ? out[S_RR] / sums[0] : 0.0;
        break;
    case FIN_CG_BETA:
        out[S_RRNEW] = sums[0];
        out[S_BETA] = out[S_RR] != 0.0 ? sums[0] / out[S_RR] : 0.0;
        out[S_RR] = sums[0];
        break;
    case FIN_GCR_DOT:
        for (int j = 0; j < ns; ++j) out[G_A + 2 * kMaxKv * k + j] = sums[j] * out[G_IB + j / 2];
        break;
    case FIN_GCR_NORM: {
        const double b = sqrt(sums[0]);
        const double ib = b > 0.0 ? 1.0 / b : 0.0;
        out[G_B + k] = b;
        out[G_C + 2 * k] = sums[1] * ib;
        out[G_C + 2 * k + 1] = sums[2] * ib;
        out[G_IB + k] = ib;
        out[G_COEF] = sums[1] * ib * ib;
        out[G_COEF + 1] = sums[2] * ib * ib;
        break;
    }
    default:
        break;
    }
}

// ---------------------------------------------------------------- reductions over the grid
//
// Every workgroup leaves its partial sums in memory; the one that arrives last adds them
// up, in an order fixed by the workgroup index, and runs the scalar program. That saves the
// launch of a second kernel and the idle machine around it. Partial sums and arrival
// counters are agent-scope atomics: each XCD has its own L2, and such accesses are coherent
// between them without writing back or invalidating a whole cache. A workgroup's counter is
// bumped only after its stores have completed (the wait below).

struct Sums {
    double* partials;   // sum j of workgroup b at [j * workgroups + b]
    unsigned* ticket;   // kTicketWords, zero between launches
    double* out;        // scalar program's block
    int fin, k;
    double* host;       // pinned host memory for the sums themselves, or nullptr
};

__device__ __forceinline__ double agent_load(const double* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Arrival `which` of n at a counter; true for the one that completes them. Arrival 0 adds
// 2^32 - (n - 1) and the others one each: the last one's addition carries, whichever it is, and
// the counter is zero again by itself. Nothing sets it back, so no arrival can be lost. (A
// counter that the last workgroup zeroed could lose one to another launch's, when two reductions
// ran at a time; they spoil each other's sums, but then no later sum was completed either.)
__device__ __forceinline__ bool arrive(unsigned* at, unsigned which, unsigned n)
{
    if (n == 1) return true;
    const unsigned mine = which == 0 ? 1u - n : 1u;
    return __hip_atomic_fetch_add(at, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > ~mine;
}

// one lane per workgroup; true for the last of nblk
__device__ __forceinline__ bool last_arrival(unsigned* ticket, unsigned blk, unsigned nblk)
{
    constexpr unsigned NG = kTickets;
    if (nblk < NG) return arrive(ticket, blk, nblk);
    const unsigned gr = blk % NG;
    return arrive(ticket + 32 * (1 + gr), blk / NG, (nblk - gr + NG - 1) / NG) && arrive(ticket, gr, NG);
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

constexpr int pow2_at_least(int n)
{
    int p = 1;
    while (p < n) p *= 2;
    return p;
}

// The sums over a wavefront of N values per lane, to dst[0 .. N). At each exchange a lane
// keeps one half of its values and hands over the other, so N values take about N + 6
// exchanges instead of 6 N (the 30 sums of a late Gram-Schmidt step cost more than the
// loads they follow otherwise).
template <int N>
__device__ __forceinline__ void wave_sums(const double* acc, int lane, double* dst)
{
    constexpr int P = pow2_at_least(N);
    static_assert(P <= 64, "one value per lane at most");
    double v[P];
#pragma unroll
    for (int j = 0; j < P; ++j) v[j] = j < N ? acc[j] : 0.0;
    int o = 32;
#pragma unroll
    for (int h = P / 2; h > 0; h /= 2, o /= 2) {
        const bool up = lane & o;
#pragma unroll
        for (int j = 0; j < h; ++j) {
            const double keep = up ? v[j + h] : v[j], send = up ? v[j] : v[j + h];
            v[j] = keep + __shfl_xor(send, o, 64);
        }
    }
    for (; o > 0; o /= 2) v[0] += __shfl_xor(v[0], o, 64);
    constexpr int L = 64 / P;  // lanes that hold the same sum
    if (lane % L == 0 && lane / L < N) dst[lane / L] = v[0];
}

// p[first] + p[first + step] + ... below n, eight loads in flight at a time
__device__ __forceinline__ double sum_strided(const double* p, unsigned first, unsigned step, unsigned n)
{
    double v = 0.0;
    for (unsigned b = first; b < n; b += 8 * step) {
        double t[8];
#pragma unroll
        for (unsigned q = 0; q < 8; ++q) {
            const unsigned at = b + q * step;
            t[q] = agent_load(p + (at < n ? at : b));
        }
#pragma unroll
        for (unsigned q = 0; q < 8; ++q) v += b + q * step < n ? t[q] : 0.0;
    }
    return v;
}

// Sums acc[NS] of every lane of the grid (whole workgroups of at most 512 lanes, all of
// whose lanes call this; workgroup blk of nblk) into s.out through s.fin.
template <int NS>
__device__ __forceinline__ void grid_sums(const double* acc, const Sums& s, unsigned blk, unsigned nblk)
{
    __shared__ double red[NS == 1 ? 8 : 4][NS];  // only single sums run in 512-lane workgroups
    __shared__ double sums[NS];
    __shared__ int last;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwv = blockDim.x >> 6;
    wave_sums<NS>(acc, lane, red[wave]);
    __syncthreads();
    if (wave == 0) {
        if (lane < NS) {
            double v = red[0][lane];
            for (int w = 1; w < nwv; ++w) v += red[w][lane];
            agent_store(s.partials + (long)lane * nblk + blk, v);
        }
        // the workgroup's partial sums are in memory before its arrival is counted
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) last = last_arrival(s.ticket, blk, nblk);
    }
    __syncthreads();
    if (!last) return;
    if constexpr (NS <= 3) {
        // few sums over possibly many workgroups: every lane takes part in each
        double v[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j)
            v[j] = sum_strided(s.partials + (long)j * nblk, threadIdx.x, blockDim.x, nblk);
        wave_sums<NS>(v, lane, red[wave]);
        __syncthreads();
        if (threadIdx.x < NS) {
            double t = red[0][threadIdx.x];
            for (int w = 1; w < nwv; ++w) t += red[w][threadIdx.x];
            sums[threadIdx.x] = t;
        }
    } else {
        // many sums: a wavefront each, side by side
        for (int j = wave; j < NS; j += nwv) {
            const double v = wave_sum(sum_strided(s.partials + (long)j * nblk, lane, 64, nblk));
            if (lane == 0) sums[j] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    scalar_program(sums, NS, s.out, s.fin, s.k);
    if (s.host)
        for (int j = 0; j < NS; ++j)
            __hip_atomic_store(s.host + j, sums[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// map over the runs of a field, a wavefront per run; F::NS doubles are summed over the grid
template <class F>
__global__ __launch_bounds__(256) void map_kernel(Runs runs, F f, Sums s)
{
    double acc[F::NS > 0 ? F::NS : 1];
#pragma unroll
    for (int k = 0; k < (F::NS > 0 ? F::NS : 1); ++k) acc[k] = 0.0;
    for (unsigned n = blockIdx.x * 4 + (threadIdx.x >> 6); n < runs.nw; n += gridDim.x * 4) {
        const Unit u = runs.unit(n);
        if (runs.holds(u)) f(u, acc);
    }
    if constexpr (F::NS > 0) grid_sums<F::NS>(acc, s, blockIdx.x, gridDim.x);
}

// Workgroups of a map: one run per wavefront until the machine is full (a small lattice then
// spreads over all CUs: 16^3 x 32 has 3072 workgroups' worth of runs), at most kMaxPartials;
// with many sums at most 512, two workgroups per CU, whose partial sums the last one reads
// with one batch of loads per sum.
template <int NS>
inline int map_blocks(unsigned nw)
{
    const unsigned cap = NS > 3 ? 512 : kMaxPartials, b = (nw + 3) / 4;
    return (int)(b < cap ? b : cap);
}

// launch F over op's lattice, or over its even half, and (if F::NS > 0) run the scalar
// program fin on its sums
template <class F>
int run_map(const qdw_op* op, const F& f, hipStream_t st, double* out = nullptr,
            int fin = FIN_STORE, int k = 0, bool even_half = false, bool back = false,
            double* host = nullptr)
{
    const Runs r = runs_of(op->g, even_half, back);
    const Sums s = {op->partials, op->tickets, out ? out : op->scalars, fin, k, host};
    map_kernel<F><<<map_blocks<F::NS>(r.nw), 256, 0, st>>>(r, f, s);
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

// ---------------------------------------------------------------- functors

template <int P>
struct Norm2 {
    static constexpr int NS = 1;
    const void* x;
    __device__ void operator()(const Unit& w, double* acc) const
    {
        cx<double> v[4];
        ld4<P, double>(x, w, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[0] += v[k].re * v[k].re + v[k].im * v[k].im;
    }
};

// y = a x + b y, a and b real host scalars (no reduction)
template <int PX, int PY>
struct Axpby {
    static constexpr int NS = 0;
    const void* x;
    void* y;
    double a, b;
    __device__ void operator()(const Unit& w, double*) const
    {
        using R = typename Traits<(PX == F64 && PY == F64) ? F64 : F32>::real;
        cx<R> vx[4], vy[4];
        ld4<PX, R>(x, w, vx);
        if (b != 0.0) ld4<PY, R>(y, w, vy);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            cx<R> t = scale(vx[k], (R)a);
            if (b != 0.0) t = t + scale(vy[k], (R)b);
            vy[k] = t;
        }
        st4<PY, R>(y, w, vy);
    }
};

// y = s x (down-conversion with scaling, one rounding)
template <int PX, int PY>
struct ScaleTo {
    static constexpr int NS = 0;
    const void* x;
    void* y;
    double s;
    __device__ void operator()(const Unit& w, double*) const
    {
        cx<double> v[4];
        ld4<PX, double>(x, w, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = scale(v[k], s);
        st4<PY, double>(y, w, v);
    }
};

// y = s x as above and |y|^2 of the stored values
template <int PX, int PY>
struct ScaleNorm {
    static constexpr int NS = 1;
    const void* x;
    void* y;
    double s;
    __device__ void operator()(const Unit& w, double* acc) const
    {
        cx<double> vx[4];
        ld4<PX, double>(x, w, vx);
        cx<double> vy[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) vy[k] = scale(vx[k], s);
        st4<PY, double>(y, w, vy);
        cx<double> back[4];
        ld4<PY, double>(y, w, back);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[0] += back[k].re * back[k].re + back[k].im * back[k].im;
    }
};

// p_next = r + beta p   (beta read from device scalars)
template <int P>
struct CgDirection {
    static constexpr int NS = 0;
    const void* r;
    const void* p;
    void* next;
    const double* sc;
    __device__ void operator()(const Unit& u, double*) const
    {
        using R = typename Traits<P>::real;
        const R b = (R)sc[S_BETA];
        cx<R> vr[4], vp[4];
        ld4<P, R>(r, u, vr);
        ld4<P, R>(p, u, vp);
#pragma unroll
        for (int k = 0; k < 4; ++k) vp[k] = vr[k] + scale(vp[k], b);
        st4<P, R>(next, u, vp);
    }
};

// x += sum of alpha_l p_l over the first n directions of the ring, one after the other; with
// TURN (a full ring) also p_0 = r + beta p_{n-1}, the next direction
template <int PX, int P, bool TURN>
struct CgMove {
    static constexpr int NS = 0;
    void* x;
    void* p[kRing];
    const void* r;
    const double* sc;
    int n;
    __device__ void operator()(const Unit& u, double*) const
    {
        using R = typename Traits<P>::real;
        cx<R> vx[4], vp[kRing][4], vr[4];
        ld4<PX, R>(x, u, vx);
#pragma unroll
        for (int l = 0; l < kRing; ++l)
            if (TURN || l < n) ld4<P, R>(p[l], u, vp[l]);
        if (TURN) ld4<P, R>(r, u, vr);
#pragma unroll
        for (int l = 0; l < kRing; ++l) {
            const R a = (R)sc[S_RING + l];
            // a zero or non-finite step length leaves the iterate as it was, so that a solve
            // that runs into a non-finite value still holds its last finite iterate
            if ((TURN || l < n) && a != (R)0 && isfinite(a)) {
#pragma unroll
                for (int k = 0; k < 4; ++k) vx[k] = vx[k] + scale(vp[l][k], a);
            }
        }
        st4<PX, R>(x, u, vx);
        if (TURN) {
            const R b = (R)sc[S_BETA];
#pragma unroll
            for (int k = 0; k < 4; ++k) vr[k] = vr[k] + scale(vp[kRing - 1][k], b);
            st4<P, R>(p[0], u, vr);
        }
    }
};

// r = eta - t ; |r|^2   (all FP64)
struct Residual {
    static constexpr int NS = 1;
    const void* eta;
    const void* t;
    void* r;
    __device__ void operator()(const Unit& u, double* acc) const
    {
        cx<double> ve[4], vt[4];
        ld4<F64, double>(eta, u, ve);
        ld4<F64, double>(t, u, vt);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            ve[k] = ve[k] - vt[k];
            acc[0] += ve[k].re * ve[k].re + ve[k].im * ve[k].im;
        }
        st4<F64, double>(r, u, ve);
    }
};

// x_hi += s x_lo ; x_lo = 0
template <int PL>
struct Accumulate {
    static constexpr int NS = 0;
    void* xhi;
    void* xlo;
    double s;
    __device__ void operator()(const Unit& u, double*) const
    {
        cx<double> vh[4], vl[4];
        ld4<F64, double>(xhi, u, vh);
        ld4<PL, double>(xlo, u, vl);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            vh[k] = vh[k] + scale(vl[k], s);
            vl[k] = {0.0, 0.0};
        }
        st4<F64, double>(xhi, u, vh);
        st4<PL, double>(xlo, u, vl);
    }
};

// x = 0
template <int P>
struct Zero {
    static constexpr int NS = 0;
    void* x;
    __device__ void operator()(const Unit& u, double*) const
    {
        cx<double> v[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
        st4<P, double>(x, u, v);
    }
};

// ---------------------------------------------------------------- host helpers

int dw_launch(qdw_op* op, const void* in, void* out, int prec, bool dag, hipStream_t st);
// the even-odd reduced operator on the even half of in (odd half of out: scratch)
int schur_launch(qdw_op* op, const void* in, void* out, int prec, bool dag, hipStream_t st);
// the two operator applications of a CG step with the step's sums and residual in them:
//   q = D p, |q|^2 -> alpha ;  r -= alpha D^+ q, |r|^2 -> beta
// (schur: the even-odd reduced operator; t is then the scratch its odd half needs; alpha is
// also kept at place `ring` of S_RING; host: where the host is to find |r|^2, or nullptr)
int cg_apply(qdw_op* op, const void* p, void* q, int prec, bool schur, int ring, hipStream_t st);
int cg_apply_dag(qdw_op* op, const void* q, void* r, void* t, int prec, bool schur, double* host,
                 hipStream_t st);

// run F and wait for its sums (also stored at `out`, by default the scratch scalars): the
// last workgroup writes them to the host block, so no copy follows the kernel (4 us and a
// launch gap each)
template <class F>
int run_sum(const qdw_op* op, const F& f, hipStream_t st, double* sums, bool even_half = false,
            double* out = nullptr)
{
    if (!out) out = op->scalars + S_TMP;
    const int rc = run_map(op, f, st, out, FIN_STORE, 0, even_half, false, op->host_dev);
    if (rc) return rc;
    if (!op->host_dev)
        QDW_HIP(hipMemcpyAsync(op->host_scalars, out, sizeof(double) * F::NS, hipMemcpyDeviceToHost, st));
    QDW_HIP(hipStreamSynchronize(st));
    for (int j = 0; j < F::NS; ++j) sums[j] = ((volatile double*)op->host_scalars)[j];
    return QDW_OK;
}

// read `n` device doubles at `src` (synchronises the stream)
inline int read_device(const qdw_op* op, const double* src, int n, double* out, hipStream_t st)
{
    QDW_CHECK(n >= 1 && n <= kHostScalars, QDW_EINVAL, "internal: read-back too large");
    QDW_HIP(hipMemcpyAsync(op->host_scalars, src, sizeof(double) * n, hipMemcpyDeviceToHost, st));
    QDW_HIP(hipStreamSynchronize(st));
    for (int k = 0; k < n; ++k) out[k] = op->host_scalars[k];
    return QDW_OK;
}

}  // namespace qdw
