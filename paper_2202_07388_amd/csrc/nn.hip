// nn.hip -- a learned gauge-covariant preconditioner for flexible GCR (not from the paper;
// the paper's solvers tolerate any preconditioner that changes from step to step).
//
// Network: three linear parallel-transport layers with 1 -> 8 -> 8 -> 1 spinor channels.
// A layer maps channels in_b to
//     out_a(x) = sum_{p=0..8} sum_b W_p[a][b] (T_p in_b)(x)
// with T_0 = 1, T_{+mu} v(x) = s U_mu(x) v(x+mu), T_{-mu} v(x) = s U_mu(x-mu)^+ v(x-mu)
// (s the fermion boundary sign) and W_p[a][b] a complex 4x4 matrix acting on spin only,
// so the network commutes with gauge transformations.
//
// GPU mapping of a layer: transports feed the channel mixing, the real product
// out[(x, c)][(a, s, re/im)] = A B with rows (site x, colour c), columns
// A[(x, c)][(p, b, t, re/im)] = (T_p in_b)(x) and B the real embedding of the complex
// weights, on the matrix cores: bf16 operands and FP32 accumulation. Backward: dA = G B^T and
// the adjoint transports give the input gradient, dB = A^T G the weight gradient (fixed-order
// sums). All of it runs in fused kernels that keep A and dA out of memory; the FP32-operand
// passes for gradient checks form them there. Adam updates FP32 master weights.
#include <cmath>
#include <type_traits>

#include "blas.h"
#include "dirac_core.h"

namespace qdw {

namespace {

constexpr int kPaths = 9;
constexpr int kLayers = 3;
constexpr int kCh[kLayers + 1] = {1, 8, 8, 1};
constexpr int kMaxK = 72 * 8;   // 9 paths x 8 channels x 4 spins x 2
constexpr int kMaxN = 64;       // 8 channels x 4 spins x 2

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// channel fields of a layer boundary, at a fixed distance in the workspace (passed by value:
// no pointer table to copy to the device, and its loads are known to be global ones)
struct Chan {
    char* base = nullptr;
    long stride = 0;
    __host__ __device__ __forceinline__ void* at(int c) const { return base + c * stride; }
};

inline int layer_K(int l) { return (kPaths * kCh[l] * 8 + 15) & ~15; }
inline int layer_N(int l) { return std::max(16, kCh[l + 1] * 8); }
inline int layer_w_offset(int l)  // in complex numbers
{
    int o = 0;
    for (int j = 0; j < l; ++j) o += kPaths * kCh[j] * kCh[j + 1] * 16;
    return o;
}
inline int total_weights() { return layer_w_offset(kLayers); }

inline long rows_of(const Geom& g) { return (long)2 * padded(g.Vh) * 3; }
inline long rows_padded(const Geom& g) { return (rows_of(g) + 63) & ~63L; }

// A and dA in panels of 8 columns: element (row m, column k) of a matrix with Mp rows
__device__ __forceinline__ long pidx(long Mp, long m, int k)
{
    return (((long)(k >> 3) * Mp + m) << 3) + (k & 7);
}

// two FP32 values rounded to bf16 (to nearest even, by the conversion instruction) and
// packed into one register, lo in the low half
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    const bf16x2_t b = __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t);
    uint32_t r;
    __builtin_memcpy(&r, &b, 4);
    return r;
}

// 8 consecutive values of one panel row
__device__ __forceinline__ void put8(float* A, long at, const float v[8])
{
    float4* d = (float4*)(A + at);
    d[0] = make_float4(v[0], v[1], v[2], v[3]);
    d[1] = make_float4(v[4], v[5], v[6], v[7]);
}

__device__ __forceinline__ uint16_t bf16_bits(float f) { return float_to_bf16(f); }

template <bool F32M>
__device__ __forceinline__ void put_el(void* A, long at, float v)
{
    if (F32M) ((float*)A)[at] = v;
    else ((uint16_t*)A)[at] = bf16_bits(v);
}

// one complex component (spin s, colour c) of an FP32 eo-SoA field at site (par, i)
__device__ __forceinline__ long f32_addr(int Vh, int par, int i, int s, int c)
{
    const int k12 = s * 3 + c;
    return chunk_at(Vh, 6, par, k12 >> 1, i) * 4 + (k12 & 1) * 2;
}

// ------------------------------------------------------------------ FP32-operand passes
//
// Gradient checks run with FP32 operands, through matrices in memory: A (transported rows),
// G (output gradients) and dA = G B^T. The bf16 passes never form them (fused layers below).
//
// A[(q, c)][((p*Cin + b)*4 + t)*2 + re/im] = (T_p in_b)(q)[t][c], q = par*Vp + i. Rows of
// padded sites and the padding columns K..Kpad-1 are written as zeros, so the matrix holds
// no stale values from earlier use of the workspace.
__global__ __launch_bounds__(256) void nn_transport_kernel(Geom g, int Cin, int Kpad, long Mp,
                                                           Chan in, float* A,
                                                           const void* links, const void* dets)
{
    const long tid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int Vp = padded(g.Vh);
    const long nq = 2L * Vp;
    if (tid >= nq * Cin) return;
    const int b = (int)(tid / nq);
    const long q = tid - (long)b * nq;
    const int par = (int)(q / Vp), i = (int)(q - (long)par * Vp);
    const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (b == Cin - 1)
        for (int kg = kPaths * Cin; kg < Kpad / 8; ++kg)
            for (int c = 0; c < 3; ++c) put8(A, pidx(Mp, q * 3 + c, kg * 8), zero);
    if (i >= g.Vh) {
        for (int p = 0; p < kPaths; ++p)
            for (int c = 0; c < 3; ++c) put8(A, pidx(Mp, q * 3 + c, (p * Cin + b) * 8), zero);
        return;
    }
    int x[4], lex;
    eo_coords(g, par, i, x, lex);
    const void* v = in.at(b);
    for (int p = 0; p < kPaths; ++p) {
        cx<float> s[12], w[12];
        if (p == 0) {
            load_spinor<F32>(v, g.Vh, par, i, s);
            for (int k = 0; k < 12; ++k) w[k] = s[k];
        } else {
            const int mu = (p - 1) >> 1;
            const bool fwd = ((p - 1) & 1) == 0;
            const int j = (fwd ? lex_fwd(g, x, lex, mu) : lex_bwd(g, x, lex, mu)) >> 1;
            load_spinor<F32>(v, g.Vh, 1 - par, j, s);
            cx<float> u[6], d;
            float sg = 1.f;
            if (fwd) {
                load_link<F32>(links, dets, g.Vh, par, i, mu, u, d);
                if (mu == 0 && x[0] == g.L[0] - 1) sg = (float)g.bc_t;
            } else {
                load_link<F32>(links, dets, g.Vh, 1 - par, j, mu, u, d);
                if (mu == 0 && x[0] == 0) sg = (float)g.bc_t;
            }
            // the SU(3) multiply of dirac_core acts on two spin components at a time
            cx<float> h[6], o[6];
            for (int half = 0; half < 2; ++half) {
                for (int k = 0; k < 6; ++k) h[k] = scale(s[6 * half + k], sg);
                if (fwd) su3_mul<float, false>(u, d, h, o);
                else su3_mul<float, true>(u, d, h, o);
                for (int k = 0; k < 6; ++k) w[6 * half + k] = o[k];
            }
        }
        // rows (q, c): 8 consecutive entries (t, re/im) of the (p, b) panel
        const int k0 = (p * Cin + b) * 8;
        for (int c = 0; c < 3; ++c) {
            float v[8];
            for (int t = 0; t < 4; ++t) {
                v[2 * t] = w[t * 3 + c].re;
                v[2 * t + 1] = w[t * 3 + c].im;
            }
            put8(A, pidx(Mp, q * 3 + c, k0), v);
        }
    }
}

// g_b(x) = sum_p T_p^+ dA[p][b](x): T_{+mu}^+ = T_{-mu}, T_{-mu}^+ = T_{+mu}
__global__ __launch_bounds__(256) void nn_transport_adj_kernel(Geom g, int Cin, long Mp,
                                                               const float* dA, Chan gout,
                                                               const void* links, const void* dets)
{
    const long tid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int Vp = padded(g.Vh);
    const long nq = 2L * Vp;
    if (tid >= nq * Cin) return;
    const int b = (int)(tid / nq);
    const long q = tid - (long)b * nq;
    const int par = (int)(q / Vp), i = (int)(q - (long)par * Vp);
    if (i >= g.Vh) return;
    int x[4], lex;
    eo_coords(g, par, i, x, lex);
    cx<float> acc[12];
    auto rows = [&](long qq, int p, cx<float> w[12]) {
        const int k0 = (p * Cin + b) * 8;
        for (int c = 0; c < 3; ++c) {
            const float4* r = (const float4*)(dA + pidx(Mp, qq * 3 + c, k0));
            const float4 lo = r[0], hi = r[1];
            w[c] = {lo.x, lo.y};
            w[3 + c] = {lo.z, lo.w};
            w[6 + c] = {hi.x, hi.y};
            w[9 + c] = {hi.z, hi.w};
        }
    };
    rows(q, 0, acc);
    for (int mu = 0; mu < 4; ++mu) {
        for (int dir = 0; dir < 2; ++dir) {
            // dir 0: the +mu path of site y = x - mu lands here through U_mu(y)^+
            // dir 1: the -mu path of site y = x + mu lands here through U_mu(x)
            const bool from_below = dir == 0;
            const int ylex = from_below ? lex_bwd(g, x, lex, mu) : lex_fwd(g, x, lex, mu);
            const long yq = (long)(1 - par) * Vp + (ylex >> 1);
            cx<float> w[12], u[6], d, h[6], o[6];
            rows(yq, from_below ? 1 + 2 * mu : 2 + 2 * mu, w);
            float sg = 1.f;
            if (from_below) {
                load_link<F32>(links, dets, g.Vh, 1 - par, ylex >> 1, mu, u, d);
                if (mu == 0 && x[0] == 0) sg = (float)g.bc_t;
            } else {
                load_link<F32>(links, dets, g.Vh, par, i, mu, u, d);
                if (mu == 0 && x[0] == g.L[0] - 1) sg = (float)g.bc_t;
            }
            for (int half = 0; half < 2; ++half) {
                for (int k = 0; k < 6; ++k) h[k] = scale(w[6 * half + k], sg);
                if (from_below) su3_mul<float, true>(u, d, h, o);
                else su3_mul<float, false>(u, d, h, o);
                for (int k = 0; k < 6; ++k) acc[6 * half + k] = acc[6 * half + k] + o[k];
            }
        }
    }
    store_spinor<F32>(gout.at(b), g.Vh, par, i, acc);
}

// ------------------------------------------------------------------ weights as matrices
//
// Real embedding of the complex weights, B[k][n] with k = ((p*Cin + b)*4 + t)*2 + ri,
// n = (a*4 + s)*2 + ro: B[(.., re)][(.., re)] = Re W, B[(.., im)][(.., re)] = -Im W,
// B[(.., re)][(.., im)] = Im W, B[(.., im)][(.., im)] = Re W, W = W_p[a][b][s][t].
// Stored transposed, Bt[n][k], for the forward GEMM, and as Bk[k][n] for dA = G B^T.
__device__ __forceinline__ float embed(const float* W, int Cin, int Cout, int k, int n)
{
    const int ri = k & 1, kk = k >> 1, t = kk & 3, pb = kk >> 2, b = pb % Cin, p = pb / Cin;
    const int ro = n & 1, nn = n >> 1, s = nn & 3, a = nn >> 2;
    if (a >= Cout || p >= kPaths) return 0.f;
    const long w = ((((long)p * Cout + a) * Cin + b) * 4 + s) * 4 + t;
    const float re = W[2 * w], im = W[2 * w + 1];
    if (ro == 0) return ri == 0 ? re : -im;
    return ri == 0 ? im : re;
}

// The same for every layer and form in one launch (blockIdx.y: 0..2 the layers; in bf16 also
// 3, the 8-channel layer as the fused kernel's LDS image -- for each path p the block of Bt
// (rows n < 64, columns k = 64 p + 0..63) as [k / 8][n][k % 8], so that a lane's eight
// consecutive k of one column n are one 16-byte read -- and 4, the last layer's path mixing
// Bm[n][k], n = (p*4 + s)*2 + re/im (72, padded to 80), k = (b*4 + t)*2 + re/im).
struct Embedded {
    void* Bt[kLayers];
    void* Bk[kLayers];
    uint16_t* Bl;
    uint16_t* Bm;
};

template <bool F32M>
__global__ void nn_embed_kernel(const float* W, Embedded E)
{
    const int tid = blockIdx.x * blockDim.x + threadIdx.x, job = blockIdx.y;
    const int off[kLayers] = {0, kPaths * kCh[0] * kCh[1] * 16, kPaths * (kCh[0] * kCh[1] + kCh[1] * kCh[2]) * 16};
    if (job < kLayers) {
        const int Cin = kCh[job], Cout = kCh[job + 1];
        const int Kpad = (kPaths * Cin * 8 + 15) & ~15, Npad = Cout * 8 < 16 ? 16 : Cout * 8;
        if (tid >= Kpad * Npad) return;
        const int n = tid / Kpad, k = tid - n * Kpad;
        const float v = (k < kPaths * Cin * 8) ? embed(W + 2 * off[job], Cin, Cout, k, n) : 0.f;
        put_el<F32M>(E.Bt[job], (long)n * Kpad + k, v);
        put_el<F32M>(E.Bk[job], (long)k * Npad + n, v);
    } else if (job == 3) {
        if (tid >= kPaths * 64 * 64) return;
        const int e = tid & 7, n = (tid >> 3) & 63, kq = (tid >> 9) & 7, p = tid >> 12;
        E.Bl[tid] = bf16_bits(embed(W + 2 * off[1], 8, 8, p * 64 + kq * 8 + e, n));
    } else {
        if (tid >= 80 * 64) return;
        const int n = tid / 64, k = tid - n * 64;
        float v = 0.f;
        if (n < 72) {
            const int p = n >> 3, sro = n & 7;            // (s, re/im) of the output
            const int b = k >> 3, tri = k & 7;            // (t, re/im) of the input
            v = embed(W + 2 * off[2], 8, 1, (p * 8 + b) * 8 + tri, sro);
        }
        E.Bm[tid] = bf16_bits(v);
    }
}

// ------------------------------------------------------------------ GEMMs on matrix cores

// acc[j] += A[m0 : m0+16][k0 : k0+4] * B[k0 : k0+4][16 j : 16 j + 16] for one wave; A
// row-major (element (m, k) at arow + k for this lane's row) or, with Mp > 0, in panels
__device__ __forceinline__ void mfma_step(const float* A, long arow, const float* Bt, long brow0,
                                          long bstride, int kofs, int nt, f4 acc[4], long Mp = 0,
                                          long row = 0)
{
    const float a = A[Mp > 0 ? pidx(Mp, row, kofs) : arow + kofs];
    for (int j = 0; j < nt; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Bt[brow0 + j * 16 * bstride + kofs], acc[j], 0, 0, 0);
}

// out channels (FP32 fields) = A Bt^T; a workgroup computes 64 rows, a wave 16 rows x Npad
__global__ __launch_bounds__(256) void nn_gemm_out_kernel(Geom g, int Kpad, int Npad, int Cout, long Mp,
                                                          const float* A, const float* Bt, Chan out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long m0 = (long)blockIdx.x * 64 + wave * 16;
    const int nt = Npad / 16;
    f4 acc[4];
    for (int j = 0; j < 4; ++j) acc[j] = f4{0.f, 0.f, 0.f, 0.f};
    const long row = m0 + (lane & 15);
    const long brow0 = (long)(lane & 15) * Kpad;
    for (int k0 = 0; k0 < Kpad; k0 += 4)
        mfma_step(A, 0, Bt, brow0, Kpad, k0 + (lane >> 4), nt, acc, Mp, row);
    const int Vp = padded(g.Vh);
    for (int j = 0; j < nt; ++j)
        for (int r = 0; r < 4; ++r) {
            const long m = m0 + 4 * (lane >> 4) + r;
            const int n = j * 16 + (lane & 15);
            const long q = m / 3;
            const int c = (int)(m - q * 3);
            const int a = n >> 3, s = (n >> 1) & 3, ri = n & 1;
            if (q >= 2L * Vp || a >= Cout) continue;
            const int par = (int)(q / Vp), i = (int)(q - (long)par * Vp);
            if (i >= g.Vh) continue;
            ((float*)out.at(a))[f32_addr(g.Vh, par, i, s, c) + ri] = acc[j][r];
        }
}

// dA[m][k] = sum_n G[m][n] Bk[k][n]  (G = gradient of the layer output, FP32 rows)
__global__ __launch_bounds__(256) void nn_gemm_da_kernel(int Kpad, int Npad, long Mp, const float* G,
                                                         const float* Bk, float* dA)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long m0 = (long)blockIdx.x * 64 + wave * 16;
    const long arow = (m0 + (lane & 15)) * Npad;
    for (int kt = 0; kt < Kpad / 16; kt += 4) {
        const int nt = std::min(4, Kpad / 16 - kt);
        f4 acc[4];
        for (int j = 0; j < 4; ++j) acc[j] = f4{0.f, 0.f, 0.f, 0.f};
        const long brow0 = (long)(kt * 16 + (lane & 15)) * Npad;
        for (int n0 = 0; n0 < Npad; n0 += 4)
            mfma_step(G, arow, Bk, brow0, Npad, n0 + (lane >> 4), nt, acc);
        for (int j = 0; j < nt; ++j)
            for (int r = 0; r < 4; ++r)
                dA[pidx(Mp, m0 + 4 * (lane >> 4) + r, (kt + j) * 16 + (lane & 15))] = acc[j][r];
    }
}

// partial dB[k][n] over a slice of rows: D[k][n] += sum_m A[m][k] G[m][n]
__global__ __launch_bounds__(256) void nn_gemm_db_kernel(long M, int Kpad, int Npad, int rows_per, long Mp,
                                                         const float* A, const float* G, float* part)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kt = blockIdx.x;     // 16 columns k of A
    const int split = blockIdx.y;  // slice of rows
    const int nt = Npad / 16;
    if (wave >= nt) return;
    const long mbeg = (long)split * rows_per;
    const long mend = std::min(M, mbeg + rows_per);
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
    const int kcol = kt * 16 + (lane & 15);
    const int ncol = wave * 16 + (lane & 15);
    for (long m = mbeg; m < mend; m += 4) {
        const long mm = m + (lane >> 4);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(A[pidx(Mp, mm, kcol)], G[mm * Npad + ncol], acc, 0, 0, 0);
    }
    for (int r = 0; r < 4; ++r) {
        const int k = kt * 16 + 4 * (lane >> 4) + r;
        part[((long)split * Kpad + k) * Npad + ncol] = acc[r];
    }
}

// G rows from a channel gradient (FP32 fields), times `scale`
__global__ __launch_bounds__(256) void nn_pack_g_kernel(Geom g, int Cout, int Npad, Chan gf, float scale,
                                                        float* G)
{
    const long tid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int Vp = padded(g.Vh);
    const long nq = 2L * Vp;
    if (tid >= nq) return;
    const int par = (int)(tid / Vp), i = (int)(tid - (long)par * Vp);
    for (int c = 0; c < 3; ++c)
        for (int n = 0; n < Npad; ++n) {
            const int a = n >> 3, s = (n >> 1) & 3, ri = n & 1;
            float v = 0.f;
            if (a < Cout && i < g.Vh) v = scale * ((const float*)gf.at(a))[f32_addr(g.Vh, par, i, s, c) + ri];
            G[(tid * 3 + c) * Npad + n] = v;
        }
}

// ------------------------------------------------------------------ fused forward layer
//
// The production forward pass (bf16 operands) fuses transport and mixing: a workgroup
// owns 64 consecutive sites q (192 rows (q, c)); for each batch of paths (one path when
// Cin = 8, all nine when Cin = 1) its lanes transport the input channels into the rows'
// columns for that batch, then the four wavefronts multiply them by the batch's rows of B
// on the matrix cores, 48 rows each, accumulating in FP32 -- with Cin = 1 through an LDS
// tile (the waves share the paths), with Cin = 8 straight from the registers the
// transports leave (each wave transports the 16 sites whose rows it multiplies). Columns
// are visited in the same order as by the unfused kernels, so both give the same sums; the
// difference is that A never goes to HBM. A lane always transports for the same site: its
// coordinates are computed once, and with Cin = 8 one link load serves the lane's two
// channels.

// neighbour index, boundary sign and link of path p (1..8) at site (par, i)
__device__ __forceinline__ void nn_path_setup(const Geom& g, int par, int i, const int x[4], int lex,
                                              int p, const void* links, const void* dets, int& j,
                                              float& sg, cx<float> u[6], cx<float>& d)
{
    const int mu = (p - 1) >> 1;
    const bool fwd = ((p - 1) & 1) == 0;
    j = (fwd ? lex_fwd(g, x, lex, mu) : lex_bwd(g, x, lex, mu)) >> 1;
    sg = 1.f;
    if (fwd) {
        load_link<F32>(links, dets, g.Vh, par, i, mu, u, d);
        if (mu == 0 && x[0] == g.L[0] - 1) sg = (float)g.bc_t;
    } else {
        load_link<F32>(links, dets, g.Vh, 1 - par, j, mu, u, d);
        if (mu == 0 && x[0] == 0) sg = (float)g.bc_t;
    }
}

// the 3x3 matrix s U of a path's link, its third row rebuilt once (s = +-1, so folding it
// into the matrix changes no rounding)
__device__ __forceinline__ void nn_link_matrix(const cx<float> u[6], cx<float> d, float sg,
                                               cx<float> m[9])
{
    m[6] = d * conj_(cmadd(u[1] * u[5], -u[2], u[4]));
    m[7] = d * conj_(cmadd(u[2] * u[3], -u[0], u[5]));
    m[8] = d * conj_(cmadd(u[0] * u[4], -u[1], u[3]));
#pragma unroll
    for (int k = 0; k < 6; ++k) m[k] = u[k];
#pragma unroll
    for (int k = 0; k < 9; ++k) m[k] = scale(m[k], sg);
}

// A path's link matrix as bf16 pairs for the dot-product instruction that multiplies two
// bf16 pairs and adds both products to an FP32 sum (v_dot2_f32_bf16): the hidden channels are
// stored as (re, im) bf16 pairs, so with a = (e.re, -e.im), b = (e.im, e.re) one complex
// product e v adds dot(a, v) to the real and dot(b, v) to the imaginary part -- two
// instructions instead of four FMAs, and no widening of the stored spinor. Entry r * 3 + k is
// the coefficient of v_k in w_r: M[r][k] for a forward path, conj(M[k][r]) for a backward one.
// The link is rounded to bf16 like the operands of the mixing that follows.
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
struct LinkBF {
    uint32_t a[9], b[9];
};

__device__ __forceinline__ void nn_link_bf16(bool fwd, const cx<float> m[9], LinkBF& L)
{
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const cx<float> e = fwd ? m[3 * r + k] : conj_(m[3 * k + r]);
            L.a[3 * r + k] = pack_bf16x2(e.re, -e.im);
            L.b[3 * r + k] = pack_bf16x2(e.im, e.re);
        }
}

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c)
{
    bf16x2v x, y;
    __builtin_memcpy(&x, &a, 4);
    __builtin_memcpy(&y, &b, 4);
    return __builtin_amdgcn_fdot2_f32_bf16(x, y, c, false);
}

// w = (M or M^+) v (ACC: w += ...) for the four spins of a spinor stored as 12 (re, im)
// bf16 pairs (three 16-byte chunks as loaded), FP32 sums
template <bool ACC = false>
__device__ __forceinline__ void nn_transport_dot2(const LinkBF& L, const u32x4 raw[3], cx<float> w[12])
{
    uint32_t v[12];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[4 * k] = raw[k].x;
        v[4 * k + 1] = raw[k].y;
        v[4 * k + 2] = raw[k].z;
        v[4 * k + 3] = raw[k].w;
    }
#pragma unroll
    for (int sd = 0; sd < 4; ++sd)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            float re = ACC ? w[3 * sd + r].re : 0.f, im = ACC ? w[3 * sd + r].im : 0.f;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                re = dot2_bf16(L.a[3 * r + k], v[3 * sd + k], re);
                im = dot2_bf16(L.b[3 * r + k], v[3 * sd + k], im);
            }
            w[3 * sd + r] = {re, im};
        }
}

// w = M sp (forward path) or M^+ sp (backward path) for the four spins
__device__ __forceinline__ void nn_apply_m(bool fwd, const cx<float> m[9], const cx<float> sp[12],
                                           cx<float> w[12])
{
#pragma unroll
    for (int sd = 0; sd < 4; ++sd) {
        const cx<float> h0 = sp[3 * sd], h1 = sp[3 * sd + 1], h2 = sp[3 * sd + 2];
#pragma unroll
        for (int r = 0; r < 3; ++r)
            w[3 * sd + r] = fwd ? cmadd(cmadd(m[3 * r] * h0, m[3 * r + 1], h1), m[3 * r + 2], h2)
                                : cmadd_conj(cmadd_conj(cmul_conj(m[r], h0), m[3 + r], h1),
                                             m[6 + r], h2);
    }
}

// one path's 64 x 64 block of the 8-channel layer's weights (bf16), as the fused kernel
// keeps it in LDS
constexpr int kWBlock = 64 * 64 * 2;
typedef __attribute__((address_space(1))) const u32x4 g_cu4;

// LDS row stride (in bf16 halves) of a tile with KB columns: at least KB + 8, rows 16-byte
// aligned, and a lane's three rows (the lane-to-lane step of the 16-byte row writes) 4 banks
// apart modulo the 64 banks, so the 64 lanes of a write hit every bank equally
constexpr int tile_stride(int kb)
{
    int ls = (kb + 8 + 7) / 8 * 8;
    while ((3 * ls / 2) % 64 != 4) ls += 8;
    return ls;
}

// first row q (site) of the 64-site block of this workgroup in the forward kernels, whose
// grid is one workgroup per block of either parity: blocks of the two parities alternate
// (the even and odd sites of one index range are lexicographic neighbours along x3), and
// each XCD takes one contiguous range of blocks, so that the neighbour windows a workgroup
// gathers were mostly loaded into its XCD's L2 by workgroups running beside it
__device__ __forceinline__ long nn_block_q0(int Vp)
{
    const int w = xcd_tile(blockIdx.x, gridDim.x);
    return (long)(w & 1) * Vp + (long)(w >> 1) * 64;
}

// the three rows (site sl, colour c) of one (path, channel) group, as bf16, into the tile
template <int LS>
__device__ __forceinline__ void nn_put_rows(uint16_t* tile, int sl, int k0, const cx<float> w[12])
{
    for (int c = 0; c < 3; ++c) {
        uint4 r;
        r.x = pack_bf16x2(w[c].re, w[c].im);
        r.y = pack_bf16x2(w[3 + c].re, w[3 + c].im);
        r.z = pack_bf16x2(w[6 + c].re, w[6 + c].im);
        r.w = pack_bf16x2(w[9 + c].re, w[9 + c].im);
        *(uint4*)&tile[(sl * 3 + c) * LS + k0] = r;
    }
}

// the same rows as the matrix-core operands of colours 0..2: (re, im) of spins 0..3 as bf16
// (the eight columns of one channel that a lane supplies for its site)
__device__ __forceinline__ void nn_rows(const cx<float> w[12], bf16x8 T[3])
{
    for (int c = 0; c < 3; ++c) {
        const uint32_t v[4] = {pack_bf16x2(w[c].re, w[c].im), pack_bf16x2(w[3 + c].re, w[3 + c].im),
                               pack_bf16x2(w[6 + c].re, w[6 + c].im), pack_bf16x2(w[9 + c].re, w[9 + c].im)};
        __builtin_memcpy(&T[c], v, 16);
    }
}

// the same straight from a spinor stored as bf16 pairs (the identity path)
__device__ __forceinline__ void nn_rows_raw(const u32x4 raw[3], bf16x8 T[3])
{
    uint32_t v[12];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[4 * k] = raw[k].x;
        v[4 * k + 1] = raw[k].y;
        v[4 * k + 2] = raw[k].z;
        v[4 * k + 3] = raw[k].w;
    }
    for (int c = 0; c < 3; ++c) {
        const uint32_t t[4] = {v[c], v[3 + c], v[6 + c], v[9 + c]};
        __builtin_memcpy(&T[c], t, 16);
    }
}

// MIXOUT (inference passes of the 8 -> 8 layer only): instead of storing the layer's eight
// output channels, the kernel goes on with the last layer's path mixing on them (the
// product nn_mix_paths_kernel forms, with the mixing matrix Bm) and stores the nine m_p
// fields to out[0..8]; its operand is the outputs rounded to bf16, as the stored hidden
// channels would be, taken from the registers that hold them, and the products sum over
// the same K steps in the same order (the forward pass's output at 32^3 x 64 was checked
// bit for bit against the two-kernel form).
// Occupancy: the one-channel layer is held to 128 registers, four waves per SIMD, where its
// gathers (two or three paths per wave, one after the other) hide behind the other waves
// (the compiler's own choice, 132, allows three); the eight-channel layers keep theirs.
template <int CIN, int COUT, int PIN, int POUT, bool MIXOUT = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CIN == 1 ? 4 : 1)))
void nn_layer_fused_kernel(Geom g, int Kpad, Chan in, const void* Bt, const void* Bl, Chan out,
                           const void* links, const void* dets, const uint16_t* Bm = nullptr)
{
    constexpr int PB = CIN == 1 ? kPaths : 1;          // paths per batch
    constexpr int KB = (PB * CIN * 8 + 15) & ~15;      // columns per batch (80 or 64)
    constexpr int LS = tile_stride(KB);                // LDS row stride (halves)
    constexpr int NT = COUT * 8 >= 16 ? COUT * 8 / 16 : 1;  // 16-column tiles of N
    static_assert(CIN == 1 || CIN == 8, "channel counts of the network");
    static_assert(CIN == 1 || (KB == 64 && NT == 4), "the LDS weight image is a 64 x 64 block");
    // LDS: Cin = 1, the transported tile of the batch; Cin = 8, two 8 KiB buffers for the
    // weight blocks of the current and the next path (its transports go to the matrix
    // cores from the registers); then the output block (COUT channels x 24 reals x 64
    // sites, bf16)
    constexpr int TILE_B = CIN == 1 ? 192 * LS * 2 : 0, W_B = CIN == 8 ? 2 * kWBlock : 0;
    // output staging in bf16: one row per (channel, 16-byte chunk) of 64 sites x 8 halves,
    // padded by one chunk so that consecutive rows start 4 banks apart
    static_assert(POUT == BF16S, "the layers' outputs are bf16 hidden channels");
    constexpr int OROW = 64 * 8 + 8;
    constexpr int OUT_B = (MIXOUT ? kPaths : COUT) * 3 * OROW * 2;
    static_assert(!MIXOUT || (CIN == 8 && COUT == 8), "the path mixing follows the 8 -> 8 layer");
    static_assert(TILE_B % 16 == 0, "weight blocks 16-byte aligned");
    __shared__ __attribute__((aligned(16))) char lds[TILE_B + W_B > OUT_B ? TILE_B + W_B : OUT_B];
    uint16_t* tile = (uint16_t*)lds;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Cin = 8: the weight block of path p is in buffer p & 1, as [k/8][n][k%8] (bf16)
    uint16_t* const wbuf = (uint16_t*)(lds + TILE_B);
    const uint16_t* wb = wbuf;
    // the site (0..63) and colour of output row 16 r + i (i < 16) of a wave's 48 rows:
    // Cin = 1, the tile's rows 3 site + colour; Cin = 8, colour-major (row tile r is colour
    // r of the wave's 16 sites), the order in which its transports reach the matrix cores
    auto row_site = [&](int r, int i, int& site, int& c) {
        if constexpr (CIN == 8) {
            site = wave * 16 + i;
            c = r;
        } else {
            const int m = wave * 48 + r * 16 + i;
            site = m / 3;
            c = m - site * 3;
        }
    };
    const int Vp = padded(g.Vh);
    const long q0 = nn_block_q0(Vp);
    // this lane's transport site: Cin = 8, the wave's own 16 sites, four lanes per site,
    // channels cg and cg + 4 per lane, so that a lane's transports are the very operand
    // registers it supplies to the wave's products (no LDS between them, and the workgroup
    // meets once per path only, for the shared weight block); Cin = 1, all 64 sites, paths
    // split over the waves
    const int sl = CIN == 8 ? wave * 16 + (lane & 15) : lane;
    const int cg = lane >> 4;
    const long qs = q0 + sl;
    const int par = (int)(qs / Vp), i = (int)(qs - (long)par * Vp);
    const bool real = i < g.Vh;
    int x[4] = {0, 0, 0, 0}, lex = 0;
    if (real) eo_coords(g, par, i, x, lex);
    const cx<float> zero12[12] = {};
    static_assert(CIN == 1 || PIN == BF16S, "hidden channels are stored in bf16");
    f4 acc[3][NT];
    for (int r = 0; r < 3; ++r)
        for (int j = 0; j < NT; ++j) acc[r][j] = f4{0.f, 0.f, 0.f, 0.f};
    // The products are formed transposed, B^T A^T (the weights as the first operand, the
    // transported rows as the second; the operand registers are the same as for A B):
    // acc[r][j] then holds, in lane l, output row 16 r + l % 16 of the wave's 48 and the
    // four columns 16 j + 4 (l / 16) + e, e = 0..3 -- the layout in which a 16x16x16
    // product takes its operands, so the last layer's mixing reads them from the
    // registers, and consecutive (re, im) columns pair up for 4-byte stores.
    // Cin = 1: rows 48*wave .. +48 of the tile times B[0 .. KB][0 .. 16 NT]
    auto mix_tile = [&]() {
        for (int kk = 0; kk < KB; kk += 16) {
            const int kl = kk + 4 * (lane >> 4);
            s4 bf[NT];
            for (int j = 0; j < NT; ++j)
                bf[j] = *(const s4*)((const uint16_t*)Bt + (long)(j * 16 + (lane & 15)) * Kpad + kl);
            for (int r = 0; r < 3; ++r) {
                const s4 a = *(const s4*)&tile[(wave * 48 + r * 16 + (lane & 15)) * LS + kl];
                for (int j = 0; j < NT; ++j)
                    acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bf[j], a, acc[r][j], 0, 0, 0);
            }
        }
    };
    if constexpr (CIN == 8) {
        // The inputs of one path for this lane -- the neighbour spinors of its two channels
        // as stored (bf16, widened when used), the link and the path's weight block -- are
        // loaded ahead of their use: the spinors two paths ahead (three stages), the link and
        // the weights one path ahead (two stages), so the gathered spinors have two paths'
        // transports and products to arrive in. Within one path the weights are issued
        // first, the link next and the spinors last: loads complete in issue order, so the
        // wait for the weights before the path's barrier leaves the link and spinor loads
        // in flight. The stages rotate by name (no indexed arrays).
        struct SpStage {
            u32x4 s0[3], s1[3];
        };
        struct LkStage {
            cx<float> u[6], d;
            float sg;
        };
        // the lane's two channel fields, accessed as global memory: loads through generic
        // pointers would be flat loads, which may complete out of order with the LDS
        // accesses, so that every wait in the path loop would become a wait for all loads in
        // flight, the prefetched ones included
        const g_cu4* const c0 = (const g_cu4*)in.at(cg);
        const g_cu4* const c1 = (const g_cu4*)in.at(cg + 4);
        // the spinors of path p: the lane's own site for p = 0, else the neighbour
        auto fetch_sp = [&](int p, SpStage& S) {
            int j = i, pp = par;
            if (p > 0) {
                const int mu = (p - 1) >> 1;
                j = ((((p - 1) & 1) == 0) ? lex_fwd(g, x, lex, mu) : lex_bwd(g, x, lex, mu)) >> 1;
                pp = 1 - par;
            }
            const long b0 = chunk_at(g.Vh, 3, pp, 0, j);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                S.s0[k] = c0[b0 + (long)k * kSB];
                S.s1[k] = c1[b0 + (long)k * kSB];
            }
        };
        // the link and boundary sign of path p (1..8)
        auto fetch_lk = [&](int p, LkStage& L) {
            int j;
            nn_path_setup(g, par, i, x, lex, p, links, dets, j, L.sg, L.u, L.d);
        };
        // the weight block of path p: each of the 256 lanes loads 32 contiguous bytes of it
        // and stores them into the block's LDS buffer once the path before it is done (one
        // workgroup barrier per path; the loads stay in registers meanwhile, in flight
        // during the transport and the matrix-core step)
        const int tid = threadIdx.x;
        auto load_w = [&](int p, u32x4 r[2]) {
            const g_cu4* src = (const g_cu4*)((const char*)Bl + (long)p * kWBlock) + 2 * tid;
            r[0] = src[0];
            r[1] = src[1];
        };
        auto store_w = [&](int p, const u32x4 r[2]) {
            u32x4* dst = (u32x4*)((char*)wbuf + (p & 1) * kWBlock) + 2 * tid;
            dst[0] = r[0];
            dst[1] = r[1];
        };
        // path p0 from the spinor stage sc and the link stage lc, while the weights and link
        // of path p0 + 1 and the spinors of path p0 + 2 are loaded; the wave writes and then
        // reads only its own rows of the tile, so a wave-level sync orders them. Every lane
        // issues the loads, the lanes of padded sites too (their site index is below the
        // padded row length and their neighbours are those of site 0, so the loads stay in
        // bounds; the data are not used): with the same loads in flight on every path
        // through the code, the compiler waits for exactly the loads an instruction needs
        auto path = [&](int p0, const SpStage& sc, SpStage& sn2, const LkStage& lc, LkStage& ln) {
            u32x4 wn[2];
            if (p0 + 1 < kPaths) {
                load_w(p0 + 1, wn);
                fetch_lk(p0 + 1, ln);
            }
            if (p0 + 2 < kPaths) fetch_sp(p0 + 2, sn2);
            // the matrix cores' second operand for row tile (colour) c: this lane's site,
            // channel cg (T0) or cg + 4 (T1), the four spins' (re, im) as bf16 -- exactly
            // the 8 consecutive columns of its row that a lane supplies in the product
            bf16x8 T0[3], T1[3];
            if (!real) {
                for (int c = 0; c < 3; ++c) T0[c] = T1[c] = bf16x8{};
            } else if (p0 == 0) {
                nn_rows_raw(sc.s0, T0);
                nn_rows_raw(sc.s1, T1);
            } else {
                const bool fwd = ((p0 - 1) & 1) == 0;
                cx<float> w[12], m[9];
                LinkBF lb;
                nn_link_matrix(lc.u, lc.d, lc.sg, m);
                nn_link_bf16(fwd, m, lb);
                nn_transport_dot2(lb, sc.s0, w);
                nn_rows(w, T0);
                nn_transport_dot2(lb, sc.s1, w);
                nn_rows(w, T1);
            }
            wb = wbuf + (p0 & 1) * (kWBlock / 2);
            // K = 64 per path in two steps of gfx950's doubled-K bf16 product (16 x 16 x 32),
            // channels 0..3 then 4..7; each lane reads 8 consecutive k of its column of the
            // path's weight block ([k/8][n][k%8] in LDS)
            for (int h = 0; h < 2; ++h) {
                const int kl = 32 * h + 8 * (lane >> 4);
                bf16x8 bf[NT];
                for (int j = 0; j < NT; ++j)
                    bf[j] = *(const bf16x8*)&wb[((kl >> 3) * 64 + j * 16 + (lane & 15)) * 8];
                for (int r = 0; r < 3; ++r)
                    for (int j = 0; j < NT; ++j)
                        acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j], h ? T1[r] : T0[r],
                                                                           acc[r][j], 0, 0, 0);
            }
            if (p0 + 1 < kPaths) {
                // the next block into the other buffer (last read by every wave before the
                // previous barrier); the barrier also keeps every wave's reads of this path's
                // block ahead of its rewrite at the end of the next path
                store_w(p0 + 1, wn);
                __syncthreads();
            }
        };
        SpStage S0, S1, S2;
        LkStage LA, LB;  // path 0 has no link: LA first holds path 2's
        {
            u32x4 w0[2];
            load_w(0, w0);
            fetch_sp(0, S0);
            fetch_sp(1, S1);
            store_w(0, w0);
        }
        __syncthreads();
        // unrolled, so that the stage of each path is fixed at compile time; the last
        // two paths issue fewer loads
#pragma unroll
        for (int p0 = 0; p0 < kPaths; ++p0) {
            const int r3 = p0 % 3;
            if (p0 & 1) {
                if (r3 == 0) path(p0, S0, S2, LB, LA);
                else if (r3 == 1) path(p0, S1, S0, LB, LA);
                else path(p0, S2, S1, LB, LA);
            } else {
                if (r3 == 0) path(p0, S0, S2, LA, LB);
                else if (r3 == 1) path(p0, S1, S0, LA, LB);
                else path(p0, S2, S1, LA, LB);
            }
        }
    } else {
        // paths wave, wave + 4, wave + 8 of the single channel, one batch
        for (int p = wave; p < kPaths; p += 4) {
            cx<float> w[12];
            if (!real) {
                nn_put_rows<LS>(tile, sl, p * 8, zero12);
                continue;
            }
            if (p == 0) {
                load_spinor<PIN>(in.base, g.Vh, par, i, w);
            } else {
                int j;
                float sg;
                cx<float> u[6], d, sp[12];
                nn_path_setup(g, par, i, x, lex, p, links, dets, j, sg, u, d);
                load_spinor<PIN>(in.base, g.Vh, 1 - par, j, sp);
                cx<float> m[9];
                nn_link_matrix(u, d, sg, m);
                nn_apply_m(((p - 1) & 1) == 0, m, sp, w);
            }
            nn_put_rows<LS>(tile, sl, p * 8, w);
        }
        // zero padding columns 72..79
        for (int rr = threadIdx.x; rr < 192; rr += 256)
            *(uint4*)&tile[rr * LS + kPaths * 8] = uint4{0u, 0u, 0u, 0u};
        __syncthreads();  // the waves filled each other's rows
        mix_tile();
    }
    __syncthreads();  // the output block below reuses the tile
    if constexpr (MIXOUT) {
        // m_p = the layer's outputs rounded to bf16 (as the stored hidden channels would be)
        // times Bm, K = 64 in four steps of 16: step j takes the lane's acc[r][j] as its
        // operand, again as the transposed product (Bm^T first), so am[r][jm] holds row
        // 16 r + l % 16 and columns 16 jm + 4 (l / 16) + e of m, column (p * 4 + s) * 2 + re/im
        constexpr int NM = 5;  // 80 columns: 9 paths x 4 spins x re/im (72), padded
        f4 am[3][NM];
        for (int r = 0; r < 3; ++r)
            for (int jm = 0; jm < NM; ++jm) am[r][jm] = f4{0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < NT; ++j) {
            const int kl = j * 16 + 4 * (lane >> 4);
            s4 bf[NM];
            for (int jm = 0; jm < NM; ++jm)
                bf[jm] = *(const s4*)(Bm + (jm * 16 + (lane & 15)) * 64 + kl);
            for (int r = 0; r < 3; ++r) {
                const uint32_t h2[2] = {pack_bf16x2(acc[r][j][0], acc[r][j][1]),
                                        pack_bf16x2(acc[r][j][2], acc[r][j][3])};
                s4 a;
                __builtin_memcpy(&a, h2, 8);
                for (int jm = 0; jm < NM; ++jm)
                    am[r][jm] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bf[jm], a, am[r][jm], 0, 0, 0);
            }
        }
        // staged as [path][chunk][site][8] like the outputs below, (re, im) pairs as one word
        uint16_t* ob = (uint16_t*)lds;
        for (int r = 0; r < 3; ++r)
            for (int jm = 0; jm < NM; ++jm)
                for (int h = 0; h < 2; ++h) {
                    int ms, c;
                    row_site(r, lane & 15, ms, c);
                    const int n = jm * 16 + 4 * (lane >> 4) + 2 * h;
                    if (n >= 72) continue;
                    const int p = n >> 3, sp = (n >> 1) & 3;
                    const int k = (sp * 3 + c) * 2;
                    *(uint32_t*)&ob[(p * 3 + (k >> 3)) * OROW + ms * 8 + (k & 7)] =
                        pack_bf16x2(am[r][jm][2 * h], am[r][jm][2 * h + 1]);
                }
        __syncthreads();
        const int mpar = (int)(q0 / Vp), mi0 = (int)(q0 - (long)mpar * Vp);
        for (int u = threadIdx.x; u < kPaths * 3 * 64; u += 256) {
            const int p = u / 192, rem = u - p * 192, ch = rem >> 6, site = rem & 63;
            if (mi0 + site >= g.Vh) continue;
            const uint4 raw = *(const uint4*)&ob[(p * 3 + ch) * OROW + site * 8];
            ((uint4*)out.at(p))[chunk_at(g.Vh, 3, mpar, ch, mi0 + site)] = raw;
        }
        return;
    }
    // outputs: row m = 3 * site + c, column n = (a * 4 + s) * 2 + re/im, rounded to bf16
    // (the conversion instruction) and staged in LDS as [channel][chunk][site][8] (the 64
    // sites are one aligned block of one parity; rows padded as in the tile), then written
    // as 16-byte chunks
    uint16_t* ob = (uint16_t*)lds;
    for (int r = 0; r < 3; ++r)
        for (int j = 0; j < NT; ++j)
            for (int h = 0; h < 2; ++h) {
                int ms, c;
                row_site(r, lane & 15, ms, c);
                const int n = j * 16 + 4 * (lane >> 4) + 2 * h;
                const int a = n >> 3, sp = (n >> 1) & 3;
                if (a >= COUT) continue;
                const int k = (sp * 3 + c) * 2;  // real index of the pair within the spinor
                *(uint32_t*)&ob[(a * 3 + (k >> 3)) * OROW + ms * 8 + (k & 7)] =
                    pack_bf16x2(acc[r][j][2 * h], acc[r][j][2 * h + 1]);
            }
    __syncthreads();
    const int opar = (int)(q0 / Vp), oi0 = (int)(q0 - (long)opar * Vp);
    for (int u = threadIdx.x; u < COUT * 3 * 64; u += 256) {
        const int a = u / 192, rem = u - a * 192, ch = rem >> 6, site = rem & 63;
        if (oi0 + site >= g.Vh) continue;
        const uint4 raw = *(const uint4*)&ob[(a * 3 + ch) * OROW + site * 8];
        ((uint4*)out.at(a))[chunk_at(g.Vh, 3, opar, ch, oi0 + site)] = raw;
    }
}

// ------------------------------------------------------------------ last layer: mix, then transport
//
// With one output channel the order of the two linear maps of a layer pays to be swapped:
// W_p acts on spin and channel, T_p on colour and site, so
//     out(x) = sum_p sum_b W_p[0][b] (T_p in_b)(x) = sum_p (T_p m_p)(x),
//     m_p(y) = sum_b W_p[0][b] in_b(y).
// Pass 1 forms the nine m_p at every site on the matrix cores (rows (site, colour), K = 8
// channels x 4 spins x re/im, N = 9 paths x 4 spins x re/im), storing them in bf16; pass 2
// is a plain stencil over them. Each site then gathers 9 spinors instead of 72.

__global__ __launch_bounds__(256) void nn_mix_paths_kernel(Geom g, Chan in, const uint16_t* Bm,
                                                           Chan mix)
{
    constexpr int KB = 64, LS = tile_stride(KB), NT = 5;
    // output staging in bf16: one row per (path, 16-byte chunk) of 64 sites x 8 halves,
    // padded by one chunk so that consecutive rows start 4 banks apart
    constexpr int ROW = 64 * 8 + 8;
    constexpr int TILE_B = 192 * LS * 2, OUT_B = 9 * 3 * ROW * 2;
    __shared__ __attribute__((aligned(16))) char lds[TILE_B > OUT_B ? TILE_B : OUT_B];
    uint16_t* tile = (uint16_t*)lds;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int Vp = padded(g.Vh);
    const long q0 = nn_block_q0(Vp);
    const int par = (int)(q0 / Vp), i0 = (int)(q0 - (long)par * Vp);
    const int i = i0 + lane;
    const cx<float> zero12[12] = {};
    // rows of the tile: the site's eight input channels (channels wave and wave + 4)
    if (i < g.Vh) {
        cx<float> w0[12], w1[12];
        load_spinor<BF16S>(in.at(wave), g.Vh, par, i, w0);
        load_spinor<BF16S>(in.at(wave + 4), g.Vh, par, i, w1);
        nn_put_rows<LS>(tile, lane, wave * 8, w0);
        nn_put_rows<LS>(tile, lane, (wave + 4) * 8, w1);
    } else {
        nn_put_rows<LS>(tile, lane, wave * 8, zero12);
        nn_put_rows<LS>(tile, lane, (wave + 4) * 8, zero12);
    }
    __syncthreads();
    f4 acc[3][NT];
    for (int r = 0; r < 3; ++r)
        for (int j = 0; j < NT; ++j) acc[r][j] = f4{0.f, 0.f, 0.f, 0.f};
    for (int kk = 0; kk < KB; kk += 16) {
        const int kl = kk + 4 * (lane >> 4);
        s4 bf[NT];
        for (int j = 0; j < NT; ++j)
            bf[j] = *(const s4*)(Bm + (j * 16 + (lane & 15)) * KB + kl);
        for (int r = 0; r < 3; ++r) {
            const s4 a = *(const s4*)&tile[(wave * 48 + r * 16 + (lane & 15)) * LS + kl];
            for (int j = 0; j < NT; ++j)
                acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bf[j], acc[r][j], 0, 0, 0);
        }
    }
    __syncthreads();
    // outputs rounded to bf16 (the conversion instruction, as for the other bf16 fields)
    // and staged as [path][chunk][site][8], then written as 16-byte chunks
    uint16_t* ob = (uint16_t*)lds;
    for (int r = 0; r < 3; ++r)
        for (int j = 0; j < NT; ++j)
            for (int e = 0; e < 4; ++e) {
                const int m = wave * 48 + r * 16 + 4 * (lane >> 4) + e;
                const int n = j * 16 + (lane & 15);
                if (n >= 72) continue;
                const int ms = m / 3, c = m - ms * 3;
                const int p = n >> 3, sp = (n >> 1) & 3, ri = n & 1;
                const int k = (sp * 3 + c) * 2 + ri;  // real index within the spinor
                ob[(p * 3 + (k >> 3)) * ROW + ms * 8 + (k & 7)] =
                    (uint16_t)(pack_bf16x2(acc[r][j][e], 0.f) & 0xFFFFu);
            }
    __syncthreads();
    for (int u = threadIdx.x; u < 9 * 3 * 64; u += 256) {
        const int p = u / 192, rem = u - p * 192, ch = rem >> 6, site = rem & 63;
        if (i0 + site >= g.Vh) continue;
        const uint4 raw = *(const uint4*)&ob[(p * 3 + ch) * ROW + site * 8];
        ((uint4*)mix.at(p))[chunk_at(g.Vh, 3, par, ch, i0 + site)] = raw;
    }
}

// out(x) = a (m_0(x) + sum_{p = 1..8} (T_p m_p)(x)), formed in FP32 and stored as FP32 or, for
// a caller's FP64 field, as the FP64 of that (no second pass to convert it)
template <int POUT>
__global__ __launch_bounds__(256) void nn_transport_sum_kernel(Geom g, Chan mix, void* out, float a,
                                                               const void* links, const void* dets)
{
    // 256-site blocks of the two parities alternate, XCD-contiguously (as nn_block_q0)
    const int w = xcd_tile(blockIdx.x, gridDim.x);
    const int par = w & 1;
    const int i = (w >> 1) * 256 + (int)threadIdx.x;
    if (i >= g.Vh) return;
    int x[4], lex;
    eo_coords(g, par, i, x, lex);
    cx<float> acc[12];
    load_spinor<BF16S>(mix.base, g.Vh, par, i, acc);
#pragma unroll 1
    for (int p = 1; p < kPaths; ++p) {
        int j;
        float sg;
        cx<float> u[6], d;
        nn_path_setup(g, par, i, x, lex, p, links, dets, j, sg, u, d);
        u32x4 raw[3];
        const long b0 = chunk_at(g.Vh, 3, 1 - par, 0, j);
#pragma unroll
        for (int k = 0; k < 3; ++k) raw[k] = ((const u32x4*)mix.at(p))[b0 + (long)k * kSB];
        cx<float> m[9];
        LinkBF lb;
        nn_link_matrix(u, d, sg, m);
        nn_link_bf16(((p - 1) & 1) == 0, m, lb);
        nn_transport_dot2<true>(lb, raw, acc);
    }
    cx<typename Traits<POUT>::real> o[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const cx<float> v = scale(acc[k], a);
        o[k] = {v.re, v.im};
    }
    store_spinor<POUT>(out, g.Vh, par, i, o);
}

// ------------------------------------------------------------------ fused backward layer
//
// The bf16 backward pass of a layer out_a = sum_p sum_b W_p[a][b] T_p in_b, without the
// matrices of transported rows and of their gradients in memory (A and dA, 1152 and 2304
// times 3 bytes per site for eight channels, each written and read once). G, the gradient of
// the layer's outputs, is a set of bf16 fields: the operand precision of the products.
//
// Input gradient: dA_p[b](y) = sum_a W_p[a][b]^+ G_a(y) is used at one site only, the one
// that T_p takes to y, so the workgroup that forms dx(x) = sum_p T_p^+ dA_p at 64 sites
// gathers G at the eight neighbours and the sites themselves, multiplies on the matrix
// cores and transports the FP32 products from the registers that hold them. The products
// are formed transposed (weights first), the 16 sites of a wave in the columns and the
// colours in the three row tiles, so a lane ends up with two spins and all colours of one
// channel: what one link multiplies. It supplies the same two spins of channels
// 2 step + lane / 32 of G, 24 contiguous bytes of a stored spinor.

// the half spinor (two spins) of G that a lane supplies in one product step, as stored
struct HalfRaw {
    u32x4 a;
    uint2 b;
};

template <int CIN, int COUT, int POUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(COUT == 8 && CIN == 8 ? 1 : 2)))
void nn_dx_kernel(Geom g, Chan G, const uint16_t* Bk, Chan out, const void* links, const void* dets)
{
    constexpr int NP = COUT * 8 < 16 ? 16 : COUT * 8;  // columns n of G (zero from COUT * 8)
    constexpr int KS = NP / 16;                        // product steps
    constexpr int NJ = CIN == 8 ? 4 : 1;               // 16-column tiles of a path's inputs
    constexpr int JH = CIN == 8 ? 2 : 1;               // tiles multiplied at a time (registers)
    constexpr int LS = NP + 8;                         // LDS row of weights (halves)
    constexpr int WQ = NJ * 16 * NP * 2 / 16;          // 16-byte pieces of a path's weights
    __shared__ __attribute__((aligned(16))) uint16_t wb[2][NJ * 16 * LS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tid = threadIdx.x;
    const int qd = lane >> 4, hf = qd & 1;
    const int Vp = padded(g.Vh);
    const long q0 = nn_block_q0(Vp), qs = q0 + wave * 16 + (lane & 15);
    const int par = (int)(qs / Vp), i = (int)(qs - (long)par * Vp);
    const bool real = i < g.Vh;
    int x[4] = {0, 0, 0, 0}, lex = 0;
    if (real) eo_coords(g, par, i, x, lex);

    // The weights of path p: rows k of Bk from p * CIN * 8, in pieces of 16 bytes, loaded one
    // path ahead and stored after the path before is done (as the forward layer does)
    constexpr int WL = (WQ + 255) / 256;
    auto load_w = [&](int p, u32x4 r[WL]) {
        const g_cu4* src = (const g_cu4*)(Bk + (long)p * CIN * 8 * NP);
#pragma unroll
        for (int k = 0; k < WL; ++k)
            if (WQ % 256 == 0 || tid + 256 * k < WQ) r[k] = src[tid + 256 * k];
    };
    auto store_w = [&](int buf, const u32x4 r[WL]) {
#pragma unroll
        for (int k = 0; k < WL; ++k) {
            const int at = tid + 256 * k, row = at / (NP / 8), col = at % (NP / 8);
            if (WQ % 256 == 0 || at < WQ) *(u32x4*)&wb[buf][row * LS + col * 8] = r[k];
        }
    };
    // Paths 1 + 2 mu come from the site below (BELOW), paths 2 + 2 mu from the one above; the
    // loop over mu keeps its indices opaque, as the D kernels do, so that the addresses of all
    // nine paths are not formed at once and held. Padded lanes load the neighbours of site 0,
    // in bounds and not used.
    auto neighbour = [&](bool below, int mu, const int xx[4], int ll) {
        const int xm = mu == 0 ? xx[0] : mu == 1 ? xx[1] : mu == 2 ? xx[2] : xx[3];
        const int wrap = (g.L[mu] - 1) * g.stride[mu];
        return (below ? (xm == 0 ? ll + wrap : ll - g.stride[mu])
                      : (xm == g.L[mu] - 1 ? ll - wrap : ll + g.stride[mu])) >> 1;
    };
    auto load_g = [&](int pp, int j, HalfRaw r[KS]) {
        const long b0 = chunk_at(g.Vh, 3, pp, 0, j);
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            if (COUT == 1 && qd >= 2) {
                r[k].a = u32x4{0u, 0u, 0u, 0u};
                r[k].b = uint2{0u, 0u};
                continue;
            }
            const char* f = (const char*)G.at(2 * k + (qd >> 1));
            r[k].a = ((const g_cu4*)f)[b0 + (hf ? 2 * kSB : 0)];
            const __attribute__((address_space(1))) uint32_t* h =
                (const __attribute__((address_space(1))) uint32_t*)f + (b0 + kSB) * 4 + 2 * hf;
            r[k].b = uint2{h[0], h[1]};
        }
    };
    struct Lk {
        cx<float> u[6], d;
        float sg;
    };
    // G and the link of the path from below / above in direction mu
    auto fetch = [&](bool below, int mu, HalfRaw r[KS], Lk& L) {
        int ii = i, ll = lex, xx[4] = {x[0], x[1], x[2], x[3]};
        asm volatile("" : "+v"(ii), "+v"(ll), "+v"(xx[0]), "+v"(xx[1]), "+v"(xx[2]), "+v"(xx[3]));
        const int j = neighbour(below, mu, xx, ll);
        load_link<F32>(links, dets, g.Vh, below ? 1 - par : par, below ? j : ii, mu, L.u, L.d);
        L.sg = mu == 0 && xx[0] == (below ? 0 : g.L[0] - 1) ? (float)g.bc_t : 1.f;
        load_g(1 - par, j, r);
    };
    cx<float> dx[NJ][6];
    // tiles j0 .. j0 + JH of the products of one path, dA in acc, from weight buffer `buf`
    auto products = [&](int buf, const HalfRaw gc[KS], int j0, f4 acc[3][JH]) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int j = 0; j < JH; ++j) acc[c][j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            // words (spin, colour) of the half spinor: the lower half starts with the 16-byte
            // piece, the upper half with the 8-byte one
            const uint32_t A[4] = {gc[k].a.x, gc[k].a.y, gc[k].a.z, gc[k].a.w};
            const uint32_t v[6] = {hf ? gc[k].b.x : A[0], hf ? gc[k].b.y : A[1], hf ? A[0] : A[2],
                                   hf ? A[1] : A[3], hf ? A[2] : gc[k].b.x, hf ? A[3] : gc[k].b.y};
            s4 w[JH];
#pragma unroll
            for (int j = 0; j < JH; ++j)
                w[j] = *(const s4*)&wb[buf][((j0 + j) * 16 + (lane & 15)) * LS + k * 16 + 4 * qd];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const uint32_t t[2] = {v[c], v[3 + c]};
                s4 b;
                __builtin_memcpy(&b, t, 8);
#pragma unroll
                for (int j = 0; j < JH; ++j)
                    acc[c][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[j], b, acc[c][j], 0, 0, 0);
            }
        }
    };
    auto half = [&](const f4 acc[3][JH], int j, cx<float> h[6]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            h[c] = {acc[c][j][0], acc[c][j][1]};
            h[3 + c] = {acc[c][j][2], acc[c][j][3]};
        }
    };
    // dx += T_p^+ dA_p
    auto path = [&](auto below_c, int buf, const HalfRaw gc[KS], const Lk& L) {
        constexpr bool BELOW = decltype(below_c)::value;
#pragma unroll
        for (int j0 = 0; j0 < NJ; j0 += JH) {
            f4 acc[3][JH];
            products(buf, gc, j0, acc);
#pragma unroll
            for (int j = 0; j < JH; ++j) {
                cx<float> h[6], o[6];
                half(acc, j, h);
#pragma unroll
                for (int k = 0; k < 6; ++k) h[k] = scale(h[k], L.sg);
                su3_mul<float, BELOW>(L.u, L.d, h, o);
#pragma unroll
                for (int k = 0; k < 6; ++k) dx[j0 + j][k] = dx[j0 + j][k] + o[k];
            }
            __builtin_amdgcn_sched_barrier(0);  // one half's registers at a time
        }
    };
    HalfRaw ga[KS], gb[KS];
    Lk la, lb;
    u32x4 w[WL];
    load_w(0, w);
    load_g(par, i, gb);
    store_w(0, w);
    __syncthreads();
    {
        load_w(1, w);
        fetch(true, 0, ga, la);
#pragma unroll
        for (int j0 = 0; j0 < NJ; j0 += JH) {
            f4 acc[3][JH];
            products(0, gb, j0, acc);
#pragma unroll
            for (int j = 0; j < JH; ++j) half(acc, j, dx[j0 + j]);
        }
        store_w(1, w);
        __syncthreads();
    }
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
        load_w(2 + 2 * mu, w);
        fetch(false, mu, gb, lb);
        path(std::true_type{}, 1, ga, la);
        store_w(0, w);
        __syncthreads();
        if (mu < 3) {
            load_w(3 + 2 * mu, w);
            fetch(true, mu + 1, ga, la);
        }
        path(std::false_type{}, 0, gb, lb);
        if (mu < 3) {
            store_w(1, w);
            __syncthreads();
        }
    }
    if (!real) return;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (CIN == 1 && qd >= 2) continue;  // columns of the next path
        void* f = out.at(CIN == 1 ? 0 : 2 * j + (qd >> 1));
        if constexpr (POUT == F32) {
            const long b0 = chunk_at(g.Vh, 6, par, 0, i);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                ((float4*)f)[b0 + (long)(3 * hf + k) * kSB] =
                    make_float4(dx[j][2 * k].re, dx[j][2 * k].im, dx[j][2 * k + 1].re, dx[j][2 * k + 1].im);
        } else {
            const long b0 = chunk_at(g.Vh, 3, par, 0, i);
            uint32_t v[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) v[k] = pack_bf16x2(dx[j][k].re, dx[j][k].im);
            uint32_t* mid = (uint32_t*)f + (b0 + kSB) * 4;
            if (hf) {
                *(uint2*)(mid + 2) = uint2{v[0], v[1]};
                ((uint4*)f)[b0 + 2 * kSB] = uint4{v[2], v[3], v[4], v[5]};
            } else {
                ((uint4*)f)[b0] = uint4{v[0], v[1], v[2], v[3]};
                *(uint2*)mid = uint2{v[4], v[5]};
            }
        }
    }
}

// Weight gradient: partial dB[k][n] = sum_m A[m][k] G[m][n] over the rows m = (site, colour)
// of a share of the 64-site blocks. A workgroup owns one path of the eight channels (or the
// whole one-channel layer), transports a block's inputs as the forward pass of these
// gradients does (FP32, rounded to bf16 once), leaves A and G transposed in LDS, row index
// fastest and colour-major, and multiplies on the matrix cores with FP32 accumulators in
// registers for its whole share. A never goes to memory; G is read once per path, mostly
// from L2 (the nine paths of a share run side by side).
template <int CIN, int COUT, int PIN>
__global__ __launch_bounds__(256)
void nn_dw_partial_kernel(Geom g, Chan in, Chan G, const void* links, const void* dets, int nsplit,
                          float* part)
{
    constexpr int KB = CIN == 8 ? 64 : 80;             // columns k of this workgroup
    constexpr int KPAD = (kPaths * CIN * 8 + 15) & ~15;
    constexpr int NP = COUT * 8 < 16 ? 16 : COUT * 8;
    constexpr int LS = 192 + 8;                        // LDS row (halves): 4 banks apart
    constexpr int NI = CIN == 8 ? 2 : 3;               // transports of a lane per block
    constexpr int NG = COUT == 8 ? 2 : 1;              // output channels a lane loads
    constexpr int KT = KB / 16;
    constexpr int MT = COUT == 8 ? KT : 1;             // accumulator tiles of a wave
    static_assert(COUT == 8 || CIN == 8, "the one-output layer has eight inputs");
    __shared__ __attribute__((aligned(16))) uint16_t At[KB * LS], Gt[NP * LS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wg = xcd_tile(blockIdx.x, gridDim.x);  // the paths of a share on one XCD
    const int path0 = CIN == 8 ? wg % kPaths : 0;
    const int split = CIN == 8 ? wg / kPaths : wg;
    const int Vp = padded(g.Vh), nblk = 2 * Vp / 64;
    // rows of LDS that no block writes: the padding columns
    for (int k = threadIdx.x; k < (KB - (CIN == 8 ? 64 : 72)) * LS; k += 256) At[72 * LS + k] = 0;
    for (int k = threadIdx.x; k < (NP - COUT * 8) * LS; k += 256) Gt[COUT * 8 * LS + k] = 0;
    f4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};

    // one word (re, im) of row (site = lane, colour c), columns k and k + 1
    auto put = [&](uint16_t* T, int k, int c, uint32_t v) {
        T[k * LS + c * 64 + lane] = (uint16_t)(v & 0xFFFFu);
        T[(k + 1) * LS + c * 64 + lane] = (uint16_t)(v >> 16);
    };
    for (int blk = split; blk < nblk; blk += nsplit) {
        // the two parities of one index range follow each other
        const int par = blk & 1, i = (blk >> 1) * 64 + lane;
        const bool real = i < g.Vh;
        int x[4] = {0, 0, 0, 0}, lex = 0;
        if (real) eo_coords(g, par, i, x, lex);
        u32x4 gr[NG][3];
#pragma unroll
        for (int n = 0; n < NG; ++n) {
            const long b0 = chunk_at(g.Vh, 3, par, 0, i);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                gr[n][k] = COUT == 8 || wave == 0 ? ((const g_cu4*)G.at(COUT == 8 ? wave + 4 * n : 0))[b0 + (long)k * kSB]
                                                  : u32x4{0u, 0u, 0u, 0u};
        }
        auto transport = [&](int p, int b, int k0) {
            cx<float> s[12], w[12];
            if (!real) {
#pragma unroll
                for (int k = 0; k < 12; ++k) w[k] = {0.f, 0.f};
            } else if (p == 0) {
                load_spinor<PIN>(in.at(b), g.Vh, par, i, w);
            } else {
                const int mu = (p - 1) >> 1;
                const bool fwd = ((p - 1) & 1) == 0;
                const int j = (fwd ? lex_fwd(g, x, lex, mu) : lex_bwd(g, x, lex, mu)) >> 1;
                load_spinor<PIN>(in.at(b), g.Vh, 1 - par, j, s);
                cx<float> u[6], d, h[6], o[6];
                float sg = 1.f;
                if (fwd) {
                    load_link<F32>(links, dets, g.Vh, par, i, mu, u, d);
                    if (mu == 0 && x[0] == g.L[0] - 1) sg = (float)g.bc_t;
                } else {
                    load_link<F32>(links, dets, g.Vh, 1 - par, j, mu, u, d);
                    if (mu == 0 && x[0] == 0) sg = (float)g.bc_t;
                }
#pragma unroll
                for (int half = 0; half < 2; ++half) {
#pragma unroll
                    for (int k = 0; k < 6; ++k) h[k] = scale(s[6 * half + k], sg);
                    if (fwd) su3_mul<float, false>(u, d, h, o);
                    else su3_mul<float, true>(u, d, h, o);
#pragma unroll
                    for (int k = 0; k < 6; ++k) w[6 * half + k] = o[k];
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    put(At, k0 + 2 * t, c, pack_bf16x2(w[3 * t + c].re, w[3 * t + c].im));
        };
        __syncthreads();  // the products of the block before have read LDS
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int b = wave + 4 * n;
            if (CIN == 8) transport(path0, b, b * 8);
            else if (b < kPaths) transport(b, 0, b * 8);
        }
#pragma unroll
        for (int n = 0; n < NG; ++n) {
            if (COUT == 1 && wave != 0) continue;
            const int a = COUT == 8 ? wave + 4 * n : 0;
            const uint32_t v[12] = {gr[n][0].x, gr[n][0].y, gr[n][0].z, gr[n][0].w, gr[n][1].x, gr[n][1].y,
                                    gr[n][1].z, gr[n][1].w, gr[n][2].x, gr[n][2].y, gr[n][2].z, gr[n][2].w};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int c = 0; c < 3; ++c) put(Gt, (a * 4 + s) * 2, c, real ? v[3 * s + c] : 0u);
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 192; m += 32) {
            const int mo = m + 8 * (lane >> 4);
            if constexpr (COUT == 8) {
                const bf16x8 gb = *(const bf16x8*)&Gt[(wave * 16 + (lane & 15)) * LS + mo];
#pragma unroll
                for (int t = 0; t < KT; ++t) {
                    const bf16x8 a = *(const bf16x8*)&At[(t * 16 + (lane & 15)) * LS + mo];
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, gb, acc[t], 0, 0, 0);
                }
            } else {
                const bf16x8 gb = *(const bf16x8*)&Gt[(lane & 15) * LS + mo];
                const bf16x8 a = *(const bf16x8*)&At[(wave * 16 + (lane & 15)) * LS + mo];
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, gb, acc[0], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = path0 * 64 + (COUT == 8 ? t : wave) * 16 + 4 * (lane >> 4) + e;
            const int n = (COUT == 8 ? wave * 16 : 0) + (lane & 15);
            part[((long)split * KPAD + k) * NP + n] = acc[t][e];
        }
}

// dW (complex, dL/dRe W + i dL/dIm W) += the partial real-embedding gradients summed over the
// shares: 64 weights a workgroup, a quarter of the shares per wavefront
__global__ __launch_bounds__(256) void nn_dw_reduce_kernel(const float* part, int nsplit, int Cin, int Cout,
                                                           int Kpad, int Npad, float* dW)
{
    __shared__ float red[4][2][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int w = blockIdx.x * 64 + lane, nw = kPaths * Cout * Cin * 16;
    float re = 0.f, im = 0.f;
    if (w < nw) {
        const int t = w & 3, s = (w >> 2) & 3, rest = w >> 4;
        const int b = rest % Cin, a = (rest / Cin) % Cout, p = rest / (Cin * Cout);
        const long at = (long)(((p * Cin + b) * 4 + t) * 2) * Npad + (a * 4 + s) * 2;
#pragma unroll 4
        for (int q = wave; q < nsplit; q += 4) {
            const float* P = part + (long)q * Kpad * Npad + at;
            const float2 lo = *(const float2*)P, hi = *(const float2*)(P + Npad);
            re += lo.x + hi.y;
            im += lo.y - hi.x;
        }
    }
    red[wave][0][lane] = re;
    red[wave][1][lane] = im;
    __syncthreads();
    if (wave == 0 && w < nw) {
        dW[2 * w] += (red[0][0][lane] + red[1][0][lane]) + (red[2][0][lane] + red[3][0][lane]);
        dW[2 * w + 1] += (red[0][1][lane] + red[1][1][lane]) + (red[2][1][lane] + red[3][1][lane]);
    }
}

__global__ void fill_kernel(uint32_t* p, long n)
{
    for (long k = (long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x)
        p[k] = 0u;
}

__global__ void adam_kernel(float* w, float* m, float* v, const float* g, int n, float lr,
                            float b1, float b2, float c1, float c2, float eps, float gscale)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const float gr = g[k] * gscale;
    m[k] = b1 * m[k] + (1.f - b1) * gr;
    v[k] = b2 * v[k] + (1.f - b2) * gr * gr;
    w[k] -= lr * (m[k] / c1) / (sqrtf(v[k] / c2) + eps);
}

// loss terms: d = out - e (stored in `d`), sum |d|^2
struct LossDiff {
    static constexpr int NS = 1;
    const void* out;
    const void* e;
    void* d;
    __device__ void operator()(const Unit& u, double* acc) const
    {
        cx<float> o[4], t[4];
        ld4<F32, float>(out, u, o);
        ld4<F32, float>(e, u, t);
        for (int k = 0; k < 4; ++k) {
            o[k] = o[k] - t[k];
            acc[0] += (double)o[k].re * o[k].re + (double)o[k].im * o[k].im;
        }
        st4<F32, float>(d, u, o);
    }
};

// ------------------------------------------------------------------ host side

struct NnWork {
    Chan act[kLayers + 1];       // channel fields per layer boundary (FP32 space; the hidden
                                 // ones hold bf16 fields in the bf16 forward pass)
    Chan grad[2];                // gradient channel fields (ping-pong)
    float* efield;               // target (FP32)
    void* A;                     // transported rows, [Mpad][Kmax]
    float* dA;                   // [Mpad][Kmax] (training only)
    void* G;                     // [Mpad][Nmax]
    Embedded E;                  // per layer Bt [Nmax][Kmax] and Bk [Kmax][Nmax]; Bl, Bm
    float* part;                 // [nsplit][Kmax][Nmax]
    Chan mix;                    // bf16 fields m_p of the last layer's path mixing
};

constexpr int kSplit = 64;  // row slices of the FP32-operand weight gradient
// Shares of the blocks in the fused weight gradients, so that one round of workgroups fills
// the machine: nine paths of the 8 -> 8 layer three workgroups per CU (what their LDS
// allows), of the 8 -> 1 layer four (their registers), the one-channel layer one per CU.
// One buffer of partial gradients, sized for the first, serves all of them and the slices.
constexpr int kShares = 85;
template <int CIN, int COUT>
constexpr int shares_of() { return CIN == 1 ? 256 : COUT == 1 ? 113 : kShares; }
static_assert(kShares >= kSplit && 113 * 16 <= kShares * kMaxN && 256 * 80 * 64 <= kShares * kMaxN * kMaxK,
              "the partial gradients fit");

// need_A: the materialised transport matrix A (FP32-operand forward passes, training)
size_t nn_layout(const qdw_op* op, bool training, char* base, NnWork* W, bool need_A = true)
{
    const Geom& g = op->g;
    const size_t fb = spinor_bytes(g, F32);
    const long Mp = rows_padded(g);
    size_t off = 0;
    auto take = [&](size_t n) {
        char* at = base ? base + off : nullptr;
        off += (n + 255) & ~(size_t)255;
        return at;
    };
    auto channels = [&](int n, size_t bytes) {
        const size_t each = (bytes + 255) & ~(size_t)255;
        return Chan{take(each * n), (long)each};
    };
    for (int l = 0; l <= kLayers; ++l) W->act[l] = channels(kCh[l], fb);
    for (int h = 0; h < 2; ++h) W->grad[h] = training ? channels(8, fb) : Chan{};
    W->efield = training ? (float*)take(fb) : nullptr;
    W->A = need_A || training ? take((size_t)Mp * kMaxK * 4) : nullptr;
    W->mix = channels(kPaths, spinor_bytes(g, BF16S));
    W->E.Bm = (uint16_t*)take(80 * 64 * 2);
    W->E.Bl = (uint16_t*)take((size_t)kPaths * kWBlock);
    W->dA = training ? (float*)take((size_t)Mp * kMaxK * 4) : nullptr;
    W->G = training ? take((size_t)Mp * kMaxN * 4) : nullptr;
    for (int l = 0; l < kLayers; ++l) {
        W->E.Bt[l] = take((size_t)kMaxN * kMaxK * 4);
        W->E.Bk[l] = take((size_t)kMaxN * kMaxK * 4);
    }
    W->part = training ? (float*)take((size_t)kShares * kMaxN * kMaxK * 4) : nullptr;
    return off + 256;
}

// the weights in every form the passes read; once per set of weights
template <bool F32M>
int embed_weights(const float* weights, const NnWork& W, hipStream_t st)
{
    nn_embed_kernel<F32M><<<dim3((kMaxK * kMaxN + 255) / 256, F32M ? kLayers : kLayers + 2), 256, 0, st>>>(
        weights, W.E);
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

int zero_dev(void* p, size_t bytes, hipStream_t st)
{
    const long n = (long)(bytes / 4);
    fill_kernel<<<1024, 256, 0, st>>>((uint32_t*)p, n);
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

// forward through all layers, input already in act[0] and the weights embedded; keeps every
// layer's input (keep_hidden, needed by the gradients), or, in bf16 inference passes without
// it, fuses the last layer's path mixing into the 8 -> 8 layer so that the second hidden
// layer's channels never go to memory. The output times `a` goes to `out64` (FP64) if given,
// else to act[kLayers] (FP32, a = 1).
template <bool F32M>
int forward(qdw_op* op, NnWork& W, hipStream_t st, bool keep_hidden = true, void* out64 = nullptr,
            float a = 1.f)
{
    const Geom& g = op->g;
    const long nq = 2L * padded(g.Vh);
    const void* L = op->links[F32];
    const void* D = op->det[F32];
    if constexpr (F32M) {
        const long Mp = rows_padded(g);
        for (int l = 0; l < kLayers; ++l) {
            const int Cin = kCh[l], Cout = kCh[l + 1], Kp = layer_K(l), Np = layer_N(l);
            nn_transport_kernel<<<(unsigned)((nq * Cin + 255) / 256), 256, 0, st>>>(
                g, Cin, Kp, Mp, W.act[l], (float*)W.A, L, D);
            QDW_LAUNCH_CHECK();
            nn_gemm_out_kernel<<<(unsigned)(Mp / 64), 256, 0, st>>>(
                g, Kp, Np, Cout, Mp, (const float*)W.A, (const float*)W.E.Bt[l], W.act[l + 1]);
            QDW_LAUNCH_CHECK();
        }
        return out64 ? run_map(op, Axpby<F32, F64>{W.act[kLayers].base, out64, a, 0.0}, st) : QDW_OK;
    }
    // hidden activations (between the layers) are stored in bf16, the network's input and
    // output in FP32
    const unsigned nb = (unsigned)(nq / 64);
    nn_layer_fused_kernel<1, 8, F32, BF16S><<<nb, 256, 0, st>>>(g, layer_K(0), W.act[0], W.E.Bt[0],
                                                                 nullptr, W.act[1], L, D);
    QDW_LAUNCH_CHECK();
    if (keep_hidden) {
        nn_layer_fused_kernel<8, 8, BF16S, BF16S><<<nb, 256, 0, st>>>(g, layer_K(1), W.act[1], W.E.Bt[1],
                                                                       W.E.Bl, W.act[2], L, D);
        QDW_LAUNCH_CHECK();
        // one output channel: mix the paths first, then transport 9 fields
        nn_mix_paths_kernel<<<nb, 256, 0, st>>>(g, W.act[2], W.E.Bm, W.mix);
    } else {
        nn_layer_fused_kernel<8, 8, BF16S, BF16S, true><<<nb, 256, 0, st>>>(
            g, layer_K(1), W.act[1], W.E.Bt[1], W.E.Bl, W.mix, L, D, W.E.Bm);
    }
    QDW_LAUNCH_CHECK();
    const unsigned ns = 2 * ((g.Vh + 255) / 256);
    if (out64)
        nn_transport_sum_kernel<F64><<<ns, 256, 0, st>>>(g, W.mix, out64, a, L, D);
    else
        nn_transport_sum_kernel<F32><<<ns, 256, 0, st>>>(g, W.mix, W.act[kLayers].base, a, L, D);
    QDW_LAUNCH_CHECK();
    return QDW_OK;
}

// dx of one layer from G (bf16 fields), and its weight gradient
template <int CIN, int COUT, int PIN, int POUT>
int backward_layer(qdw_op* op, int l, Chan in, Chan G, Chan dx, float* dW, const NnWork& W, hipStream_t st)
{
    const Geom& g = op->g;
    const int nblk = 2 * padded(g.Vh) / 64, shares = std::min(shares_of<CIN, COUT>(), nblk);
    nn_dw_partial_kernel<CIN, COUT, PIN><<<shares * (CIN == 8 ? kPaths : 1), 256, 0, st>>>(
        g, in, G, op->links[F32], op->det[F32], shares, W.part);
    QDW_LAUNCH_CHECK();
    const int nw = kPaths * COUT * CIN * 16;
    nn_dw_reduce_kernel<<<(nw + 63) / 64, 256, 0, st>>>(W.part, shares, CIN, COUT, layer_K(l), layer_N(l),
                                                       dW + 2 * layer_w_offset(l));
    QDW_LAUNCH_CHECK();
    if (dx.base) {
        nn_dx_kernel<CIN, COUT, POUT><<<nblk, 256, 0, st>>>(g, G, (const uint16_t*)W.E.Bk[l], dx,
                                                            op->links[F32], op->det[F32]);
        QDW_LAUNCH_CHECK();
    }
    return QDW_OK;
}

// backward from the real gradient of the network output (grad[0], channel 0, times gscale);
// accumulates dL/dRe W + i dL/dIm W into dW and, if asked for, leaves the input gradient in
// *gin_out. The gradients between the layers are bf16 fields, the operands of the products.
int backward_bf16(qdw_op* op, float* dW, NnWork& W, float gscale, hipStream_t st, float** gin_out)
{
    int rc;
    if ((rc = run_map(op, Axpby<F32, BF16S>{W.grad[0].base, W.grad[1].base, gscale, 0.0}, st))) return rc;
    if ((rc = backward_layer<8, 1, BF16S, BF16S>(op, 2, W.act[2], W.grad[1], W.grad[0], dW, W, st))) return rc;
    if ((rc = backward_layer<8, 8, BF16S, BF16S>(op, 1, W.act[1], W.grad[0], W.grad[1], dW, W, st))) return rc;
    if (gin_out) *gin_out = (float*)W.grad[0].base;
    return backward_layer<1, 8, F32, F32>(op, 0, W.act[0], W.grad[1], gin_out ? W.grad[0] : Chan{}, dW, W, st);
}

// the same with FP32 operands, through the matrices in memory (gradient checks)
int backward_f32(qdw_op* op, float* dW, NnWork& W, float gscale, hipStream_t st, float** gin_out)
{
    const Geom& g = op->g;
    const long Mp = rows_padded(g);
    const long nq = 2L * padded(g.Vh);
    const long M = rows_of(g);
    int cur = 0;  // grad[cur] holds the gradient of layer l's output
    for (int l = kLayers - 1; l >= 0; --l) {
        const int Cin = kCh[l], Cout = kCh[l + 1], Kp = layer_K(l), Np = layer_N(l);
        // recompute this layer's transported input rows
        nn_transport_kernel<<<(unsigned)((nq * Cin + 255) / 256), 256, 0, st>>>(
            g, Cin, Kp, Mp, W.act[l], (float*)W.A, op->links[F32], op->det[F32]);
        QDW_LAUNCH_CHECK();
        // G rows from the output gradient
        nn_pack_g_kernel<<<(unsigned)((nq + 255) / 256), 256, 0, st>>>(
            g, Cout, Np, W.grad[cur], l == kLayers - 1 ? gscale : 1.f, (float*)W.G);
        QDW_LAUNCH_CHECK();
        // weight gradient dB = A^T G
        const long rows_per = ((M + kSplit - 1) / kSplit + 15) & ~15L;
        nn_gemm_db_kernel<<<dim3(Kp / 16, kSplit), 256, 0, st>>>(
            M, Kp, Np, (int)rows_per, Mp, (const float*)W.A, (const float*)W.G, W.part);
        QDW_LAUNCH_CHECK();
        const int nw = kPaths * Cout * Cin * 16;
        nn_dw_reduce_kernel<<<(nw + 63) / 64, 256, 0, st>>>(W.part, kSplit, Cin, Cout, Kp, Np,
                                                           dW + 2 * layer_w_offset(l));
        QDW_LAUNCH_CHECK();
        // input gradient dA = G B^T, then the adjoint transport
        nn_gemm_da_kernel<<<(unsigned)(Mp / 64), 256, 0, st>>>(Kp, Np, Mp, (const float*)W.G,
                                                               (const float*)W.E.Bk[l], W.dA);
        QDW_LAUNCH_CHECK();
        nn_transport_adj_kernel<<<(unsigned)((nq * Cin + 255) / 256), 256, 0, st>>>(
            g, Cin, Mp, W.dA, W.grad[1 - cur], op->links[F32], op->det[F32]);
        QDW_LAUNCH_CHECK();
        cur = 1 - cur;
    }
    if (gin_out) *gin_out = (float*)W.grad[cur].base;
    return QDW_OK;
}

char* align_work(void* work) { return (char*)(((uintptr_t)work + 255) & ~(uintptr_t)255); }

}  // namespace

size_t nn_precond_workspace(const qdw_op* op)
{
    NnWork W;
    return nn_layout(op, false, nullptr, &W, false);  // bf16 forward only: no A
}

// the weights of a solve, embedded into the preconditioner's workspace once
int nn_prepare(qdw_op* op, const void* weights, char* work, hipStream_t st)
{
    NnWork W;
    nn_layout(op, false, work, &W, false);
    return embed_weights<false>((const float*)weights, W, st);
}

// phi = N(rho): rho, phi FP64 eo-SoA fields; |rho| given (sets the FP32 scale); after
// nn_prepare on the same workspace
int nn_precondition(qdw_op* op, const void* rho, void* phi, double rho_norm, char* work,
                    hipStream_t st)
{
    NnWork W;
    nn_layout(op, false, work, &W, false);
    const Geom& g = op->g;
    int rc;
    if (!(rho_norm > 0.0)) return run_map(op, Zero<F64>{phi}, st);
    const double s = std::sqrt(24.0 * g.V) / rho_norm;
    if ((rc = run_map(op, ScaleTo<F64, F32>{rho, W.act[0].base, s}, st))) return rc;
    return forward<false>(op, W, st, false, phi, (float)(1.0 / s));
}

}  // namespace qdw

using namespace qdw;

extern "C" int qdw_nn_weight_count(void) { return total_weights(); }

extern "C" size_t qdw_nn_workspace_bytes(const qdw_op* op, int training)
{
    if (!op) return 0;
    NnWork W;
    return nn_layout(op, training != 0, nullptr, &W);
}

extern "C" int nn_forward(qdw_op* op, const float* weights, const void* in, void* out, int f32_mixing,
                          void* work, size_t work_bytes, void* stream)
{
    QDW_CHECK(op && weights && in && out && work, QDW_EINVAL, "nn_forward: null argument");
    QDW_CHECK(work_bytes >= qdw_nn_workspace_bytes(op, 0), QDW_EWORKSPACE,
              "nn_forward: workspace smaller than qdw_nn_workspace_bytes(op, 0)");
    hipStream_t st = (hipStream_t)stream;
    NnWork W;
    nn_layout(op, false, align_work(work), &W);
    int rc;
    if ((rc = run_map(op, Axpby<F64, F32>{in, W.act[0].base, 1.0, 0.0}, st))) return rc;
    if ((rc = f32_mixing ? embed_weights<true>(weights, W, st) : embed_weights<false>(weights, W, st)))
        return rc;
    return f32_mixing ? forward<true>(op, W, st, true, out) : forward<false>(op, W, st, false, out);
}

extern "C" int nn_backward(qdw_op* op, const float* weights, const void* in, const void* gout,
                           float* dW, void* gin, int f32_mixing, void* work, size_t work_bytes,
                           void* stream)
{
    QDW_CHECK(op && weights && in && gout && dW && gin && work, QDW_EINVAL,
              "nn_backward: null argument");
    QDW_CHECK(work_bytes >= qdw_nn_workspace_bytes(op, 1), QDW_EWORKSPACE,
              "nn_backward: workspace smaller than qdw_nn_workspace_bytes(op, 1)");
    hipStream_t st = (hipStream_t)stream;
    NnWork W;
    nn_layout(op, true, align_work(work), &W);
    int rc;
    if ((rc = zero_dev(dW, sizeof(float) * 2 * total_weights(), st))) return rc;
    if ((rc = run_map(op, Axpby<F64, F32>{in, W.act[0].base, 1.0, 0.0}, st))) return rc;
    if ((rc = f32_mixing ? embed_weights<true>(weights, W, st) : embed_weights<false>(weights, W, st)))
        return rc;
    if ((rc = f32_mixing ? forward<true>(op, W, st) : forward<false>(op, W, st))) return rc;
    if ((rc = run_map(op, Axpby<F64, F32>{gout, W.grad[0].base, 1.0, 0.0}, st))) return rc;
    float* gi = nullptr;
    rc = f32_mixing ? backward_f32(op, dW, W, 1.f, st, &gi)
                    : backward_bf16(op, dW, W, 1.f, st, &gi);
    if (rc) return rc;
    return run_map(op, Axpby<F32, F64>{gi, gin, 1.0, 0.0}, st);
}

namespace {

// x (pair storage precision P) -> FP32 field times s; |x|^2 of the input when want_norm
template <int P>
int pair_to_f32(qdw_op* op, const void* x, void* y, double s, hipStream_t st)
{
    return run_map(op, Axpby<P, F32>{x, y, s, 0.0}, st);
}

int pair_norm2(qdw_op* op, const void* x, int prec, double* out, hipStream_t st)
{
    switch (prec) {
    case F64: return run_sum(op, Norm2<F64>{x}, st, out);
    case F32: return run_sum(op, Norm2<F32>{x}, st, out);
    default: return run_sum(op, Norm2<BF16S>{x}, st, out);
    }
}

int pair_convert(qdw_op* op, const void* x, int prec, void* y, double s, hipStream_t st)
{
    switch (prec) {
    case F64: return pair_to_f32<F64>(op, x, y, s, st);
    case F32: return pair_to_f32<F32>(op, x, y, s, st);
    default: return pair_to_f32<BF16S>(op, x, y, s, st);
    }
}

}  // namespace

extern "C" int nn_train_step(qdw_op* op, float* weights, float* adam, int step, double lr,
                             const void* const* rho, const void* const* err, int nbatch,
                             qdw_prec pair_prec, int loss_kind, double* loss, void* work,
                             size_t work_bytes, void* stream)
{
    QDW_CHECK(loss_kind == 0 || loss_kind == 1, QDW_EINVAL, "nn_train_step: loss_kind 0 or 1");
    QDW_CHECK(op && weights && adam && rho && err && loss && work && nbatch >= 1 && step >= 1,
              QDW_EINVAL, "nn_train_step: bad argument");
    QDW_CHECK(pair_prec == QDW_F64 || pair_prec == QDW_F32 || pair_prec == QDW_BF16S, QDW_EINVAL,
              "nn_train_step: pairs must be QDW_F64, QDW_F32 or QDW_BF16S fields");
    QDW_CHECK(work_bytes >= qdw_nn_workspace_bytes(op, 1) + sizeof(float) * 2 * total_weights() + 512,
              QDW_EWORKSPACE, "nn_train_step: workspace smaller than "
                              "qdw_nn_workspace_bytes(op, 1) + 8 * qdw_nn_weight_count() + 512");
    hipStream_t st = (hipStream_t)stream;
    NnWork W;
    char* base = align_work(work);
    const size_t nb = nn_layout(op, true, base, &W);
    float* dW = (float*)(base + ((nb + 255) & ~(size_t)255));
    const int nw2 = 2 * total_weights();
    const Geom& g = op->g;
    int rc;
    if ((rc = zero_dev(dW, sizeof(float) * nw2, st))) return rc;
    if ((rc = embed_weights<false>(weights, W, st))) return rc;
    double total = 0.0;
    for (int k = 0; k < nbatch; ++k) {
        // scale the pair so that the residual has unit component size (the map is linear)
        double r2;
        if ((rc = pair_norm2(op, rho[k], pair_prec, &r2, st))) return rc;
        QDW_CHECK(r2 > 0.0, QDW_EINVAL, "nn_train_step: a residual is zero");
        const double s = std::sqrt(24.0 * g.V / r2);
        if ((rc = pair_convert(op, rho[k], pair_prec, W.act[0].base, s, st))) return rc;
        if ((rc = pair_convert(op, err[k], pair_prec, W.efield, s, st))) return rc;
        double e2;
        if ((rc = run_sum(op, Norm2<F32>{W.efield}, st, &e2))) return rc;
        if ((rc = forward<false>(op, W, st))) return rc;
        double d2;
        if ((rc = run_sum(op, LossDiff{W.act[kLayers].base, W.efield, W.grad[0].base}, st, &d2))) return rc;
        double denom = e2;
        if (loss_kind == 1) {
            // D-norm: d = N(rho) - e  ->  t = D d, |t|^2, gradient direction D^+ t; the
            // normalisation |D e|^2 is |rho|^2 of the stored pair
            void* t = W.grad[1].at(0);
            void* De = W.grad[1].at(1);
            if ((rc = dw_launch(op, W.grad[0].base, t, F32, false, st))) return rc;
            if ((rc = run_sum(op, Norm2<F32>{t}, st, &d2))) return rc;
            if ((rc = dw_launch(op, W.efield, De, F32, false, st))) return rc;
            if ((rc = run_sum(op, Norm2<F32>{De}, st, &denom))) return rc;
            if ((rc = dw_launch(op, t, W.grad[0].base, F32, true, st))) return rc;
        }
        total += d2 / denom;
        // dL/d(out re, im) = 2 (out - e) / |e|^2, or 2 D^+ D (out - e) / |D e|^2, batch mean
        const float gs = (float)(2.0 / (denom * nbatch));
        if ((rc = backward_bf16(op, dW, W, gs, st, nullptr))) return rc;
    }
    *loss = total / nbatch;
    const float b1 = 0.9f, b2 = 0.999f;
    adam_kernel<<<(nw2 + 255) / 256, 256, 0, st>>>(weights, adam, adam + nw2, dW, nw2, (float)lr, b1,
                                                   b2, 1.f - std::pow(b1, (float)step),
                                                   1.f - std::pow(b2, (float)step), 1e-8f, 1.f);
    QDW_LAUNCH_CHECK();
    QDW_HIP(hipStreamSynchronize(st));
    return QDW_OK;
}
