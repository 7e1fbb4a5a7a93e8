// qdw_host.h -- host-side state of an operator and error plumbing of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "../../include/qdw.h"
#include "qdw_internal.h"

struct qdw_op {
    qdw::Geom g;
    double m0, csw;
    int device;
    // per precision (index = qdw::Prec): compressed links (rows 0, 1 of the U(3) link),
    // link determinants exp(3 i theta) (F64: one double each, see encode_phase; F32: float2
    // arrays; the 16-bit formats keep them inside the link chunks), clover blocks
    void* links[4];
    void* det[4];
    void* clover[4];
    void* cloverinv[4];    // per precision: inverses of the clover blocks (same format)
    void* clover54[4];     // per precision: the compact clover form the D kernels read
    void* full_links;      // optional, caller-owned: FP64 links as full 3x3 matrices
    // per precision: shape of the D kernel (sites per parity of a workgroup, time slices
    // per walk chunk, software-pipelined hop loop, walk order, marching form); other site
    // kernels use g
    struct { int ts, nt, pipe, walk, march; } dw_shape[4];
    bool dw_auto[4];       // per precision: the shape is the default one, not a caller's choice
    // reduction scratch: per-workgroup partial sums, the arrival counters of the workgroups
    // (zero between launches) and the final scalars
    double* partials;      // device, kMaxPartials * kMaxScalars doubles, or one per site workgroup
    unsigned* tickets;     // device, kTicketWords words
    double* scalars;       // device, kMaxScalars doubles
    double* host_scalars;  // pinned host, kHostScalars doubles
    double* host_dev;      // the same block as kernels address it (nullptr: not mapped)
};

namespace qdw {

constexpr int kMaxPartials = 2048;  // workgroups of a reduction launch
// arrivals are counted in two levels, kTickets counters (one per 128 bytes) and a top one,
// so that thousands of workgroups do not meet on one address
constexpr int kTickets = 32;
constexpr int kTicketWords = (kTickets + 1) * 32;
constexpr int kMaxScalars = 64;     // doubles produced by one fused reduction
constexpr int kHostScalars = 1024;  // doubles the host can read back in one copy
constexpr int kMaxRhs = 64;         // right-hand sides of one multi-right-hand-side launch

void set_error(const std::string& msg);

inline size_t spinor_bytes(const Geom& g, int prec)
{
    const size_t r = prec == F64 ? 8 : prec == F32 ? 4 : 2;
    return (size_t)2 * padded(g.Vh) * 24 * r;
}

// The walk chunk nt of the marching form on 64-site tiles. A workgroup walks nt slices after
// loading one more (0.2 of a step: its neighbour in time has mostly just loaded it), and the
// machine holds 512 workgroups (FP64, one wave per SIMD) or 1024 (FP32, two) at once, so a
// launch takes whole rounds and a rest. A step of a rest that fills a share x of the machine
// is shorter than that of a full round, down to the latency of one step: measured 0.68 (FP64)
// and 0.48 (FP32) of a full step. The chunk with the smallest sum wins. Measured against the
// longest power of two that gives 512 workgroups: FP64 24^3 x 48 183 instead of 231 us
// (nt 6 instead of 8), 24^4 81 instead of 106 us, 32^3 x 40 328 instead of 401 us; FP32
// 32^3 x 64 275 instead of 318 us (nt 16 instead of 32), 16^3 x 32 18.0 instead of 22.8 us. Several fields of one launch
// are that many times the workgroups.
inline int march_chunk(const Geom& g, int prec, int nrhs)
{
    const int room = prec == F64 ? 512 : 1024, ntile = (g.S + 63) / 64;
    double best = 0.0;
    int chunk = 0;
    for (int nt = 1; nt <= 64 && nt <= g.L[0]; ++nt) {
        if (g.L[0] % nt) continue;
        const long nwg = (long)(g.L[0] / nt) * ntile * nrhs;
        const double x = (double)(nwg % room) / room;
        const double rest = nwg % room == 0 ? 0.0
                            : prec == F64   ? std::max(0.68, 0.45 + 0.55 * x)
                                            : std::max(0.48, 0.1 + 0.9 * x);
        const double steps = (nt + 0.2) * ((double)(nwg / room) + rest);
        if (!chunk || steps < best) {
            best = steps;
            chunk = nt;
        }
    }
    return chunk;
}

}  // namespace qdw

#define QDW_HIP(call)                                                                  \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess) {                                                        \
            qdw::set_error(std::string(#call) + ": " + hipGetErrorString(e_));         \
            return QDW_EDEVICE;                                                        \
        }                                                                              \
    } while (0)

#define QDW_CHECK(cond, code, msg)                                                     \
    do {                                                                               \
        if (!(cond)) {                                                                 \
            qdw::set_error(msg);                                                       \
            return (code);                                                             \
        }                                                                              \
    } while (0)

#define QDW_LAUNCH_CHECK() QDW_HIP(hipGetLastError())
