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

// The walk chunk and pipelining of the marching form on 64-site tiles. A workgroup walks nt
// slices after loading one more (0.3 of a step in FP64, 0.2 in FP32: its neighbour in time has
// mostly just loaded it), and the machine holds `room` workgroups at once: two waves per SIMD
// (FP64, and FP32 with the pipelined hop loop) or three (FP32 without). A launch takes whole
// rounds and a rest; a step of a rest that fills a share x of the machine is shorter than that
// of a full round, down to the latency of one step. FP32 rounds of three waves are 1.5 times as
// long and 7 % slower for the same work, so that form is for launches that would leave the
// other's last round nearly empty. The choice with the smallest sum wins. The constants are
// fitted to the times of all chunks and hop loops on 280 lattices of 45,000 to 2.1 million
// sites: the choice is 0.6 % (FP64) and 0.8 % (FP32) behind the fastest on average, and against
// the longest power of two that gives 512 workgroups it is 3 % faster and on three of them more
// than 2 % slower (at most 5 %). FP64 24^3 x 48 175 instead of 230 us (nt 6 instead of 8), 32^3
// x 40 334 instead of 397 us; FP32 32^3 x 64 262 instead of 315 us (nt 16 instead of 32).
// Several fields of one launch are that many times the workgroups. In one round they keep in
// step, and the links and neighbours that they share stay in L2 (4 FP64 fields at 32^3 x 64:
// 1483 us with nt 64 and the planes of x1 side by side, 1631 with nt 64 in index order, 1690
// with nt 4, 1860 with nt 32 in two rounds); launches of more rounds are faster with short
// chunks (8 fields 3200 us with nt 4, 4180 with 64). FP32 takes its pipelined form in one round
// only (4 fields at 32^3 x 64: 755 us, three waves 823) and is 10 % further behind there than
// with one field (8 fields at 24^3 x 48: 549 us in one round, 529 with three waves and nt 8).
struct MarchShape {
    int nt, pipe, walk;
};
inline MarchShape march_shape(const Geom& g, int prec, int nrhs)
{
    const int ntile = (g.S + 63) / 64, most = prec == F64 ? 4 : 8;
    double best = 0.0;
    MarchShape s{0, 0, 0};
    for (int pipe = prec == F32 ? 1 : 0; pipe >= 0; --pipe)
        for (int nt = 1; nt <= 64 && nt <= g.L[0]; ++nt) {
            if (g.L[0] % nt) continue;
            const bool three = prec == F32 && !pipe, several = nrhs > 1;
            const long nwg = (long)(g.L[0] / nt) * ntile * nrhs, room = three ? 1536 : 1024;
            const bool one = nwg <= room;
            if (several && !one && (pipe || nt > most)) continue;
            const long last = one ? nwg : nwg % room;
            const double x = (double)last / room;
            double rounds = one ? 0.0 : (double)(nwg / room);
            // (FP64 by the workgroups on the fullest of 256 CUs: one to four take 0.38, 0.56, 0.74
            // and 0.92 of a full round's step, so 588 workgroups as long as 768)
            if (last && prec == F64) rounds += (one ? 0.2 : several ? 0.28 : 0.32) + 0.18 * ((last + 255) / 256);
            else if (last && several) rounds += three ? std::max(0.6, 0.3 + 0.7 * x) : std::max(0.48, 0.2 + 0.8 * x);
            else if (last) rounds += three ? std::max(0.6, x) : 0.4 + 0.6 * x;
            const double slower = three ? (several ? 1.56 : 1.6) : several && pipe ? 1.095 : 1.0;
            const double steps = (nt + (prec == F64 && !several ? 0.3 : 0.2)) * rounds * slower;
            if (!s.nt || steps < best) {
                best = steps;
                // (planes of x1 side by side: where they are whole tiles; chunks of fewer than
                // 16 slices and FP32 are as fast or faster in index order)
                s = {nt, pipe, several && one && prec == F64 && nt >= 16 && g.L[2] * g.L[3] / 2 % 64 == 0};
            }
        }
    return s;
}

// The D kernel's shape at creation, and the default rule for it (dw_auto): launches of few
// sites take the split form, several fields choose the chunk anew. FP64 and FP32 march on
// 64-site tiles; half-precision storage takes the plain form (one lane per site, four waves per
// SIMD) on 128-site tiles in chunks of two slices (T is even).
inline void default_dw_shape(qdw_op* op, int prec)
{
    if (prec == F64 || prec == F32) {
        const MarchShape s = march_shape(op->g, prec, 1);
        op->dw_shape[prec] = {64, s.nt, s.pipe, 0, 1};
    } else {
        op->dw_shape[prec] = {128, 2, 0, 0, 0};
    }
    op->dw_auto[prec] = true;
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
