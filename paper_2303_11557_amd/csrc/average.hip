// Channel averaging of visibilities (Sec. 2.6).  L fine channels, DC at
// c = L/2, are averaged by F into N = L / F output channels arranged
// centre-symmetrically: output channel o is centred (o - N/2) * F channels from
// DC (N/2 rounded down) and takes the channels at offsets d around its centre,
//   F odd : d = -(F-1)/2 .. (F-1)/2, weight 1;
//   F even: d = -F/2 .. F/2, the two outermost at weight 1/2 (a boundary falls
//           on a fine channel shared half and half by the two neighbours).
// The centre output channel leaves the DC channel out and is divided by the
// weight left (F - 1), every other by F.  With N even the outermost output
// channel is the half channel at the coarse-channel edges: its fine channels
// wrap round +-f_s/2.  F = 1 copies.  Optionally each pair's mean is divided by
// its occupancy weight while averaging (Sec. 2.6 allows a weight here; the
// weights are those of Sec. 4.1), where the weight is positive.
//
// One thread per two neighbouring pairs and run of consecutive output channels,
// produced in order: for even F the boundary channel a channel shares with the
// next is kept in registers, so each fine channel is read from HBM once (once
// more per run).  The sum runs in FP64 in ascending d: the weights are 1 and 1/2,
// so every product is exact and the value is the FP64 mean rounded once to
// FP32.  HBM-bound: 131,328 pairs x 1,024 channels by 8 (1.21 GB) take 251 us
// (4.8 TB/s, the rate of a large copy); one pair per thread, with a remainder to
// find every channel's index, took 301 us.  Short runs for small outputs, where a
// run's loads wait for each other (105 pairs, 32 outputs by 2).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "plan.h"

namespace mwax {
namespace {

constexpr int kAvgMaxInputs = 2048;
constexpr int kSegOut = 4;   // most output channels one thread produces in order

// Two neighbouring pairs of a channel.  Rows are 8-byte aligned only (P may be
// odd), which vector loads allow; ONE: the last pair of an odd P, read and
// written alone.
struct __attribute__((packed, aligned(8))) Two { float v[4]; };
template <bool ONE>
__device__ __forceinline__ Two load_two(const float2 *p) {
    if constexpr (ONE) return Two{{p->x, p->y, 0.0f, 0.0f}};
    else return *reinterpret_cast<const Two *>(p);
}

template <bool ONE>
__device__ __forceinline__ void fscrunch_run(const float2 *vj, const float *wj, float2 *oj, int64_t P, int L, int F,
                                             int N, int o0, int o1) {
    const int half = F / 2, oc = N / 2;
    const bool even = (F & 1) == 0;
    // occupancy weights of the pairs (1 when none are given; 0 leaves the mean)
    double scale[2] = {1.0, 1.0};
    if (wj) {
#pragma unroll
        for (int e = 0; e < (ONE ? 1 : 2); ++e) scale[e] = wj[e] > 0.0f ? (double)wj[e] : 1.0;
    }
    // the fine channels are walked in order, wrapping at L
    int c = ((L / 2 + (o0 - oc) * F - half) % L + L) % L;
    const float2 *src = vj + (int64_t)c * P;
    auto next = [&] {
        ++c;
        src += P;
        if (c == L) {
            c = 0;
            src = vj;
        }
    };
    Two edge{};          // even F: the boundary channel shared with the next output
    if (even) {
        edge = load_two<ONE>(src);
        next();
    }
    for (int o = o0; o < o1; ++o) {
        const bool centre = F > 1 && o == oc;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        auto add = [&](const Two &v, double w) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += w * (double)v.v[e];
        };
        auto run = [&](int n) {
#pragma unroll 4
            for (int k = 0; k < n; ++k) {
                add(load_two<ONE>(src), 1.0);
                next();
            }
        };
        // offsets -half .. half (even F: the outermost two at 1/2, both edges)
        if (even) add(edge, 0.5);
        const int below = even ? half - 1 : half;
        if (centre) {
            run(below);
            next();                        // DC
            run(below);
        } else {
            run(2 * below + 1);
        }
        if (even) {
            edge = load_two<ONE>(src);
            next();
            add(edge, 0.5);
        }
        const double wsum = centre ? (double)(F - 1) : (double)F;
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double m = acc[e] / wsum;
            if (wj) m /= scale[e >> 1];
            y[e] = (float)m;
        }
        float2 *dst = oj + (int64_t)o * P;
        if constexpr (ONE) *dst = make_float2(y[0], y[1]);
        else *reinterpret_cast<Two *>(dst) = Two{{y[0], y[1], y[2], y[3]}};
    }
}

__global__ __launch_bounds__(256) void fscrunch_kernel(const float2 *__restrict__ vis,
                                                       const float *__restrict__ weights, float2 *__restrict__ out,
                                                       int64_t P, int L, int F, int N, int seg, int64_t rows,
                                                       int64_t chunks) {
    const int nseg = (N + seg - 1) / seg;
    const int64_t nblk = rows * chunks;
    for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int64_t row = b / chunks;  // j * nseg + segment
        const int64_t p = ((b - row * chunks) * 256 + threadIdx.x) * 2;
        if (p >= P) continue;
        const int64_t j = row / nseg;
        const int o0 = (int)(row - j * nseg) * seg, o1 = min(N, o0 + seg);
        const float2 *vj = vis + j * L * P + p;
        const float *wj = weights ? weights + j * P + p : nullptr;
        float2 *oj = out + j * N * P + p;
        if (p + 1 < P) fscrunch_run<false>(vj, wj, oj, P, L, F, N, o0, o1);
        else fscrunch_run<true>(vj, wj, oj, P, L, F, N, o0, o1);
    }
}

}  // namespace
}  // namespace mwax

using namespace mwax;

extern "C" {

mwax_status mwax_fscrunch(const void *d_vis, const float *d_weights, int32_t n_inputs, int32_t n_chan,
                          int32_t n_ints, int32_t fscrunch, void *d_out, void *hip_stream) {
    if (n_inputs < 1 || n_inputs > kAvgMaxInputs)
        return fail(MWAX_E_INVAL, "n_inputs must be in 1..%d (got %d)", kAvgMaxInputs, n_inputs);
    if (n_chan < 1) return fail(MWAX_E_INVAL, "n_chan must be >= 1 (got %d)", n_chan);
    if (fscrunch < 1 || n_chan % fscrunch)
        return fail(MWAX_E_INVAL, "fscrunch = %d must be >= 1 and divide n_chan = %d", fscrunch, n_chan);
    if (n_ints < 0) return fail(MWAX_E_INVAL, "n_ints must be >= 0 (got %d)", n_ints);
    if (n_ints == 0) return ok();
    if (!d_vis || !d_out) return fail(MWAX_E_INVAL, "null visibility pointer");
    if (((uintptr_t)d_vis & 7) || ((uintptr_t)d_out & 7))
        return fail(MWAX_E_INVAL, "visibilities must be 8-byte aligned");
    if ((uintptr_t)d_weights & 3) return fail(MWAX_E_INVAL, "weights must be 4-byte aligned");
    const int64_t P = (int64_t)n_inputs * (n_inputs + 1) / 2;
    const int N = n_chan / fscrunch;
    const uintptr_t in0 = (uintptr_t)d_vis, in1 = in0 + (uintptr_t)((int64_t)n_ints * n_chan * P * 8);
    const uintptr_t out0 = (uintptr_t)d_out, out1 = out0 + (uintptr_t)((int64_t)n_ints * N * P * 8);
    if (in0 < out1 && out0 < in1) return fail(MWAX_E_INVAL, "output overlaps the input visibilities");
    const int64_t chunks = (P + 511) / 512;
    // runs of four only where that leaves four workgroups per CU (1,024)
    const int seg = (int)std::max<int64_t>(1, std::min<int64_t>(kSegOut, (int64_t)n_ints * N * chunks / 1024));
    const int64_t rows = (int64_t)n_ints * ((N + seg - 1) / seg);
    const unsigned grid = (unsigned)std::min<int64_t>(rows * chunks, 1 << 20);
    hipLaunchKernelGGL(fscrunch_kernel, dim3(grid), dim3(256), 0, (hipStream_t)hip_stream,
                       (const float2 *)d_vis, d_weights, (float2 *)d_out, P, n_chan, fscrunch, N, seg, rows,
                       chunks);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "channel averaging launch");
    return ok();
}

}  // extern "C"
