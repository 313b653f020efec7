// Visibility weights (Sec. 4.1, with the zeroing flags of Sec. 2.4 and the
// weight table of Sec. 2.7): the occupancy of each input pair over an
// integration, and the optional normalisation of the visibilities by it.
//
// Occupancy.  Flags mark, per input and per 50 ms sub-block, the sub-blocks
// whose samples were zeroed.  The weight of pair (n1, n2) in integration j is
// the fraction of j's sub-blocks populated in both inputs.  Each workgroup
// owns a block of the pair triangle of B = 32 or 64 inputs a side: it packs the
// populated flags of its B + B inputs into 32-bit masks in LDS, 1024 sub-blocks at
// a time, and every thread counts B / 16 x B / 16 pairs with AND + popcount.  No
// workspace.  B = 32 with all of a wave's rows in flight at once is bound by the
// latency of the flag loads: 512 inputs, 160 sub-blocks 7.6 us, where B = 64 with 8
// of a wave's 32 rows in flight takes 16.4 us.  With many blocks the number of flag
// loads counts instead, of which B = 64 has half (see the launch).
//
// Normalisation.  V[j][c][p] /= w[j][p] where w > 0; where w == 0 every
// product in the sum had a zeroed factor, so V is already 0 and is left as it
// is.  One read and one write of the visibilities: HBM-bound.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "plan.h"

namespace mwax {
namespace {

constexpr int kWWords = 32;          // mask words per LDS pass (1024 sub-blocks)
constexpr int kMaxInputs = 2048;     // n_inputs of a 1024-tile array

// B: inputs per side of a pair block; kRowBatch: flag rows a wave loads before their ballots
template <int B, int kRowBatch>
__global__ __launch_bounds__(256) void vis_weights_kernel(const uint8_t *__restrict__ flags, int n_in,
                                                          int subs, int n_ints, float *__restrict__ w) {
    static_assert(2 * B % (4 * kRowBatch) == 0, "row batches must tile the 2 B rows");
    constexpr int E = B / 16;            // pairs of a thread along each side
    __shared__ uint32_t mask[2 * B][kWWords + 2];
    // lower-triangle block (bi >= bj) of this workgroup
    const int blk = blockIdx.x;
    int bi = (int)((sqrtf(8.0f * blk + 1.0f) - 1.0f) * 0.5f);
    while ((bi + 1) * (bi + 2) / 2 <= blk) ++bi;
    while (bi * (bi + 1) / 2 > blk) --bi;
    const int bj = blk - bi * (bi + 1) / 2;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int64_t row_len = (int64_t)n_ints * subs;
    const int W = (subs + 31) / 32;
    const int64_t P = (int64_t)n_in * (n_in + 1) / 2;

    for (int j = blockIdx.y; j < n_ints; j += gridDim.y) {
        int cnt[E][E] = {};
        for (int w0 = 0; w0 < W; w0 += kWWords) {
            __syncthreads();
            // one wave per input row: 64 lanes read 64 consecutive flags and a
            // ballot of "populated" is two mask words.  A wave owns the rows
            // r = wave (mod 4) and loads kRowBatch of them before their ballots, so the
            // loads overlap; addresses are clamped into the flag array.
            const int nw = min(kWWords, W - w0);
            const int lane = tid & 63, wave = tid >> 6;
            for (int k = 0; k < nw; k += 2) {
                const int sub = (w0 + k) * 32 + lane;
                const int bc = min(sub, subs - 1);
                for (int r0 = wave; r0 < 2 * B; r0 += 4 * kRowBatch) {
                    bool pop[kRowBatch];
#pragma unroll
                    for (int u = 0; u < kRowBatch; ++u) {
                        const int r = r0 + 4 * u;
                        const int n = r < B ? bi * B + r : bj * B + (r - B);
                        const uint8_t v = flags[(int64_t)min(n, n_in - 1) * row_len + (int64_t)j * subs + bc];
                        pop[u] = (n < n_in) & (sub < subs) & (v == 0);
                    }
#pragma unroll
                    for (int u = 0; u < kRowBatch; ++u) {
                        const uint64_t m = __ballot(pop[u]);
                        if (lane == 0) mask[r0 + 4 * u][k] = (uint32_t)m;
                        if (lane == 1) mask[r0 + 4 * u][k + 1] = (uint32_t)(m >> 32);
                    }
                }
            }
            __syncthreads();
            for (int k = 0; k < nw; ++k) {
                uint32_t a[E], b[E];
#pragma unroll
                for (int i = 0; i < E; ++i) {
                    a[i] = mask[ty * E + i][k];
                    b[i] = mask[B + tx * E + i][k];
                }
#pragma unroll
                for (int i = 0; i < E; ++i)
#pragma unroll
                    for (int jj = 0; jj < E; ++jj) cnt[i][jj] += __popc(a[i] & b[jj]);
            }
        }
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const int n1 = bi * B + ty * E + i;
#pragma unroll
            for (int jj = 0; jj < E; ++jj) {
                const int n2 = bj * B + tx * E + jj;
                if (n1 < n_in && n2 <= n1)
                    w[(int64_t)j * P + (int64_t)n1 * (n1 + 1) / 2 + n2] = (float)cnt[i][jj] / (float)subs;
            }
        }
    }
}

constexpr int kApplyPerThread = 4;
constexpr int kApplyChunk = 256 * kApplyPerThread;

__global__ __launch_bounds__(256) void apply_weights_kernel(float2 *__restrict__ vis, const float *__restrict__ w,
                                                            int64_t P, int L, int64_t rows, int64_t chunks) {
    const int64_t nblk = rows * chunks;
    for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int64_t row = b / chunks;          // j * L + c
        const int64_t p0 = (b - row * chunks) * kApplyChunk + threadIdx.x;
        float2 *v = vis + row * P;
        const float *wr = w + (row / L) * P;
        float2 x[kApplyPerThread];
        float s[kApplyPerThread];
#pragma unroll
        for (int e = 0; e < kApplyPerThread; ++e) {
            const int64_t p = p0 + e * 256;
            if (p < P) {
                x[e] = v[p];
                s[e] = wr[p];
            }
        }
#pragma unroll
        for (int e = 0; e < kApplyPerThread; ++e) {
            const int64_t p = p0 + e * 256;
            if (p < P && s[e] > 0.0f) v[p] = make_float2(x[e].x / s[e], x[e].y / s[e]);
        }
    }
}

}  // namespace
}  // namespace mwax

using namespace mwax;

extern "C" {

mwax_status mwax_vis_weights(const uint8_t *d_flags, int32_t n_inputs, int32_t subs_per_int, int32_t n_ints,
                             float *d_weights, void *hip_stream) {
    if (n_inputs < 1 || n_inputs > kMaxInputs)
        return fail(MWAX_E_INVAL, "n_inputs must be in 1..%d (got %d)", kMaxInputs, n_inputs);
    if (subs_per_int < 1) return fail(MWAX_E_INVAL, "subs_per_int must be >= 1 (got %d)", subs_per_int);
    if (n_ints < 0) return fail(MWAX_E_INVAL, "n_ints must be >= 0 (got %d)", n_ints);
    if (n_ints == 0) return ok();
    if (!d_flags || !d_weights) return fail(MWAX_E_INVAL, "null flags or weights pointer");
    if ((uintptr_t)d_weights & 3) return fail(MWAX_E_INVAL, "weights must be 4-byte aligned");
    auto blocks = [&](int B) {
        const int nb = (n_inputs + B - 1) / B;
        return dim3((unsigned)(nb * (nb + 1) / 2), (unsigned)std::min(n_ints, 65535));
    };
    // Blocks of 32 up to some 24 per CU: in us at B = 32 / 64, 1,024 inputs, 160 sub-blocks, 8 integrations (4,224 blocks)
    // 36.0 / 37.7; 2,048 inputs, 2 of 1,200 sub-blocks (4,160) 149 / 161; but 2,048
    // inputs, 4 of 160 (8,320) 58.8 / 54.4, 1,536, 8 of 160 (9,408) 62.6 / 58.6.
    const dim3 small = blocks(32);
    if ((int64_t)small.x * n_ints <= 6144)
        hipLaunchKernelGGL((vis_weights_kernel<32, 16>), small, dim3(256), 0, (hipStream_t)hip_stream, d_flags,
                           n_inputs, subs_per_int, n_ints, d_weights);
    else
        hipLaunchKernelGGL((vis_weights_kernel<64, 8>), blocks(64), dim3(256), 0, (hipStream_t)hip_stream, d_flags,
                           n_inputs, subs_per_int, n_ints, d_weights);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "weights launch");
    return ok();
}

mwax_status mwax_apply_weights(void *d_vis, const float *d_weights, int32_t n_inputs, int32_t n_chan,
                               int32_t n_ints, void *hip_stream) {
    if (n_inputs < 1 || n_inputs > kMaxInputs)
        return fail(MWAX_E_INVAL, "n_inputs must be in 1..%d (got %d)", kMaxInputs, n_inputs);
    if (n_chan < 1) return fail(MWAX_E_INVAL, "n_chan must be >= 1 (got %d)", n_chan);
    if (n_ints < 0) return fail(MWAX_E_INVAL, "n_ints must be >= 0 (got %d)", n_ints);
    if (n_ints == 0) return ok();
    if (!d_vis || !d_weights) return fail(MWAX_E_INVAL, "null visibility or weights pointer");
    if (((uintptr_t)d_vis & 7) || ((uintptr_t)d_weights & 3))
        return fail(MWAX_E_INVAL, "visibilities must be 8-byte and weights 4-byte aligned");
    const int64_t P = (int64_t)n_inputs * (n_inputs + 1) / 2;
    const int64_t rows = (int64_t)n_ints * n_chan;
    const int64_t chunks = (P + kApplyChunk - 1) / kApplyChunk;
    const int64_t nblk = rows * chunks;
    const unsigned grid = (unsigned)std::min<int64_t>(nblk, 1 << 20);
    hipLaunchKernelGGL(apply_weights_kernel, dim3(grid), dim3(256), 0, (hipStream_t)hip_stream,
                       (float2 *)d_vis, d_weights, P, n_chan, rows, chunks);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "weight normalisation launch");
    return ok();
}

}  // extern "C"
