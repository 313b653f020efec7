// Integration output (Morrison et al. 2023, Sec. 2.5.2 and 2.7): turn one
// completed integration's device integrators into the output visibilities and
// (unless the next integration in the slot overwrites them anyway) clear them
// for reuse.  Done on the device rather than on the host CPU.
//
//   CHAN_TRI: out[c][p] = complex64(scale(V[c][p])), p = n1(n1+1)/2 + n2
//   TILE_BL : out[bl][c][pp] for tile baselines a >= b (bl = a(a+1)/2 + b) and
//             products pp = 2 p1 + p2 in the order XX, XY, YX, YY, taken from
//             input pair (2a+p1, 2b+p2); above the diagonal (auto-tile XY) the
//             conjugate of the mirrored entry.
//   raw     : out[c][p] = the exact int64 sums (INT8 integrators).
// scale: INT8 V_int * s_c * s_c (computed in FP64), FP16 and FP32 V * post.
//
// INT8 integrators hold Im V[n1,n2] - sum_m re_n1[m] (the X-engine forms its
// imaginary operand from one's complements); the autos, whose imaginary parts
// are zero, therefore hold -sum_m re_n1[m], and every entry of row n1 is
// corrected exactly by subtracting its auto's imaginary part.  Slots are cleared
// (where they have to be) by a separate fill after the pack, never while it reads
// them.
#include <algorithm>

#include "mwax_internal.h"

namespace mwax {
namespace {

__device__ __forceinline__ int64_t tri_row(int64_t t) {
    int64_t i = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    while (i * (i + 1) / 2 > t) --i;
    return i;
}

// What the integrators hold.
enum Source { kI32, kI64, kF64 };
constexpr bool is_int(int S) { return S == kI32 || S == kI64; }

// Entry p of the channel whose integrators start at base (elements of the
// source); d: the auto of p's row (sources that need it).
template <int S>
__device__ __forceinline__ auto entry(const void *base, int64_t p, int64_t d) {
    if constexpr (S == kI32) {       // within range, see kInt32MaxSpectra
        const int2 *v = reinterpret_cast<const int2 *>(base);
        const int2 x = v[p];
        return make_longlong2(x.x, (long long)x.y - v[d].y);
    } else if constexpr (S == kI64) {
        const longlong2 *v = reinterpret_cast<const longlong2 *>(base);
        longlong2 x = v[p];
        x.y -= v[d].y;
        return x;
    } else {
        return reinterpret_cast<const double2 *>(base)[p];
    }
}
template <int S>
__device__ __forceinline__ const void *channel(const PackArgs &a, int c) {
    return reinterpret_cast<const uint8_t *>(a.integ) + (int64_t)c * a.P * (S == kI32 ? 8 : 16);
}
// The scaled value in FP64: INT8 V_int s s (s = s_c), FP16 and FP32 V post.
template <int S>
__device__ __forceinline__ double2 scaled(const PackArgs &a, int c, int64_t p, int64_t d) {
    const auto v = entry<S>(channel<S>(a, c), p, d);
    if constexpr (is_int(S)) {
        const double s = (double)a.scales[c];
        return make_double2((double)v.x * s * s, (double)v.y * s * s);
    } else {
        return make_double2(v.x * a.post, v.y * a.post);
    }
}
__device__ __forceinline__ int64_t auto_of(int64_t n1) { return n1 * (n1 + 1) / 2 + n1; }

// A thread emits one pair over up to kPackCh channels: its row (a square root in
// FP64) is found once, and the loads of four channels are in flight together.
// Bound by HBM: the 2.98 GB of six uneven instances take 551 us (5.4 TB/s, part of
// it from the last-level cache); one element per thread, with a 64-bit division to
// find its channel, took 880 us.
constexpr int kPackCh = 8;
template <int S, bool RAW>
__global__ __launch_bounds__(256) void pack_tri_kernel(PackArgs a, int per_thread) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int c0 = blockIdx.y * per_thread, c1 = min(a.L, c0 + per_thread);
    if (p < a.P) {
        const int64_t d = is_int(S) ? auto_of(tri_row(p)) : 0;
#pragma unroll 4
        for (int c = c0; c < c1; ++c) {
            if constexpr (RAW) {
                reinterpret_cast<longlong2 *>(a.out)[(int64_t)c * a.P + p] = entry<S>(channel<S>(a, c), p, d);
            } else {
                const double2 v = scaled<S>(a, c, p, d);
                reinterpret_cast<float2 *>(a.out)[(int64_t)c * a.P + p] = make_float2((float)v.x, (float)v.y);
            }
        }
    }
    if (a.scales_out && blockIdx.x == 0 && c0 + (int)threadIdx.x < c1)
        a.scales_out[c0 + threadIdx.x] = a.scales[c0 + threadIdx.x];
}

// Emission with channel averaging in the same pass (Sec. 2.6): output channel o
// of N = L / F holds the weighted mean of its fine channels' scaled integrator
// values (the rule of average.hip: offsets |d| <= F/2 around its centre, the
// outermost two at weight 1/2 for even F, DC left out of the centre channel),
// optionally divided by the pair's occupancy weight; FP64 sums, one rounding.
// Reading the integrators once replaces a pack to 6,400-channel visibilities
// and a second pass over them.
template <int S>
__global__ __launch_bounds__(256) void pack_avg_kernel(PackArgs a) {
    const int N = a.L / a.F, oc = N / 2, half = a.F / 2, o = blockIdx.y;
    const bool even = (a.F & 1) == 0, centre = a.F > 1 && o == oc;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= a.P) return;
    const int64_t d = is_int(S) ? auto_of(tri_row(p)) : 0;
    double re = 0.0, im = 0.0, wsum = 0.0;
    int c = ((a.L / 2 + (o - oc) * a.F - half) % a.L + a.L) % a.L;
    auto add = [&](double w) {
        const double2 v = scaled<S>(a, c, p, d);
        re += w * v.x;
        im += w * v.y;
        wsum += w;
        c = c + 1 == a.L ? 0 : c + 1;
    };
    auto run = [&](int n) {
#pragma unroll 4
        for (int k = 0; k < n; ++k) add(1.0);
    };
    const double we = even ? 0.5 : 1.0;   // the outermost two
    if (a.F == 1) {
        add(1.0);
    } else {
        add(we);
        run(half - 1);
        if (centre) c = c + 1 == a.L ? 0 : c + 1;
        else add(1.0);
        run(half - 1);
        add(we);
    }
    double div = wsum;
    if (a.avg_w) {
        const double wp = (double)a.avg_w[p];
        if (wp > 0.0) div *= wp;
    }
    reinterpret_cast<float2 *>(a.out)[(int64_t)o * a.P + p] = make_float2((float)(re / div), (float)(im / div));
}

// Tile-baseline order: a workgroup moves kBlB consecutive baselines x kBlC channels
// through LDS.  The products of the baselines of a tile row are two rows of the
// triangle (the inputs of its tile), contiguous over the inputs of their second tiles,
// so reads run along the inputs and writes along the channels.  Integer sources, which
// read the auto of a row beside every value, have the loads of all of a thread's
// channels in flight; the others are as fast without.
constexpr int kBlB = 16, kBlC = 16;
template <int S>
__global__ __launch_bounds__(256) void pack_tilebl_kernel(PackArgs a) {
    __shared__ float2 img[kBlB][kBlC][5];    // [baseline][channel][product], padded
    const int nt = a.n_in / 2, nbl = nt * (nt + 1) / 2;
    const int bl0 = blockIdx.x * kBlB, nb = min(kBlB, nbl - bl0);
    const int c0 = blockIdx.y * kBlC, nc = min(kBlC, a.L - c0);
    // lanes along the 2 kBlB inputs of the baselines' second tiles; 8 (channel, input of
    // the first tile) at a time
    const int s = threadIdx.x % (2 * kBlB), k0 = threadIdx.x / (2 * kBlB);
    // tile row of the first baseline (uniform; FP32 holds every index exactly), then of the lane's
    int ta = (int)((sqrtf(8.0f * (float)bl0 + 1.0f) - 1.0f) * 0.5f);
    while (ta * (ta + 1) / 2 > bl0) --ta;
    const int bl = bl0 + (s >> 1);
    while ((ta + 1) * (ta + 2) / 2 <= bl) ++ta;
    if (s < 2 * nb) {
        const int n2 = 2 * (bl - ta * (ta + 1) / 2) + (s & 1);
        // channels past the last are read as it
        constexpr int kUnroll = is_int(S) ? 2 * kBlC / (256 / (2 * kBlB)) : 1;
#pragma unroll kUnroll
        for (int k = k0; k < 2 * kBlC; k += 256 / (2 * kBlB)) {
            const int c = min(c0 + (k >> 1), a.L - 1), p1 = k & 1;
            const int r = 2 * ta + p1;
            double2 v;
            if (n2 <= r) {
                v = scaled<S>(a, c, (int64_t)r * (r + 1) / 2 + n2, auto_of(r));
            } else {   // auto-tile XY: the conjugate of the mirrored entry
                v = scaled<S>(a, c, (int64_t)n2 * (n2 + 1) / 2 + r, auto_of(n2));
                v.y = -v.y;
            }
            img[s >> 1][k >> 1][2 * p1 + (s & 1)] = make_float2((float)v.x, (float)v.y);
        }
    }
    __syncthreads();
    for (int u = threadIdx.x; u < nb * nc * 4; u += 256) {
        const int b = u / (nc * 4), rest = u - b * nc * 4;
        reinterpret_cast<float2 *>(a.out)[((int64_t)(bl0 + b) * a.L + c0) * 4 + rest] = img[b][rest >> 2][rest & 3];
    }
}

__global__ void fill_zero_kernel(uint4 *p, int64_t n16) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n16;
         t += (int64_t)gridDim.x * blockDim.x)
        p[t] = make_uint4(0, 0, 0, 0);
}

unsigned grid_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b < 1) b = 1;
    if (b > 16384) b = 16384;
    return (unsigned)b;
}

}  // namespace

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if ((bytes & 15) || ((uintptr_t)p & 15)) return hipErrorInvalidValue;
    const int64_t n16 = (int64_t)(bytes / 16);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(n16)), dim3(256), 0, s, (uint4 *)p, n16);
    return hipGetLastError();
}

// integrator bytes of the slot, rounded up to whole 16-byte units (slots are
// padded to 256 bytes)
static size_t clear_bytes(const PackArgs &a) {
    return ((size_t)a.L * a.P * (a.i32 ? 8 : 16) + 15) / 16 * 16;
}

template <int S>
static hipError_t launch_pack_source(const PackArgs &a, hipStream_t s) {
    const unsigned gx = (unsigned)((a.P + 255) / 256);
    if (a.order == 3) {
        if (a.F < 1 || a.L % a.F != 0) return hipErrorInvalidValue;
        hipLaunchKernelGGL(pack_avg_kernel<S>, dim3(gx, (unsigned)(a.L / a.F)), dim3(256), 0, s, a);
    } else if (a.order == MWAX_ORDER_TILE_BL) {
        const int nt = a.n_in / 2, nbl = nt * (nt + 1) / 2;
        hipLaunchKernelGGL(pack_tilebl_kernel<S>, dim3((unsigned)((nbl + kBlB - 1) / kBlB), (unsigned)((a.L + kBlC - 1) / kBlC)),
                           dim3(256), 0, s, a);
    } else {
        // small outputs: fewer channels per thread, at least eight workgroups per CU
        // (4 tiles: 2.8 us with one channel per thread, 5.0 with eight)
        const int per = (int)std::max<int64_t>(1, std::min<int64_t>(kPackCh, (int64_t)gx * a.L / 2048));
        const dim3 grid(gx, (unsigned)((a.L + per - 1) / per));
        if (a.order != 2) {
            hipLaunchKernelGGL((pack_tri_kernel<S, false>), grid, dim3(256), 0, s, a, per);
        } else {
            if constexpr (!is_int(S)) return hipErrorInvalidValue;
            else hipLaunchKernelGGL((pack_tri_kernel<S, true>), grid, dim3(256), 0, s, a, per);
        }
    }
    return hipGetLastError();
}

hipError_t launch_pack(const PackArgs &a, hipStream_t s) {
    hipError_t e = a.is_int ? (a.i32 ? launch_pack_source<kI32>(a, s) : launch_pack_source<kI64>(a, s))
                            : launch_pack_source<kF64>(a, s);
    if (e != hipSuccess || !a.clear) return e;
    return launch_fill_zero(a.integ, clear_bytes(a), s);
}

}  // namespace mwax
