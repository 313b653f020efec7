// Tied-array beamforming (Sec. 4.4) from the channelised voltages a plan holds
// in its channel-major buffer (the F-engine output the X-engine reads).
//
// Coherent beams: per channel c, the beams of a block are the complex product
// B_c = W_c X_c (W_c: [beams][inputs] weights that phase the signal paths up
// for each pointing; X_c: [inputs][spectra]), as real products on the matrix
// cores.  The channel's scale (INT8 s_c, FP16 2^e) is common to all inputs of
// the channel and is applied to the sums.
//   INT8, binary16 (beamform_kernel): bf16 instructions with FP32 sums.  An FP32
//     weight is the exact sum of three bf16 pieces of 8 significant bits, an
//     int8 code is one bf16 value and a binary16 value the exact sum of two, so
//     every product is exact and only the FP32 sums round: three (six)
//     instructions at 16 times the FP32 rate.
//   FP32 (beamform_f32_kernel): v_mfma_f32_32x32x2_f32 with K = (input, re/im):
//     Re B = [Re W, -Im W] . [Re X; Im X],   Im B = [Im W, Re W] . [Re X; Im X],
//     lanes 0..31 carrying the re/re and lanes 32..63 the im parts of one input.
//
// Incoherent beam: the detected power of the inputs of each polarisation,
// summed over t_avg spectra and f_avg channels (FP64 sums, fixed reduction
// order).
#include "mwax_internal.h"

namespace mwax {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

typedef __bf16 v8b __attribute__((ext_vector_type(8)));

// Spectrum t (0 .. G-1) of a 32-byte row, decoded to FP32 (before the scale).
template <int ES>
__device__ __forceinline__ float2 row_value(const uint8_t *row, int t) {
    const int re = row_re_off(t, ES), im = re + row_im_gap(ES);
    if constexpr (ES == 1) return make_float2((float)(int8_t)row[re], (float)(int8_t)row[im]);
    else if constexpr (ES == 2)
        return make_float2((float)__builtin_bit_cast(_Float16, *reinterpret_cast<const uint16_t *>(row + re)),
                           (float)__builtin_bit_cast(_Float16, *reinterpret_cast<const uint16_t *>(row + im)));
    else return make_float2(*reinterpret_cast<const float *>(row + re), *reinterpret_cast<const float *>(row + im));
}

// The upper halves of x and y as one dword (x low): two bf16 values by truncation.
__device__ __forceinline__ uint32_t pack_hi(float x, float y) {
    return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
}
// What truncation to bf16 leaves of x (exact); 0 for infinities and NaNs, whose
// truncation already carries the value.
__device__ __forceinline__ float rest_of(float x) {
    const float h = __uint_as_float(__float_as_uint(x) & 0xffff0000u);
    return fabsf(x) < __builtin_inff() ? x - h : 0.0f;
}
__device__ __forceinline__ v16f mma_bf16(const uint4 &a, const uint4 &b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), c, 0, 0, 0);
}

// Coherent beams of int8 codes (ES = 1) or binary16 values (ES = 2).  One
// workgroup = one channel x 32 WB beams x kMT = 32 NC (4 / WB) spectra: WB waves
// along the beams, 4 / WB along the spectra, a wave 32 beams x 32 NC spectra (rows
// of the product = spectra, columns = beams, so that a wave stores runs of 32
// beams).  K runs over stages of KI inputs in two LDS buffers, one stage ahead:
// the voltages' rows are copied as they are (16 bytes per lane, straight into
// LDS), each lane picking and converting the samples of its spectrum from there;
// the weights are split into their pieces on the way into LDS.  Row n of a row
// group sits at n ^ s within its eight rows, s = the 8-input half and the group's
// low bits, so that the lanes of a read fall in distinct banks.
// 32 beams, 256 tiles, 128 channels, 10,000 INT8 spectra: 0.57 ms (295 TFLOP/s of
// the FP32 product, 2.9 TB/s of the 1.66 GB it cannot do without) against 1.86 ms
// on the FP32 instructions, and half their error (2.9e-7 of the rms against
// 5.7e-7: a sum rounds once per 16 inputs and piece, not once per input and
// component).  Binary16, 8 to 96 beams: 1.5 to 2 times as fast.
// These instructions take bf16 denormals as zeros, so a weight's pieces and their
// products with the voltages' (2^-24 at the least) have to be normal: its last bit,
// 2^-23 of it, at least 2^(24 - 126), the weight at least 2^-79 (kLeastWeight).  And
// an infinity times another value's piece of zero is a NaN where the whole product
// is not.  So the beams of a smaller weight, and sums that are not finite, take their
// values from the whole weights and voltages as in the FP32 plans' kernel.
constexpr uint32_t kLeastWeight = (127u - 79u) << 23;   // bits of 2^-79
// (Binary16, more than 32 beams: held to four or, with the doubled tile, three
// workgroups per CU, which the compiler misses by some registers: 225 / 253 us
// without, 48 beams of 256 inputs, 128 channels, 2,000 spectra.)
template <int ES, int WB, int NC>
__global__ __launch_bounds__(256, (ES == 2 && WB == 2 ? 5 - NC : 2)) void beamform_kernel(BeamArgs a) {
    constexpr int G = 16 / ES;
    constexpr int KI = 32 / ES, KB = KI / 16;               // inputs and 16-input blocks per stage
    constexpr int kMT = 32 * NC * (4 / WB), GL = kMT / G;   // spectra and row groups per workgroup
    constexpr int NX = ES == 1 ? 1 : 2;                     // bf16 pieces of a voltage
    constexpr int kX = GL * KI * kRowBytes, kW = KB * 2 * 3 * 2 * 32 * WB * 16;
    __shared__ __align__(16) uint8_t xb0[kX], xb1[kX], wb0[kW], wb1[kW];
    const int c = blockIdx.z;
    const int64_t m0 = (int64_t)blockIdx.x * kMT;
    const int b0 = blockIdx.y * 32 * WB;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wb = wave / (4 / WB), wm = wave % (4 / WB);
    const int64_t gstride = (int64_t)a.n_in * kRowBytes;
    const uint8_t *base = a.chan + ((int64_t)c * a.NG + a.grp0) * gstride;
    const int64_t g0 = m0 / G, glast = (a.nframes - 1) / G;
    const float2 *wbase = a.w + ((int64_t)c * a.nb + b0) * a.n_in;
    const int nst = (a.n_in + KI - 1) / KI;

    // voltages: 16-byte units [row group][slot row][half row]; groups past the block
    // and inputs past the last are read from clamped addresses (the groups' outputs
    // are not stored, the inputs' weights are zero)
    constexpr int kUnits = kX / 16, kCopies = kUnits / 256;
    auto copy_x = [&](int s, uint8_t *xb) {
#pragma unroll
        for (int j = 0; j < kCopies; ++j) {
            const int u0 = (wave * kCopies + j) * 64, u = u0 + lane;
            const int gl = u / (2 * KI), slot = u % (2 * KI) / 2;
            const int sw = ((slot >> 3) & 1) | ((gl & (2 * ES - 1)) << 1);
            const int n = s * KI + ((slot & ~7) | ((slot ^ sw) & 7));
            const uint8_t *src = base + min(g0 + gl, glast) * gstride + (int64_t)min(n, a.n_in - 1) * kRowBytes +
                                 (u & 1) * 16;
            __builtin_amdgcn_global_load_lds(src, xb + u0 * 16, 16, 0, 0);
        }
    };
    // weights: quads of four inputs of one beam, as two pairs (n_in is even) from
    // clamped addresses, zeroed past the beams and inputs when they are split (a
    // load behind a branch would be waited for at once)
    struct __attribute__((packed, aligned(8))) Pair { float v[4]; };
    constexpr int kQuads = 32 * WB * KI / 4, kQ = (kQuads + 255) / 256;
    float wq[kQ][8];   // (re, im) of four inputs
    auto load_w = [&](int s) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int u = tid + q * 256, bl = u / (KI / 4), n = s * KI + u % (KI / 4) * 4;
            const float2 *row = wbase + (int64_t)min(bl, a.nb - 1 - b0) * a.n_in;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const Pair p = *reinterpret_cast<const Pair *>(row + min(n + 2 * h, a.n_in - 2));
#pragma unroll
                for (int e = 0; e < 4; ++e) wq[q][4 * h + e] = p.v[e];
            }
        }
    };
    uint32_t below = 0;   // bit q: the beam of this thread's quad q has a weight below kLeastWeight
    // LDS units of 16 bytes (8 inputs): [block][half][piece][re, im][beam]
    auto store_w = [&](int s, uint8_t *wbuf) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int u = tid + q * 256, bl = u / (KI / 4), kq = u % (KI / 4);
            if (kQuads % 256 != 0 && u >= kQuads) break;
            const int n = s * KI + kq * 4;
            uint8_t *dst = wbuf + (kq / 2 * 6 * 32 * WB + bl) * 16 + (kq & 1) * 8;
            uint32_t least = 0xffffffffu;   // least nonzero weight: bits, sign dropped, times two, less one
#pragma unroll
            for (int comp = 0; comp < 2; ++comp) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float w = __builtin_canonicalizef(wq[q][2 * e + comp]);   // a quiet NaN keeps its top half
                    v[e] = b0 + bl < a.nb && n + e < a.n_in ? w : 0.0f;
                    least = min(least, (__float_as_uint(v[e]) << 1) - 1u);
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    *reinterpret_cast<uint2 *>(dst + (p * 2 + comp) * 32 * WB * 16) =
                        make_uint2(pack_hi(v[0], v[1]), pack_hi(v[2], v[3]));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = rest_of(v[e]);
                }
            }
            below |= least < (kLeastWeight << 1) - 1u ? 1u << q : 0u;
        }
    };

    v16f acc_r[NC], acc_i[NC];
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) acc_r[nc] = acc_i[nc] = v16f{};
    // this lane's place in a row group: spectrum t, group t's low bits
    const int t = l32 % G, gsub = l32 / G;
    const int sw = half | ((gsub & (2 * ES - 1)) << 1);
    const int toff = ES == 1 ? (t >> 3) * 16 + ((t >> 2) & 1) * 4 : (t >> 2) * 16 + ((t >> 1) & 1) * 4;
    const int shift = ES == 1 ? (t & 3) * 8 : (t & 1) * 16;
    const int xoff = (wm * NC * (32 / G) + gsub) * KI * kRowBytes + half * 8 * kRowBytes + toff;
    auto compute = [&](const uint8_t *xb, const uint8_t *wbuf) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            uint4 wr[3], wi[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint8_t *src = wbuf + (((kb * 2 + half) * 6 + p * 2) * 32 * WB + wb * 32 + l32) * 16;
                wr[p] = *reinterpret_cast<const uint4 *>(src);
                wi[p] = *reinterpret_cast<const uint4 *>(src + 32 * WB * 16);
            }
#pragma unroll
            for (int nc = 0; nc < NC; ++nc) {
                uint32_t xr[NX][4], xi[NX][4];
                const uint8_t *src = xb + xoff + nc * (32 / G) * KI * kRowBytes + kb * 16 * kRowBytes;
#pragma unroll
                for (int i = 0; i < 8; i += 2) {
                    float r[2], m[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const uint8_t *row = src + ((i + e) ^ sw) * kRowBytes;
                        const uint32_t dr = *reinterpret_cast<const uint32_t *>(row);
                        const uint32_t di = *reinterpret_cast<const uint32_t *>(row + 8);
                        if constexpr (ES == 1) {
                            r[e] = (float)(int)__builtin_amdgcn_sbfe(dr, shift, 8);
                            m[e] = (float)(int)__builtin_amdgcn_sbfe(di, shift, 8);
                        } else {
                            r[e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(dr >> shift));
                            m[e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(di >> shift));
                        }
                    }
                    xr[0][i / 2] = pack_hi(r[0], r[1]);
                    xi[0][i / 2] = pack_hi(m[0], m[1]);
                    if constexpr (NX == 2) {
                        xr[1][i / 2] = pack_hi(rest_of(r[0]), rest_of(r[1]));
                        xi[1][i / 2] = pack_hi(rest_of(m[0]), rest_of(m[1]));
                    }
                }
                // the small products first
#pragma unroll
                for (int x = NX - 1; x >= 0; --x) {
                    const uint4 vr = make_uint4(xr[x][0], xr[x][1], xr[x][2], xr[x][3]);
                    const uint4 vi = make_uint4(xi[x][0], xi[x][1], xi[x][2], xi[x][3]);
                    const uint4 vn = make_uint4(vi.x ^ 0x80008000u, vi.y ^ 0x80008000u, vi.z ^ 0x80008000u,
                                                vi.w ^ 0x80008000u);
#pragma unroll
                    for (int p = 2; p >= 0; --p) {
                        acc_r[nc] = mma_bf16(vr, wr[p], acc_r[nc]);
                        acc_i[nc] = mma_bf16(vr, wi[p], acc_i[nc]);
                        acc_r[nc] = mma_bf16(vn, wi[p], acc_r[nc]);
                        acc_i[nc] = mma_bf16(vi, wr[p], acc_i[nc]);
                    }
                }
            }
        }
    };

    copy_x(0, xb0);
    load_w(0);
    store_w(0, wb0);
    drain_barrier();
    // stage s from one pair of buffers while stage s + 1 lands in the other (last
    // read one iteration ago, behind a barrier); past the end a stage is copied from
    // clamped addresses and not used
    auto iteration = [&](int s, uint8_t *xc, uint8_t *wc, uint8_t *xn, uint8_t *wn) {
        copy_x(s + 1, xn);
        load_w(s + 1);
        if (s < nst) compute(xc, wc);
        store_w(s + 1, wn);
        drain_barrier();
    };
    for (int s = 0; s < nst; s += 2) {
        iteration(s, xb0, wb0, xb1, wb1);
        iteration(s + 1, xb1, wb1, xb0, wb0);
    }
    // sums to form again?  (the LDS of the stages is free now)
    float z = 0.0f;   // stays zero if every sum is finite
#pragma unroll
    for (int nc = 0; nc < NC; ++nc)
#pragma unroll
        for (int r = 0; r < 16; ++r) z = fmaf(acc_i[nc][r], 0.0f, fmaf(acc_r[nc][r], 0.0f, z));
    int *flags = reinterpret_cast<int *>(xb0);   // per beam, then per wave
    const uint64_t found = __ballot(below != 0 || z != 0.0f);
    if (lane == 0) flags[32 * WB + wave] = found != 0;
    __syncthreads();
    const int *any = flags + 32 * WB;
    if (any[0] | any[1] | any[2] | any[3]) {
        // on the FP32 instructions, K = (re, im) of one input, straight from global memory
        if (tid < 32 * WB) flags[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kQ; ++q)
            if (below >> q & 1u) flags[(tid + q * 256) / (KI / 4)] = 1;
        __syncthreads();
        const bool small = flags[wb * 32 + l32] != 0;
        const float2 *row = wbase + (int64_t)min(wb * 32 + l32, a.nb - 1 - b0) * a.n_in;
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
            const int64_t m = m0 + (wm * NC + nc) * 32 + l32;
            const uint8_t *x0 = base + min(m / G, glast) * gstride;
            auto odd = [&](float v) { return small || !(fabsf(v) < __builtin_inff()); };
            v16f er{}, ei{};
#pragma unroll 1
            for (int n = 0; n < a.n_in; ++n) {
                const float2 w = row[n], x = row_value<ES>(x0 + (int64_t)n * kRowBytes, (int)(m % G));
                er = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? x.y : x.x, half ? -w.y : w.x, er, 0, 0, 0);
                ei = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? x.y : x.x, half ? w.x : w.y, ei, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (odd(acc_r[nc][r])) acc_r[nc][r] = er[r];
                if (odd(acc_i[nc][r])) acc_i[nc][r] = ei[r];
            }
        }
    }

    // out[m][c][b]: lane l32 is beam l32 of the wave's block, rows are spectra
    const float sc = a.scales ? a.scales[c] * a.post : a.post;
    const int b = b0 + wb * 32 + l32;
    if (b >= a.nb) return;
#pragma unroll
    for (int nc = 0; nc < NC; ++nc)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t m = m0 + (wm * NC + nc) * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
            if (m < a.nframes)
                a.out[((a.m0 + m) * a.L + c) * (int64_t)a.nb + b] = make_float2(acc_r[nc][r] * sc, acc_i[nc][r] * sc);
        }
}

constexpr int kKC = 32;     // inputs per LDS stage of the FP32 kernel
constexpr int kWP = kKC + 1;   // float2 pitch of a beam's weights in LDS

// WB waves along the beams, 4 / WB along the spectra: a tile of 32 WB beams x
// 128 / WB spectra (WB = 1 when a launch has at most 32 beams, so that no wave
// multiplies empty beams).
template <int WB>
__global__ __launch_bounds__(256) void beamform_f32_kernel(BeamArgs a) {
    constexpr int G = 4;
    constexpr int kBT = 32 * WB, kMT = 128 / WB;
    // one LDS block: the stage (weights [beam][input], voltages [input][spectrum])
    // and, after the K loop, the output tile [spectrum][beam] (pitch kBT + 1)
    constexpr int kStage = kBT * kWP + kKC * kMT, kOut = kMT * (kBT + 1);
    __shared__ float2 lds[kStage > kOut ? kStage : kOut];
    float2 *ws = lds, *xs = lds + kBT * kWP;
    const int c = blockIdx.z;
    const int m0 = blockIdx.x * kMT, b0 = blockIdx.y * kBT;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = tid >> 6, wb = wave / (4 / WB), wm = wave % (4 / WB);
    v16f acc_r, acc_i;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_r[r] = acc_i[r] = 0.0f;

    for (int n0 = 0; n0 < a.n_in; n0 += kKC) {
        __syncthreads();   // the previous stage has been read
        // weights: thread -> beam tid / 4, inputs (tid % 4) * 8 .. + 7 (WB = 2), or
        // beam tid / 8, inputs (tid % 8) * 4 .. + 3 (WB = 1)
        {
            constexpr int PER = kBT * kKC / 256;
            const int bl = tid / (kKC / PER), nl0 = (tid % (kKC / PER)) * PER;
            const int b = b0 + bl;
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                const int n = n0 + nl0 + e;
                float2 w = make_float2(0.0f, 0.0f);
                if (b < a.nb && n < a.n_in) w = a.w[((int64_t)c * a.nb + b) * a.n_in + n];
                ws[bl * kWP + nl0 + e] = w;
            }
        }
        // voltages: the kMT spectra of the tile for kKC inputs
        for (int u = tid; u < kKC * (kMT / G); u += 256) {
            const int nl = u % kKC, gl = u / kKC;
            const int n = n0 + nl;
            const int64_t tloc = (int64_t)m0 + gl * G;          // first spectrum of this row group
            float2 v[G];
            if (n < a.n_in && tloc < a.nframes) {
                const uint8_t *row = a.chan + (((int64_t)c * a.NG + a.grp0 + tloc / G) * a.n_in + n) * kRowBytes;
                uint4 h0 = *reinterpret_cast<const uint4 *>(row), h1 = *reinterpret_cast<const uint4 *>(row + 16);
                uint8_t buf[kRowBytes];
                __builtin_memcpy(buf, &h0, 16);
                __builtin_memcpy(buf + 16, &h1, 16);
#pragma unroll
                for (int t = 0; t < G; ++t) v[t] = row_value<4>(buf, t);
            } else {
#pragma unroll
                for (int t = 0; t < G; ++t) v[t] = make_float2(0.0f, 0.0f);
            }
#pragma unroll
            for (int t = 0; t < G; ++t) xs[nl * kMT + gl * G + t] = v[t];
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < kKC; ++k) {
            const float2 w = ws[(wb * 32 + l32) * kWP + k];
            const float2 x = xs[k * kMT + wm * 32 + l32];
            const float ar = half ? -w.y : w.x, ai = half ? w.x : w.y, bx = half ? x.y : x.x;
            acc_r = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, bx, acc_r, 0, 0, 0);
            acc_i = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, bx, acc_i, 0, 0, 0);
        }
    }

    // out[m][c][b]: stage the tile [spectrum][beam] through LDS, store rows of beams
    __syncthreads();
    float2 *os = lds;
    const float sc = a.scales ? a.scales[c] * a.post : a.post;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = (r >> 2) * 8 + half * 4 + (r & 3);   // beam within the wave's block
        const int j = l32;                                 // spectrum within the wave's block
        os[(wm * 32 + j) * (kBT + 1) + wb * 32 + i] = make_float2(acc_r[r] * sc, acc_i[r] * sc);
    }
    __syncthreads();
    for (int u = tid; u < kMT * kBT; u += 256) {
        const int ml = u / kBT, bl = u % kBT;
        const int64_t t = (int64_t)m0 + ml;
        if (t < a.nframes && b0 + bl < a.nb)
            a.out[((a.m0 + t) * a.L + c) * (int64_t)a.nb + b0 + bl] = os[ml * (kBT + 1) + bl];
    }
}

// Power of the frames [f0, f1) of one 32-byte row (G frames of one input):
// sum over those frames of re^2 + im^2.  INT8: exact, with signed 4-byte dot
// products on the bytes kept by a per-dword mask (a dword holds the re or the
// im parts of 4 frames); binary16 / FP32: FP64 sums of the exact squares.
template <int ES>
__device__ __forceinline__ double row_power(uint4 h0, uint4 h1, int f0, int f1) {
    const uint32_t w[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
    if constexpr (ES == 1) {
        // dword k: frames (k >> 2) * 8 + (k & 1) * 4 + 0 .. 3, re (k & 2 == 0) or im
        int acc = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int fb = (k >> 2) * 8 + (k & 1) * 4;
            uint32_t m = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) m |= (fb + e >= f0 && fb + e < f1) ? (0xffu << (8 * e)) : 0u;
            const int v = (int)(w[k] & m);
            acc = __builtin_amdgcn_sdot4(v, v, acc, false);
        }
        return (double)acc;
    } else if constexpr (ES == 2) {
        double acc = 0.0;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (t >= f0 && t < f1) {
                const float2 v = row_value<2>(reinterpret_cast<const uint8_t *>(w), t);
                acc += (double)v.x * v.x + (double)v.y * v.y;
            }
        }
        return acc;
    } else {
        double acc = 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t >= f0 && t < f1) {
                const float2 v = row_value<4>(reinterpret_cast<const uint8_t *>(w), t);
                acc += (double)v.x * v.x + (double)v.y * v.y;
            }
        }
        return acc;
    }
}

// One workgroup per output bin (o, j): channels o f_avg .. and spectra j t_avg
// .. of the block.  The bin's spectra are walked segment by segment and row
// group by row group; for each (row group, channel) the threads read whole
// 32-byte rows of consecutive inputs (thread tid takes inputs tid, tid + 256,
// .., all of one polarisation, so a wave reads 2 KB contiguous) and sum the
// power of the frames inside the bin; each (row group, channel) sum is scaled
// by the square of its channel's scale (INT8 s_c of the segment; binary16
// 2^e) and added to the thread's FP64 total.  The totals are reduced per
// polarisation in a fixed order.
template <int ES>
__global__ __launch_bounds__(256) void incoherent_kernel(IncohArgs a) {
    constexpr int G = 16 / ES;
    __shared__ double red[256];
    const int o = blockIdx.x;
    const int64_t j = blockIdx.y;
    const int tid = threadIdx.x;
    const int64_t m_lo = j * a.t_avg, m_hi = m_lo + a.t_avg;   // block spectra of the bin
    const int64_t m_end = a.n_j * a.t_avg;                       // block spectra
    const int64_t rstride = (int64_t)a.n_in * kRowBytes;         // bytes between row groups
    double acc = 0.0;
    for (int s = 0; s < a.nseg; ++s) {
        const int64_t s0 = a.seg_m0[s], s1 = s + 1 < a.nseg ? a.seg_m0[s + 1] : m_end;
        const int64_t lo = m_lo > s0 ? m_lo : s0, hi = m_hi < s1 ? m_hi : s1;
        if (lo >= hi) continue;
        const int64_t t0 = lo - s0, t1 = hi - s0;                 // spectra of the segment
        for (int64_t g = t0 / G; g * G < t1; ++g) {
            const int f0 = (int)(t0 > g * G ? t0 - g * G : 0), f1 = (int)(t1 - g * G < G ? t1 - g * G : G);
            for (int ci = 0; ci < a.f_avg; ++ci) {
                const int c = o * a.f_avg + ci;
                const uint8_t *rows = a.chan + ((int64_t)c * a.NG + a.seg_grp0[s] + g) * rstride;
                double pw = 0.0;
                for (int n = tid; n < a.n_in; n += 256) {
                    const uint4 *r = reinterpret_cast<const uint4 *>(rows + (int64_t)n * kRowBytes);
                    pw += row_power<ES>(r[0], r[1], f0, f1);
                }
                const double f = a.seg_scales[s] ? (double)a.seg_scales[s][c] * a.post : (double)a.post;
                acc += pw * f * f;
            }
        }
    }
    // inputs tid + 256 k have the polarisation tid & 1: even strides keep it
    red[tid] = acc;
    __syncthreads();
    for (int h = 128; h > 1; h >>= 1) {
        if (tid < h) red[tid] += red[tid + h];
        __syncthreads();
    }
    if (tid < 2) a.out[(j * a.n_o + o) * 2 + tid] = (float)red[tid];
}

}  // namespace

template <int WB, int NC>
hipError_t launch_beamform_nc(int esize, const BeamArgs &a, hipStream_t s) {
    constexpr int kBT = 32 * WB, kMT = 32 * NC * (4 / WB);
    const dim3 grid((unsigned)((a.nframes + kMT - 1) / kMT), (unsigned)((a.nb + kBT - 1) / kBT), (unsigned)a.L);
    if (esize == 1) hipLaunchKernelGGL((beamform_kernel<1, WB, NC>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((beamform_kernel<2, WB, NC>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int WB>
hipError_t launch_beamform_wb(int esize, const BeamArgs &a, hipStream_t s) {
    constexpr int kBT = 32 * WB, kMT = 128 / WB;
    if (esize == 4) {
        const dim3 grid((unsigned)((a.nframes + kMT - 1) / kMT), (unsigned)((a.nb + kBT - 1) / kBT), (unsigned)a.L);
        hipLaunchKernelGGL((beamform_f32_kernel<WB>), grid, dim3(256), 0, s, a);
        return hipGetLastError();
    }
    // the doubled spectra tile halves the weights' share of the loads and of the
    // splitting; a block that fits the single one would multiply empty spectra
    return a.nframes <= kMT ? launch_beamform_nc<WB, 1>(esize, a, s) : launch_beamform_nc<WB, 2>(esize, a, s);
}

hipError_t launch_beamform(int esize, const BeamArgs &a, hipStream_t s) {
    if (a.nframes <= 0 || a.nb <= 0) return hipSuccess;
    if (esize != 1 && esize != 2 && esize != 4) return hipErrorInvalidValue;
    // one block of 32 beams: no wave multiplies empty beams
    return a.nb <= 32 ? launch_beamform_wb<1>(esize, a, s) : launch_beamform_wb<2>(esize, a, s);
}

hipError_t launch_incoherent(int esize, const IncohArgs &a, hipStream_t s) {
    if (a.n_o <= 0 || a.n_j <= 0) return hipSuccess;
    const dim3 grid((unsigned)a.n_o, (unsigned)a.n_j);
    switch (esize) {
        case 1: hipLaunchKernelGGL(incoherent_kernel<1>, grid, dim3(256), 0, s, a); break;
        case 2: hipLaunchKernelGGL(incoherent_kernel<2>, grid, dim3(256), 0, s, a); break;
        case 4: hipLaunchKernelGGL(incoherent_kernel<4>, grid, dim3(256), 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mwax
