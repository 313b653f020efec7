// F-engine of the FX correlator (Morrison et al. 2023, Sec. 2.5 and 2.5.1):
// per input and per contiguous frame of L complex int8 samples, an
// unnormalised forward FFT in FP32, channels re-ordered so DC sits at
// c = L/2 (centre-symmetric channels, Sec. 2.6), then requantised (INT8 /
// binary16) or kept (FP32) and transposed through LDS into the channel-major
// layout the X-engine reads (the transpose of Sec. 2.5.1).
//
// One workgroup owns R inputs x G consecutive frames of one integration
// segment = one 32-byte row group per (channel, input).  The raw int8 frames
// are staged in LDS with coalesced 16-byte loads (L = 1024: loaded by the FFT
// lanes themselves, see FCfg::DIRECT); each FFT is computed by a group of L2 lanes holding L1 = L / L2 points each:
//   X[k1 + L1 k2] = sum_r W_L2^(r k2) W_L^(r k1) sum_n1 x[r + L2 n1] W_L1^(n1 k1)
// (a two-pass Cooley-Tukey split): pass 1 in registers per lane, twiddle,
// exchange of the L1 x L2 block through LDS, pass 2 in registers.  The
// quantised outputs are written to an LDS image of the workgroup's output rows,
// which is then stored with coalesced 16-byte writes.
#include <algorithm>
#include <type_traits>

#include "fft_common.h"
#include "mwax_internal.h"

namespace mwax {
namespace {

using namespace fft;

// Two-pass split L = L1 * L2 over an FFT group of L2 lanes.  Pass 2 (length L2)
// is done by each lane on U columns when L2 <= L1.  At L >= 512 a lane keeps 16
// points (L2 = 32 or 64 > L1 = 16): each pass-2 transform is shared by
// P = L2 / 16 neighbouring lanes, an in-lane 16-point DFT, a second exchange and
// in-lane P-point DFTs (see fengine_body).  Measured against 32 points per lane:
// 1.2x (L = 1024) and 1.1x (L = 512) for INT8, 1.12x / 1.13x for binary16,
// 1.06x / 1.12x for FP32 (about 150 instead of 230-280 VGPRs).
template <int L, int XP>
struct FftShape {
    static constexpr bool kLaneSplit = L >= 512;
    static constexpr int L2 = L <= 16 ? 1
                              : (L == 32 ? 4
                              : (L <= 128 ? 8 : (L == 256 ? 16 : (kLaneSplit ? L / 16 : (L == 512 ? 16 : 32)))));
    static constexpr int L1 = L / L2;
    static constexpr int P = L2 > L1 ? L2 / L1 : 1;
    static constexpr int U = (L2 > 1 && P == 1) ? L1 / L2 : 1;
};

template <int XP>
struct PrecTraits;
template <>
struct PrecTraits<MWAX_X_INT8> { static constexpr int G = 16, ES = 1; };
template <>
struct PrecTraits<MWAX_X_FP16> { static constexpr int G = 8, ES = 2; };
template <>
struct PrecTraits<MWAX_X_FP32> { static constexpr int G = 4, ES = 4; };

// Channel of output slot i of lane r (see the kernel comment): bin
// k = (r U + u) + L1 k2 with i = u L2 + k2; with P lanes per pass-2 transform,
// lane r = k1 P + g holds k = k1 + L1 (g + P j + L1 q) in slot i = j P + q.
// Channel (k + L/2) mod L.
template <int L, int XP>
__device__ __forceinline__ int bin_of(int r, int i) {
    using SH = FftShape<L, XP>;
    if constexpr (SH::P > 1) return r / SH::P + SH::L1 * (r % SH::P + SH::P * (i / SH::P) + SH::L1 * (i % SH::P));
    else if constexpr (SH::L2 > 1) return (r * SH::U + i / SH::L2) + SH::L1 * (i % SH::L2);
    else return i;
}
template <int L, int XP>
__device__ __forceinline__ int chan_of(int r, int i) {
    return (bin_of<L, XP>(r, i) + L / 2) & (L - 1);
}

// Gain of the fractional delay correction for signed bin ks (channel offset
// c - L/2): exp(-2 pi i (ks alpha + phi)), alpha = d / L, phi = the frame's
// phase offset (nu_c / f_s) d reduced to [-1/2, 1/2] revolutions.
__device__ __forceinline__ float2 delay_gain(int ks, float alpha, float phi) {
    float sn, cs;
    sincospif(-2.0f * fmaf((float)ks, alpha, phi), &sn, &cs);
    return make_float2(cs, sn);
}
// exp(-2 pi i x), and the product of two of these, in FP64.
__device__ __forceinline__ double2 turn(double x) {
    double sn, cs;
    sincospi(-2.0 * x, &sn, &cs);
    return make_double2(cs, sn);
}
__device__ __forceinline__ double2 turn_by(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

constexpr int kThreads = 256;   // workgroup size

// Output-image padding per channel (bytes beyond R * 32), chosen so the packed
// output writes of a wave fall in distinct LDS banks.
constexpr int cp_pad(int L, int XP) {
    return L <= 16 ? 4 : (L == 32 ? (XP == MWAX_X_INT8 ? 8 : 4)
                       : (L == 64 ? (XP == MWAX_X_INT8 ? 8 : 16)
                       : (L <= 256 ? (XP == MWAX_X_INT8 ? 4 : 8) : 4)));
}

constexpr int64_t kLeast = 2048;   // workgroups that fill the device (about all that can be resident)

// Work decomposition of one workgroup (THREADS threads) for length L and
// output precision XP.  An FFT group is L2 lanes; a wave holds GPW groups.
// Each group transforms FPG consecutive frames of one input, so that the
// results of FPG frames leave in one packed LDS write; the workgroup covers
// R inputs x G frames (one 32-byte row group per channel and input).
template <int L, int XP>
struct FCfg {
    using SH = FftShape<L, XP>;
    static constexpr int L1 = SH::L1, L2 = SH::L2, U = SH::U;
    static constexpr int G = PrecTraits<XP>::G, ES = PrecTraits<XP>::ES;
    // INT8 at 16 <= L <= 256: one frame per group (byte writes) holds fewer
    // registers than packing two frames' codes, for more waves per SIMD.  At
    // L >= 512 (32 or 64 lanes per FFT) an INT8 group transforms two frames, so
    // that its codes leave two at a time.  Binary16 keeps one frame per group (two
    // would need 86 KB of LDS at L = 128, one workgroup per CU).
    static constexpr int FPG = XP == MWAX_X_INT8 ? (L >= 16 && L <= 256 ? 1 : 2) : 1;
    // L = 1024 (one FFT per wave): the lanes load their own samples straight from HBM
    // (a lane's samples r + 64 n1 of a frame are one 128-byte line per load
    // instruction), INT8 two packs of an item per wave in turn, binary16 two frames.
    // Without the staging area two (INT8) or three workgroups fit a CU, and one's
    // barriers and image store overlap the others' FFTs: INT8 2.34 instead of 1.86
    // TB/s, binary16 and FP32 see SPLIT.  (At L = 512, two 32-lane groups per wave,
    // INT8 ran at 2.04 instead of 2.37 TB/s this way.)
    static constexpr bool DIRECT = L == 1024;
    static constexpr int THREADS = kThreads;
    static constexpr int P = SH::P;
    static constexpr int GPW = 64 / L2;
    static constexpr int NGWG = THREADS / 64 * GPW;   // FFT groups per workgroup
    static constexpr int PACKS = G / FPG;         // frame packs per input
    static constexpr int R = NGWG >= PACKS ? NGWG / PACKS : 1;   // inputs per workgroup item
    static constexpr int PPG = PACKS * R / NGWG;  // packs per group and item
    static constexpr int CP = R * kRowBytes + cp_pad(L, XP);
    static constexpr int SP = 2 * L + 16;         // staged frame pitch (bytes)
    // SPLIT: the lanes exchange the real and the imaginary parts one after the
    // other through half the LDS (conflict-free as the float2 exchange is).  At L >=
    // 128 binary16 and FP32, whose images are two and four times the INT8 one, then
    // fit three workgroups on a CU instead of two (one at L = 1024): these launches
    // wait for LDS and barriers (VALU 39 % busy), so a third wave per SIMD pays.
    // 256 inputs x 0.5 s at L = 128 / 256 / 512 / 1024: binary16 388, 394, 553, 664
    // -> 293, 339, 430, 422 us; 128 inputs FP32 217, 244, 274, 358 -> 188, 208,
    // 249, 332 us.  INT8 has the third wave already (L <= 256) or cannot hold it in
    // registers (L >= 512).
    static constexpr bool SPLIT = XP != MWAX_X_INT8 && L >= 128;
    // exchange area per group (float2, or float if SPLIT): L + L2 (8 at least, so
    // that the groups of a wave start in distinct banks), or L1 rows of L2 + P (P > 1)
    static constexpr int EXR = L2 + P;
    static constexpr int EXG = P > 1 ? L1 * EXR : L + (SPLIT ? L2 : 8);
    // ALIAS: a wave exchanges where its own staged frames were (each group
    // transforms one frame per item, held in registers by then)
    static constexpr bool ALIAS = SPLIT && FPG == 1 && PPG == 1 && !DIRECT;
    static constexpr int WAVE_STAGE = GPW * SP, WAVE_EX = GPW * EXG * (SPLIT ? 4 : 8);
    static constexpr int WAVE_PITCH = ALIAS ? (WAVE_STAGE > WAVE_EX ? WAVE_STAGE : (WAVE_EX + 15) / 16 * 16) : WAVE_STAGE;
    static constexpr int OUT_BYTES = L * CP;
    static constexpr int STAGE_BYTES = L2 > 1 && !DIRECT ? (ALIAS ? THREADS / 64 * WAVE_PITCH : R * G * SP) : 0;
    static constexpr int EX_BYTES = L2 > 1 && !ALIAS ? THREADS / 64 * WAVE_EX : 0;
    // statistics pass: per-lane channel sums (L1 floats) and the populated-frame count
    static constexpr int RED_BYTES = THREADS * L1 * 4 + 16;
    // waves per SIMD the registers are held to (0: the compiler's choice); four
    // would spill 7 to 15 registers and is slower (L = 256: 482 us)
    static constexpr int MINW = SPLIT ? 3 : 0;
    // load the next item's frames while transforming the current one (where the
    // extra registers keep the occupancy)
    static constexpr bool PREFETCH = XP != MWAX_X_FP32 && L2 > 1 && (L <= 256 || XP == MWAX_X_INT8) && !DIRECT;
    static_assert(R >= 1 && NGWG * PPG == PACKS * R && (PPG == 1 || GPW == 1), "bad decomposition");
    // most workgroups of a single-plan launch (main_grid): each takes items in
    // rounds, and in too many rounds the workgroups holding adjacent items (their rows
    // share output lines) drift apart.  Measured at 256 tiles, 8 s: 65,536 at every
    // length but 256, where 131,072 is 10 % faster (32,768 - 262,144 swept).
    static constexpr int64_t GRID_CAP = L == 256 ? 131072 : 65536;
    // most rounds of a single-plan launch (main_grid): eight, but where the drift costs
    // more than the set-up.  FP32 at L >= 512, whose items write 64 or 32 bytes of a
    // channel's 128-byte lines: at L = 512 two, at L = 1024 one once three do not hold the
    // launch to kLeast.  us in eight rounds / these: L = 512, 128 inputs x 400 spectra
    // 90 / 82, 512 x 400 340 / 307; L = 1024, 128 x 520 317 / 269, 256 x 1,200 1,509 /
    // 1,192 (64 x 320: 71 in three, 90 in one).  And L = 8, 16, an FFT to a lane, which
    // has next to no set-up: two and one.  20 tiles x 0.5 s, L = 8 INT8 27.0 / 25.4,
    // binary16 31.0 / 28.2, FP32 47.2 / 41.4; L = 16, 64 tiles x 1 s 140 / 134, 207 /
    // 199, 342 / 325.
    static constexpr int64_t most_rounds(int64_t items) {
        if (L == 8 || L == 16) return 16 / L;
        return XP != MWAX_X_FP32 || L < 512 ? 8 : (L == 512 ? 2 : (items <= 3 * kLeast ? 3 : 1));
    }
};

// One complex int8 sample, converted exactly.  Written with arithmetic shifts of
// the halfword placed in the upper half of a word so that each component is one
// sign-extending byte-select convert (the int8_t casts of a 16-bit load compile
// to a separate extract per component).
__device__ __forceinline__ float2 load_pair(const uint8_t *p) {
    const int32_t w = (int32_t)((uint32_t)*reinterpret_cast<const uint16_t *>(p) << 16);
    return make_float2((float)((w << 8) >> 24), (float)(w >> 24));
}

// Exchange within one FFT group through its LDS area of floats ex, real parts,
// then imaginary parts: dst[m] = the value some lane holds as src[k] with write(k)
// == read(m).  The caller orders it against earlier and later uses of the area.
template <int N, int M, class Write, class Read>
__device__ __forceinline__ void split_exchange(uint8_t *ex, const float2 (&src)[N], float2 (&dst)[M], Write &&write,
                                               Read &&read) {
    float *e = reinterpret_cast<float *>(ex);
#pragma unroll
    for (int k = 0; k < N; ++k) e[write(k)] = src[k].x;
    wave_sync();
#pragma unroll
    for (int m = 0; m < M; ++m) dst[m].x = e[read(m)];
    wave_sync();
#pragma unroll
    for (int k = 0; k < N; ++k) e[write(k)] = src[k].y;
    wave_sync();
#pragma unroll
    for (int m = 0; m < M; ++m) dst[m].y = e[read(m)];
}

// The work of workgroup wg of nwg workgroups on the segment described by a;
// DELAY: apply the fractional delay and phase correction before requantising.
template <int L, int XP, bool STATS, bool DELAY = false>
__device__ __forceinline__ void fengine_body(const FArgs &a, const int wg, const int nwg, const int xoff,
                                             uint8_t *smem) {
    using C = FCfg<L, XP>;
    constexpr int L1 = C::L1, L2 = C::L2, U = C::U, G = C::G, ES = C::ES, FPG = C::FPG;
    constexpr int GPW = C::GPW, PACKS = C::PACKS, R = C::R, CP = C::CP, SP = C::SP, EXG = C::EXG;
    uint8_t *outbuf = smem;
    uint8_t *stage = smem + (STATS ? 0 : C::OUT_BYTES);
    uint8_t *exbase = stage + (C::ALIAS ? 0 : C::STAGE_BYTES);
    // staged frame q = input slot G + f of the item
    auto stage_at = [&](int q) {
        if constexpr (C::ALIAS) return stage + q / GPW * C::WAVE_PITCH + q % GPW * SP;
        else return stage + q * SP;
    };

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane / L2, r = lane % L2;
    const int gg = wave * GPW + gi;            // FFT group within the workgroup
    constexpr int PPG = C::PPG;                // packs gg PPG + pp of the item are group gg's
    const int nblk = (a.n_in + R - 1) / R;
    const int items = a.ngrp * nblk;

    // Per-lane constants.  Output slot i of a lane (i = u * L2 + k2 for the
    // two-pass split) holds FFT bin k = (r U + u) + L1 k2, channel (k + L/2) mod L.
    constexpr bool kTwReg = L1 <= 16;
    constexpr int P = C::P;
    float2 twr[kTwReg && L2 > 1 ? L1 : 1];
    if constexpr (kTwReg && L2 > 1) {
#pragma unroll
        for (int i = 1; i < L1; ++i) twr[i] = a.tw[(r * i) % L];        // W_L^(r k1)
    }
    // W_L2^(q m2) for the values q = 1 .. P-1 of the columns m2 = g + P j that
    // lane (k1, g) = (r / P, r % P) transforms after the second exchange
    constexpr int kTw2 = P > 1 ? (P - 1) * (L1 / P) : 1;
    float2 tw2[kTw2];
    if constexpr (P > 1) {
#pragma unroll
        for (int q = 1; q < P; ++q)
#pragma unroll
            for (int j = 0; j < L1 / P; ++j)
                tw2[(q - 1) * (L1 / P) + j] = a.tw[((q * (r % P + P * j)) % L2) * (L / L2)];
    }
    float sc[XP == MWAX_X_INT8 && kTwReg && !STATS ? L1 : 1];
    if constexpr (XP == MWAX_X_INT8 && kTwReg && !STATS) {
#pragma unroll
        for (int i = 0; i < L1; ++i) sc[i] = a.inv_s[chan_of<L, XP>(r, i)];
    }
    float acc[STATS ? L1 : 1];
#pragma unroll
    for (int i = 0; i < (STATS ? L1 : 1); ++i) acc[i] = 0.0f;
    int popc = 0;   // statistics pass: populated frames this lane counted

    // Staging of the raw frames (two-pass split) through registers; with
    // PREFETCH the global loads of the next item are issued before the current
    // item is transformed, so their latency hides behind the FFT work.
    constexpr int UPF = 2 * L / 16;                      // 16-byte units per frame
    constexpr int NUNITS = L2 > 1 && !C::DIRECT ? R * G * UPF : 0;
    constexpr int NU = (NUNITS + C::THREADS - 1) / C::THREADS;
    uint4 pre[NU > 0 ? NU : 1];
    auto fetch = [&](int it) {
        if constexpr (NU > 0) {
            const int gs = it / nblk;
            const int m0 = (it - gs * nblk) * R;
            const int nr = min(R, a.n_in - m0);
            const int64_t l0 = (int64_t)gs * G;
            const int fv = (int)min((int64_t)G, a.nframes - l0);
            // the item's first sample (uniform); a unit adds its row and offset
            const int8_t *ib = a.volts + ((int64_t)m0 * a.ld + (a.frame0 + l0) * L) * 2;
#pragma unroll
            for (int j = 0; j < NU; ++j) {
                const int u = tid + j * C::THREADS;
                const int sl = u / (G * UPF);
                const int rem = u - sl * G * UPF;
                const int f = rem / UPF;
                pre[j] = make_uint4(0u, 0u, 0u, 0u);     // frames past the end are zero
                if (u < NUNITS && sl < nr && f < fv)
                    pre[j] = *reinterpret_cast<const uint4 *>(ib + (int64_t)sl * (2 * a.ld) + rem * 16);
            }
        }
    };
    // Item of round t.  Workgroup b of a launch runs on XCD b mod 8, and each
    // XCD has its own L2.  The output rows of consecutive items (adjacent inputs
    // of one row group) share cache lines, so a round hands each XCD one
    // contiguous range of items: a line is then completed in one L2 instead of
    // leaving several L2s as partial 32- or 64-byte writes.  xoff: the XCD of
    // workgroup 0 of this work (batched launches).
    const bool xmap = (nwg & 7) == 0;
    auto item_at = [&](int t) {
        return t * nwg + (xmap ? ((wg + xoff) & 7) * (nwg >> 3) + (wg >> 3) : wg);
    };
    const int rounds = (items + nwg - 1) / nwg;
    if constexpr (C::PREFETCH) {
        if (item_at(0) < items) fetch(item_at(0));
    }
    // DIRECT: the 16-bit samples of the group's next frame (q = pp FPG + t of
    // item it), loaded while the current frame is transformed; zeros past the
    // segment or the inputs
    uint32_t raw[C::DIRECT ? L1 : 1];
    auto fetch_frame = [&](int it, int q) {
        if constexpr (C::DIRECT) {
            const int gs = it / nblk;
            const int pg = gg * PPG + q / FPG;
            const int ni = (it - gs * nblk) * R + pg / PACKS;
            const int f = (pg % PACKS) * FPG + q % FPG;
            const int64_t l0 = (int64_t)gs * G;
            if (ni < a.n_in && f < (int)min((int64_t)G, a.nframes - l0)) {
                const uint16_t *src = reinterpret_cast<const uint16_t *>(
                                          a.volts + ((int64_t)ni * a.ld + (a.frame0 + l0 + f) * L) * 2) + r;
#pragma unroll
                for (int n1 = 0; n1 < L1; ++n1) raw[n1] = src[L2 * n1];
            } else {
#pragma unroll
                for (int n1 = 0; n1 < L1; ++n1) raw[n1] = 0u;
            }
        }
    };
    if constexpr (C::DIRECT) {
        if (item_at(0) < items) fetch_frame(item_at(0), 0);
    }

    for (int round = 0; round < rounds; ++round) {
        const int item = item_at(round);
        if (item >= items) continue;   // the last round's tail (uniform per workgroup)
        const int gsel = item / nblk;
        const int n0 = (item - gsel * nblk) * R;
        const int nrows = min(R, a.n_in - n0);

        __syncthreads();  // LDS of the previous item fully consumed
        if constexpr (L2 > 1 && !C::DIRECT) {
            if constexpr (!C::PREFETCH) fetch(item);
#pragma unroll
            for (int j = 0; j < NU; ++j) {
                const int u = tid + j * C::THREADS;
                if (u < NUNITS) {
                    const int sl = u / (G * UPF);
                    const int rem = u - sl * G * UPF;
                    const int f = rem / UPF, o = rem - f * UPF;
                    *reinterpret_cast<uint4 *>(stage_at(sl * G + f) + o * 16) = pre[j];
                }
            }
            __syncthreads();
            if constexpr (C::PREFETCH) {
                if (round + 1 < rounds && item_at(round + 1) < items) fetch(item_at(round + 1));
            }
        }
        const int64_t lf0 = (int64_t)gsel * G;
        const int fvalid = (int)min((int64_t)G, a.nframes - lf0);
        const int64_t src_frame = a.frame0 + lf0;

        for (int pp = 0; pp < PPG; ++pp) {
        const int nl = (gg * PPG + pp) / PACKS;           // the pack's input within the item
        const int pk = (gg * PPG + pp) - nl * PACKS;      // and its frames pk FPG + t
        // first frame of the pack: binary16 bits per slot, or int8 codes packed four
        // to a word (re words, then im words)
        constexpr int kQ0 = XP == MWAX_X_INT8 ? 2 * ((L1 + 3) / 4) : 2 * L1;
        uint32_t q0[XP != MWAX_X_FP32 && FPG == 2 && !STATS ? kQ0 : 1];
        if constexpr (XP == MWAX_X_INT8 && FPG == 2 && !STATS) {
#pragma unroll
            for (int w = 0; w < kQ0; ++w) q0[w] = 0u;
        }
        for (int t = 0; t < FPG; ++t) {
            const int f = pk * FPG + t;
            // this frame's delay (signal path n0 + nl) and phase offset
            float dl_alpha = 0.0f, dl_phi = 0.0f;
            // CHAIN (binary16): a lane's bins of a column are evenly spaced, so its
            // gains turn by the same angle from one to the next: in FP64, whose roundings
            // do not reach FP32, two sincos per column and four multiply-adds per bin
            // instead of a sincos per bin (that of a bin in FP32 is off by 6e-8 rms, for
            // delays of many samples by more; these by the one rounding to FP32).  Taken
            // before the frame is loaded, when registers are free.  186 inputs, 1 s at L =
            // 256 / 1024: 461, 697 us; with a sincos per bin and two workgroups per CU
            // 752, 1,227.  INT8 and FP32 plans evaluate every bin.
            constexpr bool CHAIN = DELAY && XP == MWAX_X_FP16 && L2 > 1;
            constexpr int NT = P > 1 || L2 == 1 ? L1 : L2, NC = L1 / NT;   // bins of a column, columns
            double2 first[CHAIN ? NC : 1], by;
            auto take_delay = [&] {
                float d = 0.0f;
                if (nl < nrows && f < fvalid)
                    d = a.dl[(int64_t)(n0 + nl) * a.dl_ld + (a.dl_f0 + lf0 + f) / a.dl_fps];
                const double ph = (double)d * a.dl_nu;
                dl_phi = (float)(ph - rint(ph));
                dl_alpha = d * (1.0f / (float)L);
                if constexpr (CHAIN) {
                    // column u: bins k0 + L / NT t; t >= NT / 2 are the negative
                    // frequencies t - NT: from -NT / 2 on
#pragma unroll
                    for (int u = 0; u < NC; ++u)
                        first[u] = turn((bin_of<L, XP>(r, u * NT) - L / 2) * ((double)d / L) + (ph - rint(ph)));
                    by = turn((double)d / NT);
                }
            };
            if constexpr (CHAIN) take_delay();

            float2 v[L1];
            if constexpr (C::DIRECT) {
#pragma unroll
                for (int n1 = 0; n1 < L1; ++n1) {
                    const int32_t w = (int32_t)(raw[n1] << 16);
                    v[n1] = make_float2((float)((w << 8) >> 24), (float)(w >> 24));
                }
                // start the loads of the group's next frame (in this item or the next)
                const int q = pp * FPG + t + 1;
                if (q < PPG * FPG) fetch_frame(item, q);
                else if (round + 1 < rounds && item_at(round + 1) < items) fetch_frame(item_at(round + 1), 0);
            } else if constexpr (L2 == 1) {
                if (nl < nrows && f < fvalid) {
                    const uint8_t *src = reinterpret_cast<const uint8_t *>(a.volts) +
                                         ((int64_t)(n0 + nl) * a.ld + (src_frame + f) * L) * 2;
                    if constexpr (L == 1) {
                        v[0] = load_pair(src);
                    } else {
#pragma unroll
                        for (int q = 0; q < L / 2; ++q) {
                            const uint32_t wv = *reinterpret_cast<const uint32_t *>(src + 4 * q);
                            v[2 * q] = make_float2((float)(int8_t)wv, (float)(int8_t)(wv >> 8));
                            v[2 * q + 1] = make_float2((float)(int8_t)(wv >> 16), (float)(int8_t)(wv >> 24));
                        }
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < L; ++q) v[q] = make_float2(0.0f, 0.0f);
                }
            } else {
                const uint8_t *fr = stage_at(nl * G + f);
#pragma unroll
                for (int n1 = 0; n1 < L1; ++n1) v[n1] = load_pair(fr + 2 * (r + L2 * n1));
            }
            if constexpr (STATS) {
                // a frame is populated if any of its samples is nonzero (zeroed
                // frames, from lost packets, are left out of the calibration);
                // frames past the segment or input range were loaded as zeros
                bool nz = false;
#pragma unroll
                for (int n1 = 0; n1 < L1; ++n1) nz = nz || v[n1].x != 0.0f || v[n1].y != 0.0f;
                if constexpr (L2 == 1) {
                    popc += nz ? 1 : 0;
                } else {
                    const uint64_t m = __ballot(nz);
                    const uint64_t gm = L2 == 64 ? m : (m >> (gi * L2)) & ((1ull << (L2 & 63)) - 1ull);
                    popc += (r == 0 && gm != 0ull) ? 1 : 0;
                }
            }
            dft_regs<L1>(v);
            if constexpr (DELAY && !CHAIN) take_delay();

            // consume output slot i (FFT bin of this lane) with value X and, if CHAIN, gain
            // g; tc: the frame's place in its pack as a compile-time constant (see emit_frame)
            auto emit = [&](int i, float2 X, float2 g, auto tc) {
                constexpr int T = decltype(tc)::value;
                if constexpr (DELAY) {
                    if constexpr (!CHAIN) {
                        const int k = bin_of<L, XP>(r, i);
                        g = delay_gain(k < L / 2 ? k : k - L, dl_alpha, dl_phi);
                    }
                    X = make_float2(X.x * g.x - X.y * g.y, X.x * g.y + X.y * g.x);
                }
                if constexpr (STATS) {
                    acc[i] += X.x * X.x + X.y * X.y;
                } else {
                    const int c = chan_of<L, XP>(r, i);
                    uint8_t *row = outbuf + c * CP + nl * kRowBytes + row_re_off(pk * FPG, ES);
                    constexpr int IM = row_im_gap(ES);
                    if constexpr (XP == MWAX_X_INT8) {
                        float s;
                        if constexpr (kTwReg) s = sc[i];
                        else s = a.inv_s[c];
                        const uint32_t br = quant8_bits(X.x, s), bi = quant8_bits(X.y, s);
                        if constexpr (FPG == 1) {
                            // one frame per group: the code's low byte goes straight out
                            row[0] = (uint8_t)br;
                            row[IM] = (uint8_t)bi;
                        } else {
                            // frame 0: keep the code's low byte in byte i % 4 of a word;
                            // frame 1: pair it with the new code, one 16-bit write per half
                            constexpr int kW = (L1 + 3) / 4;
                            const int w = i / 4, p = i % 4;
                            if constexpr (T == 0) {
                                const uint32_t ins = (0x03020100u & ~(0xffu << (8 * p))) | (0x04u << (8 * p));
                                q0[w] = __builtin_amdgcn_perm(br, q0[w], ins);
                                q0[kW + w] = __builtin_amdgcn_perm(bi, q0[kW + w], ins);
                            } else {
                                const uint32_t pair = 0x0c0c0400u | (uint32_t)p;
                                *reinterpret_cast<uint16_t *>(row) = (uint16_t)__builtin_amdgcn_perm(br, q0[w], pair);
                                *reinterpret_cast<uint16_t *>(row + IM) = (uint16_t)__builtin_amdgcn_perm(bi, q0[kW + w], pair);
                            }
                        }
                    } else if constexpr (XP == MWAX_X_FP16) {
                        const _Float16 hr = (_Float16)(X.x * a.half_scale), hi = (_Float16)(X.y * a.half_scale);
                        const uint32_t br = (uint32_t)__builtin_bit_cast(uint16_t, hr);
                        const uint32_t bi = (uint32_t)__builtin_bit_cast(uint16_t, hi);
                        if constexpr (FPG == 2) {
                            if constexpr (T == 0) {
                                q0[2 * i] = br;
                                q0[2 * i + 1] = bi;
                            } else {
                                *reinterpret_cast<uint32_t *>(row) = q0[2 * i] | (br << 16);
                                *reinterpret_cast<uint32_t *>(row + IM) = q0[2 * i + 1] | (bi << 16);
                            }
                        } else {
                            *reinterpret_cast<uint16_t *>(row) = (uint16_t)br;
                            *reinterpret_cast<uint16_t *>(row + IM) = (uint16_t)bi;
                        }
                    } else {
                        *reinterpret_cast<float *>(row) = X.x;
                        *reinterpret_cast<float *>(row + IM) = X.y;
                    }
                }
            };
            // run body(tc) with the frame's place in the pack as a constant, so that
            // the emission of a two-frame pack has no per-slot branch on t
            auto emit_frame = [&](auto body) {
                if (FPG == 1 || t == 0) body(std::integral_constant<int, 0>{});
                else body(std::integral_constant<int, 1>{});
            };

            // emit the column of slots i0 .. i0 + NT - 1 with values w
            auto emit_column = [&](int i0, const float2 *w, auto tc) {
                if constexpr (CHAIN) {
                    double2 g = first[i0 / NT];
#pragma unroll
                    for (int e = 0; e < NT; ++e) {
                        const int t = (e + NT / 2) % NT;
                        const int i = P > 1 ? t % (L1 / P) * P + t / (L1 / P) : t;
                        emit(i0 + i, w[i], make_float2((float)g.x, (float)g.y), tc);
                        if (e + 1 < NT) g = turn_by(g, by);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < NT; ++i) emit(i0 + i, w[i], float2{}, tc);
                }
            };

            if constexpr (L2 == 1) {
                emit_frame([&](auto tc) { emit_column(0, v, tc); });
            } else {
#pragma unroll
                for (int k1 = 1; k1 < L1; ++k1) {      // W_L^0 = 1
                    float2 w;
                    if constexpr (kTwReg) w = twr[k1];
                    else w = a.tw[(r * k1) % L];
                    v[k1] = make_float2(v[k1].x * w.x - v[k1].y * w.y, v[k1].x * w.y + v[k1].y * w.x);
                }
                uint8_t *eg = exbase + (C::ALIAS ? wave * C::WAVE_PITCH + gi * EXG * 4 : gg * EXG * (C::SPLIT ? 4 : 8));
                if constexpr (C::ALIAS) wave_sync();   // the wave's frames have been read
                if constexpr (P > 1) {
                    // lane r writes its column of the L1 x L2 block (row pitch
                    // L2 + P keeps the writes and the strided reads below free of
                    // bank conflicts); lane (k1, h) = (r / P, r % P) then takes
                    // rows h + P m of column k1 and an in-lane 16-point DFT over m.
                    // A second exchange hands lane (k1, g) the P values over h of the
                    // columns m2 = g + P j; each takes the twiddle W_L2^(h m2) (none
                    // for h = 0) and their P-point DFTs complete the column's
                    // transform: slot j P + q of the lane holds bin k1 + L1 (g + P j + L1 q)
                    // (the two forms compile to differently contracted products: INT8, whose
                    // codes and scales would show it, keeps the one it always had)
                    const int k1 = r / P, h = r % P;
                    // lane rows of L1 + 1 values in the second exchange: writes (fixed m)
                    // and reads (fixed h, j) both fall in distinct banks
                    constexpr int XR = L1 + 1;
                    static_assert(C::L2 * XR <= EXG, "second exchange exceeds the group's area");
                    float2 w[L1];
                    if constexpr (C::SPLIT) {
                        split_exchange(eg, v, w, [&](int k) { return k * C::EXR + r; },
                                       [&](int m) { return k1 * C::EXR + h + P * m; });
                        dft_regs<L1>(w);
                        wave_sync();   // the first exchange has been read
                        float2 y[L1];
                        split_exchange(eg, w, y, [&](int m) { return r * XR + m; },
                                       [&](int i) { return (k1 * P + i % P) * XR + h + P * (i / P); });
#pragma unroll
                        for (int j = 0; j < L1 / P; ++j) {
#pragma unroll
                            for (int q = 0; q < P; ++q) {
                                float2 u = y[j * P + q];
                                if (q > 0) {
                                    const float2 t = tw2[(q - 1) * (L1 / P) + j];
                                    u = make_float2(u.x * t.x - u.y * t.y, u.x * t.y + u.y * t.x);
                                }
                                w[j * P + q] = u;
                            }
                            dft_regs<P>(w + j * P);
                        }
                    } else {
                        float2 *e = reinterpret_cast<float2 *>(eg);
#pragma unroll
                        for (int k = 0; k < L1; ++k) e[k * C::EXR + r] = v[k];
                        wave_sync();
#pragma unroll
                        for (int m = 0; m < L1; ++m) w[m] = e[k1 * C::EXR + h + P * m];
                        dft_regs<L1>(w);
                        wave_sync();   // the first exchange has been read
#pragma unroll
                        for (int m = 0; m < L1; ++m) e[r * XR + m] = w[m];
                        wave_sync();
#pragma unroll
                        for (int j = 0; j < L1 / P; ++j) {
#pragma unroll
                            for (int q = 0; q < P; ++q) {
                                float2 y = e[(k1 * P + q) * XR + h + P * j];
                                if (q > 0) {
                                    const float2 t = tw2[(q - 1) * (L1 / P) + j];
                                    y = make_float2(y.x * t.x - y.y * t.y, y.x * t.y + y.y * t.x);
                                }
                                w[j * P + q] = y;
                            }
                            dft_regs<P>(w + j * P);
                        }
                    }
                    emit_frame([&](auto tc) { emit_column(0, w, tc); });
                } else {
                    // exchange through LDS; column swizzle r ^ (k1 / U) keeps both the
                    // writes (fixed k1) and the reads (fixed r2) free of bank conflicts
                    // (all U columns of a lane are read before their transforms if
                    // the parts are exchanged in turn)
                    if constexpr (C::SPLIT) {
                        float2 w[U * L2];
                        split_exchange(eg, v, w, [&](int k) { return k * L2 + (r ^ (k / U)); },
                                       [&](int m) { return (r * U + m / L2) * L2 + (m % L2 ^ r); });
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            dft_regs<L2>(w + u * L2);
                            emit_frame([&](auto tc) { emit_column(u * L2, w + u * L2, tc); });
                        }
                    } else {
                        float2 *e = reinterpret_cast<float2 *>(eg);
#pragma unroll
                        for (int k1 = 0; k1 < L1; ++k1) e[k1 * L2 + (r ^ (k1 / U))] = v[k1];
                        wave_sync();
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int k1 = r * U + u;
                            float2 w[L2];
#pragma unroll
                            for (int r2 = 0; r2 < L2; ++r2) w[r2] = e[k1 * L2 + (r2 ^ r)];
                            dft_regs<L2>(w);
                            emit_frame([&](auto tc) { emit_column(u * L2, w, tc); });
                        }
                    }
                }
                wave_sync();
            }
        }
        }   // packs of the group

        if constexpr (!STATS) {
            __syncthreads();
            // store the image: per channel, nrows rows of 32 bytes, 16 bytes per
            // thread; unit u = (c, 16-byte piece e of the channel's nrows rows)
            const int64_t cstride = a.NG * a.n_in * kRowBytes;    // bytes per channel
            uint8_t *db = a.chan + ((a.grp0 + gsel) * a.n_in + n0) * kRowBytes;
            auto store_unit = [&](int c, int e) {
                const uint32_t *src = reinterpret_cast<const uint32_t *>(outbuf + c * CP + e * 16);
                *reinterpret_cast<uint4 *>(db + c * cstride + e * 16) = make_uint4(src[0], src[1], src[2], src[3]);
            };
            constexpr int SU = L * R * 2, NJ = (SU + C::THREADS - 1) / C::THREADS;
            if (nrows == R && NJ <= 2) {
                // unrolled (more units per thread would hold their loads in registers)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int u = tid + j * C::THREADS;
                    if (SU % C::THREADS == 0 || u < SU) store_unit(u / (2 * R), u % (2 * R));
                }
            } else if (nrows == R) {
                for (int u = tid; u < SU; u += C::THREADS) store_unit(u / (2 * R), u % (2 * R));
            } else {
                for (int u = tid; u < L * nrows * 2; u += C::THREADS) store_unit(u / (nrows * 2), u % (nrows * 2));
            }
        }
    }

    if constexpr (STATS) {
        // Deterministic reduction of the per-lane channel sums: lanes with the same r
        // hold the same channel set; sum them in a fixed order.
        __syncthreads();
        float *red = reinterpret_cast<float *>(smem);   // [THREADS / L2 slots][L2][L1]
        int *redp = reinterpret_cast<int *>(red + C::THREADS * L1);
#pragma unroll
        for (int i = 0; i < L1; ++i) red[(gg * L2 + r) * L1 + i] = acc[i];
        if (tid == 0) *redp = 0;
        __syncthreads();
        if (popc) atomicAdd(redp, popc);
        constexpr int NSLOT = C::THREADS / L2;
        // partial row of this workgroup: L channel sums, then the populated count
        double *row = a.stats + (int64_t)wg * (L + 1);
        for (int t = tid; t < L; t += C::THREADS) {
            const int rr = t / L1, i = t - rr * L1;
            double sum = 0.0;
            for (int sl = 0; sl < NSLOT; ++sl) sum += (double)red[(sl * L2 + rr) * L1 + i];
            row[chan_of<L, XP>(rr, i)] = sum;
        }
        __syncthreads();
        if (tid == 0) row[L] = (double)*redp;
    }
}

template <int L, int XP, bool STATS, bool DELAY>
__global__ __launch_bounds__((FCfg<L, XP>::THREADS), (STATS || (DELAY && (XP != MWAX_X_FP16 || L == 1024)) ? 1 : std::max(1, FCfg<L, XP>::MINW))) void fengine_kernel(FArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    fengine_body<L, XP, STATS, DELAY>(a, blockIdx.x, gridDim.x, 0, smem);
}

// Batched form: workgroups [block0[d], block0[d+1]) of the launch work on
// descriptor d (a segment of one plan of the batch); the rest return at once.
// Not held to MINW waves: binary16 compiles to three per SIMD up to L = 512 as it is,
// and at L = 1024 (two) a third changes nothing (60 and 96 tiles, 195 spectra: 165.5
// us, held to three 164.9).
template <int L, int XP, bool STATS>
__global__ __launch_bounds__((FCfg<L, XP>::THREADS)) void fengine_batch_kernel(FBatchArgs b) {
    extern __shared__ __align__(16) uint8_t smem[];
    // the tables are read through the constant address space (scalar loads)
    const int nd = load_uniform(b.ndesc);
    const int blk = blockIdx.x;
    if (blk >= load_uniform(b.block0 + nd)) return;
    int d = 0;
    while (load_uniform(b.block0 + d + 1) <= blk) ++d;
    const FArgs a = load_uniform(b.desc + d);
    const int first = load_uniform(b.block0 + d), count = load_uniform(b.block0 + d + 1) - first;
    fengine_body<L, XP, STATS>(a, blk - first, count, first & 7, smem);
}

template <int L, int XP>
constexpr int cfg_value_lds(bool stats) {
    using C = FCfg<L, XP>;
    return stats ? (C::STAGE_BYTES + C::EX_BYTES > C::RED_BYTES ? C::STAGE_BYTES + C::EX_BYTES : C::RED_BYTES)
                 : C::OUT_BYTES + C::STAGE_BYTES + C::EX_BYTES;
}

// Workgroups of a single-plan launch over `items` items: whole rounds (a last round
// of a few items costs as much as a full one), so that each workgroup's set-up
// (twiddles, scales) is spread over several items, and no more than cap.  As many
// rounds as bring the launch to kLeast workgroups or fewer, but no more than `most`,
// with which large launches have more workgroups.
// Up to an eighth past kLeast a round of one item each is the faster: 64 inputs,
// 2,112 items, INT8, L = 512 / 1024: 40.0, 69.4 us in two rounds, 38.5, 66.6 in one
// (2,560 items: 41.2, 71.5 in two, 42.8, 74.8 in one).  Rounds of the 8 XCDs.  256
// tiles, 1 s INT8 at L = 128 / 256: 881, 983 -> 720, 809 us with 65,536 workgroups
// (2.4 rounds) before; 64 tiles: 242 -> 175; 128 tiles at L = 512 / 1024: 564, 580 ->
// 482, 502; 256 tiles, 8 s: 19.5 -> 20 rounds, 5.59 -> 5.41 ms.
int main_grid(int64_t items, int64_t cap, int64_t most) {
    if (items <= kLeast) return (int)items;
    const int64_t fill = items < kLeast / 8 * 9 ? 1 : (items + kLeast - 1) / kLeast;
    const int64_t rounds = std::max((items + cap - 1) / cap, std::min(most, fill));
    return (int)(((items + rounds - 1) / rounds + 7) / 8 * 8);
}

template <int L, int XP>
hipError_t launch_L(const FArgs &a, hipStream_t s) {
    using C = FCfg<L, XP>;
    const bool stats = a.stats_mode != 0;
    if (a.R != C::R) return hipErrorInvalidValue;
    const int lds = fengine_lds_bytes(L, XP, a.R, stats);
    int grid = fengine_grid(a.n_in, a.R, a.ngrp, stats);
    if (!stats) {
        const int64_t items = (int64_t)a.ngrp * ((a.n_in + C::R - 1) / C::R);
        grid = main_grid(items, C::GRID_CAP, C::most_rounds(items));
    }
    if (grid < 1) return hipSuccess;
    // allow dynamic LDS beyond the default limit (once per instantiation)
    const int variant = stats ? 1 : (a.dl ? 2 : 0);
    const void *fns[3] = {reinterpret_cast<const void *>(&fengine_kernel<L, XP, false, false>),
                          reinterpret_cast<const void *>(&fengine_kernel<L, XP, true, false>),
                          reinterpret_cast<const void *>(&fengine_kernel<L, XP, false, true>)};
    static bool attr_done[3] = {false, false, false};
    if (!attr_done[variant]) {
        (void)hipFuncSetAttribute(fns[variant], hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
        attr_done[variant] = true;
    }
    if (variant == 1)
        hipLaunchKernelGGL((fengine_kernel<L, XP, true, false>), dim3((unsigned)grid), dim3(C::THREADS), lds, s, a);
    else if (variant == 2)
        hipLaunchKernelGGL((fengine_kernel<L, XP, false, true>), dim3((unsigned)grid), dim3(C::THREADS), lds, s, a);
    else
        hipLaunchKernelGGL((fengine_kernel<L, XP, false, false>), dim3((unsigned)grid), dim3(C::THREADS), lds, s, a);
    return hipGetLastError();
}

template <int L, int XP>
hipError_t prepare_batch_L() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&fengine_batch_kernel<L, XP, true>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&fengine_batch_kernel<L, XP, false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    return e;
}

template <int L, int XP>
hipError_t launch_batch_L(bool stats, const FBatchArgs &b, int grid, hipStream_t s) {
    const int lds = cfg_value_lds<L, XP>(stats);
    if (stats)
        hipLaunchKernelGGL((fengine_batch_kernel<L, XP, true>), dim3((unsigned)grid), dim3(FCfg<L, XP>::THREADS), lds, s, b);
    else
        hipLaunchKernelGGL((fengine_batch_kernel<L, XP, false>), dim3((unsigned)grid), dim3(FCfg<L, XP>::THREADS), lds, s, b);
    return hipGetLastError();
}

#define MWAX_L_SWITCH(CALL)                         \
    switch (L) {                                    \
        case 1: return CALL(1);                     \
        case 2: return CALL(2);                     \
        case 4: return CALL(4);                     \
        case 8: return CALL(8);                     \
        case 16: return CALL(16);                   \
        case 32: return CALL(32);                   \
        case 64: return CALL(64);                   \
        case 128: return CALL(128);                 \
        case 256: return CALL(256);                 \
        case 512: return CALL(512);                 \
        case 1024: return CALL(1024);               \
        default: return hipErrorInvalidValue;       \
    }

template <int XP>
hipError_t launch_batch_xp(int L, bool stats, const FBatchArgs &b, int grid, hipStream_t s) {
#define MWAX_CALL(LL) launch_batch_L<LL, XP>(stats, b, grid, s)
    MWAX_L_SWITCH(MWAX_CALL)
#undef MWAX_CALL
}

template <int XP>
hipError_t prepare_batch_xp(int L) {
#define MWAX_CALL(LL) prepare_batch_L<LL, XP>()
    MWAX_L_SWITCH(MWAX_CALL)
#undef MWAX_CALL
}

template <int XP>
hipError_t launch_xp(int L, const FArgs &a, hipStream_t s) {
    switch (L) {
        case 1: return launch_L<1, XP>(a, s);
        case 2: return launch_L<2, XP>(a, s);
        case 4: return launch_L<4, XP>(a, s);
        case 8: return launch_L<8, XP>(a, s);
        case 16: return launch_L<16, XP>(a, s);
        case 32: return launch_L<32, XP>(a, s);
        case 64: return launch_L<64, XP>(a, s);
        case 128: return launch_L<128, XP>(a, s);
        case 256: return launch_L<256, XP>(a, s);
        case 512: return launch_L<512, XP>(a, s);
        case 1024: return launch_L<1024, XP>(a, s);
        default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
__global__ void twiddle_kernel(float2 *tw, int L) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= L) return;
    // exp(-2 pi i k / L) in FP64, rounded to FP32; quarter turns exact.
    const int q4 = (4 * k) % L == 0 ? (4 * k) / L : -1;
    if (q4 >= 0) {
        const float re[4] = {1.0f, 0.0f, -1.0f, 0.0f};
        const float im[4] = {0.0f, -1.0f, 0.0f, 1.0f};
        tw[k] = make_float2(re[q4], im[q4]);
        return;
    }
    double sn, cs;
    sincospi(-2.0 * (double)k / (double)L, &sn, &cs);
    tw[k] = make_float2((float)cs, (float)sn);
}

// Scales of channel c from its power sum and populated-frame count over the
// calibration window:
//   sigma^2 = power / (2 populated),  s = 5 sigma / 127,  inv_s = 127 / (5 sigma)
// (s = inv_s = 1 for a channel of zero power).  With no populated frame the
// window holds only zeroed samples: the channel keeps last[] (the scales of the
// plan's most recent calibrated integration).  Otherwise last[] is updated.
__device__ __forceinline__ void finish_scale(double sum, double count, int L, float *scales, float *last, int c) {
    float s = last[c], inv = last[L + c];
    if (count > 0.0) {
        const double var = sum / (2.0 * count);
        s = 1.0f;
        inv = 1.0f;
        if (var > 0.0) {
            const double sd = sqrt(var);
            s = (float)(5.0 * sd / 127.0);
            inv = (float)(127.0 / (5.0 * sd));
        }
        last[c] = s;
        last[L + c] = inv;
    }
    scales[c] = s;
    scales[L + c] = inv;
}

// Scales of channel c from the partial rows of nwg workgroups ([nwg][L + 1]: L
// power sums, then the populated-frame count), reduced in a fixed order so the
// result is bitwise reproducible.
__device__ void calib_finish_channel(const double *stats, int nwg, int L, float *scales, float *last, int c) {
    __shared__ double part[256], cnt[256];
    __syncthreads();   // part/cnt of a previous call on this workgroup fully read
    double t = 0.0, n = 0.0;
    for (int w = threadIdx.x; w < nwg; w += 256) {
        t += stats[(int64_t)w * (L + 1) + c];
        n += stats[(int64_t)w * (L + 1) + L];
    }
    part[threadIdx.x] = t;
    cnt[threadIdx.x] = n;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            part[threadIdx.x] += part[threadIdx.x + h];
            cnt[threadIdx.x] += cnt[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    finish_scale(part[0], cnt[0], L, scales, last, c);
}

__global__ void calib_finish_kernel(const double *stats, int nwg, int L, float *scales, float *last) {
    calib_finish_channel(stats, nwg, L, scales, last, blockIdx.x);
}

// Wide transforms (L = 6400): one workgroup per 16 channels.  Thread (channel
// cl, slice sl) sums the partial rows sl, sl + 16, ... into eight running sums
// (row sl + 16 (8 k + i) into sum i, so eight loads are in flight); the eight
// sums, then the sixteen slices (and the frame counts) are added in a fixed
// order.
constexpr int kWideCh = 16, kWideSl = 256 / kWideCh;
__global__ __launch_bounds__(256) void calib_finish_wide_kernel(const double *stats, int nwg, int L, float *scales,
                                                                float *last) {
    constexpr int kAcc = 8;
    __shared__ double part[kWideSl][kWideCh], cnt[kWideSl];
    const int cl = threadIdx.x % kWideCh, sl = threadIdx.x / kWideCh, c = blockIdx.x * kWideCh + cl;
    const int cc = c < L ? c : L;   // channels past L read the count column instead
    double ts[kAcc] = {}, ns[kAcc] = {};
    int w = sl;
    for (; w + kWideSl * (kAcc - 1) < nwg; w += kWideSl * kAcc) {
#pragma unroll
        for (int i = 0; i < kAcc; ++i) {
            ts[i] += stats[(int64_t)(w + kWideSl * i) * (L + 1) + cc];
            ns[i] += stats[(int64_t)(w + kWideSl * i) * (L + 1) + L];
        }
    }
#pragma unroll
    for (int i = 0; i < kAcc; ++i) {
        if (w + kWideSl * i < nwg) {
            ts[i] += stats[(int64_t)(w + kWideSl * i) * (L + 1) + cc];
            ns[i] += stats[(int64_t)(w + kWideSl * i) * (L + 1) + L];
        }
    }
    double t = 0.0, n = 0.0;
#pragma unroll
    for (int i = 0; i < kAcc; ++i) {
        t += ts[i];
        n += ns[i];
    }
    part[sl][cl] = t;
    if (cl == 0) cnt[sl] = n;
    __syncthreads();
    if (sl != 0 || c >= L) return;
    t = 0.0;
    n = 0.0;
    for (int k = 0; k < kWideSl; ++k) {
        t += part[k][cl];
        n += cnt[k];
    }
    finish_scale(t, n, L, scales, last, c);
}

// One workgroup per (channel, descriptor).  The descriptors of one instance are
// consecutive and its first one carries their number (n_chain); that workgroup
// processes them in order, so an integration whose window holds no populated
// frame takes the scales of the instance's previous calibrated integration,
// also within one call.  Other descriptors and channels past L return at once.
__global__ void calib_batch_kernel(const CalDesc *desc, const int32_t *ndesc) {
    const int d = blockIdx.y, c = blockIdx.x;
    if (d >= *ndesc) return;
    const CalDesc head = desc[d];
    if (head.n_chain == 0 || c >= head.L) return;
    for (int k = 0; k < head.n_chain; ++k) {
        const CalDesc cd = desc[d + k];
        if (cd.copy_src) {
            if (threadIdx.x == 0) {
                cd.scales[c] = cd.copy_src[c];
                cd.scales[cd.L + c] = cd.copy_src[cd.L + c];
            }
        } else {
            calib_finish_channel(cd.stats, cd.nwg, cd.L, cd.scales, cd.last, c);
        }
    }
}

__global__ void copy_scales_kernel(const float *src, float *dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

__global__ void fill_f32_kernel(float *dst, float v, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = v;
}

// Bytes of four dwords regrouped: out[k] = byte k of a, b, c, d.
__device__ __forceinline__ void transpose4x4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t out[4]) {
    const uint32_t p = __builtin_amdgcn_perm(b, a, 0x05010400u), q = __builtin_amdgcn_perm(b, a, 0x07030602u);
    const uint32_t r = __builtin_amdgcn_perm(d, c, 0x05010400u), t = __builtin_amdgcn_perm(d, c, 0x07030602u);
    out[0] = __builtin_amdgcn_perm(r, p, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(r, p, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(t, q, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(t, q, 0x07060302u);
}

// Each byte equal to -128 becomes -127.
__device__ __forceinline__ uint32_t clamp_m128(uint32_t x) {
    const uint32_t z = x ^ 0x80808080u;                                        // zero bytes are the ones
    return x + (~(((z & 0x7f7f7f7fu) + 0x7f7f7f7fu) | z | 0x7f7f7f7fu) >> 7);
}

// Canonical [m][c][n][re, im] (elements of ES bytes) <-> row groups.  A thread
// moves the two inputs of one tile over one row group of one channel: G loads
// (load) or stores (read) of 4 ES bytes, consecutive threads consecutive tiles,
// and two whole 32-byte rows, regrouped in registers.  Bound by HBM: 256 inputs x
// 128 channels x 10,000 spectra INT8 (1.31 GB moved) took 2.41 ms with one
// element per thread and byte-wide row accesses, now 0.276 ms (4.75 TB/s, the
// rate of a large copy).  The canonical data are only
// aligned to an element, which vector loads allow.
template <int ES, bool LOAD>
__global__ __launch_bounds__(256) void repack_kernel(RepackArgs a) {
    constexpr int G = 16 / ES;
    struct __attribute__((packed, aligned(ES))) Two { uint32_t d[ES]; };   // both inputs of one spectrum
    const uint32_t ntile = (uint32_t)a.n_in / 2;
    const uint32_t u = blockIdx.x * 256 + threadIdx.x;
    if (u >= ntile * (uint32_t)a.L) return;
    const int c = (int)(u / ntile), n = 2 * (int)(u - c * ntile);
    const int64_t mstride = (int64_t)a.L * a.n_in * 2 * ES;   // bytes between spectra
    uint8_t *cv0 = reinterpret_cast<uint8_t *>(a.canon) + a.m0 * mstride + (int64_t)u * 4 * ES;
    const int64_t ngrp = (a.nframes + G - 1) / G;
    for (int64_t g = blockIdx.y; g < ngrp; g += gridDim.y) {
        const int valid = (int)min((int64_t)G, a.nframes - g * G);
        uint8_t *cv = cv0 + g * G * mstride;
        uint4 *row = reinterpret_cast<uint4 *>(a.chan + (((int64_t)c * a.NG + a.grp0 + g) * a.n_in + n) * kRowBytes);
        uint32_t w[2][8];    // the two rows
        uint32_t v[G][ES];   // spectrum f: (re, im) of both inputs
        if constexpr (LOAD) {
            // addresses clamped to the last spectrum, so that every load is in flight at once
#pragma unroll
            for (int f = 0; f < G; ++f) {
                const Two t = *reinterpret_cast<const Two *>(cv + min(f, valid - 1) * mstride);
#pragma unroll
                for (int e = 0; e < ES; ++e) v[f][e] = f < valid ? t.d[e] : 0u;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint4 lo = row[2 * q], hi = row[2 * q + 1];
                w[q][0] = lo.x, w[q][1] = lo.y, w[q][2] = lo.z, w[q][3] = lo.w;
                w[q][4] = hi.x, w[q][5] = hi.y, w[q][6] = hi.z, w[q][7] = hi.w;
            }
        }
        // dwords re, re + 2 of a row: the real and imaginary parts of frames
        // 4 fb .. (INT8) or 2 fb .. (binary16)
        if constexpr (ES == 1) {
#pragma unroll
            for (int fb = 0; fb < 4; ++fb) {
                const int re = (fb >> 1) * 4 + (fb & 1);
                uint32_t t[4];
                if constexpr (LOAD) {
                    transpose4x4(clamp_m128(v[4 * fb][0]), clamp_m128(v[4 * fb + 1][0]), clamp_m128(v[4 * fb + 2][0]),
                                 clamp_m128(v[4 * fb + 3][0]), t);
                    w[0][re] = t[0], w[0][re + 2] = t[1], w[1][re] = t[2], w[1][re + 2] = t[3];
                } else {
                    transpose4x4(w[0][re], w[0][re + 2], w[1][re], w[1][re + 2], t);
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[4 * fb + k][0] = t[k];
                }
            }
        } else if constexpr (ES == 2) {
#pragma unroll
            for (int fb = 0; fb < 4; ++fb) {
                const int re = (fb >> 1) * 4 + (fb & 1);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if constexpr (LOAD) {
                        const uint32_t x = v[2 * fb][q], y = v[2 * fb + 1][q];
                        w[q][re] = (x & 0xffffu) | (y << 16);
                        w[q][re + 2] = (x >> 16) | (y & 0xffff0000u);
                    } else {
                        const uint32_t r = w[q][re], i = w[q][re + 2];
                        v[2 * fb][q] = (r & 0xffffu) | (i << 16);
                        v[2 * fb + 1][q] = (r >> 16) | (i & 0xffff0000u);
                    }
                }
            }
        } else {
#pragma unroll
            for (int f = 0; f < 4; ++f)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if constexpr (LOAD) w[q][f] = v[f][2 * q], w[q][4 + f] = v[f][2 * q + 1];
                    else v[f][2 * q] = w[q][f], v[f][2 * q + 1] = w[q][4 + f];
                }
        }
        if constexpr (LOAD) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                row[2 * q] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
                row[2 * q + 1] = make_uint4(w[q][4], w[q][5], w[q][6], w[q][7]);
            }
        } else {
#pragma unroll
            for (int f = 0; f < G; ++f) {
                if (f < valid) {
                    Two t;
#pragma unroll
                    for (int e = 0; e < ES; ++e) t.d[e] = v[f][e];
                    *reinterpret_cast<Two *>(cv + f * mstride) = t;
                }
            }
        }
    }
}

template <int ES>
void launch_repack_es(const RepackArgs &a, dim3 grid, hipStream_t s) {
    if (a.to_internal) hipLaunchKernelGGL((repack_kernel<ES, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((repack_kernel<ES, false>), grid, dim3(256), 0, s, a);
}

}  // namespace

template <int XP>
static int cfg_value(int L, int what) {
#define MWAX_CFG_CASE(LL)                                                                     \
    case LL:                                                                                  \
        return what == 0 ? FCfg<LL, XP>::R                                                    \
                         : (what == 1 ? FCfg<LL, XP>::OUT_BYTES + FCfg<LL, XP>::STAGE_BYTES + \
                                            FCfg<LL, XP>::EX_BYTES                            \
                                      : std::max(FCfg<LL, XP>::STAGE_BYTES + FCfg<LL, XP>::EX_BYTES, \
                                                 FCfg<LL, XP>::RED_BYTES));
    switch (L) {
        MWAX_CFG_CASE(1) MWAX_CFG_CASE(2) MWAX_CFG_CASE(4) MWAX_CFG_CASE(8) MWAX_CFG_CASE(16)
        MWAX_CFG_CASE(32) MWAX_CFG_CASE(64) MWAX_CFG_CASE(128) MWAX_CFG_CASE(256)
        MWAX_CFG_CASE(512) MWAX_CFG_CASE(1024)
        default: return -1;
    }
#undef MWAX_CFG_CASE
}

static int cfg_of(int L, int xprec, int what) {
    switch (xprec) {
        case MWAX_X_INT8: return cfg_value<MWAX_X_INT8>(L, what);
        case MWAX_X_FP16: return cfg_value<MWAX_X_FP16>(L, what);
        default: return cfg_value<MWAX_X_FP32>(L, what);
    }
}

int fengine_grid(int n_in, int R, int ngrp, bool stats) {
    const int64_t items = (int64_t)ngrp * ((n_in + R - 1) / R);
    // stats mode writes one partial row per workgroup: keep that buffer small
    const int64_t cap = stats ? kStatsMaxWG : 65536;
    return (int)(items < cap ? items : cap);
}

int fengine_pick_R(int L, int xprec, int /*n_in*/, int /*lds_limit*/) { return cfg_of(L, xprec, 0); }

int fengine_lds_bytes(int L, int xprec, int /*R*/, bool stats) { return cfg_of(L, xprec, stats ? 2 : 1); }

hipError_t launch_fengine(int L, int xprec, const FArgs &a, hipStream_t s) {
    switch (xprec) {
        case MWAX_X_INT8: return launch_xp<MWAX_X_INT8>(L, a, s);
        case MWAX_X_FP16: return launch_xp<MWAX_X_FP16>(L, a, s);
        case MWAX_X_FP32: return launch_xp<MWAX_X_FP32>(L, a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fengine_batch(int L, int xprec, bool stats, const FBatchArgs &b, int grid, hipStream_t s) {
    if (grid < 1) return hipSuccess;
    switch (xprec) {
        case MWAX_X_INT8: return launch_batch_xp<MWAX_X_INT8>(L, stats, b, grid, s);
        case MWAX_X_FP16: return launch_batch_xp<MWAX_X_FP16>(L, stats, b, grid, s);
        case MWAX_X_FP32: return launch_batch_xp<MWAX_X_FP32>(L, stats, b, grid, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t fengine_prepare_batch(int L, int xprec) {
    switch (xprec) {
        case MWAX_X_INT8: return prepare_batch_xp<MWAX_X_INT8>(L);
        case MWAX_X_FP16: return prepare_batch_xp<MWAX_X_FP16>(L);
        case MWAX_X_FP32: return prepare_batch_xp<MWAX_X_FP32>(L);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_calib_batch(const CalDesc *desc, const int32_t *ndesc, int max_desc, int max_L, hipStream_t s) {
    if (max_desc < 1) return hipSuccess;
    hipLaunchKernelGGL(calib_batch_kernel, dim3((unsigned)max_L, (unsigned)max_desc), dim3(256), 0, s, desc, ndesc);
    return hipGetLastError();
}

hipError_t launch_twiddles(float2 *tw, int L, hipStream_t s) {
    hipLaunchKernelGGL(twiddle_kernel, dim3((L + 255) / 256), dim3(256), 0, s, tw, L);
    return hipGetLastError();
}

hipError_t launch_calib_finish(const double *stats, int nwg, int L, float *scales, float *last, hipStream_t s) {
    if (L == kUltraFineL)
        hipLaunchKernelGGL(calib_finish_wide_kernel, dim3((L + kWideCh - 1) / kWideCh), dim3(256), 0, s, stats, nwg, L,
                           scales, last);
    else
        hipLaunchKernelGGL(calib_finish_kernel, dim3(L), dim3(256), 0, s, stats, nwg, L, scales, last);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *dst, float v, int n, hipStream_t s) {
    hipLaunchKernelGGL(fill_f32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, dst, v, n);
    return hipGetLastError();
}

hipError_t launch_copy_scales(const float *src, float *dst, int n, hipStream_t s) {
    hipLaunchKernelGGL(copy_scales_kernel, dim3((n + 255) / 256), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

hipError_t launch_repack(const RepackArgs &a, hipStream_t s) {
    if (a.nframes <= 0 || a.n_in & 1) return a.n_in & 1 ? hipErrorInvalidValue : hipSuccess;
    const int64_t units = (int64_t)a.L * (a.n_in / 2), ngrp = (a.nframes + a.G - 1) / a.G;
    const dim3 grid((unsigned)((units + 255) / 256), (unsigned)std::min<int64_t>(ngrp, 65535));
    switch (a.esize) {
        case 1: launch_repack_es<1>(a, grid, s); break;
        case 2: launch_repack_es<2>(a, grid, s); break;
        case 4: launch_repack_es<4>(a, grid, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mwax
