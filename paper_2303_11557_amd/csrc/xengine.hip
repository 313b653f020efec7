// X-engine of the FX correlator (Morrison et al. 2023, Sec. 2.5.2): for each
// fine channel c and every input pair n1 >= n2 (autos included),
//   V[c][n1,n2] += sum_m X_n1[m,c] conj(X_n2[m,c]),
// accumulated into per-integration device integrators (Sec. 2.5.2, time
// integration) in the packed lower-triangle order p = n1(n1+1)/2 + n2.
//
// The complex Hermitian rank-k update is run as two real GEMMs over the
// channel-major rows of each input (real and imaginary parts of G frames):
//   Re V[n1,n2] = sum (re1 re2 + im1 im2) = A_n1 . A_n2,   A = the row
//   Im V[n1,n2] = sum (im1 re2 - re1 im2) = A_n1 . B_n2,   B = the row with
//                 each frame's (re, im) replaced by (-im, re)
// so every complex multiply-accumulate is four real ones and nothing is
// wasted on the real expansion.  Each 16-byte half of a row holds the real
// parts of 8 (FP16: 4) frames followed by their imaginary parts, so B is made
// from A in registers by swapping the two 8-byte quarters of a half and
// negating one of them.  Work is split into 64 x 64 blocks of the lower triangle,
// four to a workgroup.
//
//   INT8: v_mfma_i32_32x32x32_i8, int32 partials flushed to int64 integrators
//         at most every 65536 spectra (|partial| < 518160 * 4096 < 2^31).
//   FP16: v_mfma_f32_32x32x16_f16, FP32 partials flushed to FP64 integrators.
//   FP32: v_mfma_f32_32x32x2_f32, two-level FP32 partials (see xengine_f32)
//         flushed to FP64 integrators every 2048 spectra.
#include <type_traits>

#include "mwax_internal.h"

namespace mwax {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

constexpr int kTile = kXTile;       // tile edge in inputs (single-plan launches of more than
                                    // kXSmallInputs; a batch instance may take kTileSmall)
constexpr int kTileSmall = kXTileSmall;
constexpr int kThreads = 256;       // 4 waves

// Lower-triangle tile index t -> (I, J), I >= J, t = I(I+1)/2 + J.
__device__ __forceinline__ void tile_ij(int t, int &I, int &J) {
    int i = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    while (i * (i + 1) / 2 > t) --i;
    I = i;
    J = t - i * (i + 1) / 2;
}

// Lower triangle of m x m blocks, one block per wave, four to a workgroup.
// Workgroup t of a channel, with nt = m / 2 tiles of 2 x 2 blocks along an edge:
//   t < nt (nt - 1) / 2: the four blocks of an off-diagonal tile;
//   then, for each of g sets of four diagonal tiles (three blocks each), three
//   workgroups: the blocks of one tile and one block of the set's last tile;
//   then the diagonal tiles left, three blocks and an idle wave each;
//   for odd m, the last row of blocks, three columns to a workgroup, its diagonal
//   block with the last of them.
// An idle wave does not only leave its SIMD empty: the other SIMDs, which have
// more to do, hold back the waves it would run instead.
// Four LDS slots hold the rows of a block each; wave w copies slot w.
struct TriBlock {
    int ra, rb;          // row blocks of the wave's rows and columns (ra >= rb), or ra < 0: idle
    int sa, sb;          // the slots that hold them
    int copy;            // row block this wave copies into its slot
};
__host__ __device__ inline int tri_sets(int m) { return m / 8; }
__host__ __device__ inline int tri_groups(int m, int g) {
    const int nt = m / 2, strips = (m + 1) / 3 > 1 ? (m + 1) / 3 : 1;
    return nt * (nt - 1) / 2 + nt - g + (m & 1 ? strips : 0);
}
__device__ __forceinline__ TriBlock tri_block(int m, int g, int t, int role, int wave) {
    const int nt = m / 2, noff = nt * (nt - 1) / 2;
    TriBlock b;
    if (t < noff) {
        int I, J;
        tile_ij(t, I, J);
        ++I;
        b.ra = 2 * I + (role >> 1), b.rb = 2 * J + (role & 1);
        b.sa = role >> 1, b.sb = 2 + (role & 1);
        b.copy = wave < 2 ? 2 * I + wave : 2 * J + (wave & 1);
        return b;
    }
    const int u = t - noff, w = u - (nt - g);
    if (w >= 0) {
        const int r = m - 1, col = 3 * w + role;
        const bool diag = role == 3 && 3 * w + 3 >= r;
        b.ra = diag || (role < 3 && col < r) ? r : -1, b.rb = diag ? r : col;
        b.sa = 0, b.sb = diag ? 0 : 1 + role;
        b.copy = wave == 0 ? r : min(3 * w + wave - 1, r);
        return b;
    }
    const int j = u % 3;
    const bool group = u < 3 * g;
    const int d = group ? u / 3 * 4 + j : 4 * g + (u - 3 * g), e = group ? u / 3 * 4 + 3 : d;
    // blocks of a diagonal tile: 0 (0, 0), 1 (1, 0), 2 (1, 1)
    const int k = role < 3 ? role : j, x = role < 3 ? d : e, s0 = role < 3 ? 0 : 2;
    b.ra = 2 * x + (k > 0), b.rb = 2 * x + (k > 1);
    b.sa = s0 + (k > 0), b.sb = s0 + (k > 1);
    if (role == 3 && !group) b.ra = -1;
    b.copy = 2 * (wave < 2 ? d : e) + (wave & 1);
    return b;
}

// Workgroups are handed to the 8 XCDs round-robin.  Renumber them so the
// workgroups one XCD receives carry consecutive logical indices: the tiles of a
// channel then share that XCD's L2 for the input panels they all read.
__device__ __forceinline__ int xcd_logical(int b, int nb) {
    const int full = nb & ~7;
    if (b >= full) return b;
    return (b & 7) * (full >> 3) + (b >> 3);
}

// Negation of four int8 values in [-127, 127].
__device__ __forceinline__ uint32_t neg_i8x4(uint32_t x) {
    return (0x80808080u - (x & 0x7f7f7f7fu)) ^ (~x & 0x80808080u);
}

template <int XP>
struct MfmaT;
template <>
struct MfmaT<MWAX_X_INT8> {
    using acc_t = v16i;                          // 16 spectra per row group
    // a row group adds at most (127 * 128 + 127^2) * 16 = 518160 to a partial
    // (the Im operand holds one's complements, see below), so 4096 groups
    // (65536 spectra) stay below 2^31
    static constexpr int kFlushGroups = 4096;
    __device__ static acc_t mma(uint4 a, uint4 b, acc_t c) {
        v4i av, bv;
        __builtin_memcpy(&av, &a, 16);
        __builtin_memcpy(&bv, &b, 16);
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, c, 0, 0, 0);
    }
};
template <>
struct MfmaT<MWAX_X_FP16> {
    using acc_t = v16f;                           // 8 spectra per row group
    static constexpr int kFlushGroups = 8192;     // 65536 spectra per FP32 partial
    __device__ static acc_t mma(uint4 a, uint4 b, acc_t c) {
        v8h av, bv;
        __builtin_memcpy(&av, &a, 16);
        __builtin_memcpy(&bv, &b, 16);
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv, c, 0, 0, 0);
    }
};

// The B operand of Im V (see the file comment) from that of Re V.  INT8: EXACT or by
// one's complements (see below).
template <int XP, bool EXACT>
__device__ __forceinline__ uint4 im_operand(uint4 v) {
    if constexpr (XP == MWAX_X_FP16) return make_uint4(v.z ^ 0x80008000u, v.w ^ 0x80008000u, v.x, v.y);
    else if constexpr (EXACT) return make_uint4(neg_i8x4(v.z), neg_i8x4(v.w), v.x, v.y);
    else return make_uint4(~v.z, ~v.w, v.x, v.y);
}

// One workgroup = one channel x four 64 x 64 blocks of the lower triangle (see
// TriBlock; off the diagonal a 128 x 128 tile), one per wave in 2 x 2 parts of
// 32 x 32, with real and imaginary accumulators for every part (128 accumulator
// registers).  Channelise to emission, 128 x 128 tiles only / this: INT8, 512 inputs,
// 80,000 spectra 11.22 / 10.99 ms; 140 inputs, 20,000 spectra 739 / 680 us; FP16, 186
// inputs, 1,024 channels, 1,250 spectra 1,067 / 1,024 us; 440 inputs, 5,000 spectra
// 1,155 / 1,084 us.
// Two workgroups share a CU (two waves per SIMD), so one workgroup's barrier
// latency is covered by the other's matrix work.
//
// The K loop runs over stages of kXG row groups.  Stages are copied from global
// memory straight into LDS (16 bytes per lane, no register staging and no LDS
// store instructions) into a ring of kNBuf stage buffers, kDist stages
// ahead of the matrix work, with one barrier per stage.  Each wave copies the
// rows of one slot, 32 whole rows (1 KB of global memory) at a time into an LDS block
// laid out [16-byte half][row], the layout the fragment reads want.  The ring buffers
// are separate LDS objects, so the compiler can tell a read of one buffer from the copies still
// landing in the others and does not wait for those.
//
// The Im operand B2 is formed in registers from the B fragment: its two 8-byte
// quarters (real parts, imaginary parts of the same frames) are swapped and the
// imaginary one is flipped -- FP16 by its sign bits, INT8 by its one's
// complement ~x = -x - 1.  The INT8 integrators therefore hold Im V[n1,n2] -
// sum_m re_n1[m], and the autos (whose imaginary parts are zero) hold exactly
// -sum_m re_n1[m]: the pack step subtracts an entry's auto from it, which makes
// the result exact without any extra work in this loop.  With ~im in
// [-128, 126] a row group adds at most 127 * 128 * 16 + 127^2 * 16 to a partial,
// and 65536 spectra stay below 2^31.
constexpr int kXG = 2;                      // row groups per stage
constexpr int kNBuf = 4;                    // stage buffers
constexpr int kDist = 2;                    // stages copied ahead of the matrix work (< kNBuf)
constexpr int kBlock = 32 * kRowBytes;      // LDS bytes of 32 rows: [half][row][16 B]
static_assert((kNBuf == 2 || kNBuf == 4) && kDist >= 1 && kDist < kNBuf, "ring of 2 or 4 stage buffers");

// Stage geometry of a TE x TE tile (TE = 128 or 64).  A 128-edge tile gives each
// of the four waves 64 x 64 outputs (2 x 2 blocks of 32 x 32) and each wave
// copies 64 rows; a 64-edge tile gives each wave one 32 x 32 block and each wave
// copies 32 rows.
template <int TE, int DIST = kDist>
struct TileGeo {
    static_assert(TE == 128 || TE == 64, "tile edge");
    static_assert(DIST >= 1 && DIST < kNBuf, "copies run at most kNBuf - 1 stages ahead");
    static constexpr int MB = TE / 64;                   // 32 x 32 blocks per wave and dimension
    static constexpr int kGroupPitch = TE / 32 * kBlock;
    static constexpr int kPanel = kXG * kGroupPitch;     // one panel (A or B) of a stage
    static constexpr int kStage = 2 * kPanel;
    // first byte of slot w (TE / 2 rows) in a row group: two slots to a panel
    __host__ __device__ static constexpr int slot(int w) { return (w >> 1) * kPanel + (w & 1) * MB * kBlock; }
    static constexpr int kCopiesPerStage = MB * kXG;     // copies per wave per stage
    // s_waitcnt immediate: vmcnt(copies of the DIST - 1 later stages), lgkmcnt(0)
    static constexpr int kWaitCopies = kCopiesPerStage * (DIST - 1);
    static_assert(kWaitCopies < 16, "vmcnt immediate");
    static constexpr int kStageWait = kWaitCopies | (7 << 4);
};
constexpr int kStage = TileGeo<kTile>::kStage;          // stage buffers are sized for the larger tile

struct XLds {
    uint8_t *buf[4];   // the first kNBuf are used
};
constexpr int kStage23 = kNBuf > 2 ? kStage : 16;

// Source of the row groups past the end of a segment (they must read as zero).
__device__ __align__(16) const uint8_t kZeroGroup[kTile * kRowBytes] = {};

// End of a stage: this wave's copies of the next stage have landed (the
// kDist - 1 later stages stay in flight) and its LDS reads have returned; then the
// workgroup barrier.  The barrier carries no memory fence of its own (a fence
// would wait for every copy in flight); the wait provides the ordering, and the
// memory clobber keeps the compiler from moving LDS accesses across it.
template <int TE, int DIST = kDist>
__device__ __forceinline__ void stage_barrier() {
    __builtin_amdgcn_s_waitcnt(TileGeo<TE, DIST>::kStageWait);
    asm volatile("s_barrier" ::: "memory");
}

// ATOMIC: flush with int64 atomic adds (another workgroup may be flushing other
// row groups of the same tile at the same time).
template <int XP, int TE, bool ACTIVE, bool ATOMIC, bool BATCH>
__device__ __forceinline__ void xengine_tile_loop(const XArgs &a, const XLds &lds, int c, const TriBlock &tb) {
    static_assert(!ATOMIC || XP == MWAX_X_INT8, "atomic flushes are exact for integer partials only");
    using GEO = TileGeo<TE>;
    constexpr int MB = GEO::MB, kGroupPitch = GEO::kGroupPitch;
    using T = MfmaT<XP>;
    using acc_t = typename T::acc_t;
    constexpr bool INT8 = XP == MWAX_X_INT8;
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    // Copies: wave w moves the TE / 2 rows of slot w, 32 at a time; lane l takes half
    // l / 32 of its row and lands at byte l * 16 of the rows' block.
    // Rows past the last input are read from a clamped (valid) address and not
    // cleared: row i of A and column j of B reach only output (i, j), and outputs
    // past the last input are never flushed.
    uint32_t off[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
        off[m] = (uint32_t)min((tb.copy * MB + m) * 32 + l32, a.n_in - 1) * kRowBytes + half * 16;
    const uint32_t offZ = (uint32_t)l32 * kRowBytes + half * 16;
    const int64_t gstride = (int64_t)a.n_in * kRowBytes;   // bytes between row groups
    const uint8_t *base = a.chan + ((int64_t)c * a.NG + a.grp0) * gstride;
    const int ldst = GEO::slot(wave);
    const int nstages = (a.ngrp + kXG - 1) / kXG;

    // CHECK: the stage may reach past the segment end (its last stage)
    auto copy_stage = [&](int s, uint8_t *buf, auto check_c) {
        constexpr bool CHECK = decltype(check_c)::value;
#pragma unroll
        for (int k = 0; k < kXG; ++k) {
            const int g = s * kXG + k;
            const bool in = !CHECK || g < a.ngrp;
            const uint8_t *gb = in ? base + (int64_t)g * gstride : kZeroGroup;
#pragma unroll
            for (int m = 0; m < MB; ++m)
                __builtin_amdgcn_global_load_lds(gb + (in ? off[m] : offZ), buf + k * kGroupPitch + ldst + m * kBlock,
                                                 16, 0, 0);
        }
    };

    acc_t re[MB][MB], im[MB][MB];
    // fragment m of a slot's 32 MB rows is its block m; lane (half, l32) reads half
    // `half` of its row l32
    const int fa_off = GEO::slot(tb.sa) + half * 512 + l32 * 16;
    const int fb_off = GEO::slot(tb.sb) + half * 512 + l32 * 16;

    // One stage of matrix-core work from one buffer; the fragments of row group
    // k+1 are read while the MFMAs of group k run.
    auto compute = [&](const uint8_t *st) {
        uint4 fa[2][MB], fb[2][MB];
        auto read = [&](int k, int slot) {
            const int ko = k * kGroupPitch;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                fa[slot][m] = *reinterpret_cast<const uint4 *>(st + ko + fa_off + m * kBlock);
                fb[slot][m] = *reinterpret_cast<const uint4 *>(st + ko + fb_off + m * kBlock);
            }
        };
        read(0, 0);
#pragma unroll
        for (int k = 0; k < kXG; ++k) {
            if (k + 1 < kXG) read(k + 1, (k + 1) & 1);
            const int sl = k & 1;
            uint4 fb2[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m) fb2[m] = im_operand<XP, false>(fb[sl][m]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb2 = 0; nb2 < MB; ++nb2) {
                    re[mb][nb2] = T::mma(fa[sl][mb], fb[sl][nb2], re[mb][nb2]);
                    im[mb][nb2] = T::mma(fa[sl][mb], fb2[nb2], im[mb][nb2]);
                }
        }
        // 2 MB reads and 2 MB^2 MFMAs per row group: the reads of group k+1 are
        // interleaved with the first MFMAs of group k
        constexpr int kReads = 2 * MB, kMfma = 2 * MB * MB;
        __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);    // reads, group 0
#pragma unroll
        for (int k = 0; k + 1 < kXG; ++k) {
#pragma unroll
            for (int q = 0; q < kReads; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one read of group k+1
            }
            if constexpr (kMfma > kReads) __builtin_amdgcn_sched_group_barrier(0x008, kMfma - kReads, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, kMfma, 0);     // MFMAs, last group
    };

    // Iteration on stage s held in buffer B: copy stage s + kDist into a buffer
    // last read by an earlier iteration, matrix work on stage s, wait for
    // stage s + 1, barrier.  Every iteration copies a stage (past the segment end
    // from the zero page), so exactly kCopiesPerStage copies per stage are in
    // flight and no copy sits behind a branch: for a copy behind a branch the
    // compiler would wait for every copy in flight before the next LDS read.
    // CHECK: tail iterations, which may reach past the segment end and skip the
    // matrix work of stages at or past s1.
    using Yes = std::true_type;
    using No = std::false_type;
    auto iteration = [&](int s, int s1, auto b_c, auto check_c) {
        constexpr int B = decltype(b_c)::value;
        constexpr bool CHECK = decltype(check_c)::value;
        copy_stage(s + kDist, lds.buf[(B + kDist) % kNBuf], check_c);
        if constexpr (ACTIVE) {
            if (!CHECK || s < s1) compute(lds.buf[B]);
        }
        stage_barrier<TE>();
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    using B2 = std::integral_constant<int, 2>;
    using B3 = std::integral_constant<int, 3>;

#pragma unroll
    for (int b = 0; b < kDist; ++b) copy_stage(b, lds.buf[b], Yes{});
    stage_barrier<TE>();

    constexpr int kChunkStages = T::kFlushGroups / kXG;
    static_assert(kChunkStages % kNBuf == 0, "flush chunks must start on buffer 0");
    for (int s0 = 0; s0 < nstages; s0 += kChunkStages) {
        // s1 is a multiple of kNBuf or the segment end
        const int s1 = min(nstages, s0 + kChunkStages);
        if constexpr (ACTIVE) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb2 = 0; nb2 < MB; ++nb2) {
                    re[mb][nb2] = acc_t{};
                    im[mb][nb2] = acc_t{};
                }
        }
        // steady state: every stage copied is whole and before the last one
        const int sfull = min(s1, nstages - kDist - 1);
        int s = s0;
        for (; s + kNBuf <= sfull; s += kNBuf) {
            iteration(s, s1, B0{}, No{});
            iteration(s + 1, s1, B1{}, No{});
            if constexpr (kNBuf > 2) {
                iteration(s + 2, s1, B2{}, No{});
                iteration(s + 3, s1, B3{}, No{});
            }
        }
        for (; s < s1; s += kNBuf) {
            iteration(s, s1, B0{}, Yes{});
            iteration(s + 1, s1, B1{}, Yes{});
            if constexpr (kNBuf > 2) {
                iteration(s + 2, s1, B2{}, Yes{});
                iteration(s + 3, s1, B3{}, Yes{});
            }
        }
        if constexpr (ACTIVE) {
            // flush this chunk's partial sums into the integrators.  The base is made
            // opaque here so the compiler cannot hoist 64 integrator addresses out of
            // the K loop (they would occupy half the register file).
            uint8_t *ibase = reinterpret_cast<uint8_t *>(a.integ);
            int fr0 = tb.ra * (TE / 2), fc0 = tb.rb * (TE / 2);
            if constexpr (BATCH) asm volatile("" : "+v"(ibase), "+v"(fr0), "+v"(fc0));
            else asm volatile("" : "+s"(ibase), "+v"(fr0), "+v"(fc0));
            // the first flush of a segment that starts its integration writes the
            // integrators instead of adding to them (no read)
            const bool store = a.first && s0 == 0;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
                for (int nb2 = 0; nb2 < MB; ++nb2) {
                    const int n2 = fc0 + nb2 * 32 + l32;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int n1 = fr0 + mb * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
                        if (n1 < a.n_in && n2 <= n1) {
                            const int64_t p = (int64_t)n1 * (n1 + 1) / 2 + n2;
                            if constexpr (ATOMIC) {
                                if (a.i32) {
                                    int *dst = reinterpret_cast<int *>(ibase) + 2 * ((int64_t)c * a.P + p);
                                    atomicAdd(dst, (int)re[mb][nb2][r]);
                                    atomicAdd(dst + 1, (int)im[mb][nb2][r]);
                                } else {
                                    unsigned long long *dst =
                                        reinterpret_cast<unsigned long long *>(ibase) + 2 * ((int64_t)c * a.P + p);
                                    atomicAdd(dst, (unsigned long long)(long long)re[mb][nb2][r]);
                                    atomicAdd(dst + 1, (unsigned long long)(long long)im[mb][nb2][r]);
                                }
                            } else if constexpr (INT8) {
                                if (a.i32) {
                                    int2 *dst = reinterpret_cast<int2 *>(ibase) + (int64_t)c * a.P + p;
                                    int2 v = make_int2(re[mb][nb2][r], im[mb][nb2][r]);
                                    if (!store) {
                                        const int2 o = *dst;
                                        v.x += o.x;
                                        v.y += o.y;
                                    }
                                    *dst = v;
                                } else {
                                    longlong2 *dst = reinterpret_cast<longlong2 *>(ibase) + (int64_t)c * a.P + p;
                                    longlong2 v = make_longlong2(re[mb][nb2][r], im[mb][nb2][r]);
                                    if (!store) {
                                        const longlong2 o = *dst;
                                        v.x += o.x;
                                        v.y += o.y;
                                    }
                                    *dst = v;
                                }
                            } else {
                                double2 *dst = reinterpret_cast<double2 *>(ibase) + (int64_t)c * a.P + p;
                                double2 v = make_double2((double)re[mb][nb2][r], (double)im[mb][nb2][r]);
                                if (!store) {
                                    const double2 o = *dst;
                                    v.x += o.x;
                                    v.y += o.y;
                                }
                                *dst = v;
                            }
                        }
                    }
                }
            }
        }
    }
    // the copies past the segment end must land before the LDS is reused (next
    // work item) or released (workgroup end)
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
}

// The wave's block of a workgroup; an idle wave still copies its slot and meets the
// barriers.
template <int XP, int TE, bool BATCH>
__device__ __forceinline__ void run_blocks(const XArgs &a, const XLds &lds, int c, const TriBlock &tb, bool atomic) {
    if constexpr (XP == MWAX_X_INT8) {
        if (atomic) {
            if (tb.ra < 0) xengine_tile_loop<XP, TE, false, true, BATCH>(a, lds, c, tb);
            else xengine_tile_loop<XP, TE, true, true, BATCH>(a, lds, c, tb);
            return;
        }
    }
    if (tb.ra < 0) xengine_tile_loop<XP, TE, false, false, BATCH>(a, lds, c, tb);
    else xengine_tile_loop<XP, TE, true, false, BATCH>(a, lds, c, tb);
}

// Workgroup -> (chunk, channel, tile): the tiles of one channel are consecutive,
// so they land on one XCD and share its L2; the chunks of a tile read disjoint
// row groups and run one after another (measured: 25 % less HBM traffic than
// interleaving them).
template <int XP>
__global__ __launch_bounds__(kThreads, 2) void xengine_mfma(XArgs a) {
    __shared__ __align__(16) uint8_t lds0[kStage], lds1[kStage], lds2[kStage23], lds3[kStage23];
    const XLds lds{{lds0, lds1, lds2, lds3}};
    const int nb = gridDim.x;
    const int lin = xcd_logical(blockIdx.x, nb);
    const int per_k = a.ntiles * a.L;
    const int ks = lin / per_k;
    const int rem = lin - ks * per_k;
    const int c = rem / a.ntiles;
    int t = rem - c * a.ntiles;
    // The workgroups of a channel are not alike, and an XCD deals consecutive ones to
    // its 32 CUs in turn: with an even number to a channel a CU would get only one
    // kind.  The order turns every 16 channels (INT8, 134 inputs, 1,024 channels, two
    // calls of 232 spectra, channelise to emission: 386 us without, 337 with).
    if (!(a.ntiles & 1) && ((c >> 4) & 1)) t = a.ntiles - 1 - t;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the wave of each block turns with the workgroup: an idle one is on another
    // SIMD from workgroup to workgroup
    const TriBlock tb = tri_block((a.n_in + 63) / 64, a.sets, t, (wave + lin) & 3, wave);
    XArgs b = a;
    b.grp0 = a.grp0 + (int64_t)ks * a.kchunk;
    b.ngrp = min(a.kchunk, a.ngrp - ks * a.kchunk);
    run_blocks<XP, kTile, false>(b, lds, c, tb, a.nks > 1);
}

// ---------------------------------------------------------------------------
// Small arrays (up to kXSmallInputs inputs): a 128-edge tile would leave most of a
// workgroup's waves idle and a launch with one workgroup per channel, each behind
// one long K loop.  Instead one workgroup runs one 32 x 32 block and its waves
// share the K loop, straight from global memory (a row group of 32 inputs is 1 KB
// contiguous; no panel is shared that LDS could hold).  The row groups are dealt in
// stages of kSmallG to kSmallSlices slices; the slices' sums are added in order, in
// int64 or FP64, so the result does not depend on how many waves share them: a
// batch item (four waves) gives the same bits as a plan of its own (eight).
// Bound by latency.  32 inputs, 128 channels, 10,000 spectra, channelise to emission,
// 128-edge tiles / this: INT8 123 / 85 us, FP16 279 / 106 us; 64 inputs, 512 channels,
// 4 x 64 spectra in one launch: INT8 189 / 121 us, FP16 115 / 74 us (a launch per
// segment: 132 and 83 us).
// ---------------------------------------------------------------------------
constexpr int kSmallSlices = 8, kSmallG = 8;
template <int XP>
using SmallSum = typename std::conditional<XP == MWAX_X_INT8, longlong2, double2>::type;

// Fragments of kSmallG row groups of a block (rows from pa and pb), from group g0 on;
// groups at or past gend read as zeros.
struct SmallStage {
    uint4 a[kSmallG], b[kSmallG];
    __device__ __forceinline__ void fetch(const uint8_t *pa, const uint8_t *pb, int64_t gstride, int g0, int gend) {
#pragma unroll
        for (int k = 0; k < kSmallG; ++k) {
            const int64_t o = (int64_t)min(g0 + k, gend - 1) * gstride;
            a[k] = *reinterpret_cast<const uint4 *>(pa + o);
            b[k] = *reinterpret_cast<const uint4 *>(pb + o);
        }
    }
    template <int XP, bool EXACT>
    __device__ __forceinline__ void multiply(int g0, int gend, typename MfmaT<XP>::acc_t &re,
                                             typename MfmaT<XP>::acc_t &im) const {
        const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int k = 0; k < kSmallG; ++k) {
            const bool in = g0 + k < gend;
            const uint4 x = in ? a[k] : zero, y = in ? b[k] : zero;
            re = MfmaT<XP>::mma(x, y, re);
            im = MfmaT<XP>::mma(x, im_operand<XP, EXACT>(y), im);
        }
    }
};

// Block (I, J) of channel c over the segment of a, by the W waves of a workgroup;
// sum: LDS for the running sums.  W = 1 takes segments of one stage.
template <int XP, int W>
__device__ __forceinline__ void small_block(const XArgs &a, int c, int I, int J, int wave, SmallSum<XP> (*sum)[64]) {
    static_assert(kSmallSlices % W == 0, "whole passes of the slices");
    using T = MfmaT<XP>;
    using acc_t = typename T::acc_t;
    using Sum = SmallSum<XP>;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int64_t gstride = (int64_t)a.n_in * kRowBytes;
    const uint8_t *base = a.chan + ((int64_t)c * a.NG + a.grp0) * gstride + half * 16;
    const uint8_t *pa = base + min(I * 32 + l32, a.n_in - 1) * kRowBytes;
    const uint8_t *pb = base + min(J * 32 + l32, a.n_in - 1) * kRowBytes;
    // row r of the lane's sixteen sums
    auto put = [&](int r, Sum v) {
        const int n1 = I * 32 + (r >> 2) * 8 + half * 4 + (r & 3), n2 = J * 32 + l32;
        if (n1 >= a.n_in || n2 > n1) return;
        const int64_t e = (int64_t)c * a.P + (int64_t)n1 * (n1 + 1) / 2 + n2;
        if (XP == MWAX_X_INT8 && a.i32) {
            int2 *dst = reinterpret_cast<int2 *>(a.integ) + e;
            int2 w = make_int2((int)v.x, (int)v.y);
            if (!a.first) {
                const int2 o = *dst;
                w.x += o.x;
                w.y += o.y;
            }
            *dst = w;
        } else {
            Sum *dst = reinterpret_cast<Sum *>(a.integ) + e;
            if (!a.first) {
                const Sum o = *dst;
                v.x += o.x;
                v.y += o.y;
            }
            *dst = v;
        }
    };
    if constexpr (W == 1) {
        acc_t re{}, im{};
        SmallStage st;
        st.fetch(pa, pb, gstride, 0, a.ngrp);
        st.template multiply<XP, false>(0, a.ngrp, re, im);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            Sum v;
            v.x = re[r];
            v.y = im[r];
            put(r, v);
        }
        return;
    }
    const int nst = (a.ngrp + kSmallG - 1) / kSmallG;
#pragma unroll 1
    for (int first = 0; first < min(kSmallSlices, nst); first += W) {
        const int slice = first + wave;
        acc_t re{}, im{};
        Sum mine[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[r].x = mine[r].y = 0;
        auto collect = [&] {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                mine[r].x += re[r];
                mine[r].y += im[r];
            }
            re = acc_t{};
            im = acc_t{};
        };
        SmallStage next;
        if (slice < nst) next.fetch(pa, pb, gstride, slice * kSmallG, a.ngrp);
        int groups = 0;
        for (int s = slice; s < nst; s += kSmallSlices) {
            const SmallStage cur = next;
            if (s + kSmallSlices < nst) next.fetch(pa, pb, gstride, (s + kSmallSlices) * kSmallG, a.ngrp);
            cur.template multiply<XP, false>(s * kSmallG, a.ngrp, re, im);
            groups += kSmallG;
            if (groups == T::kFlushGroups) {
                collect();
                groups = 0;
            }
        }
        collect();
#pragma unroll 1
        for (int k = 0; k < W; ++k) {
            if (wave == k) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    Sum v = mine[r];
                    if (slice > 0) {
                        v.x += sum[r][lane].x;
                        v.y += sum[r][lane].y;
                    }
                    sum[r][lane] = v;
                }
            }
            __syncthreads();
        }
    }
    for (int r = wave; r < 16; r += W) put(r, sum[r][lane]);
}

template <int XP, int W>
__global__ __launch_bounds__(64 * W, 2) void xengine_small(XArgs a, XSegList segs) {
    __shared__ SmallSum<XP> sum[W > 1 ? 16 : 1][64];
    const int lin = xcd_logical(blockIdx.x, gridDim.x);
    const int cs = lin / a.ntiles, seg = cs / a.L, c = cs - seg * a.L;
    const XSeg sg = segs.s[seg];
    a.grp0 = sg.grp0;
    a.ngrp = sg.ngrp;
    a.integ = sg.integ;
    a.first = sg.first;
    int I, J;
    tile_ij(lin - cs * a.ntiles, I, J);
    small_block<XP, W>(a, c, I, J, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), sum);
}

// Persistent batched form (see XBatchArgs): each workgroup takes items from the
// queue of its XCD until it is empty, then from the other queues in turn, and
// exits when all are empty.  Every item is one tile of one channel over one chunk
// of row groups, run by the same loop as the single-plan kernel.
template <int XP>
__global__ __launch_bounds__(kThreads, 2) void xengine_batch(XBatchArgs b) {
    __shared__ __align__(16) uint8_t lds0[kStage], lds1[kStage], lds2[kStage23], lds3[kStage23];
    __shared__ int s_item;
    const XLds lds{{lds0, lds1, lds2, lds3}};
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int home = blockIdx.x & (kXQueues - 1);
    for (int v = 0; v < kXQueues; ++v) {
        const int q = (home + v) & (kXQueues - 1);
        const int q0 = load_uniform(b.qbeg + q), qn = load_uniform(b.qbeg + q + 1) - q0;
        for (;;) {
            if (threadIdx.x == 0) s_item = atomicAdd(&b.counters[q * kXCounterStride], 1);
            __syncthreads();
            const int k = __builtin_amdgcn_readfirstlane(s_item);
            __syncthreads();
            if (k >= qn) break;
            const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)b.items[q0 + k]);
            const int d = (int)(it >> 24), c = (int)((it >> 14) & 1023), t = (int)((it >> 6) & 255);
            const int ks = (int)(it & 63);
            const XDesc xd = load_uniform(b.desc + d);
            XArgs a{};
            a.chan = xd.chan;
            a.NG = xd.NG;
            a.grp0 = xd.grp0 + (int64_t)ks * xd.kchunk;
            a.ngrp = min(xd.kchunk, xd.ngrp - ks * xd.kchunk);
            a.n_in = xd.n_in;
            a.integ = xd.integ;
            a.P = xd.P;
            a.first = xd.first;
            a.i32 = xd.i32;
            if (xd.te == kXTileTiny) {
                if constexpr (XP == MWAX_X_FP16) {
                    int I, J;
                    tile_ij(t, I, J);
                    small_block<XP, 4>(a, c, I, J, wave, reinterpret_cast<SmallSum<XP> (*)[64]>(lds0));
                    __syncthreads();   // the sums have been read
                }
            } else if (xd.te == kTileSmall) {
                const TriBlock tb = tri_block((a.n_in + 31) / 32, tri_sets((a.n_in + 31) / 32), t, (wave + k) & 3, wave);
                run_blocks<XP, kTileSmall, true>(a, lds, c, tb, xd.ksplit > 1);
            } else {
                const TriBlock tb = tri_block((a.n_in + 63) / 64, tri_sets((a.n_in + 63) / 64), t, (wave + k) & 3, wave);
                run_blocks<XP, kTile, true>(a, lds, c, tb, xd.ksplit > 1);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Averaging X-engine (Sec. 2.6 applied inside the correlation): one workgroup =
// one output channel o of N = L / F x four 32 x 32 blocks.  It correlates the fine
// channels of o one after another -- offsets |d| <= F / 2 around o's centre
// (the rule of average.hip: the outermost pair at weight 1/2 for even F, DC left
// out of the centre channel) -- with the MFMA K loop running over the
// channel-major rows of (channel, row group), stages never straddling two
// channels.  When a channel's last stage is done its partial sums are scaled
// (INT8: s_c^2) and weighted into FP32 sums held in registers, which are
// divided by the weight total and added (or, for the first segment of an
// integration, stored) once into FP64 integrators [N][P].  The fine-channel
// integrators are never written: per 250 ms integration at 256 tiles and
// L = 6400 that is 6.7 GB of flushes and 6.7 GB of pack reads avoided.
// The INT8 Im operand is the exact negation (-im, re), not the one's complement of
// the per-channel kernel: the sums are FP32 here, and with sum_m re_n1[m] in them
// would take its rounding too, which is many times theirs where an input has a large
// mean (the one's complement takes 2 % less at 512 inputs).  Bound by the copies from
// L2 into LDS: 512 inputs at 40 kHz read every row nine times, 15 GB per four 250 ms
// integrations, 12 TB/s at 1.28 ms (the copies of the per-channel kernel reach no more
// alone); the VALU's conversion and weighted addition of every partial comes next.
// 1.40 ms with cleared partials and an idle wave on every diagonal tile; 1.74 ms with
// a launch per integration.
// ---------------------------------------------------------------------------
// Copies run three stages ahead here (two in the per-channel kernel): a work
// item's stages are short (4 MFMAs per wave at 250 ms integrations) and every
// workgroup of a launch is resident at once, so the copies in flight are what
// hides the L2 latency.
constexpr int kAvgDist = 3;

template <int XP>
__global__ __launch_bounds__(kThreads, 4) void xengine_avg(XAvgArgs a) {
    constexpr int TE = kTileSmall;
    using GEO = TileGeo<TE, kAvgDist>;
    constexpr int kGroupPitch = GEO::kGroupPitch, kPanel = GEO::kPanel;
    using T = MfmaT<XP>;
    using acc_t = typename T::acc_t;
    __shared__ __align__(16) uint8_t lds0[GEO::kStage], lds1[GEO::kStage], lds2[GEO::kStage], lds3[GEO::kStage];
    uint8_t *const bufs[4] = {lds0, lds1, lds2, lds3};
    static_assert(kNBuf == 4, "four stage buffers");

    const int lin = xcd_logical(blockIdx.x, gridDim.x);
    const int os = lin / a.ntiles, seg = os / a.N, o = os - seg * a.N;
    const XSeg sg = a.segs.s[seg];
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const TriBlock tb = tri_block((a.n_in + 31) / 32, tri_sets((a.n_in + 31) / 32), lin - os * a.ntiles, (wave + lin) & 3, wave);
    const bool active = tb.ra >= 0;

    // the fine channels of o: offsets d = -h .. h (DC skipped in the centre one),
    // channel (L/2 + (o - N/2) F + d) mod L.  They are walked with cursors: no
    // division or remainder in the loop, whose scalar work per stage is what
    // bounds a stage of four MFMAs per wave.
    const int h = a.F / 2, oc = a.N / 2;
    const bool even = (a.F & 1) == 0, centre = a.F > 1 && o == oc;
    const int nch = 2 * h + 1 - (centre ? 1 : 0);
    const float inv_wsum = 1.0f / (centre ? (float)(a.F - 1) : (float)a.F);
    const int c_first = ((a.L / 2 + (o - oc) * a.F - h) % a.L + a.L) % a.L;
    // next channel after c at offset d (skipping DC in the centre channel)
    auto next_channel = [&](int c, int d) {
        int n = c + ((centre && d == -1) ? 2 : 1);
        return n >= a.L ? n - a.L : n;
    };

    // copies: wave w moves the 32 rows of slot w
    const uint32_t offR = (uint32_t)min(tb.copy * 32 + l32, a.n_in - 1) * kRowBytes + half * 16;
    const uint32_t offZ = (uint32_t)l32 * kRowBytes + half * 16;
    const int64_t gstride = (int64_t)a.n_in * kRowBytes;
    const int64_t cstride = a.NG * gstride;       // bytes between channels
    const int ldst = (wave >> 1) * kPanel + (wave & 1) * kBlock;
    const int spc = (sg.ngrp + kXG - 1) / kXG;     // stages per channel
    const int nst = nch * spc;

    // copy cursor: channel index, its channel and offset, stage within it, and the
    // address of the stage's first row group
    int cp_ci = 0, cp_c = c_first, cp_d = -h, cp_g = 0;
    if (centre && cp_d == 0) cp_d = 1;            // (h = 0 only when F = 1: no centre rule)
    const uint8_t *cp_base = a.chan + ((int64_t)cp_c * a.NG + sg.grp0) * gstride;
    const uint8_t *cp_src = cp_base;
    const int64_t stage_bytes = (int64_t)kXG * gstride;
    auto copy_next = [&](uint8_t *buf) {
        const bool live = cp_ci < nch;
#pragma unroll
        for (int k = 0; k < kXG; ++k) {
            const bool in = live && cp_g + k < sg.ngrp;
            // (selected as a whole: with a selected base the compiler puts the copies
            // behind a branch and waits for all of them at every stage)
            const uint8_t *src = in ? cp_src + k * gstride + offR : kZeroGroup + offZ;
            __builtin_amdgcn_global_load_lds(src, buf + k * kGroupPitch + ldst, 16, 0, 0);
        }
        cp_g += kXG;
        cp_src += stage_bytes;
        if (cp_g >= sg.ngrp) {
            cp_g = 0;
            ++cp_ci;
            const int nc = next_channel(cp_c, cp_d);
            cp_base += (int64_t)(nc - cp_c) * cstride;
            cp_src = cp_base;
            cp_c = nc;
            cp_d += (centre && cp_d == -1) ? 2 : 1;
        }
    };

    acc_t re{}, im{};
    float sr[16], si[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) sr[r] = si[r] = 0.0f;
    const int fa_off = (tb.sa >> 1) * kPanel + (tb.sa & 1) * kBlock + half * 512 + l32 * 16;
    const int fb_off = (tb.sb >> 1) * kPanel + (tb.sb & 1) * kBlock + half * 512 + l32 * 16;

    // FIRST: the stage starts new partial sums (no cleared registers)
    auto compute = [&](const uint8_t *st, auto first_c) {
        constexpr bool FIRST = decltype(first_c)::value;
        uint4 fa[2], fb[2];
        fa[0] = *reinterpret_cast<const uint4 *>(st + fa_off);
        fb[0] = *reinterpret_cast<const uint4 *>(st + fb_off);
#pragma unroll
        for (int k = 0; k < kXG; ++k) {
            if (k + 1 < kXG) {
                fa[(k + 1) & 1] = *reinterpret_cast<const uint4 *>(st + (k + 1) * kGroupPitch + fa_off);
                fb[(k + 1) & 1] = *reinterpret_cast<const uint4 *>(st + (k + 1) * kGroupPitch + fb_off);
            }
            const uint4 v = fb[k & 1];
            const uint4 fb2 = im_operand<XP, true>(v);
            re = T::mma(fa[k & 1], v, FIRST && k == 0 ? acc_t{} : re);
            im = T::mma(fa[k & 1], fb2, FIRST && k == 0 ? acc_t{} : im);
        }
    };
    // Weight of every channel index ci (weight / weight total, times s_c^2): a
    // table held across the lanes, lane l holding ci = w0 + 64 t + l (t < 4) of
    // the window of 256 indices from w0, read with v_readlane when a channel is
    // done -- no memory access in the loop, whose vector-memory counter belongs
    // to the copies in flight.
    float ctab[4];
    auto load_window = [&](int w0) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int ci = w0 + 64 * t + lane;
            const int d = -h + ci + (centre && ci >= h ? 1 : 0);
            const int c = (((a.L / 2 + (o - oc) * a.F + d) % a.L) + a.L) % a.L;
            float coef = (even && (d == -h || d == h) ? 0.5f : 1.0f) * inv_wsum;
            if (sg.scales && ci < nch) {
                const float sc = sg.scales[c];
                coef *= sc * sc;
            }
            ctab[t] = coef;
        }
    };
    load_window(0);
    // compute cursor: channel index, the stage within the stages after which its partial
    // sums are taken (all of the channel's, or kTake: INT8 partials are int32, see
    // MfmaT), their number and that of the channel's stages that follow them
    constexpr int kTake = T::kFlushGroups / kXG;
    int cm_ci = 0, cm_ls = 0, cm_len = min(spc, kTake), cm_rest = spc - cm_len;
    auto iteration = [&](int s, auto b_c) {
        constexpr int B = decltype(b_c)::value;
        copy_next(bufs[(B + kAvgDist) % kNBuf]);
        if (s < nst) {
            if (active) {
                if (cm_ls == 0) compute(bufs[B], std::true_type{});
                else compute(bufs[B], std::false_type{});
            }
            if (++cm_ls == cm_len) {
                // the channel's partials, scaled and weighted, into the sums
                if (active) {
                    const int t = (cm_ci >> 6) & 3;
                    const float tv = t == 0 ? ctab[0] : (t == 1 ? ctab[1] : (t == 2 ? ctab[2] : ctab[3]));
                    const float coef = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tv), cm_ci & 63));
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        sr[r] = fmaf(coef, (float)re[r], sr[r]);
                        si[r] = fmaf(coef, (float)im[r], si[r]);
                    }
                }
                cm_ls = 0;
                if (cm_rest == 0) {
                    cm_rest = spc;
                    if ((++cm_ci & 255) == 0 && cm_ci < nch) load_window(cm_ci);
                }
                cm_len = min(cm_rest, kTake);
                cm_rest -= cm_len;
            }
        }
        stage_barrier<TE, kAvgDist>();
    };

#pragma unroll
    for (int b = 0; b < kAvgDist; ++b) copy_next(bufs[b]);
    stage_barrier<TE, kAvgDist>();
    for (int s = 0; s < nst; s += kNBuf) {
        iteration(s, std::integral_constant<int, 0>{});
        iteration(s + 1, std::integral_constant<int, 1>{});
        iteration(s + 2, std::integral_constant<int, 2>{});
        iteration(s + 3, std::integral_constant<int, 3>{});
    }
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0): copies past the end have landed

    if (active) {
        double2 *dst0 = reinterpret_cast<double2 *>(sg.integ) + (int64_t)o * a.P;
        const int n2 = tb.rb * 32 + l32;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int n1 = tb.ra * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
            if (n1 < a.n_in && n2 <= n1) {
                double2 *dst = dst0 + (int64_t)n1 * (n1 + 1) / 2 + n2;
                double2 v = make_double2((double)sr[r], (double)si[r]);
                if (!sg.first) {
                    const double2 old = *dst;
                    v.x += old.x;
                    v.y += old.y;
                }
                *dst = v;
            }
        }
    }
}

// The averaging X-engine for few output channels or inputs (compare small_block):
// one workgroup = one segment, one output channel and one 32 x 32 block; its eight
// waves take units of up to kAvgUnit row groups of one fine channel in turn and add
// the weighted partials to FP64 sums, which are added over the waves in order.
// Bound by latency.  Channelise to emission, 64-edge form / this: 12 inputs, 1,024
// channels by 16, FP16, 2 x 18,802 spectra 9,370 / 2,060 us; 18 inputs, 512 by 8,
// INT8, 99,719 spectra 7,310 / 2,700 us.
constexpr int kAvgUnit = 8 * kSmallG;
template <int XP>
__global__ __launch_bounds__(64 * kSmallSlices, 2) void xengine_avg_small(XAvgArgs a) {
    __shared__ double2 sum[16][64];
    using acc_t = typename MfmaT<XP>::acc_t;
    const int lin = xcd_logical(blockIdx.x, gridDim.x);
    const int os = lin / a.ntiles, seg = os / a.N, o = os - seg * a.N;
    const XSeg sg = a.segs.s[seg];
    int I, J;
    tile_ij(lin - os * a.ntiles, I, J);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int h = a.F / 2, oc = a.N / 2;
    const bool even = (a.F & 1) == 0, centre = a.F > 1 && o == oc;
    const int nch = 2 * h + 1 - (centre ? 1 : 0);
    const float inv_wsum = 1.0f / (centre ? (float)(a.F - 1) : (float)a.F);
    const int64_t gstride = (int64_t)a.n_in * kRowBytes;
    const int rowA = min(I * 32 + l32, a.n_in - 1) * kRowBytes + half * 16;
    const int rowB = min(J * 32 + l32, a.n_in - 1) * kRowBytes + half * 16;
    const int upc = (sg.ngrp + kAvgUnit - 1) / kAvgUnit, units = nch * upc;
    double2 mine[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) mine[r] = make_double2(0.0, 0.0);
    for (int u = wave; u < units; u += kSmallSlices) {
        const int ci = u / upc, g0 = (u - ci * upc) * kAvgUnit, g1 = min(sg.ngrp, g0 + kAvgUnit);
        const int d = -h + ci + (centre && ci >= h ? 1 : 0);
        const int c = (((a.L / 2 + (o - oc) * a.F + d) % a.L) + a.L) % a.L;
        float coef = (even && (d == -h || d == h) ? 0.5f : 1.0f) * inv_wsum;
        if (sg.scales) coef *= sg.scales[c] * sg.scales[c];
        const uint8_t *base = a.chan + ((int64_t)c * a.NG + sg.grp0) * gstride;
        acc_t re{}, im{};
        SmallStage next;
        next.fetch(base + rowA, base + rowB, gstride, g0, g1);
        for (int g = g0; g < g1; g += kSmallG) {
            const SmallStage cur = next;
            if (g + kSmallG < g1) next.fetch(base + rowA, base + rowB, gstride, g + kSmallG, g1);
            cur.template multiply<XP, true>(g, g1, re, im);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            mine[r].x += (double)coef * (double)re[r];
            mine[r].y += (double)coef * (double)im[r];
        }
    }
#pragma unroll 1
    for (int k = 0; k < kSmallSlices; ++k) {
        if (wave == k) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                double2 v = mine[r];
                if (k > 0) {
                    v.x += sum[r][lane].x;
                    v.y += sum[r][lane].y;
                }
                sum[r][lane] = v;
            }
        }
        __syncthreads();
    }
    const int n2 = J * 32 + l32;
    for (int r = wave; r < 16; r += kSmallSlices) {
        const int n1 = I * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
        if (n1 < a.n_in && n2 <= n1) {
            double2 *dst = reinterpret_cast<double2 *>(sg.integ) + (int64_t)o * a.P + (int64_t)n1 * (n1 + 1) / 2 + n2;
            double2 v = sum[r][lane];
            if (!sg.first) {
                const double2 old = *dst;
                v.x += old.x;
                v.y += old.y;
            }
            *dst = v;
        }
    }
}

__global__ void zero_i32_kernel(int32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------
// FP32 X-engine on the FP32 matrix cores (v_mfma_f32_32x32x2_f32).  One
// instruction takes one spectrum: K = (re, im), lanes 0..31 carrying the real
// and lanes 32..63 the imaginary parts, so
//   Re V: A = (re1, im1), B = (re2, im2);  Im V: the same A, B2 = (-im2, re2).
// A planar FP32 row half (4 spectra of one component) is one lane's operand of
// four instructions; B2 is the other half of B's row, read from there.
//
// Two-level FP32 accumulation: each 16-spectrum stage is summed into an inner
// accumulator, which is then added to an outer one; the outer one is flushed
// to FP64 every 2048 spectra.  A single FP32 running sum is biased: in the
// channels whose bin is a multiple of L/4 the spectra of integer voltages are
// exact integers, their squares are 0 or 1 mod 4, and once the running sum
// passes 2^24 every addition rounds the same way.  The inner sums stay far
// below 2^24 (exact for those channels) and have evenly spread low bits, so the
// outer additions round without a bias.
// ---------------------------------------------------------------------------
constexpr int kFT = kTileSmall;               // tile edge: 2 x 2 waves of one 32 x 32 block
constexpr int kFG = 4;                        // row groups per stage: 16 spectra, one inner sum
constexpr int kFGroup = kFT / 32 * kBlock;    // LDS bytes of one panel's row group
constexpr int kFPanel = kFG * kFGroup;
constexpr int kFStage = 2 * kFPanel;
constexpr int kFFlush = 2048 / (4 * kFG);     // inner sums per FP32 outer sum

// One 32 x 32 block over one row group (4 spectra): a, b the lane's halves of
// its A and B rows, b2 the other half of its B row; sign: 0x80000000 for the
// lanes of the real parts (their B2 operand is -im), else 0.
__device__ __forceinline__ void mma_f32_group(float4 a, float4 b, float4 b2, uint32_t sign, v16f &re, v16f &im) {
    const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w}, cv[4] = {b2.x, b2.y, b2.z, b2.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        re = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], bv[e], re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], __uint_as_float(__float_as_uint(cv[e]) ^ sign), im, 0, 0, 0);
    }
}

// One workgroup = one channel x one 64 x 64 tile: the stages of both panels are
// copied straight into LDS, one ahead of the matrix work, into two buffers
// (separate LDS objects, so that a read of one does not wait for the copies
// landing in the other).  A stage is 32 instructions of 64 cycles per wave, long
// enough to cover the copies with one barrier per stage; 32 KB of LDS and at most
// 128 registers put four workgroups on a CU.  Bound by the matrix cores (75 % of
// their cycles busy; the rest is the last, partly filled round of workgroups and
// the flushes): 256 inputs, 128 channels, 5,000 spectra take 1.7-1.8 ms, 96
// TFLOP/s of the 151 a large library product reaches, where 4 x 8 outputs per
// thread on the vector ALUs took 4.6 ms.
__global__ __launch_bounds__(kThreads, 4) void xengine_f32(XArgs a, XSegList segs) {
    __shared__ __align__(16) uint8_t buf0[kFStage], buf1[kFStage];
    const int lin = xcd_logical(blockIdx.x, gridDim.x);
    const int cs = lin / a.ntiles, seg = cs / a.L, c = cs - seg * a.L;
    const XSeg sg = segs.s[seg];
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // the wave of each block turns with the workgroup: an idle one is on another
    // SIMD from workgroup to workgroup
    const TriBlock tb = tri_block((a.n_in + 31) / 32, tri_sets((a.n_in + 31) / 32), lin - cs * a.ntiles, (wave + lin) & 3, wave);
    const bool active = tb.ra >= 0;

    // copies: wave w moves the 32 rows of slot w.  Rows past the last input are read
    // from a clamped address: they reach only outputs that are never flushed.
    const uint32_t offR = (uint32_t)min(tb.copy * 32 + l32, a.n_in - 1) * kRowBytes + half * 16;
    const uint32_t offZ = (uint32_t)l32 * kRowBytes + half * 16;
    const int64_t gstride = (int64_t)a.n_in * kRowBytes;
    const uint8_t *base = a.chan + ((int64_t)c * a.NG + sg.grp0) * gstride;
    const int ldst = (wave >> 1) * kFPanel + (wave & 1) * kBlock;
    const int nstages = (sg.ngrp + kFG - 1) / kFG;
    auto copy_stage = [&](int s, uint8_t *buf) {
#pragma unroll
        for (int k = 0; k < kFG; ++k) {
            const int g = s * kFG + k;
            const uint8_t *src = g < sg.ngrp ? base + g * gstride + offR : kZeroGroup + offZ;
            __builtin_amdgcn_global_load_lds(src, buf + k * kFGroup + ldst, 16, 0, 0);
        }
    };

    const int fa_off = (tb.sa >> 1) * kFPanel + (tb.sa & 1) * kBlock + half * 512 + l32 * 16;
    const int fb_off = (tb.sb >> 1) * kFPanel + (tb.sb & 1) * kBlock + half * 512 + l32 * 16;
    const int fb2_off = fb_off + (half ? -512 : 512);
    const uint32_t sign = half ? 0u : 0x80000000u;
    v16f outr{}, outi{};
    auto compute = [&](const uint8_t *st) {
        v16f re{}, im{};
#pragma unroll
        for (int k = 0; k < kFG; ++k)
            mma_f32_group(*reinterpret_cast<const float4 *>(st + k * kFGroup + fa_off),
                          *reinterpret_cast<const float4 *>(st + k * kFGroup + fb_off),
                          *reinterpret_cast<const float4 *>(st + k * kFGroup + fb2_off), sign, re, im);
        outr += re;
        outi += im;
    };
    // the outer sums into the FP64 integrators; the first flush of a segment that
    // starts its integration stores instead of adding
    bool store = sg.first != 0;
    auto flush = [&]() {
        // opaque, so that the 16 addresses are not formed ahead of the K loop and
        // held in registers through it
        int fr0 = __builtin_amdgcn_readfirstlane(tb.ra * 32), fc0 = __builtin_amdgcn_readfirstlane(tb.rb * 32);
        asm volatile("" : "+s"(fr0), "+s"(fc0));
        double2 *dst0 = reinterpret_cast<double2 *>(sg.integ) + (int64_t)c * a.P;
        const int n2 = fc0 + l32;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int n1 = fr0 + (r >> 2) * 8 + half * 4 + (r & 3);
            if (n1 < a.n_in && n2 <= n1) {
                double2 *dst = dst0 + (int64_t)n1 * (n1 + 1) / 2 + n2;
                double2 v = make_double2((double)outr[r], (double)outi[r]);
                if (!store) {
                    const double2 old = *dst;
                    v.x += old.x;
                    v.y += old.y;
                }
                *dst = v;
            }
        }
        outr = v16f{};
        outi = v16f{};
        store = false;
    };

    copy_stage(0, buf0);
    drain_barrier();
    auto iteration = [&](int s, uint8_t *cur, uint8_t *next) {
        copy_stage(s + 1, next);           // last read one iteration ago, behind a barrier
        if (active && s < nstages) compute(cur);
        drain_barrier();
    };
    static_assert(kFFlush % 2 == 0, "flushes fall between pairs of stages");
    for (int s0 = 0; s0 < nstages; s0 += kFFlush) {
        const int s1 = min(nstages, s0 + kFFlush);
        for (int s = s0; s < s1; s += 2) {
            iteration(s, buf0, buf1);
            iteration(s + 1, buf1, buf0);
        }
        if (active) flush();
    }
}

// Small launches (few tiles or channels, where 64 x 64 tiles would leave CUs
// idle behind one long serial K loop each): one workgroup = one channel x one
// 32 x 32 block, its eight waves taking the 16-spectrum stages in turn, straight
// from global memory (a row group of a block is 1 KB contiguous).  Each wave
// keeps FP64 totals of its flushed outer sums; they are added over the waves in a
// fixed order, so the result does not depend on timing.  32 inputs, 128 channels,
// 1,000 spectra: a 535 us step became 38 us (one 128-edge workgroup per channel
// ran its 63 stages one after another on half of the CUs).
constexpr int kFSWaves = 8;
__global__ __launch_bounds__(64 * kFSWaves, 2) void xengine_f32_small(XArgs a, XSegList segs) {
    __shared__ double2 part[kFSWaves / 2][16][64];
    const int lin = xcd_logical(blockIdx.x, gridDim.x);
    const int cs = lin / a.ntiles, seg = cs / a.L, c = cs - seg * a.L;
    const XSeg sg = segs.s[seg];
    int I, J;
    tile_ij(lin - cs * a.ntiles, I, J);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t gstride = (int64_t)a.n_in * kRowBytes;
    const uint8_t *base = a.chan + ((int64_t)c * a.NG + sg.grp0) * gstride;
    const uint8_t *pa = base + min(I * 32 + l32, a.n_in - 1) * kRowBytes + half * 16;
    const uint8_t *pb = base + min(J * 32 + l32, a.n_in - 1) * kRowBytes;
    const uint32_t sign = half ? 0u : 0x80000000u;
    const int nstages = (sg.ngrp + kFG - 1) / kFG;

    float4 fa[kFG], fb[kFG], fb2[kFG];
    auto fetch = [&](int s) {
#pragma unroll
        for (int k = 0; k < kFG; ++k) {
            const int g = s * kFG + k;
            const int64_t o = (int64_t)min(g, sg.ngrp - 1) * gstride;
            fa[k] = *reinterpret_cast<const float4 *>(pa + o);
            fb[k] = *reinterpret_cast<const float4 *>(pb + o + half * 16);
            fb2[k] = *reinterpret_cast<const float4 *>(pb + o + (16 - half * 16));
            if (g >= sg.ngrp) fa[k] = make_float4(0.f, 0.f, 0.f, 0.f), fb[k] = fa[k], fb2[k] = fa[k];
        }
    };
    v16f outr{}, outi{};
    double2 tot[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) tot[r] = make_double2(0.0, 0.0);
    auto collect = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            tot[r].x += (double)outr[r];
            tot[r].y += (double)outi[r];
        }
        outr = v16f{};
        outi = v16f{};
    };
    int inner = 0;
    if (wave < nstages) fetch(wave);
    for (int s = wave; s < nstages; s += kFSWaves) {
        float4 xa[kFG], xb[kFG], xb2[kFG];
#pragma unroll
        for (int k = 0; k < kFG; ++k) xa[k] = fa[k], xb[k] = fb[k], xb2[k] = fb2[k];
        if (s + kFSWaves < nstages) fetch(s + kFSWaves);
        v16f re{}, im{};
#pragma unroll
        for (int k = 0; k < kFG; ++k) mma_f32_group(xa[k], xb[k], xb2[k], sign, re, im);
        outr += re;
        outi += im;
        if (++inner == kFFlush) {
            collect();
            inner = 0;
        }
    }
    collect();
    // waves 4 .. 7 hand their totals to waves 0 .. 3, then 2, 3 to 0, 1, then 1 to 0
#pragma unroll
    for (int h = kFSWaves / 2; h > 0; h >>= 1) {
        if (wave >= h && wave < 2 * h) {
#pragma unroll
            for (int r = 0; r < 16; ++r) part[wave - h][r][lane] = tot[r];
        }
        __syncthreads();
        if (wave < h) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const double2 v = part[wave][r][lane];
                tot[r].x += v.x;
                tot[r].y += v.y;
            }
        }
        __syncthreads();
    }
    if (wave != 0) return;
    double2 *dst0 = reinterpret_cast<double2 *>(sg.integ) + (int64_t)c * a.P;
    const int n2 = J * 32 + l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int n1 = I * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
        if (n1 < a.n_in && n2 <= n1) {
            double2 *dst = dst0 + (int64_t)n1 * (n1 + 1) / 2 + n2;
            double2 v = tot[r];
            if (!sg.first) {
                const double2 old = *dst;
                v.x += old.x;
                v.y += old.y;
            }
            *dst = v;
        }
    }
}

}  // namespace

int xengine_tile_count(int n_in, int te) {
    if (te != kXTileTiny) {
        const int m = (n_in + te / 2 - 1) / (te / 2);
        return tri_groups(m, tri_sets(m));
    }
    const int t = (n_in + te - 1) / te;
    return t * (t + 1) / 2;
}

namespace {
// Compute units of the device (read once; every device of a node is the same).
int device_cus() {
    static const int cus = [] {
        int dev = 0, n = 0;
        (void)hipGetDevice(&dev);
        return hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0 ? n : 256;
    }();
    return cus;
}

// Chunks per tile of an INT8 launch of items workgroups over ngrp row groups and pairs
// integrators: those of the least cost, with at least kMinChunkGroups row groups to a
// chunk.  Cost in row groups of a workgroup, as long as they take with two workgroups
// on a CU (0.21 us for each): the K loops of the CU that gets the most chunks, one alone
// on its CU running at 4/5 of the rate; and the flushes, of which a split launch has one
// of atomic additions per chunk (less what runs beside other workgroups' K loops) and a
// slot to clear.  Chunks even out the last round of workgroups, but only few or long
// segments are worth it.  us from load to correlated, 1 / 2 / 4 / 8 chunks: 512 inputs,
// 128 channels, 4,000 spectra 299 / 546 / 868 / 1,613, 40,000 2,465 / 2,376 / 2,451 /
// 2,656; 256 channels, 2,500 382 / 933 / 1,666 / 3,180; 256 inputs, 128 channels, 10,000
// 228 / 312 / 361 / 501, 40,000 851 / 786 / 789 / 885; 128 inputs, 40,000 558 / 358 /
// 320 / 378; 80 inputs, 64 channels, 20,000 241 / 153 / 99 / 82.
constexpr int kMinChunkGroups = 64;
int pick_chunks(int64_t items, int64_t pairs, int ngrp) {
    const int cus = device_cus();
    int best = 1;
    double best_cost = 1e300;
    for (int k = 1; k <= 8; ++k) {
        if (k > 1 && (ngrp + k - 1) / k < kMinChunkGroups) break;
        const double most = (double)((items * k + cus - 1) / cus), share = (double)pairs / cus;
        const double loops = (most > 1.0 ? most : 1.25) * ngrp / k;
        const double flushes = k == 1 ? 0.0022 * share : 0.0097 * share * k + 60.0;
        if (loops + flushes < best_cost - 1e-9) {
            best_cost = loops + flushes;
            best = k;
        }
    }
    return best;
}
}  // namespace

namespace {
// Workgroups per channel of a single-plan launch, chunks per workgroup (INT8 only;
// a.nks == 1 on entry asks for whole segments) and their size.
void set_chunks(int xprec, XArgs &a) {
    const int m = (a.n_in + kTile / 2 - 1) / (kTile / 2);
    a.sets = tri_sets(m);
    a.ntiles = tri_groups(m, a.sets);
    if (a.nks != 1) a.nks = xprec == MWAX_X_INT8 ? pick_chunks((int64_t)a.ntiles * a.L, a.P * a.L, a.ngrp) : 1;
    // Unsplit, the last round of workgroups is shorter with some waves idle if that
    // brings as many workgroups to every CU (each has the same number of blocks then).
    // FP16, 512 inputs, 128 channels, two calls of 10,000 spectra: 10 workgroups per
    // channel, five per CU, 4,724 us channelise to emission; 9, 4.5 per CU, 4,751 us.
    if (a.nks == 1) {
        const int cus = device_cus(), alone = tri_groups(m, 0);
        auto most_blocks = [&](int64_t n) { return (double)((n * a.L + cus - 1) / cus) / (double)n; };
        if (most_blocks(alone) < most_blocks(a.ntiles)) {
            a.sets = 0;
            a.ntiles = alone;
        }
    }
    a.kchunk = (a.ngrp + a.nks - 1) / a.nks;
    a.nks = (a.ngrp + a.kchunk - 1) / a.kchunk;   // no empty chunk
}
}  // namespace

bool xengine_accumulates(int xprec, const XArgs &args) {
    XArgs a = args;
    set_chunks(xprec, a);
    return a.nks > 1;
}

hipError_t launch_xengine(int xprec, const XArgs &args, hipStream_t s) {
    XArgs a = args;
    set_chunks(xprec, a);
    const int64_t blocks = (int64_t)a.ntiles * a.L * a.nks;
    if (blocks <= 0 || a.ngrp <= 0) return hipSuccess;
    switch (xprec) {
        case MWAX_X_INT8:
            hipLaunchKernelGGL(xengine_mfma<MWAX_X_INT8>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
            break;
        case MWAX_X_FP16:
            hipLaunchKernelGGL(xengine_mfma<MWAX_X_FP16>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int XP>
static hipError_t launch_small(const XArgs &args, const XSegList &segs, hipStream_t s) {
    XArgs a = args;
    int ngrp = 0;
    for (int k = 0; k < segs.n; ++k) ngrp = segs.s[k].ngrp > ngrp ? segs.s[k].ngrp : ngrp;
    a.ntiles = xengine_tile_count(a.n_in, kXTileTiny);
    const unsigned blocks = (unsigned)(a.ntiles * a.L * segs.n);
    // As many waves as the device holds at two per SIMD, but no more than stages and
    // no fewer than two (one takes a single stage).  32 tiles FP16, 8,000 spectra x 2,
    // whole step in us at 8 / 4 / 2 waves: 64 channels 182 / 204 / 263, 128 channels
    // 360 / 355 / 385, 256 channels 702 / 723 / 685; 512 spectra x 2, 1,024 channels
    // 359 / 308 / 289.
    int w = kSmallSlices;
    while (w > 1 && ngrp <= w / 2 * kSmallG) w /= 2;
    while (w > 2 && (int64_t)blocks * w > 8 * device_cus()) w /= 2;
    if (w == 1) hipLaunchKernelGGL((xengine_small<XP, 1>), dim3(blocks), dim3(64), 0, s, a, segs);
    else if (w == 2) hipLaunchKernelGGL((xengine_small<XP, 2>), dim3(blocks), dim3(128), 0, s, a, segs);
    else if (w == 4) hipLaunchKernelGGL((xengine_small<XP, 4>), dim3(blocks), dim3(256), 0, s, a, segs);
    else hipLaunchKernelGGL((xengine_small<XP, 8>), dim3(blocks), dim3(512), 0, s, a, segs);
    return hipGetLastError();
}

hipError_t launch_xengine_small(int xprec, const XArgs &a, const XSegList &segs, hipStream_t s) {
    if (segs.n < 1 || segs.n > kXSegs || a.n_in > kXSmallInputs) return hipErrorInvalidValue;
    if (xprec == MWAX_X_INT8) return launch_small<MWAX_X_INT8>(a, segs, s);
    if (xprec == MWAX_X_FP16) return launch_small<MWAX_X_FP16>(a, segs, s);
    return hipErrorInvalidValue;
}

hipError_t launch_xengine_f32(const XArgs &args, const XSegList &segs, hipStream_t s) {
    XArgs a = args;
    if (segs.n < 1 || segs.n > kXSegs) return hipErrorInvalidValue;
    a.ntiles = xengine_tile_count(a.n_in, kXTileSmall);
    const int64_t tiles = (int64_t)a.ntiles * a.L * segs.n;
    // fewer 64 x 64 tiles than the four per CU that are resident together
    // would leave matrix cores idle; the small form has twice the waves per
    // workgroup and up to four times the workgroups
    if (tiles < 4 * device_cus()) {
        a.ntiles = xengine_tile_count(a.n_in, 32);
        hipLaunchKernelGGL(xengine_f32_small, dim3((unsigned)(a.ntiles * a.L * segs.n)), dim3(64 * kFSWaves), 0, s, a, segs);
    } else {
        hipLaunchKernelGGL(xengine_f32, dim3((unsigned)tiles), dim3(kThreads), 0, s, a, segs);
    }
    return hipGetLastError();
}

hipError_t launch_xengine_batch(int xprec, const XBatchArgs &b, int grid, hipStream_t s) {
    if (grid < 1) return hipSuccess;
    switch (xprec) {
        case MWAX_X_INT8:
            hipLaunchKernelGGL(xengine_batch<MWAX_X_INT8>, dim3((unsigned)grid), dim3(kThreads), 0, s, b);
            break;
        case MWAX_X_FP16:
            hipLaunchKernelGGL(xengine_batch<MWAX_X_FP16>, dim3((unsigned)grid), dim3(kThreads), 0, s, b);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_xengine_avg(int xprec, const XAvgArgs &args, hipStream_t s) {
    XAvgArgs a = args;
    a.ntiles = xengine_tile_count(a.n_in, kXTileSmall);
    if (a.segs.n < 1 || a.segs.n > kXSegs) return hipErrorInvalidValue;
    const int64_t blocks = (int64_t)a.N * a.ntiles * a.segs.n;
    // Fewer 64-edge workgroups than CUs: waves that share the K loop instead.  Whole
    // step in us, 64-edge form / this one, FP16, 200 spectra: 16 workgroups 244 / 90
    // (64 inputs, 1,024 channels by 64), 128 workgroups 467 / 408 (64 inputs, 6,400
    // by 50), 144 workgroups 325 / 213 (200 inputs, 1,024 by 64); but 256 workgroups
    // 63 / 77 (64 inputs, 1,024 by 4) and 288 workgroups 62 / 82 (200 inputs, 256 by 8).
    if (blocks < device_cus()) {
        a.ntiles = xengine_tile_count(a.n_in, kXTileTiny);
        const dim3 grid((unsigned)(a.N * a.ntiles * a.segs.n)), threads(64 * kSmallSlices);
        if (xprec == MWAX_X_INT8) hipLaunchKernelGGL(xengine_avg_small<MWAX_X_INT8>, grid, threads, 0, s, a);
        else if (xprec == MWAX_X_FP16) hipLaunchKernelGGL(xengine_avg_small<MWAX_X_FP16>, grid, threads, 0, s, a);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    switch (xprec) {
        case MWAX_X_INT8:
            hipLaunchKernelGGL(xengine_avg<MWAX_X_INT8>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
            break;
        case MWAX_X_FP16:
            hipLaunchKernelGGL(xengine_avg<MWAX_X_FP16>, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_zero_i32(int32_t *p, int n, hipStream_t s) {
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(zero_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

int xengine_batch_max_grid(int xprec, int device) {
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1)
        cus = 256;
    const void *fn = xprec == MWAX_X_INT8 ? reinterpret_cast<const void *>(&xengine_batch<MWAX_X_INT8>)
                                          : reinterpret_cast<const void *>(&xengine_batch<MWAX_X_FP16>);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kThreads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return cus * per_cu;
}

}  // namespace mwax
