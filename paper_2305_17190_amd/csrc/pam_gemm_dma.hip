// PAM matrix products on gfx950, for float32 and bfloat16 operands.
//
// PAM (Kosson & Jaggi, Sec. 2.2): the product of two float32 numbers is
// replaced by the int32 sum of their encodings minus one exponent bias
// (127 << 23); the sign is the exclusive or of the signs, zero / denormal
// operands and underflowing results give signed zeros, overflowing results
// saturate at +-FLT_MAX, NaN / inf follow IEEE multiplication with a
// canonical quiet NaN.  PAM matrix products (Sec. 3.2) keep float32
// accumulation.
//
// The product is a vector-ALU contraction (PAM is not a product, so the
// matrix cores do not apply).  Each workgroup owns a BM x BN output tile,
// each thread an 8 x 8 register micro-tile, and K advances in LDS chunks of
// 16 steps per k-group.  On gfx950 the integer add and the float32 add, mul
// and fma issue at twice the rate of other vector ops, so the per-MAC work is
// built from those four only.
//
// Encodings in LDS, written once per chunk: A as it is; B as b' = b -
// 0x3F800000 (a denormal b first flushed to its signed zero).
//   S1 (per MAC: v_add_u32, v_add_f32): acc += a + b'.  When both exponent
//      fields are in [64, 190] the int32 sum is PAM(a, b)'s encoding itself
//      (Sec. 2.2's addition; the magnitude sum cannot leave the normal range
//      and the carry out of the sign bits leaves their exclusive or): no
//      multiply at all.
//   SCALED form, for the other finite operands: with aM the encoding of
//   1 + M_A (exponent field 127, a's mantissa) and m = a with its mantissa
//   cleared (the float +-2^E_A, or +-0), t = aM + b' is the encoding of
//   PAM(1 + M_A, b); PAM is exact under power-of-two scaling (Fig. 2: the
//   pattern repeats per octave), so t * m = PAM(a, b) whenever the result is
//   a normal number, the float multiply supplying the sign.  A zero b makes t
//   a denormal encoding, which the float unit (denormals flushed) reads as 0.
//   aM and m are derived per row from A's encoding (two bit operations).
//   S2 (per MAC: v_add_u32, v_fmac_f32): acc = fma(t, m, acc).  Exact when
//      no product underflows: every nonzero operand has exponent field in
//      [64, 190].
//   S3 (per MAC: v_add_u32, v_mul_f32, v_add_f32): p = t * m rounded on its
//      own, so an underflowing product flushes to the signed zero PAM
//      defines; exact for all finite operands with |x| < 2^64.
//   Each wave takes S1, S2 or S3 per k step from bit masks of the operands
//   it reads at that k: S1 unless one has exponent field below 64, S3 if one
//   of those is a normal number ("tiny", field 1..63), S2 otherwise (zeros
//   and denormals only); the S1 steps first, then S2, then S3.
//   SPECIAL: a chunk holding inf, NaN or |x| >= 2^64 takes the complete
//   per-MAC definition (never on finite data below 2^64).
//
// Staging:
//
// * Each chunk's operand pieces (16 bytes: four float32 or eight bfloat16
//   elements consecutive in memory) are copied by the memory pipeline
//   (gfx950's global_load_lds_dwordx4) into an LDS landing buffer.  No
//   register holds a chunk while its copy is in flight, so the kernel keeps
//   only the accumulators and the compute step's operands live across the K
//   loop, and the 128 x 128 tile fits four waves per SIMD.
// * At the chunk boundary each thread re-reads segments of four elements
//   its own wave copied (so no barrier is needed for them), widens bfloat16
//   elements exactly to float32 encodings, scans and encodes them, and writes
//   them k-major into the compute buffer.  A thread holds L rows of one k
//   quad of a K-contiguous operand and writes each k as one L-word store;
//   the lanes of a wave write consecutive columns of one k row, so the
//   stores are free of bank conflicts.  Float32 and bfloat16 operands are
//   staged into the same segments, so a bfloat16 product equals the float32
//   product of its widened operands bit for bit.
// * The next chunk is copied while a chunk is computed, at any alignment of
//   the operand; at the end of K and past the last columns the pieces start
//   earlier, so that each lies whole inside the operand (pam_dma_tile.h), and
//   steps past K are not run.  Before, unaligned operands and such ends were
//   loaded element by element at the chunk boundary: the two products of a
//   197-token attention (192 matrices, head 64) took 99 us, now 78 us.
//
// With k-groups (KW > 1) the groups other than the first write their
// partial tiles to LDS, and the first group adds them in group order and
// stores the tile.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pam_dma_tile.h"
#include "pam_internal.h"
#include "pam_scalar.h"

namespace pamk {

// One micro-tile row of an S3 step from A's own encoding a: first 1 + M_A
// (exponent field 127, a's mantissa) and +-2^E_A (a with its mantissa
// cleared, +-0 for zero / denormal a), then the SCALED products with the
// eight b' values, each rounded on its own (an underflowing product flushes
// to zero), then added.  One asm block per row keeps the derived values'
// lifetime to the row.
#define PAM_DMA_ROW_OPERANDS                                                                               \
    : [am] "=&v"(am), [m] "=&v"(m), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3),       \
      [t4] "=&v"(t4), [t5] "=&v"(t5), [t6] "=&v"(t6), [t7] "=&v"(t7), [c0] "+v"(acc[0]), [c1] "+v"(acc[1]), \
      [c2] "+v"(acc[2]), [c3] "+v"(acc[3]), [c4] "+v"(acc[4]), [c5] "+v"(acc[5]), [c6] "+v"(acc[6]),        \
      [c7] "+v"(acc[7])                                                                                    \
    : [a] "v"(a), [b0] "v"(bb[0]), [b1] "v"(bb[1]), [b2] "v"(bb[2]), [b3] "v"(bb[3]), [b4] "v"(bb[4]),     \
      [b5] "v"(bb[5]), [b6] "v"(bb[6]), [b7] "v"(bb[7]), [mant] "v"(kMant), [bias] "v"(kBias),              \
      [se] "v"(kSignExp)
#define PAM_DMA_ROW_HEAD                                                                                   \
    "v_and_or_b32 %[am], %[a], %[mant], %[bias]\n\tv_and_b32 %[m], %[a], %[se]\n\t"                        \
    "v_add_u32 %[t0], %[am], %[b0]\n\tv_add_u32 %[t1], %[am], %[b1]\n\t"                                   \
    "v_add_u32 %[t2], %[am], %[b2]\n\tv_add_u32 %[t3], %[am], %[b3]\n\t"                                   \
    "v_add_u32 %[t4], %[am], %[b4]\n\tv_add_u32 %[t5], %[am], %[b5]\n\t"                                   \
    "v_add_u32 %[t6], %[am], %[b6]\n\tv_add_u32 %[t7], %[am], %[b7]\n\t"

__device__ __forceinline__ void dma_s3_row(float (&acc)[8], uint32_t a, const uint32_t (&bb)[8]) {
    uint32_t am, m, t0, t1, t2, t3, t4, t5, t6, t7;
    asm(PAM_DMA_ROW_HEAD
        "v_mul_f32 %[t0], %[t0], %[m]\n\tv_mul_f32 %[t1], %[t1], %[m]\n\t"
        "v_mul_f32 %[t2], %[t2], %[m]\n\tv_mul_f32 %[t3], %[t3], %[m]\n\t"
        "v_mul_f32 %[t4], %[t4], %[m]\n\tv_mul_f32 %[t5], %[t5], %[m]\n\t"
        "v_mul_f32 %[t6], %[t6], %[m]\n\tv_mul_f32 %[t7], %[t7], %[m]\n\t"
        "v_add_f32 %[c0], %[c0], %[t0]\n\tv_add_f32 %[c1], %[c1], %[t1]\n\t"
        "v_add_f32 %[c2], %[c2], %[t2]\n\tv_add_f32 %[c3], %[c3], %[t3]\n\t"
        "v_add_f32 %[c4], %[c4], %[t4]\n\tv_add_f32 %[c5], %[c5], %[t5]\n\t"
        "v_add_f32 %[c6], %[c6], %[t6]\n\tv_add_f32 %[c7], %[c7], %[t7]"
        PAM_DMA_ROW_OPERANDS);
}
#undef PAM_DMA_ROW_HEAD
#undef PAM_DMA_ROW_OPERANDS

// A whole S1 step (acc[i][j] += a_i + b'_j for the 8 x 8 micro-tile) as one
// instruction sequence.
#define PAM_DMA_S1_ROW(R, A)                                                                               \
    "v_add_u32 %[t0], %[" #A "], %[b0]\n\tv_add_u32 %[t1], %[" #A "], %[b1]\n\t"                           \
    "v_add_u32 %[t2], %[" #A "], %[b2]\n\tv_add_u32 %[t3], %[" #A "], %[b3]\n\t"                           \
    "v_add_u32 %[t4], %[" #A "], %[b4]\n\tv_add_u32 %[t5], %[" #A "], %[b5]\n\t"                           \
    "v_add_u32 %[t6], %[" #A "], %[b6]\n\tv_add_u32 %[t7], %[" #A "], %[b7]\n\t"                           \
    "v_add_f32 %[c" #R "0], %[c" #R "0], %[t0]\n\tv_add_f32 %[c" #R "1], %[c" #R "1], %[t1]\n\t"           \
    "v_add_f32 %[c" #R "2], %[c" #R "2], %[t2]\n\tv_add_f32 %[c" #R "3], %[c" #R "3], %[t3]\n\t"           \
    "v_add_f32 %[c" #R "4], %[c" #R "4], %[t4]\n\tv_add_f32 %[c" #R "5], %[c" #R "5], %[t5]\n\t"           \
    "v_add_f32 %[c" #R "6], %[c" #R "6], %[t6]\n\tv_add_f32 %[c" #R "7], %[c" #R "7], %[t7]\n\t"
#define PAM_DMA_ACC_ROW(R)                                                                                 \
    [c##R##0] "+v"(acc[R][0]), [c##R##1] "+v"(acc[R][1]), [c##R##2] "+v"(acc[R][2]),                       \
        [c##R##3] "+v"(acc[R][3]), [c##R##4] "+v"(acc[R][4]), [c##R##5] "+v"(acc[R][5]),                   \
        [c##R##6] "+v"(acc[R][6]), [c##R##7] "+v"(acc[R][7])

__device__ __forceinline__ void dma_s1_step(float (&acc)[8][8], const uint4 &al, const uint4 &ah,
                                            const uint32_t (&bb)[8]) {
    uint32_t t0, t1, t2, t3, t4, t5, t6, t7;
    asm(PAM_DMA_S1_ROW(0, a0) PAM_DMA_S1_ROW(1, a1) PAM_DMA_S1_ROW(2, a2) PAM_DMA_S1_ROW(3, a3)
            PAM_DMA_S1_ROW(4, a4) PAM_DMA_S1_ROW(5, a5) PAM_DMA_S1_ROW(6, a6) PAM_DMA_S1_ROW(7, a7)
        : PAM_DMA_ACC_ROW(0), PAM_DMA_ACC_ROW(1), PAM_DMA_ACC_ROW(2), PAM_DMA_ACC_ROW(3), PAM_DMA_ACC_ROW(4),
          PAM_DMA_ACC_ROW(5), PAM_DMA_ACC_ROW(6), PAM_DMA_ACC_ROW(7), [t0] "=&v"(t0), [t1] "=&v"(t1),
          [t2] "=&v"(t2), [t3] "=&v"(t3), [t4] "=&v"(t4), [t5] "=&v"(t5), [t6] "=&v"(t6), [t7] "=&v"(t7)
        : [a0] "v"(al.x), [a1] "v"(al.y), [a2] "v"(al.z), [a3] "v"(al.w), [a4] "v"(ah.x), [a5] "v"(ah.y),
          [a6] "v"(ah.z), [a7] "v"(ah.w), [b0] "v"(bb[0]), [b1] "v"(bb[1]), [b2] "v"(bb[2]), [b3] "v"(bb[3]),
          [b4] "v"(bb[4]), [b5] "v"(bb[5]), [b6] "v"(bb[6]), [b7] "v"(bb[7]));
}
#undef PAM_DMA_S1_ROW

// A whole S2 step, acc[i][j] = fma(aM_i + b'_j, m_i, acc[i][j]): per row 1 + M_A
// (1.0 is the bias) and +-2^E_A, then the SCALED products.  (Three full-rate
// ops in place of the and-or and the and ran 3% slower on ReLU operands.)
#define PAM_DMA_S2_ROW(R, A)                                                                               \
    "v_and_or_b32 %[am], %[" #A "], %[mant], 1.0\n\tv_and_b32 %[m], 0xff800000, %[" #A "]\n\t"              \
    "v_add_u32 %[t0], %[am], %[b0]\n\tv_add_u32 %[t1], %[am], %[b1]\n\t"                                   \
    "v_add_u32 %[t2], %[am], %[b2]\n\tv_add_u32 %[t3], %[am], %[b3]\n\t"                                   \
    "v_add_u32 %[t4], %[am], %[b4]\n\tv_add_u32 %[t5], %[am], %[b5]\n\t"                                   \
    "v_add_u32 %[t6], %[am], %[b6]\n\tv_add_u32 %[t7], %[am], %[b7]\n\t"                                   \
    "v_fmac_f32 %[c" #R "0], %[t0], %[m]\n\tv_fmac_f32 %[c" #R "1], %[t1], %[m]\n\t"                       \
    "v_fmac_f32 %[c" #R "2], %[t2], %[m]\n\tv_fmac_f32 %[c" #R "3], %[t3], %[m]\n\t"                       \
    "v_fmac_f32 %[c" #R "4], %[t4], %[m]\n\tv_fmac_f32 %[c" #R "5], %[t5], %[m]\n\t"                       \
    "v_fmac_f32 %[c" #R "6], %[t6], %[m]\n\tv_fmac_f32 %[c" #R "7], %[t7], %[m]\n\t"

__device__ __forceinline__ void dma_s2_step(float (&acc)[8][8], const uint4 &al, const uint4 &ah,
                                            const uint32_t (&bb)[8]) {
    uint32_t am, m, t0, t1, t2, t3, t4, t5, t6, t7;
    asm(PAM_DMA_S2_ROW(0, a0) PAM_DMA_S2_ROW(1, a1) PAM_DMA_S2_ROW(2, a2) PAM_DMA_S2_ROW(3, a3)
            PAM_DMA_S2_ROW(4, a4) PAM_DMA_S2_ROW(5, a5) PAM_DMA_S2_ROW(6, a6) PAM_DMA_S2_ROW(7, a7)
        : PAM_DMA_ACC_ROW(0), PAM_DMA_ACC_ROW(1), PAM_DMA_ACC_ROW(2), PAM_DMA_ACC_ROW(3), PAM_DMA_ACC_ROW(4),
          PAM_DMA_ACC_ROW(5), PAM_DMA_ACC_ROW(6), PAM_DMA_ACC_ROW(7), [am] "=&v"(am), [m] "=&v"(m), [t0] "=&v"(t0),
          [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [t4] "=&v"(t4), [t5] "=&v"(t5), [t6] "=&v"(t6),
          [t7] "=&v"(t7)
        : [a0] "v"(al.x), [a1] "v"(al.y), [a2] "v"(al.z), [a3] "v"(al.w), [a4] "v"(ah.x), [a5] "v"(ah.y),
          [a6] "v"(ah.z), [a7] "v"(ah.w), [b0] "v"(bb[0]), [b1] "v"(bb[1]), [b2] "v"(bb[2]), [b3] "v"(bb[3]),
          [b4] "v"(bb[4]), [b5] "v"(bb[5]), [b6] "v"(bb[6]), [b7] "v"(bb[7]), [mant] "s"(kMant));
}
#undef PAM_DMA_S2_ROW
#undef PAM_DMA_ACC_ROW

// Eight values of one k row of a compute buffer: four at p, four at p + half.
__device__ __forceinline__ void dma_frag(const uint32_t *p, int half, uint32_t (&out)[8]) {
    const uint4 lo = *reinterpret_cast<const uint4 *>(p);
    const uint4 hi = *reinterpret_cast<const uint4 *>(p + half);
    out[0] = lo.x; out[1] = lo.y; out[2] = lo.z; out[3] = lo.w;
    out[4] = hi.x; out[5] = hi.y; out[6] = hi.z; out[7] = hi.w;
}

// Waves per SIMD the tile is compiled for (registers per wave 512 / waves),
// matching what its LDS footprint allows on a 160 KB compute unit.
constexpr int dma_waves_per_simd(int bm, int bn, int kw) {
    return (bm == 128 && bn == 128 && kw == 1) ? 4 : (bm == 128 && bn == 64 && kw == 2) ? 3 : 2;
}

// A chunk with more S2 steps than this (zeros in most of its k steps: ReLU
// activations, masked probabilities, dropout) takes its S1 and S2 steps in
// one unrolled pass of S2 steps, operands read one step ahead; with fewer,
// the S2 steps come one by one after the S1 pass.  A ReLU block's six products
// (8192 tokens, 512 -> 2048 -> 512, four of them on half-zero operands) took
// 2346 us; 2317 us with this pass, 2112 us with the step masks combined over
// lanes as well (DmaTile::mark).
constexpr int kDenseS2 = 8;

// Minimum LDS words per workgroup.  Workgroups of one or two waves can be
// placed unevenly on a compute unit's four SIMDs when more fit than the
// launch fills (measured: one workgroup in a launch with three waves on a
// SIMD ran 1.4x as long as the others).  Their LDS is padded so that no more
// than two waves per SIMD fit: four 128 x 64 or eight 64 x 64 workgroups.
// The 128 x 64 two-group tile built for two waves per SIMD is padded to two
// workgroups per compute unit for the same reason.
constexpr int dma_min_lds_words(int bm, int bn, int kw, int wps) {
    return (bm == 128 && bn == 64 && kw == 1)   ? (33 << 10) / 4
           : (bm == 64 && bn == 64 && kw == 1)  ? (18 << 10) / 4
           : (bm == 128 && bn == 64 && kw == 2 && wps == 2) ? (54 << 10) / 4
                                                           : 0;
}

// WPS: waves per SIMD the kernel is compiled for.  At two (256 registers a
// wave), and at three for a row-major A (168 registers, measured to fit), the
// per-thread staging addresses are computed once, before the K loop;
// otherwise they are recomputed per chunk, since registers held across the
// loop would not fit beside the accumulators.
// EDGE: what of the edges the launch needs (DmaTile::copy); kernels of their
// own: compiled in one, the edges' scalar values spilled into vector lanes
// across the K loop and cost the other launches 3%, the clamp and blanks of
// whole pieces past the last column (1) alone 1-3%.
template <int BM, int BN, int KW, bool TA, bool TB, int WPS, int EDGE, typename T>
__global__ void __launch_bounds__(BM * BN / 64 * KW) __attribute__((amdgpu_waves_per_eu(WPS)))
pam_gemm_dma_kernel(GemmParams p) {
    constexpr bool kKeepAddresses = WPS <= 2 || (WPS == 3 && !TA);
    // k steps per group per chunk (the step masks hold one bit per step of a
    // chunk in each half of a 32-bit word).
    constexpr int KPG = kChunkK;
    constexpr int BK = KPG * KW;
    constexpr int NTG = BM * BN / 64;
    constexpr int NT = NTG * KW;
    constexpr int NRW = NTG / 64;
    constexpr int WC = BN / 64;
    constexpr int WR = NRW / WC;
    constexpr int NSLOT = WR + WC;
    static_assert(WC >= 1 && WR * WC == NRW && BM / 64 == WR, "waves do not tile the output tile");
    constexpr int HM = BM / 2;
    constexpr int HN = BN / 2;
    constexpr int LDR = BN;                // partial-tile rows (KW > 1)
    using TileA = DmaTile<BM, BK, NT, !TA, T>;
    using TileB = DmaTile<BN, BK, NT, TB, T>;
    constexpr int kRawA = TileA::CL * NT * 4;   // 16 bytes per copy
    constexpr int kRawB = TileB::CL * NT * 4;
    constexpr int kStage = kRawA + kRawB + BK * BM + BK * BN;
    // Partial tiles held at once by the LDS after the K loop (KW > 1).
    constexpr int kRedTiles = KW == 1 ? 0 : (kStage / (BM * LDR) >= KW - 1 ? KW - 1 : kStage / (BM * LDR));
    static_assert(KW == 1 || kRedTiles >= 1, "no room for a partial tile");
    constexpr int kRed = kRedTiles * BM * LDR;
    // Landing buffers, then the k-major compute buffers; for KW > 1 the
    // partial tiles reuse the same bytes after the K loop.
    constexpr int kWords0 = kStage > kRed ? kStage : kRed;
    constexpr int kMinWords = dma_min_lds_words(BM, BN, KW, WPS);
    __shared__ __attribute__((aligned(16))) uint32_t smem[kWords0 > kMinWords ? kWords0 : kMinWords];
    // Step masks of the two chunks in flight (k-group g's slot words at
    // g * NSLOT), and after them the chunk's SPECIAL vote.
    __shared__ uint32_t sMask[2][KW * NSLOT + 1];
    static_assert(2 * (KW * NSLOT + 1) <= NT, "the mask words are cleared one per thread");
    uint32_t *rawA = smem;
    uint32_t *rawB = smem + kRawA;
    uint32_t *encA = smem + kRawA + kRawB;
    uint32_t *encB = encA + BK * BM;

    const int tid = threadIdx.x;
    const int grp = tid / NTG;
    const int t = tid % NTG;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane(lds_addr(smem) + (uint32_t)wave * 1024u);
    const int gwave = t >> 6;
    const int wr = gwave / WC;
    const int wc = gwave % WC;
    const int lane = tid & 63;
    const int tx = wc * 8 + (lane & 7);
    const int ty = wr * 8 + (lane >> 3);
    const uint32_t item = blockIdx.x;
    const bool whole = item < (uint32_t)p.whole;
    const uint32_t rel = item - (uint32_t)p.whole;
    const uint32_t nsplit = (uint32_t)max(p.split_tiles, 1);
    const uint32_t st = whole ? 0u : rel % nsplit;
    const int split = whole ? 0 : (int)(rel / nsplit);
    const uint32_t tile_lin = whole ? item : (uint32_t)p.whole + st;
    const int64_t bz = tile_lin / (uint32_t)p.tiles;
    const int tile = (int)(tile_lin % (uint32_t)p.tiles);
    const int tm = tile / p.tiles_n;
    const int tn = tile % p.tiles_n;
    const int m0 = tm * BM;
    const int n0 = tn * BN;
    const int kb = whole ? 0 : split * p.k_per_split;
    const int ke = whole ? p.k : min(p.k, kb + p.k_per_split);
    const int nchunks = ke > kb ? (ke - kb + BK - 1) / BK : 0;

    const T *a_base = reinterpret_cast<const T *>(p.A) + bz * p.strideA +
                      (TA ? (int64_t)kb * p.lda + m0 : (int64_t)m0 * p.lda + kb);
    const T *b_base = reinterpret_cast<const T *>(p.B) + bz * p.strideB +
                      (TB ? (int64_t)n0 * p.ldb + kb : (int64_t)kb * p.ldb + n0);
    const int64_t a_step = TA ? (int64_t)BK * p.lda : BK;
    const int64_t b_step = TB ? BK : (int64_t)BK * p.ldb;
    TileA la;
    TileB lb;
    auto a_slot = [](int o) { return (int)(((uint32_t)o % HM) / 32u); };
    auto b_slot = [](int o) { return WR + (int)(((uint32_t)o % HN) / 32u); };

    float acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
            acc[i][j] = 0.0f;

    if (tid < 2 * (KW * NSLOT + 1))
        (&sMask[0][0])[tid] = 0u;

    // The copies' kinds (A's, then B's) as one scalar word, tested afresh in
    // each chunk (conditions kept across the loop took lane masks, spilled).
    const uint32_t kinds = EDGE < 2 ? 0u : TileA::kind(ke, m0, p.m, p.lda) | TileB::kind(ke, n0, p.n, p.ldb) << 2;
    if (nchunks > 0) {
        TileA::template copy<0, EDGE>(a_base, lds_w, tid, p.lda, m0, p.m, ke - kb, kinds & 3u);
        TileB::template copy<kRawA * 4, EDGE>(b_base, lds_w, tid, p.ldb, n0, p.n, ke - kb, kinds >> 2);
    }

    const int k_first = grp * KPG;
    auto chunk = [&](auto edge, int c) {
        constexpr int E = decltype(edge)::value;   // of this chunk and the next
        const int k_rem = ke - kb - c * BK;   // k steps left, this chunk's included
        uint32_t kd = 0u;
        if constexpr (E == 2) {
            kd = __builtin_amdgcn_readfirstlane(kinds);
            asm volatile("" : "+s"(kd));
        }
        // The thread index through an empty asm: staging addresses derived
        // from it are recomputed per chunk instead of being hoisted out of
        // the loop into registers that would stay live during the steps.
        int tid_c = tid;
        if constexpr (!kKeepAddresses)
            asm volatile("" : "+v"(tid_c));
        __builtin_amdgcn_s_setprio(1);
        // This thread's copies of chunk c have landed (the only vector-memory
        // operations outstanding).
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        la.template fetch<E>(rawA, wave, p.lda, m0, p.m, k_rem, kd & 3u, tid_c);
        lb.template fetch<E>(rawB, wave, p.ldb, n0, p.n, k_rem, kd >> 2, tid_c);

        if (p.round_drop != 0) {
            la.round_mantissa(p.round_drop);
            lb.round_mantissa(p.round_drop);
        }
        uint32_t smin_a[TileA::L], smin_b[TileB::L];
        const uint32_t mx = max(la.scan(smin_a), lb.scan(smin_b));
        uint32_t low_b = smin_b[0];
#pragma unroll
        for (int r = 1; r < TileB::L; ++r)
            low_b = min(low_b, smin_b[r]);
        if (TileB::low_seg(low_b))   // rare per thread: B's denormals to zero
            lb.flush_denormals();
        uint32_t *mask = sMask[c & 1];
        __syncthreads();   // every wave is done reading the previous chunk (and zeroing this mask)
        la.store_values(encA, false, tid_c);
        la.template mark<KPG>(tid_c, smin_a, mask, NSLOT, a_slot);
        lb.store_values(encB, true, tid_c);
        lb.template mark<KPG>(tid_c, smin_b, mask, NSLOT, b_slot);
        // The workgroup's SPECIAL vote: one more mask word.
        if (mx >= (191u << 24))
            atomicOr(&mask[KW * NSLOT], 1u);
        __syncthreads();

        const bool special = __builtin_amdgcn_readfirstlane(mask[KW * NSLOT]) != 0u;
        const uint32_t low =
            __builtin_amdgcn_readfirstlane(mask[grp * NSLOT + wr] | mask[grp * NSLOT + WR + wc]);
        if (tid < KW * NSLOT + 1)
            (&sMask[0][0])[(((uint32_t)c + 1u) & 1u) * (KW * NSLOT + 1) + (uint32_t)tid] = 0u;

        // The next chunk's copies land while this one is computed (the
        // landing slots are this thread's own and were read above).
        if (c + 1 < nchunks) {
            TileA::template copy<0, E>(a_base + (c + 1) * a_step, lds_w, tid_c, p.lda, m0, p.m, k_rem - BK, kd & 3u);
            TileB::template copy<kRawA * 4, E>(b_base + (c + 1) * b_step, lds_w, tid_c, p.ldb, n0, p.n, k_rem - BK, kd >> 2);
        }

        __builtin_amdgcn_s_setprio(0);

        // The group's steps of this chunk (those past K take none).
        const uint32_t steps = (1u << (E == 2 ? min(max(k_rem - k_first, 0), KPG) : KPG)) - 1u;
        uint32_t s1_bits = special ? 0u : (~low & steps);
        uint32_t s2_bits = special ? 0u : (low & ~(low >> 16) & steps);
        const uint32_t s3_bits = special ? 0u : ((low >> 16) & steps);
        const uint32_t sp_bits = special ? steps : 0u;
        const uint32_t *a_row = encA + k_first * BM + ty * 4;
        const uint32_t *b_row = encB + k_first * BN + tx * 4;
        {
            uint4 al[2], ah[2];
            uint32_t bq[2][8];
            auto rd = [&](int k, int slot) {
                al[slot] = *reinterpret_cast<const uint4 *>(a_row + k * BM);
                ah[slot] = *reinterpret_cast<const uint4 *>(a_row + k * BM + HM);
                const uint4 lo = *reinterpret_cast<const uint4 *>(b_row + k * BN);
                const uint4 hi = *reinterpret_cast<const uint4 *>(b_row + k * BN + HN);
                bq[slot][0] = lo.x; bq[slot][1] = lo.y; bq[slot][2] = lo.z; bq[slot][3] = lo.w;
                bq[slot][4] = hi.x; bq[slot][5] = hi.y; bq[slot][6] = hi.z; bq[slot][7] = hi.w;
            };
            if (__builtin_popcount(s2_bits) > kDenseS2) {
                s2_bits |= s1_bits;
                rd(0, 0);
#pragma unroll
                for (int k = 0; k < KPG; ++k) {
                    const int cur = k & 1;
                    if (k + 1 < KPG)
                        rd(k + 1, cur ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if ((s2_bits >> k) & 1u)
                        dma_s2_step(acc, al[cur], ah[cur], bq[cur]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                s1_bits = 0u;
                s2_bits = 0u;
            }
            if (s1_bits != 0u) {
                rd(0, 0);
#pragma unroll
                for (int k = 0; k < KPG; ++k) {
                    const int cur = k & 1;
                    if (k + 1 < KPG)
                        rd(k + 1, cur ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if ((s1_bits >> k) & 1u)
                        dma_s1_step(acc, al[cur], ah[cur], bq[cur]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // S2 steps, then S3 steps.
        for (uint32_t todo = s2_bits; todo != 0u; todo &= todo - 1u) {
            const int kk = __builtin_ctz(todo);
            const uint4 al = *reinterpret_cast<const uint4 *>(a_row + kk * BM);
            const uint4 ah = *reinterpret_cast<const uint4 *>(a_row + kk * BM + HM);
            uint32_t bb[8];
            dma_frag(b_row + kk * BN, HN, bb);
            dma_s2_step(acc, al, ah, bb);
        }
        for (uint32_t todo = s3_bits; todo != 0u; todo &= todo - 1u) {
            const int kk = __builtin_ctz(todo);
            uint32_t aa[8], bb[8];
            dma_frag(a_row + kk * BM, HM, aa);
            dma_frag(b_row + kk * BN, HN, bb);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                dma_s3_row(acc[i], aa[i], bb);
        }
        // SPECIAL: the complete definition per MAC (B: b' + bias, denormals
        // already zero).
#pragma unroll 1
        for (uint32_t todo = sp_bits; todo != 0u; todo &= todo - 1u) {
            const int kk = __builtin_ctz(todo);
            uint32_t aa[8], bb[8];
            dma_frag(a_row + kk * BM, HM, aa);
            dma_frag(b_row + kk * BN, HN, bb);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    acc[i][j] += __uint_as_float(pam_full(aa[i], bb[j] + kBias));
            }
        }
    };
    // In a launch with cut chunks the others run a loop without their code
    // (1250 x 7870 x 6276 2344 -> 2246 us, 768 x 192 x 12601 95.8 -> 92.6 us).
    constexpr int kInner = EDGE < 2 ? EDGE : 1;
    const int inner = EDGE < 2 || (ke - kb) % BK == 0 ? nchunks : max(nchunks - 2, 0);
    const int first = kinds != 0u ? 0 : inner;
    for (int c = 0; c < first; ++c)
        chunk(std::integral_constant<int, kInner>{}, c);
    if constexpr (EDGE == 2) {
        for (int c = first; c < nchunks; ++c)
            chunk(std::integral_constant<int, 2>{}, c);
    }

    // Epilogue: the output tile in C, or this K slice's partial tile (packed,
    // written whole).
    float *out;
    int64_t ld;
    int lim_m, lim_n;
    if (whole) {
        out = p.C + bz * p.strideC + (int64_t)m0 * p.ldc + n0;
        ld = p.ldc;
        lim_m = p.m - m0;
        lim_n = p.n - n0;
    } else {
        out = p.W + ((int64_t)split * p.split_tiles + st) * (BM * BN);
        ld = BN;
        lim_m = BM;
        lim_n = BN;
    }
    if constexpr (KW > 1) {
        // Groups 1.. write their partial tiles, as many at a time as the LDS
        // holds (kRedTiles); group 0 adds them, in group order, to its own.
        float *red = reinterpret_cast<float *>(smem);
#pragma unroll
        for (int g0 = 1; g0 < KW; g0 += kRedTiles) {
            __syncthreads();   // the LDS is free: every wave is past its last chunk / the previous round's adds
            if (grp >= g0 && grp < g0 + kRedTiles) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int row = i < 4 ? ty * 4 + i : HM + ty * 4 + (i - 4);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int col = h == 0 ? tx * 4 : HN + tx * 4;
                        *reinterpret_cast<float4 *>(&red[((grp - g0) * BM + row) * LDR + col]) =
                            make_float4(acc[i][4 * h], acc[i][4 * h + 1], acc[i][4 * h + 2], acc[i][4 * h + 3]);
                    }
                }
            }
            __syncthreads();
            if (grp == 0) {
                // Row by row: the row's partial values, then its adds (in
                // inline asm, in group order, so that the compiler neither
                // loads every partial tile up front nor moves the adds past
                // the next row's loads).
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    asm volatile("" ::: "memory");
                    const int row = i < 4 ? ty * 4 + i : HM + ty * 4 + (i - 4);
#pragma unroll
                    for (int g = g0; g < g0 + kRedTiles && g < KW; ++g) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int col = h == 0 ? tx * 4 : HN + tx * 4;
                            const float4 x =
                                *reinterpret_cast<const float4 *>(&red[((g - g0) * BM + row) * LDR + col]);
                            asm volatile("v_add_f32 %0, %0, %4\n\tv_add_f32 %1, %1, %5\n\t"
                                         "v_add_f32 %2, %2, %6\n\tv_add_f32 %3, %3, %7"
                                         : "+v"(acc[i][4 * h]), "+v"(acc[i][4 * h + 1]), "+v"(acc[i][4 * h + 2]),
                                           "+v"(acc[i][4 * h + 3])
                                         : "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w));
                        }
                    }
                }
            }
        }
        if (grp > 0)
            return;
    }
    // Four outputs a store, at any address.
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = i < 4 ? ty * 4 + i : HM + ty * 4 + (i - 4);
        if (row >= lim_m)
            continue;
        float *orow = out + (int64_t)row * ld;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int col = h == 0 ? tx * 4 : HN + tx * 4;
            if (col + 3 < lim_n) {
                const f32x4 v = {acc[i][4 * h], acc[i][4 * h + 1], acc[i][4 * h + 2], acc[i][4 * h + 3]};
                // The final C with the non-temporal hint (written once);
                // split partial sums without it (the reduce reads them soon).
                if (whole)
                    __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(orow + col));
                else
                    *reinterpret_cast<f32x4 *>(orow + col) = v;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (col + j < lim_n)
                        orow[col + j] = acc[i][4 * h + j];
            }
        }
    }
}

template <typename T, int BM, int BN, int KW, int WPS, int EDGE>
static hipError_t launch_dma_kernel(bool ta, bool tb, const GemmParams &p, dim3 grid, hipStream_t stream) {
    const dim3 block(BM * BN / 64 * KW);
    if (!ta && !tb)
        hipLaunchKernelGGL((pam_gemm_dma_kernel<BM, BN, KW, false, false, WPS, EDGE, T>), grid, block, 0, stream, p);
    else if (!ta && tb)
        hipLaunchKernelGGL((pam_gemm_dma_kernel<BM, BN, KW, false, true, WPS, EDGE, T>), grid, block, 0, stream, p);
    else if (ta && !tb)
        hipLaunchKernelGGL((pam_gemm_dma_kernel<BM, BN, KW, true, false, WPS, EDGE, T>), grid, block, 0, stream, p);
    else
        hipLaunchKernelGGL((pam_gemm_dma_kernel<BM, BN, KW, true, true, WPS, EDGE, T>), grid, block, 0, stream, p);
    return hipGetLastError();
}

// The launch of one (element type, EDGE) pair: a translation unit each
// (PAM_GEMM_PART 0..5), compiled side by side.
template <typename T, int EDGE>
hipError_t launch_dma_shape(int tile_m, int tile_n, int kgroups, bool ta, bool tb, const GemmParams &p, int64_t items,
                            hipStream_t stream) {
    const dim3 grid((unsigned)items);
    if (tile_m == 128 && tile_n == 128 && kgroups == 1)
        return launch_dma_kernel<T, 128, 128, 1, dma_waves_per_simd(128, 128, 1), EDGE>(ta, tb, p, grid, stream);
    if (tile_m == 128 && tile_n == 64 && kgroups == 1)
        return launch_dma_kernel<T, 128, 64, 1, dma_waves_per_simd(128, 64, 1), EDGE>(ta, tb, p, grid, stream);
    if (tile_m == 128 && tile_n == 64 && kgroups == 2) {
        // A launch that two workgroups per compute unit hold at once runs
        // the build for two waves per SIMD (staging addresses kept in
        // registers); its occupancy is two anyway.
        if (items <= 2 * 256)
            return launch_dma_kernel<T, 128, 64, 2, 2, EDGE>(ta, tb, p, grid, stream);
        return launch_dma_kernel<T, 128, 64, 2, dma_waves_per_simd(128, 64, 2), EDGE>(ta, tb, p, grid, stream);
    }
    if (tile_m == 64 && tile_n == 64 && kgroups == 1)
        return launch_dma_kernel<T, 64, 64, 1, dma_waves_per_simd(64, 64, 1), EDGE>(ta, tb, p, grid, stream);
    if (tile_m == 64 && tile_n == 64 && kgroups == 4)
        return launch_dma_kernel<T, 64, 64, 4, dma_waves_per_simd(64, 64, 4), EDGE>(ta, tb, p, grid, stream);
    return hipErrorInvalidValue;
}

#define PAM_DMA_SHAPE(T, EDGE)                                                                                   \
    template hipError_t launch_dma_shape<T, EDGE>(int, int, int, bool, bool, const GemmParams &, int64_t, hipStream_t)

#if PAM_GEMM_PART == 0
extern PAM_DMA_SHAPE(float, 1);
extern PAM_DMA_SHAPE(float, 2);
extern PAM_DMA_SHAPE(uint16_t, 0);
extern PAM_DMA_SHAPE(uint16_t, 1);
extern PAM_DMA_SHAPE(uint16_t, 2);

hipError_t launch_pam_gemm(int tile_m, int tile_n, int kgroups, bool trans_a, bool trans_b, bool bf16,
                               const GemmParams &p, hipStream_t stream) {
    const int64_t items = (int64_t)p.whole + (int64_t)p.split_tiles * p.splits;
    if (items <= 0 || items > kMaxLaunchItems)
        return hipErrorInvalidValue;
    const int bk = kChunkK * kgroups;
    const int piece = bf16 ? 8 : 4;   // elements
    const bool cut = p.k % bk != 0 || (p.split_tiles > 0 && p.k_per_split % bk != 0) ||
                     (trans_a && p.m % piece != 0) || (!trans_b && p.n % piece != 0);
    const bool past = (trans_a && p.m % tile_m != 0) || (!trans_b && p.n % tile_n != 0);
    auto launch = bf16 ? (cut    ? launch_dma_shape<uint16_t, 2>
                          : past ? launch_dma_shape<uint16_t, 1>
                                 : launch_dma_shape<uint16_t, 0>)
                       : (cut    ? launch_dma_shape<float, 2>
                          : past ? launch_dma_shape<float, 1>
                                 : launch_dma_shape<float, 0>);
    return launch(tile_m, tile_n, kgroups, trans_a, trans_b, p, items, stream);
}
#elif PAM_GEMM_PART == 1
PAM_DMA_SHAPE(float, 1);
#elif PAM_GEMM_PART == 2
PAM_DMA_SHAPE(float, 2);
#elif PAM_GEMM_PART == 3
PAM_DMA_SHAPE(uint16_t, 0);
#elif PAM_GEMM_PART == 4
PAM_DMA_SHAPE(uint16_t, 1);
#elif PAM_GEMM_PART == 5
PAM_DMA_SHAPE(uint16_t, 2);
#else
#error "PAM_GEMM_PART is 0 to 5"
#endif
#undef PAM_DMA_SHAPE

}  // namespace pamk
