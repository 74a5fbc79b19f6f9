// Internal interface between the C-ABI layer (pam_api.cpp) and the HIP
// kernels (pam_gemm_dma.hip, pam_skinny.hip, pam_small.hip, pam_kernels.hip,
// pa_ops.hip, pam_exact_grad.hip).  Not installed; not part of the public ABI.
#pragma once

#include <stdint.h>
#include <hip/hip_runtime_api.h>

namespace pamk {

// K extent of one LDS chunk.
constexpr int kChunkK = 16;

// Arguments of one (batched, possibly split-K) PAM matrix product launch.
//
// Matrix product launches run whole + split_tiles * splits work items: tiles
// are numbered batch-major, then by tile row, then tile column (`tiles` per
// matrix, `tiles_n` per tile row); item i < whole computes tile i over the
// whole K into C; item whole + s * split_tiles + t computes K slice s (k in
// [s * k_per_split, (s + 1) * k_per_split)) of tile whole + t into the
// tile-packed partial sums W[s][t][tile_m][tile_n].
struct GemmParams {
    const float *A;    // operands (bfloat16 elements for the bfloat16 products)
    const float *B;
    float *C;          // final output
    float *W;          // partial sums of the split tiles, or nullptr (layout per kernel)
    int64_t lda, ldb, ldc;
    int64_t strideA, strideB, strideC;
    int32_t m, n, k;
    int32_t k_per_split;  // multiple of kChunkK
    int32_t splits;
    int32_t tiles_n;
    int32_t tiles;        // matrix products: tiles per matrix
    int32_t whole;        // matrix products: whole-K work items
    int32_t split_tiles;  // matrix products: tiles split into `splits` K slices
    int32_t round_drop;   // 0, or 23 - m: round every input to m mantissa bits first
    // Exact-derivative products only: the output-shaped operand whose
    // mantissas set each term's carry (row-major, leading dimension ldm).
    const float *Mod;
    int64_t ldm;
};

hipError_t launch_pam_mul(const float *a, const float *b, float *out, int64_t n, hipStream_t stream);

// Elementwise PAD, palog2 and paexp2 (pa_ops.hip).
hipError_t launch_pad(const float *a, const float *b, float *out, int64_t n, hipStream_t stream);
hipError_t launch_palog2(const float *a, float *out, int64_t n, hipStream_t stream);
hipError_t launch_paexp2(const float *a, float *out, int64_t n, hipStream_t stream);
// Round to 23 - drop mantissa bits, nearest even (drop in [1, 23]).
hipError_t launch_round_mantissa(const float *a, float *out, int64_t n, int drop, hipStream_t stream);

// The tiled product (pam_gemm_dma.hip): operand chunks copied into LDS by the
// memory pipeline.  (tile_m, tile_n, kgroups) in {(128,128,1), (128,64,1),
// (128,64,2), (64,64,1), (64,64,4)}; a one-dimensional grid of p.whole +
// p.split_tiles * p.splits workgroups.
// bf16: p.A and p.B hold bfloat16 elements (leading dimensions and strides
// in elements), widened exactly to float32 as they are loaded.
hipError_t launch_pam_gemm(int tile_m, int tile_n, int kgroups, bool trans_a, bool trans_b, bool bf16,
                           const GemmParams &p, hipStream_t stream);

// Products of K-contiguous operands (op N, op T) with at most kSkinnyRows rows
// of op(A) (rows) or columns of op(B) (otherwise): pam_skinny.hip.  One launch
// for the batch; takes no plan and no workspace.
constexpr int kSkinnyRows = 32;
constexpr int64_t kMaxSkinnyItems = 8388607;   // workgroups of 512 threads: below 2^32 threads
// How a launch is cut: a workgroup takes `rows` of the s few rows and, `kwaves`
// waves along K (while each keeps at least one chunk of kSkinnyStep k steps),
// d_rows of the d others.
constexpr int kSkinnyStep = 64;
constexpr int kSkinnyWaves = 8;
struct SkinnyShape {
    int rows, kwaves, d_rows;
    int64_t d_tiles, s_tiles;
};
inline SkinnyShape skinny_shape(int64_t s, int64_t d, int64_t k) {
    SkinnyShape r{};
    r.rows = s <= 4 ? 4 : s <= 8 ? 8 : 16;
    r.kwaves = 1;
    while (r.kwaves < kSkinnyWaves && (int64_t)r.kwaves * kSkinnyStep < k)
        r.kwaves *= 2;
    r.d_rows = 16 * (kSkinnyWaves / r.kwaves);
    r.d_tiles = (d + r.d_rows - 1) / r.d_rows;
    r.s_tiles = (s + r.rows - 1) / r.rows;
    return r;
}
hipError_t launch_pam_skinny(bool rows, bool bf16, const GemmParams &p, int64_t batch, hipStream_t stream);

// Small products (pam_small.hip): 32 x 32 tiles, kSmallWaves waves sharing each
// chunk's k steps.  One launch for the batch; takes no plan and no workspace.
constexpr int kSmallWaves = 8;
hipError_t launch_pam_small(bool trans_a, bool trans_b, bool bf16, GemmParams p, int64_t batch, hipStream_t stream);

// C of the split tiles of a product launch: element by element the sum over s
// of W[s][t][.][.], in an order fixed by the number of slices.
hipError_t launch_split_tile_reduce(int tile_m, int tile_n, const GemmParams &p, hipStream_t stream);

// Bytes of the static split-K scratch pam_gemm_batched_noalloc uses, and its
// device address on the current device (looked up once per device).
constexpr size_t kScratchBytes = (size_t)64 << 20;
hipError_t scratch_address(void **out);

// Workgroups one product launch may hold (its grid, in threads, stays
// below 2^32).
constexpr int64_t kMaxLaunchItems = 16777215;

// Exact-derivative product (pam_exact_grad.hip): C(r, c) = sum_q op(A)(r, q)
// d(Mod(r, c) .^ B(q, c)) / dMod(r, c); tiles of kExactTileM x kExactTileN,
// work items and partial sums as in a matrix product launch.
constexpr int kExactTileM = 128, kExactTileN = 64;
hipError_t launch_pam_exact_grad(bool trans_a, const GemmParams &p, hipStream_t stream);

// C[b][i][j] = +0.0f for a k == 0 product.
hipError_t launch_fill_zero(float *C, int32_t m, int32_t n, int64_t ldc, int64_t strideC,
                            int64_t batch, hipStream_t stream);

}  // namespace pamk
