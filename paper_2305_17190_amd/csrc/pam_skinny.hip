// PAM matrix products with few rows (or columns) on gfx950: both operands
// K-contiguous (op N, op T) and at most kSkinnyRows rows of op(A) or columns
// of op(B), as when a few tokens go through a layer's weights.
//
// What bounds it: reading the wide operand once.  The tiled kernel pads the
// few rows to 64 and gives each workgroup a few chunks between barriers.
// Measured against it (one call after the other, other weights each time): 8
// x 4096 x 4096 20.6 us (52.5; its 67 MB take 14 us at a copy's rate), 1 x 4096
// x 4096 18.8 us (53.0), 16 x 4096 x 4096 25.9 us (53.9), 32 x 4096 x 4096
// 47.9 us (54.1; two passes of 16 rows), 8 x 2048 x 512 4.9 us (27.7), 32 x 768 x
// 192 6.0 us (20.7); bfloat16, 4096 x 4096 weights: 1 row 11.0 us (61.4), 8 rows
// 14.9 us (61.7), 16 rows 22.5 us (62.1), 32 rows 43.6 us (62.1).  Where it is
// taken: skinny_product in pam_api.cpp.
//
// No wave waits for another until the end: a lane holds four consecutive k of
// kJ rows of the wide operand, loaded straight into registers one chunk ahead
// (16 lanes read 256 consecutive bytes of a row), and keeps a sum for each of S
// skinny rows and its kJ wide rows, folded into the outputs every kFoldChunks
// chunks; the skinny operand's chunk comes from LDS, written by the wave
// itself.  The waves of a workgroup take parts of K (long K) or further wide rows.
//
// Arithmetic: the SCALED form with the product and sum in one fma (S2 of
// pam_gemm_dma.hip): t = (1 + M_x) + w' is the encoding of PAM(1 + M_x, w),
// acc = fma(t, +-2^E_x, acc); a zero x gives the factor 0, a zero w a t that
// reads as 0.  It is exact while every nonzero operand has exponent field in
// [64, 190].  A wave's chunk holding a tiny normal (field below 64) rounds each
// product on its own (S3 there); one holding |x| >= 2^64, inf or NaN takes the
// complete definition (as tiny normals did: with 0.1% of them among the weights
// 32 x 4096 x 4096 took 491 us, now 58 us; on clean operands 47 us).  bfloat16
// operands widen to the same encodings, so their product equals the float32 one
// bit for bit.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pam_internal.h"
#include "pam_scalar.h"

namespace pamk {
namespace {

constexpr int kJ = 4;            // wide rows per lane
constexpr int kWaveRows = 4 * kJ;   // wide rows per wave: lane / 16 picks four groups of kJ
constexpr int kWaves = kSkinnyWaves;   // waves per workgroup
constexpr int kStep = kSkinnyStep;     // k per chunk: 16 lanes of four
constexpr int kFoldChunks = 32;        // a lane's longest sum: 128 terms (long K)
static_assert(kStep == 64 && kWaveRows == 16, "skinny_shape's cut");

struct SkinnyParams {
    const void *X;   // skinny operand, s rows
    const void *D;   // wide operand, d rows
    float *C;
    int64_t ldx, ldd, strideX, strideD, strideC;
    int64_t cs, cd;   // C's strides along the skinny and the wide index
    int32_t s, d, k;
    int32_t kwaves;   // waves of a workgroup that share one set of wide rows (1, 2, 4 or 8)
    int32_t d_tiles, s_tiles;
    int32_t round_drop;
};

__device__ __forceinline__ uint32_t round_bits(uint32_t u, int drop) {
    const uint32_t low = (1u << drop) - 1u;
    const uint32_t r = (u + (low >> 1) + ((u >> drop) & 1u)) & ~low;
    return (u & kExpMask) == kExpMask ? u : r;
}

// Four consecutive elements of a row from element k, at any address, as they
// are in memory; elements past the row's end are zero.  Nothing is computed from
// them here, so that a load stays in flight until its chunk is used: bfloat16
// elements, widened as they were loaded, were waited for at once (8 x 4096 x 4096
// took 28.8 us, now 15.9 us).
__device__ __forceinline__ void load4(const float *row, int k, int n, uint32_t (&w)[4]) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    if (k + 4 <= n) {
        const u32x4 x = *reinterpret_cast<const u32x4 *>(row + k);
        w[0] = x[0]; w[1] = x[1]; w[2] = x[2]; w[3] = x[3];
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            w[c] = k + c < n ? __float_as_uint(row[k + c]) : 0u;
    }
}
__device__ __forceinline__ void load4(const uint16_t *row, int k, int n, uint32_t (&w)[2]) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(2)));
    if (k + 4 <= n) {
        const u32x2 x = *reinterpret_cast<const u32x2 *>(row + k);
        w[0] = x[0]; w[1] = x[1];
    } else {
#pragma unroll
        for (int c = 0; c < 4; c += 2)
            w[c / 2] = (k + c < n ? (uint32_t)row[k + c] : 0u) | (k + c + 1 < n ? (uint32_t)row[k + c + 1] << 16 : 0u);
    }
}
// The elements as float32 encodings.
__device__ __forceinline__ void widen4(const uint32_t (&w)[4], uint32_t (&e)[4]) {
    e[0] = w[0]; e[1] = w[1]; e[2] = w[2]; e[3] = w[3];
}
__device__ __forceinline__ void widen4(const uint32_t (&w)[2], uint32_t (&e)[4]) {
    e[0] = w[0] << 16; e[1] = w[0] & 0xFFFF0000u; e[2] = w[1] << 16; e[3] = w[1] & 0xFFFF0000u;
}

// Running bounds of the operands' magnitudes: the least nonzero one less one
// (a zero or denormal, flushed by the multiplication, wraps to the top) and
// the largest, both times 2^63.
struct Range {
    uint32_t least = 0xFFFFFFFFu, most = 0u;
    __device__ __forceinline__ void add(uint32_t u) {
        uint32_t f;
        asm("v_mul_f32 %0, |%1|, %2" : "=v"(f) : "v"(u), "v"(0x5F000000u));   // 2^63
        least = min(least, f - 1u);
        most = max(most, f & kMag);
    }
    // Some nonzero magnitude is below 2^-63; some is at or above 2^64 or not
    // finite (times 2^63 one of 2^65 or more is inf).
    __device__ __forceinline__ bool tiny() const { return least < kBias - 1u; }
    __device__ __forceinline__ bool wild() const { return most >= 0x7F000000u; }
};

template <int S, typename T>
__global__ void __launch_bounds__(64 * kWaves) pam_skinny_kernel(SkinnyParams p) {
    // A wave's skinny chunk: 1 + M_x and +-2^E_x, [plane][row][k].  After the
    // K loop the same bytes hold the waves' partial sums [wave][row][wide row].
    constexpr int kChunkWords = 2 * S * kStep;
    static_assert(kChunkWords >= S * kWaveRows, "the partial sums fit the chunk buffers");
    __shared__ __attribute__((aligned(16))) uint32_t smem[kWaves * kChunkWords];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kq = lane & 15;
    const int dr = lane >> 4;
    const int kwaves = p.kwaves;
    const int kw = wave % kwaves;
    const uint32_t per_matrix = (uint32_t)p.d_tiles * (uint32_t)p.s_tiles;
    const int64_t bz = blockIdx.x / per_matrix;
    const int rel = (int)(blockIdx.x % per_matrix);
    const int s0 = (rel / p.d_tiles) * S;
    const int d0 = ((rel % p.d_tiles) * (kWaves / kwaves) + wave / kwaves) * kWaveRows + dr * kJ;
    const T *x = reinterpret_cast<const T *>(p.X) + bz * p.strideX;
    const T *w = reinterpret_cast<const T *>(p.D) + bz * p.strideD;
    uint32_t *mine = smem + wave * kChunkWords;
    const int n = p.k;

    const T *wrow[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j)
        wrow[j] = w + (int64_t)min(d0 + j, p.d - 1) * p.ldd;
    // This lane's quads of the skinny chunk: (row q / 16, k quad q % 16), q =
    // lane + 64 i; rows past s repeat the last one, their sums are dropped.
    constexpr int XQ = (S * 16 + 63) / 64;
    const T *xrow[XQ];
#pragma unroll
    for (int i = 0; i < XQ; ++i)
        xrow[i] = x + (int64_t)min(s0 + dr + 4 * i, p.s - 1) * p.ldx;

    float acc[S][kJ];
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
        for (int j = 0; j < kJ; ++j)
            acc[i][j] = 0.0f;

    // The lanes' sums so far, added over the 16 lanes of a row group (the result
    // in all of them), to the running outputs: lane kq = i holds row i's.
    static_assert(S <= 16, "one lane per row");
    float mineacc[kJ] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto fold = [&]() {
        float row[kJ];
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
            for (int j = 0; j < kJ; ++j) {
                float v = acc[i][j];
                v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x128, 0xF, 0xF, true));
                v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x124, 0xF, 0xF, true));
                v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x122, 0xF, 0xF, true));
                v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x121, 0xF, 0xF, true));
                row[j] = i == 0 || kq == i ? v : row[j];
                acc[i][j] = 0.0f;
            }
#pragma unroll
        for (int j = 0; j < kJ; ++j)
            mineacc[j] += row[j];
    };

    uint32_t wr[kJ][sizeof(T)], xr[XQ][sizeof(T)];   // the next chunk's elements
    auto fetch = [&](int k0) {
#pragma unroll
        for (int j = 0; j < kJ; ++j)
            load4(wrow[j], k0 + kq * 4, n, wr[j]);
#pragma unroll
        for (int i = 0; i < XQ; ++i)
            load4(xrow[i], k0 + kq * 4, n, xr[i]);
    };
    const int step = kStep * kwaves;
    if (kw * kStep < n)
        fetch(kw * kStep);
#pragma unroll 1
    for (int kf = kw * kStep; kf < n; kf += kFoldChunks * step) {
        const int kend = n - kf > kFoldChunks * step ? kf + kFoldChunks * step : n;
#pragma unroll 1
        for (int k0 = kf; k0 < kend; k0 += step) {
            uint32_t wn[kJ][4], xn[XQ][4], wc[kJ][4];
#pragma unroll
            for (int j = 0; j < kJ; ++j)
                widen4(wr[j], wn[j]);
#pragma unroll
            for (int i = 0; i < XQ; ++i)
                widen4(xr[i], xn[i]);
            Range range;
            if (p.round_drop != 0) {
#pragma unroll
                for (int j = 0; j < kJ; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        wn[j][c] = round_bits(wn[j][c], p.round_drop);
#pragma unroll
                for (int i = 0; i < XQ; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        xn[i][c] = round_bits(xn[i][c], p.round_drop);
            }
#pragma unroll
            for (int j = 0; j < kJ; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    range.add(wn[j][c]);
                    // A denormal to its signed zero, then less one bias.
                    asm("v_mul_f32 %0, 1.0, %1" : "=v"(wc[j][c]) : "v"(wn[j][c]));
                    wc[j][c] -= kBias;
                }
#pragma unroll
            for (int i = 0; i < XQ; ++i) {
                uint4 am, m;
                am.x = (xn[i][0] & kMant) | kBias; m.x = xn[i][0] & kSignExp;
                am.y = (xn[i][1] & kMant) | kBias; m.y = xn[i][1] & kSignExp;
                am.z = (xn[i][2] & kMant) | kBias; m.z = xn[i][2] & kSignExp;
                am.w = (xn[i][3] & kMant) | kBias; m.w = xn[i][3] & kSignExp;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    range.add(xn[i][c]);
                const int row = dr + 4 * i;
                if (S % 4 == 0 || row < S) {
                    *reinterpret_cast<uint4 *>(mine + row * kStep + kq * 4) = am;
                    *reinterpret_cast<uint4 *>(mine + (S + row) * kStep + kq * 4) = m;
                }
            }
            if (k0 + step < n)
                fetch(k0 + step);
            const bool wild = __builtin_amdgcn_ballot_w64(range.wild()) != 0u;
            const bool tiny = __builtin_amdgcn_ballot_w64(range.tiny()) != 0u;
            // The wave's own writes, read by its other lanes: LDS operations of a
            // wave complete in order, and the compiler keeps them in order here.
            asm volatile("" ::: "memory");
            auto terms = [&](auto own) {
                constexpr bool kOwn = decltype(own)::value;   // each product rounded on its own
#pragma unroll
                for (int i = 0; i < S; ++i) {
                    const uint4 am = *reinterpret_cast<const uint4 *>(mine + i * kStep + kq * 4);
                    const uint4 m = *reinterpret_cast<const uint4 *>(mine + (S + i) * kStep + kq * 4);
                    const uint32_t a4[4] = {am.x, am.y, am.z, am.w}, m4[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int j = 0; j < kJ; ++j) {
                            if constexpr (kOwn) {
                                float t;   // in asm: the compiler would fuse the product and the sum
                                asm("v_mul_f32 %0, %1, %2" : "=v"(t) : "v"(a4[c] + wc[j][c]), "v"(m4[c]));
                                acc[i][j] += t;
                            } else {
                                acc[i][j] = __builtin_fmaf(__uint_as_float(a4[c] + wc[j][c]), __uint_as_float(m4[c]),
                                                           acc[i][j]);
                            }
                        }
                }
            };
            if (!wild && !tiny) {
                terms(std::false_type{});
            } else if (!wild) {
                terms(std::true_type{});
            } else {
#pragma unroll
                for (int i = 0; i < S; ++i) {
#pragma unroll 1
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t xe = (mine[i * kStep + kq * 4 + c] & kMant) | mine[(S + i) * kStep + kq * 4 + c];
#pragma unroll
                        for (int j = 0; j < kJ; ++j) {
                            const uint32_t we = c == 0 ? wc[j][0] : c == 1 ? wc[j][1] : c == 2 ? wc[j][2] : wc[j][3];
                            acc[i][j] += __uint_as_float(pam_full(xe, we + kBias));
                        }
                    }
                }
            }
            asm volatile("" ::: "memory");
        }
        fold();
    }
    if (kwaves > 1) {
        float *part = reinterpret_cast<float *>(smem);
        __syncthreads();   // every wave is past its chunks
        if (kw != 0 && kq < S) {
#pragma unroll
            for (int j = 0; j < kJ; ++j)
                part[(wave * S + kq) * kWaveRows + dr * kJ + j] = mineacc[j];
        }
        __syncthreads();
        if (kw != 0)
            return;
        if (kq < S) {
            for (int q = 1; q < kwaves; ++q)
#pragma unroll
                for (int j = 0; j < kJ; ++j)
                    mineacc[j] += part[((wave + q) * S + kq) * kWaveRows + dr * kJ + j];
        }
    }
    if (kq < S && s0 + kq < p.s) {
        float *out = p.C + bz * p.strideC + (int64_t)(s0 + kq) * p.cs + (int64_t)d0 * p.cd;
#pragma unroll
        for (int j = 0; j < kJ; ++j)
            if (d0 + j < p.d)
                out[j * p.cd] = mineacc[j];
    }
}

}  // namespace

hipError_t launch_pam_skinny(bool rows, bool bf16, const GemmParams &g, int64_t batch, hipStream_t stream) {
    SkinnyParams p{};
    // rows: op(A)'s few rows against B's; otherwise B's few rows (op(B)'s
    // columns) against A's (PAM is commutative), and C is written by columns.
    p.X = rows ? g.A : g.B;
    p.D = rows ? g.B : g.A;
    p.ldx = rows ? g.lda : g.ldb;
    p.ldd = rows ? g.ldb : g.lda;
    p.strideX = rows ? g.strideA : g.strideB;
    p.strideD = rows ? g.strideB : g.strideA;
    p.s = rows ? g.m : g.n;
    p.d = rows ? g.n : g.m;
    p.cs = rows ? g.ldc : 1;
    p.cd = rows ? 1 : g.ldc;
    p.C = g.C;
    p.strideC = g.strideC;
    p.k = g.k;
    p.round_drop = g.round_drop;
    const SkinnyShape cut = skinny_shape(p.s, p.d, p.k);
    p.kwaves = cut.kwaves;
    p.d_tiles = (int32_t)cut.d_tiles;
    p.s_tiles = (int32_t)cut.s_tiles;
    const int64_t items = (int64_t)p.d_tiles * p.s_tiles * batch;
    if (items <= 0 || items > kMaxSkinnyItems)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)items), block(64 * kWaves);
    if (bf16) {
        if (cut.rows == 4)
            hipLaunchKernelGGL((pam_skinny_kernel<4, uint16_t>), grid, block, 0, stream, p);
        else if (cut.rows == 8)
            hipLaunchKernelGGL((pam_skinny_kernel<8, uint16_t>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((pam_skinny_kernel<16, uint16_t>), grid, block, 0, stream, p);
    } else {
        if (cut.rows == 4)
            hipLaunchKernelGGL((pam_skinny_kernel<4, float>), grid, block, 0, stream, p);
        else if (cut.rows == 8)
            hipLaunchKernelGGL((pam_skinny_kernel<8, float>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((pam_skinny_kernel<16, float>), grid, block, 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace pamk
