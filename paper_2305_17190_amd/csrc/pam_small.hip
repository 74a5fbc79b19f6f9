// Small PAM matrix products on gfx950: outputs of so few 64 x 64 tiles that
// the tiled kernel's plan leaves most of the chip idle.
//
// What bounds them: the chain of one workgroup (first copies, the chunks one
// after the other, the reduction), since there is less than a round of them.
// A wave of the tiled kernel computes 64 x 64 outputs, 256 x 256 outputs are 16
// workgroups, and each wave runs alone on its SIMD at half the issue rate.
// Here a workgroup owns 32 x 32 outputs and its KW waves take 16 k steps each of
// a chunk of 16 KW (micro-tiles of 4 x 4 per thread): four times the
// workgroups, a quarter of the steps in a row, and two waves per SIMD that
// pair their adds.  Chunks are copied into LDS by the memory pipeline while
// the previous one is computed, as in pam_gemm_dma.hip.
//
// Per chunk the workgroup takes one of that kernel's forms for all steps: S1
// (acc += a + b') when every element has exponent field in [64, 190], S2 (add
// and fma) when some are zero or denormal, S3 (the product rounded on its
// own) when one is a tiny normal, the complete definition when one is inf,
// NaN or |x| >= 2^64.
//
// Measured against the tiled kernel's plans: 256^3 6.9 us (26.7 us), 512 x 512
// x 256 7.7 us (27.0), 1024 x 1024 x 256 19.2 us (27.3), 256 x 256 x 1024 19.1 us
// (27.5), 128 x 128 x 64 5.2 us (10.9), 16 matrices of 197 x 197 x 64 11.7 us (13.4);
// half-zero operands 256^3 8.2 us (36.8), 256 x 256 x 1024 25.1 us (35.6); 2048 x 1024
// x 256 34.9 us (27.8) and 128 x 128 x 4096 65 us (28.5, K in slices) stay with the
// plan (small_product in pam_api.cpp).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pam_dma_tile.h"
#include "pam_internal.h"
#include "pam_scalar.h"

namespace pamk {
namespace {

constexpr int kTile = 32;

__device__ __forceinline__ void quad(const uint32_t *p, uint32_t (&e)[4]) {
    const uint4 x = *reinterpret_cast<const uint4 *>(p);
    e[0] = x.x; e[1] = x.y; e[2] = x.z; e[3] = x.w;
}

template <int KW, bool TA, bool TB, typename T>
__global__ void __launch_bounds__(64 * KW) __attribute__((amdgpu_waves_per_eu(4))) pam_small_kernel(GemmParams p) {
    constexpr int D = kTile, KPG = kChunkK, BK = KPG * KW, NT = 64 * KW;
    using TileA = DmaTile<D, BK, NT, !TA, T>;
    using TileB = DmaTile<D, BK, NT, TB, T>;
    constexpr int kRawA = TileA::CL * NT * 4;
    constexpr int kRawB = TileB::CL * NT * 4;
    constexpr int kEnc = BK * D;
    constexpr int kWords = kRawA + kRawB + 2 * kEnc > KW * D * D ? kRawA + kRawB + 2 * kEnc : KW * D * D;
    __shared__ __attribute__((aligned(16))) uint32_t smem[kWords];
    __shared__ uint32_t sVote[2];   // [chunk parity]: 1 a low element, 2 a tiny normal, 4 SPECIAL
    uint32_t *rawA = smem;
    uint32_t *rawB = smem + kRawA;
    uint32_t *encA = rawB + kRawB;
    uint32_t *encB = encA + kEnc;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane(lds_addr(smem) + (uint32_t)wave * 1024u);
    const int lane = tid & 63;
    const int r0 = (lane >> 3) * 4, c0 = (lane & 7) * 4;   // the micro-tile's first row and column
    const int64_t bz = blockIdx.x / (uint32_t)p.tiles;
    const int tile = (int)(blockIdx.x % (uint32_t)p.tiles);
    const int m0 = (tile / p.tiles_n) * D;
    const int n0 = (tile % p.tiles_n) * D;
    const T *a_base = reinterpret_cast<const T *>(p.A) + bz * p.strideA + (TA ? (int64_t)m0 : (int64_t)m0 * p.lda);
    const T *b_base = reinterpret_cast<const T *>(p.B) + bz * p.strideB + (TB ? (int64_t)n0 * p.ldb : (int64_t)n0);
    const int64_t a_step = TA ? (int64_t)BK * p.lda : BK;
    const int64_t b_step = TB ? BK : (int64_t)BK * p.ldb;
    const uint32_t kind_a = TileA::kind(p.k, m0, p.m, p.lda), kind_b = TileB::kind(p.k, n0, p.n, p.ldb);
    const int nchunks = (p.k + BK - 1) / BK;

    TileA::template copy<0, 2>(a_base, lds_w, tid, p.lda, m0, p.m, p.k, kind_a);
    TileB::template copy<kRawA * 4, 2>(b_base, lds_w, tid, p.ldb, n0, p.n, p.k, kind_b);
    if (tid < 2)
        sVote[tid] = 0u;

    // A chunk's sums start at zero and are added to the running ones: chains
    // of 16 roundings, so that eight waves' parts of K round no more than the
    // plans' many K slices did.
    float acc[4][4], total[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            total[i][j] = 0.0f;

    TileA la;
    TileB lb;
#pragma unroll 1
    for (int c = 0; c < nchunks; ++c) {
        const int k_rem = p.k - c * BK;   // k steps left, this chunk's included
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's copies have landed
        la.template fetch<2>(rawA, wave, p.lda, m0, p.m, k_rem, kind_a, tid);
        lb.template fetch<2>(rawB, wave, p.ldb, n0, p.n, k_rem, kind_b, tid);
        if (p.round_drop != 0) {
            la.round_mantissa(p.round_drop);
            lb.round_mantissa(p.round_drop);
        }
        uint32_t smin_a[TileA::L], smin_b[TileB::L];
        const uint32_t mx = max(la.scan(smin_a), lb.scan(smin_b));
        // The zeros past K have no say in the form of the steps.
        uint32_t low_a = 0xFFFFFFFFu, low_b = 0xFFFFFFFFu;
#pragma unroll
        for (int r = 0; r < TileA::L; ++r)
            low_a = TileA::seg_k(tid, r) < k_rem ? min(low_a, smin_a[r]) : low_a;
#pragma unroll
        for (int r = 0; r < TileB::L; ++r)
            low_b = TileB::seg_k(tid, r) < k_rem ? min(low_b, smin_b[r]) : low_b;
        uint32_t vote = 0u;
        if (TileA::low_seg(low_a) || TileB::low_seg(low_b)) {
            vote = 1u | (la.any_tiny() || lb.any_tiny() ? 2u : 0u);
            lb.flush_denormals();
        }
        vote |= mx >= (191u << 24) ? 4u : 0u;
        __syncthreads();   // every wave is done reading the previous chunk (and clearing this vote)
        la.store_values(encA, false, tid);
        lb.store_values(encB, true, tid);
        // One LDS atomic a wave.  (With one a lane, all to one word, 256 x 256 x 1024
        // on ReLU activations took 41.9 us, now 25.2 us; 19.3 us on clean ones.)
        if (__builtin_amdgcn_ballot_w64(vote != 0u) != 0u) {
            uint32_t all = 0u;
#pragma unroll
            for (uint32_t bit = 1u; bit <= 4u; bit *= 2u)
                all |= __builtin_amdgcn_ballot_w64((vote & bit) != 0u) != 0u ? bit : 0u;
            if (lane == 0)
                atomicOr(&sVote[c & 1], all);
        }
        __syncthreads();
        const uint32_t votes = __builtin_amdgcn_readfirstlane(sVote[c & 1]);
        if (tid == 0)
            sVote[(c + 1) & 1] = 0u;
        if (c + 1 < nchunks) {
            TileA::template copy<0, 2>(a_base + (c + 1) * a_step, lds_w, tid, p.lda, m0, p.m, k_rem - BK, kind_a);
            TileB::template copy<kRawA * 4, 2>(b_base + (c + 1) * b_step, lds_w, tid, p.ldb, n0, p.n, k_rem - BK,
                                                  kind_b);
        }
        const uint32_t *a_row = encA + wave * KPG * D + r0;
        const uint32_t *b_row = encB + wave * KPG * D + c0;
        const int steps = min(k_rem - wave * KPG, KPG);   // this wave's (none past K)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = 0.0f;
        // One k step in form F (1: S1, 2: S2, 3: S3).
        auto step = [&](auto form, int k) {
            constexpr int F = decltype(form)::value;
            uint32_t a[4], b[4];
            quad(a_row + k * D, a);
            quad(b_row + k * D, b);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t m = a[i] & kSignExp, am = (a[i] ^ m) | kBias;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (F == 1) {
                        acc[i][j] += __uint_as_float(a[i] + b[j]);
                    } else if constexpr (F == 2) {
                        acc[i][j] = __builtin_fmaf(__uint_as_float(am + b[j]), __uint_as_float(m), acc[i][j]);
                    } else {
                        float t;   // rounded on its own: an underflowing product flushes to zero
                        asm("v_mul_f32 %0, %1, %2" : "=v"(t) : "v"(am + b[j]), "v"(m));
                        acc[i][j] += t;
                    }
                }
            }
        };
        auto all_steps = [&](auto form) {
#pragma unroll
            for (int k = 0; k < KPG; ++k)
                step(form, k);
        };
        if (votes < 4u && steps == KPG) {
            if (votes == 0u)
                all_steps(std::integral_constant<int, 1>{});
            else if (votes < 2u)
                all_steps(std::integral_constant<int, 2>{});
            else
                all_steps(std::integral_constant<int, 3>{});
        } else if (votes < 2u) {
#pragma unroll 4
            for (int k = 0; k < steps; ++k)
                step(std::integral_constant<int, 2>{}, k);
        } else if (votes < 4u) {
#pragma unroll 2
            for (int k = 0; k < steps; ++k)
                step(std::integral_constant<int, 3>{}, k);
        } else {
#pragma unroll 1
            for (int k = 0; k < steps; ++k) {
                uint32_t a[4], b[4];
                quad(a_row + k * D, a);
                quad(b_row + k * D, b);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] += __uint_as_float(pam_full(a[i], b[j] + kBias));
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                total[i][j] += acc[i][j];
    }

    // The waves' partial tiles in LDS, added in wave order by all threads.
    float *red = reinterpret_cast<float *>(smem);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
        *reinterpret_cast<float4 *>(&red[(wave * D + r0 + i) * D + c0]) =
            make_float4(total[i][0], total[i][1], total[i][2], total[i][3]);
    __syncthreads();
    float *out = p.C + bz * p.strideC + (int64_t)m0 * p.ldc + n0;
#pragma unroll
    for (int o = tid; o < D * D; o += NT) {
        float s = red[o];
#pragma unroll
        for (int g = 1; g < KW; ++g)
            s += red[g * D * D + o];
        const int row = o / D, col = o % D;
        if (m0 + row < p.m && n0 + col < p.n)
            out[(int64_t)row * p.ldc + col] = s;
    }
}

template <int KW, typename T>
hipError_t launch(bool ta, bool tb, const GemmParams &p, dim3 grid, hipStream_t stream) {
    const dim3 block(64 * KW);
    if (!ta && !tb)
        hipLaunchKernelGGL((pam_small_kernel<KW, false, false, T>), grid, block, 0, stream, p);
    else if (!ta && tb)
        hipLaunchKernelGGL((pam_small_kernel<KW, false, true, T>), grid, block, 0, stream, p);
    else if (ta && !tb)
        hipLaunchKernelGGL((pam_small_kernel<KW, true, false, T>), grid, block, 0, stream, p);
    else
        hipLaunchKernelGGL((pam_small_kernel<KW, true, true, T>), grid, block, 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_pam_small(bool trans_a, bool trans_b, bool bf16, GemmParams p, int64_t batch, hipStream_t stream) {
    p.tiles_n = (p.n + kTile - 1) / kTile;
    const int64_t tiles = (int64_t)((p.m + kTile - 1) / kTile) * p.tiles_n;
    const int64_t items = tiles * batch;
    if (items <= 0 || items > kMaxSkinnyItems)
        return hipErrorInvalidValue;
    p.tiles = (int32_t)tiles;
    const dim3 grid((unsigned)items);
    return bf16 ? launch<kSmallWaves, uint16_t>(trans_a, trans_b, p, grid, stream)
                : launch<kSmallWaves, float>(trans_a, trans_b, p, grid, stream);
}

}  // namespace pamk
