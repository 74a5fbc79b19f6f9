// Exact-derivative PAM products on gfx950 (Kosson & Jaggi, Table 1).
//
// The exact derivative of A .^ B with respect to A is the slope of the
// piecewise affine function: sgn(B) 2^(E_B + c), c = 1{M_A + M_B >= 1}, where
// A .^ B is not clamped, and 0 where it is (a zero or denormal operand, a
// result that underflows to a signed zero or saturates at +-FLT_MAX): the
// function is constant there.  For Y = X .^ W^T the two gradients are
// contractions in which every term also depends on an output-shaped operand:
//
//   dX[i,k] = sum_j dY[i,j] d(X[i,k] .^ W[j,k]) / dX[i,k]
//   dW[j,k] = sum_i dY[i,j] d(W[j,k] .^ X[i,k]) / dW[j,k]
//
// Both are C(r, c) = sum_q op(A)(r, q) g(B(q, c), Mod(r, c)) with g(b, mod) =
// d(mod .^ b) / d mod: dX is (A = dY, B = W, Mod = X), dW is (A = dY^T,
// B = X, Mod = W).  Each term A * g is exact (g is a power of two) and added
// with one rounding (fma); a denormal A counts as zero.
//
// Fast path.  Call a normal value "safe" when its exponent field is in
// [64, 190].  For safe b and safe mod the product mod .^ b can never leave the
// normal range and 2^(E_b + c) <= 2^64, so per term: t = b + M_mod (one int
// add: it carries into b's exponent exactly when M_b + M_mod >= 1), clearing
// t's mantissa (one and) leaves the float sgn(b) 2^(E_b + c), and one fma adds
// A * g.  Zero and denormal b are staged as 0, which gives g = 0.
//
// The rest, taken by the complete definition (general_fma):
//   * b that is normal but not safe ("extreme"): staged as 0 for the fast
//     path, and the LDS chunk's steps holding one are flagged; in a flagged
//     step each thread adds the general term for its columns whose b is
//     extreme (a second plane of B keeps the extreme values).
//   * mod that is normal but not safe: the output's fast-path sum is
//     discarded; the workgroup lists such outputs in LDS (up to 512 of the
//     tile's 8192) and deals them out evenly over its threads, each keeping
//     the sums of at most two, over every k with the general term.  A tile
//     with more takes the general term for every term.
//   * zero / denormal mod: the output is zero.
// The general term needs mod's exponent; mod's mantissa stays in registers
// for the fast path, so flagged steps read mod again from memory.
//
// What bounds it: vector-ALU issue, three full-rate ops per term (v_and_b32
// with register operands issues at the rate of the adds; with a scalar
// register operand at half of it).  The bare three-op sequence ran at
// 22.4e12 terms/s over the whole chip.  Tiling: 128 x 64 outputs per
// 256-thread workgroup, 8 x 4 register micro-tiles: accumulators and mod
// mantissas together take 64 registers, so four waves fit a SIMD (an 8 x 8
// micro-tile takes 128 and left two).  Chunks of 16 k steps are copied into
// LDS by the memory pipeline while the previous one is computed
// (pam_dma_tile.h), and each step's operands are read one step ahead.
// Measured, with the reduction of the K slices, against the earlier kernel
// (128 x 128 tiles staged through registers, two waves per SIMD): 8192 x 512
// outputs over K = 2048 486 us (628 us), 2048 x 512 over K = 8192 454 us (623),
// 12608 x 192 over K = 768 133 us (366), 768 x 192 over K = 12608 122 us (301),
// 4096 x 4096 x 4096 19.5e12 terms/s.  What is left over the chunks is a
// workgroup's Mod tile read and its output written, 13 us a round.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pam_dma_tile.h"
#include "pam_internal.h"

namespace pamk {
namespace {

constexpr uint32_t kSafeLo = 64u;    // exponent fields [64, 190]: the fast path is exact
constexpr uint32_t kSafeHi = 190u;

// Normal (field 1..254; inf / NaN count too) but outside the safe band.
__device__ __forceinline__ bool extreme(uint32_t u) {
    const uint32_t f = (u >> 23) & 0xFFu;
    return f != 0u && (f < kSafeLo || f > kSafeHi);
}

// acc += a * d(mod .^ b)/d mod, the complete definition for finite operands:
// zero when b or mod is zero / denormal or mod .^ b is clamped (magnitude sum
// |b| + |mod| - bias outside [2^-126's, FLT_MAX's encoding]); otherwise
// sgn(b) 2^(E_b + c).  2^128 (E_b = 127 with the carry) is applied as
// (2a) * 2^127 (exact: a doubling).
__device__ __forceinline__ void general_fma(float &acc, float a, uint32_t b, uint32_t mod) {
    const uint32_t mb = b & kMag;
    const uint32_t md = mod & kMag;
    const uint32_t sum = mb + md;   // < 2^32: both magnitudes are below 2^31
    const bool live = mb >= kMinNormal && md >= kMinNormal && sum >= kBias + kMinNormal && sum <= kBias + kFltMax;
    uint32_t g = (b + (md & kMant)) & kSignExp;
    const bool top = (g & kExpMask) == kExpMask;
    g = top ? g - (1u << 23) : g;
    const float a2 = top ? a * 2.0f : a;
    g = live ? g : 0u;
    acc = fmaf(a2, __uint_as_float(g), acc);
}

// One k step of the micro-tile, acc[i][j] += a_i * ((b_j + mm[i][j]) & sign and
// exponent), two rows at a time: eight independent ops of each kind.
#define PAM_EXACT_ROWS(R, S, A, B)                                                                              \
    "v_add_u32 %[t0], %[m" #R "0], %[b0]\n\tv_add_u32 %[t1], %[m" #R "1], %[b1]\n\t"                           \
    "v_add_u32 %[t2], %[m" #R "2], %[b2]\n\tv_add_u32 %[t3], %[m" #R "3], %[b3]\n\t"                           \
    "v_add_u32 %[t4], %[m" #S "0], %[b0]\n\tv_add_u32 %[t5], %[m" #S "1], %[b1]\n\t"                           \
    "v_add_u32 %[t6], %[m" #S "2], %[b2]\n\tv_add_u32 %[t7], %[m" #S "3], %[b3]\n\t"                           \
    "v_and_b32 %[t0], %[se], %[t0]\n\tv_and_b32 %[t1], %[se], %[t1]\n\t"                                     \
    "v_and_b32 %[t2], %[se], %[t2]\n\tv_and_b32 %[t3], %[se], %[t3]\n\t"                                     \
    "v_and_b32 %[t4], %[se], %[t4]\n\tv_and_b32 %[t5], %[se], %[t5]\n\t"                                     \
    "v_and_b32 %[t6], %[se], %[t6]\n\tv_and_b32 %[t7], %[se], %[t7]\n\t"                                     \
    "v_fmac_f32 %[c" #R "0], %[" #A "], %[t0]\n\tv_fmac_f32 %[c" #R "1], %[" #A "], %[t1]\n\t"                 \
    "v_fmac_f32 %[c" #R "2], %[" #A "], %[t2]\n\tv_fmac_f32 %[c" #R "3], %[" #A "], %[t3]\n\t"                 \
    "v_fmac_f32 %[c" #S "0], %[" #B "], %[t4]\n\tv_fmac_f32 %[c" #S "1], %[" #B "], %[t5]\n\t"                 \
    "v_fmac_f32 %[c" #S "2], %[" #B "], %[t6]\n\tv_fmac_f32 %[c" #S "3], %[" #B "], %[t7]\n\t"
#define PAM_EXACT_ACC(R)                                                                                        \
    [c##R##0] "+v"(acc[R][0]), [c##R##1] "+v"(acc[R][1]), [c##R##2] "+v"(acc[R][2]), [c##R##3] "+v"(acc[R][3])
#define PAM_EXACT_MOD(R)                                                                                        \
    [m##R##0] "v"(mm[R][0]), [m##R##1] "v"(mm[R][1]), [m##R##2] "v"(mm[R][2]), [m##R##3] "v"(mm[R][3])

__device__ __forceinline__ void exact_step(float (&acc)[8][4], const uint32_t (&mm)[8][4], const uint4 &al,
                                           const uint4 &ah, const uint4 &b, uint32_t sign_exp) {
    uint32_t t0, t1, t2, t3, t4, t5, t6, t7;
    asm(PAM_EXACT_ROWS(0, 1, a0, a1) PAM_EXACT_ROWS(2, 3, a2, a3) PAM_EXACT_ROWS(4, 5, a4, a5)
            PAM_EXACT_ROWS(6, 7, a6, a7)
        : PAM_EXACT_ACC(0), PAM_EXACT_ACC(1), PAM_EXACT_ACC(2), PAM_EXACT_ACC(3), PAM_EXACT_ACC(4), PAM_EXACT_ACC(5),
          PAM_EXACT_ACC(6), PAM_EXACT_ACC(7), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3),
          [t4] "=&v"(t4), [t5] "=&v"(t5), [t6] "=&v"(t6), [t7] "=&v"(t7)
        : PAM_EXACT_MOD(0), PAM_EXACT_MOD(1), PAM_EXACT_MOD(2), PAM_EXACT_MOD(3), PAM_EXACT_MOD(4), PAM_EXACT_MOD(5),
          PAM_EXACT_MOD(6), PAM_EXACT_MOD(7), [a0] "v"(al.x), [a1] "v"(al.y), [a2] "v"(al.z), [a3] "v"(al.w),
          [a4] "v"(ah.x), [a5] "v"(ah.y), [a6] "v"(ah.z), [a7] "v"(ah.w), [b0] "v"(b.x), [b1] "v"(b.y), [b2] "v"(b.z),
          [b3] "v"(b.w), [se] "v"(sign_exp));
}
#undef PAM_EXACT_ROWS
#undef PAM_EXACT_ACC
#undef PAM_EXACT_MOD

// Four words of a row of Mod from column col (zero past n), at any address.
__device__ __forceinline__ uint4 mod_quad(const float *row, int col, int n) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    if (col + 3 < n) {
        const u32x4 x = *reinterpret_cast<const u32x4 *>(row + col);
        return make_uint4(x[0], x[1], x[2], x[3]);
    }
    uint32_t u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        u[j] = col + j < n ? __float_as_uint(row[col + j]) : 0u;
    return make_uint4(u[0], u[1], u[2], u[3]);
}

template <bool TA>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
pam_exact_grad_kernel(GemmParams p) {
    constexpr int BM = kExactTileM, BN = kExactTileN, BK = kChunkK;
    constexpr int NT = 256;
    constexpr int HM = BM / 2;
    using TileA = DmaTile<BM, BK, NT, !TA, float>;
    using TileB = DmaTile<BN, BK, NT, false, float>;
    constexpr int kRawA = TileA::CL * NT * 4;
    constexpr int kRawB = TileB::CL * NT * 4;
    constexpr int kListCap = 2 * NT;   // extreme-Mod outputs a tile lists
    __shared__ __attribute__((aligned(16))) uint32_t smem[kRawA + kRawB + BK * BM + 2 * BK * BN];
    __shared__ uint32_t sSlow[2];      // [chunk parity] steps holding an extreme b
    __shared__ uint32_t sCount;        // extreme-Mod outputs of the tile
    __shared__ uint32_t sList[2][kListCap];   // their (row << 16 | column) and Mod words
    uint32_t *rawA = smem;
    uint32_t *rawB = smem + kRawA;
    uint32_t *sA = smem + kRawA + kRawB;   // A as it is, k-major
    uint32_t *sB = sA + BK * BM;           // B with zero, denormal and extreme values as 0
    uint32_t *sBx = sB + BK * BN;          // B with zero and denormal values as 0

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane(lds_addr(smem) + (uint32_t)wave * 1024u);
    const int lane = tid & 63;
    const int tx = (wave % 2) * 8 + (lane & 7);
    const int ty = (wave / 2) * 8 + (lane >> 3);
    const uint32_t item = blockIdx.x;
    const bool whole = item < (uint32_t)p.whole;
    const uint32_t rel = item - (uint32_t)p.whole;
    const uint32_t nsplit = (uint32_t)max(p.split_tiles, 1);
    const uint32_t st = whole ? 0u : rel % nsplit;
    const int split = whole ? 0 : (int)(rel / nsplit);
    const uint32_t tile = whole ? item : (uint32_t)p.whole + st;
    const int m0 = (int)(tile / (uint32_t)p.tiles_n) * BM;
    const int n0 = (int)(tile % (uint32_t)p.tiles_n) * BN;
    const int kb = whole ? 0 : split * p.k_per_split;
    const int ke = whole ? p.k : min(p.k, kb + p.k_per_split);
    const int nchunks = ke > kb ? (ke - kb + BK - 1) / BK : 0;

    // op(A) rows m0.. and B columns n0.. (B is k-major: B[q * ldb + c]).
    const float *a_base = p.A + (TA ? (int64_t)kb * p.lda + m0 : (int64_t)m0 * p.lda + kb);
    const float *b_base = p.B + (int64_t)kb * p.ldb + n0;
    const int64_t a_step = TA ? (int64_t)BK * p.lda : BK;
    const int64_t b_step = (int64_t)BK * p.ldb;

    // The copies' kinds (A's, then B's) as one scalar word, tested afresh in
    // each chunk (conditions kept across the loop took lane masks, spilled).
    const uint32_t kinds = TileA::kind(ke, m0, p.m, p.lda) | TileB::kind(ke, n0, p.n, p.ldb) << 2;
    if (nchunks > 0) {
        TileA::template copy<0, 2>(a_base, lds_w, tid, p.lda, m0, p.m, ke - kb, kinds & 3u);
        TileB::template copy<kRawA * 4, 2>(b_base, lds_w, tid, p.ldb, n0, p.n, ke - kb, kinds >> 2);
    }
    if (tid < 2)
        sSlow[tid] = 0u;
    if (tid == 0)
        sCount = 0u;
    __syncthreads();

    // The micro-tile's Mod words.  One bit per output (4 i + j): its Mod is zero
    // or denormal; its Mod is extreme (then it goes to the tile's list).
    const int c0 = tx * 4;                                                  // first tile column
    uint32_t mm[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int lr = i < 4 ? ty * 4 + i : HM + ty * 4 + (i - 4);
        uint4 q = make_uint4(0u, 0u, 0u, 0u);
        if (m0 + lr < p.m)
            q = mod_quad(p.Mod + (int64_t)(m0 + lr) * p.ldm, n0 + c0, p.n);
        mm[i][0] = q.x;
        mm[i][1] = q.y;
        mm[i][2] = q.z;
        mm[i][3] = q.w;
    }
    uint32_t zero_mod = 0u, extreme_mod = 0u;
    uint32_t least = 0xFFFFFFFFu, most = 0u;   // exponent fields in the top byte
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            least = min(least, mm[i][j] << 1);
            most = max(most, mm[i][j] << 1);
        }
    if (least < (kSafeLo << 24) || most >= ((kSafeHi + 1u) << 24)) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t u = mm[i][j];
                zero_mod |= (u & kExpMask) == 0u ? 1u << (4 * i + j) : 0u;
                if (extreme(u)) {
                    extreme_mod |= 1u << (4 * i + j);
                    const uint32_t e = atomicAdd(&sCount, 1u);
                    if (e < (uint32_t)kListCap) {
                        const int lr = i < 4 ? ty * 4 + i : HM + ty * 4 + (i - 4);
                        sList[0][e] = ((uint32_t)lr << 16) | (uint32_t)(c0 + j);
                        sList[1][e] = u;
                    }
                }
            }
    }
    __syncthreads();
    const uint32_t nlist = __builtin_amdgcn_readfirstlane(sCount);
    const bool dense = nlist > (uint32_t)kListCap;
    // The fast path takes the mantissas alone (a dense tile the whole words).
    uint32_t keep = dense ? 0xFFFFFFFFu : kMant;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            // kept as computed: re-deriving it inside the loop would cost an
            // op per term
            asm volatile("v_and_b32 %0, %1, %0" : "+v"(mm[i][j]) : "v"(keep));

    float acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = 0.0f;

    // This thread's list entries: e = s * NT + slot(tid), slots dealt so that
    // consecutive entries go to different waves.
    const uint32_t slot = (uint32_t)(lane * (NT / 64) + wave);
    const uint32_t nside = dense ? 0u : nlist;   // the same for the whole workgroup
    float side_acc[2] = {0.0f, 0.0f};

    TileA la;
    TileB lb;
    for (int c = 0; c < nchunks; ++c) {
        const int k_rem = ke - kb - c * BK;   // k steps left, this chunk's included
        uint32_t kd = __builtin_amdgcn_readfirstlane(kinds);
        asm volatile("" : "+s"(kd));
        // Staging addresses are recomputed per chunk from the thread index
        // instead of staying in registers across the steps.
        int tid_c = tid;
        asm volatile("" : "+v"(tid_c));
        __builtin_amdgcn_s_setprio(1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's copies of chunk c have landed
        la.template fetch<2>(rawA, wave, p.lda, m0, p.m, k_rem, kd & 3u, tid_c);
        lb.template fetch<2>(rawB, wave, p.ldb, n0, p.n, k_rem, kd >> 2, tid_c);
        uint32_t smin[TileB::L];
        const uint32_t mx = lb.scan(smin);
        static_assert(TileB::L == 1, "one B segment per thread");
        const bool odd = TileB::low_seg(smin[0]) || mx >= (191u << 24);   // a zero, denormal or extreme b
        __syncthreads();   // every wave is done reading the previous chunk
        la.store_values(sA, false, tid_c);
        uint4 fast = lb.v[0], full = lb.v[0];
        if (odd) {
            const uint32_t e[4] = {lb.v[0].x, lb.v[0].y, lb.v[0].z, lb.v[0].w};
            uint32_t f0[4], f1[4];
            bool any = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool zero = (e[j] & kExpMask) == 0u;
                const bool ext = extreme(e[j]);
                f1[j] = zero ? 0u : e[j];
                f0[j] = (zero || ext) ? 0u : e[j];
                any = any || ext;
            }
            fast = make_uint4(f0[0], f0[1], f0[2], f0[3]);
            full = make_uint4(f1[0], f1[1], f1[2], f1[3]);
            if (any)
                atomicOr(&sSlow[c & 1], 1u << TileB::seg_k(tid_c, 0));
        }
        const int b_at = TileB::seg_k(tid_c, 0) * BN + TileB::seg_o(tid_c, 0);
        *reinterpret_cast<uint4 *>(sB + b_at) = fast;
        *reinterpret_cast<uint4 *>(sBx + b_at) = full;
        __syncthreads();
        const uint32_t slow = __builtin_amdgcn_readfirstlane(sSlow[c & 1]);
        if (tid == 0)
            sSlow[(c + 1) & 1] = 0u;   // next chunk's flags; last read one chunk ago
        // The next chunk's copies land while this one is computed.
        if (c + 1 < nchunks) {
            TileA::template copy<0, 2>(a_base + (c + 1) * a_step, lds_w, tid_c, p.lda, m0, p.m, k_rem - BK, kd & 3u);
            TileB::template copy<kRawA * 4, 2>(b_base + (c + 1) * b_step, lds_w, tid_c, p.ldb, n0, p.n, k_rem - BK, kd >> 2);
        }
        __builtin_amdgcn_s_setprio(0);

        if (!dense) {
            const uint32_t *a_row = sA + ty * 4;
            const uint32_t *b_row = sB + c0;
            uint4 al[2], ah[2], bq[2];
            auto rd = [&](int k, int s) {
                al[s] = *reinterpret_cast<const uint4 *>(a_row + k * BM);
                ah[s] = *reinterpret_cast<const uint4 *>(a_row + k * BM + HM);
                bq[s] = *reinterpret_cast<const uint4 *>(b_row + k * BN);
            };
            uint32_t se = kSignExp;
            asm volatile("" : "+v"(se));
            rd(0, 0);
#pragma unroll
            for (int k = 0; k < BK; ++k) {
                const int cur = k & 1;
                if (k + 1 < BK)
                    rd(k + 1, cur ^ 1);
                __builtin_amdgcn_sched_barrier(0);
                exact_step(acc, mm, al[cur], ah[cur], bq[cur], se);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // Steps with an extreme b (every step in a dense workgroup): the
        // general term for the columns whose b is extreme (every column).
#pragma unroll 1
        for (uint32_t todo = dense ? 0xFFFFu : slow; todo != 0u; todo &= todo - 1u) {
            const int kk = __builtin_ctz(todo);
            int rs = ty * 4, cs = c0;   // nothing of this rare path is kept across the chunks
            asm volatile("" : "+v"(rs), "+v"(cs));
            const uint4 al = *reinterpret_cast<const uint4 *>(sA + kk * BM + rs);
            const uint4 ah = *reinterpret_cast<const uint4 *>(sA + kk * BM + HM + rs);
            const uint4 bq = *reinterpret_cast<const uint4 *>(sBx + kk * BN + cs);
            const uint32_t av[8] = {al.x, al.y, al.z, al.w, ah.x, ah.y, ah.z, ah.w};
            const uint32_t bv[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (dense || extreme(bv[j])) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        uint32_t mod = mm[i][j];
                        const int row = m0 + (i < 4 ? rs + i : HM + rs + i - 4), col = n0 + cs + j;
                        if (!dense && row < p.m && col < p.n)
                            mod = __float_as_uint(p.Mod[(int64_t)row * p.ldm + col]);
                        general_fma(acc[i][j], __uint_as_float(av[i]), bv[j], mod);
                    }
                }
            }
        }
        // Outputs with an extreme Mod, every step.
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t idx = (uint32_t)e * NT + slot;
            if (idx < nside) {
                const int lr = (int)(sList[0][idx] >> 16);
                const int lc = (int)(sList[0][idx] & 0xFFFFu);
                const uint32_t mod = sList[1][idx];
#pragma unroll 4
                for (int kk = 0; kk < BK; ++kk)
                    general_fma(side_acc[e], __uint_as_float(sA[kk * BM + lr]), sBx[kk * BN + lc], mod);
            }
        }
    }

    // The output tile in C, or this K slice's partial tile (packed, written
    // whole).
    float *out;
    int64_t ld;
    int lim_m, lim_n;
    if (whole) {
        out = p.C + (int64_t)m0 * p.ldc + n0;
        ld = p.ldc;
        lim_m = p.m - m0;
        lim_n = p.n - n0;
    } else {
        out = p.W + ((int64_t)split * p.split_tiles + st) * (BM * BN);
        ld = BN;
        lim_m = BM;
        lim_n = BN;
    }
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));   // stored at any address
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        int rs = ty * 4;   // rows are worked out one by one, not held for all
        asm volatile("" : "+v"(rs));
        const int lr = i < 4 ? rs + i : HM + rs + i - 4;
        if (lr >= lim_m)
            continue;
        float *orow = out + (int64_t)lr * ld;
        f32x4 v = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
        if ((zero_mod >> (4 * i)) & 15u) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = (zero_mod >> (4 * i + j)) & 1u ? 0.0f : v[j];
        }
        // extreme-Mod outputs are written by the owner of their list entry
        const uint32_t listed = dense ? 0u : (extreme_mod >> (4 * i)) & 15u;
        if (listed == 0u && c0 + 3 < lim_n) {
            if (whole)
                __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(orow + c0));
            else
                *reinterpret_cast<f32x4 *>(orow + c0) = v;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (c0 + j < lim_n && !((listed >> j) & 1u))
                    orow[c0 + j] = v[j];
        }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint32_t idx = (uint32_t)e * NT + slot;
        if (idx < nside)   // listed outputs lie inside the output
            out[(int64_t)(sList[0][idx] >> 16) * ld + (sList[0][idx] & 0xFFFFu)] = side_acc[e];
    }
}

}  // namespace

hipError_t launch_pam_exact_grad(bool trans_a, const GemmParams &p, hipStream_t stream) {
    const int64_t items = (int64_t)p.whole + (int64_t)p.split_tiles * p.splits;
    if (items <= 0 || items > kMaxLaunchItems)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)items);
    if (trans_a)
        hipLaunchKernelGGL(pam_exact_grad_kernel<true>, grid, dim3(256), 0, stream, p);
    else
        hipLaunchKernelGGL(pam_exact_grad_kernel<false>, grid, dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace pamk
