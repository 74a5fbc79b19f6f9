// Operand tile staging through LDS, shared by the matrix product kernel
// (pam_gemm_dma.hip) and the exact-derivative kernel (pam_exact_grad.hip): a
// D x BK chunk of an operand is copied by the memory pipeline into a landing
// buffer, read back in segments of four elements and written k-major into a
// compute buffer.  Included by the HIP sources only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pam_internal.h"
#include "pam_scalar.h"

namespace pamk {

// One 16-byte copy per lane from global memory into LDS: lane i's bytes at
// base + off land at LDS byte address lds_base + IMM + 16 i (the block
// address in M0, the same for the whole wave).  Issued from inline asm, so
// that the compiler does not make later LDS reads of other buffers wait for
// the copy (it cannot tell the landing buffer from the compute buffers of
// the same array); every read of the landing buffer is preceded by an
// explicit wait for the vector-memory counter.  The kernels' compiled code uses M0 for nothing else (no other
// LDS copies, no indexed register moves), so setting it here disturbs no
// value the compiler keeps there.
template <int IMM>
__device__ __forceinline__ void dma_copy16(const char *base, uint32_t off, uint32_t lds_base) {
    // base and lds_base are the same for the whole wave; reading them from
    // the first lane puts them in scalar registers, as the instruction
    // requires.
    const uint2 b = __builtin_bit_cast(uint2, base);
    const uint64_t sb = __builtin_bit_cast(
        uint64_t, make_uint2(__builtin_amdgcn_readfirstlane(b.x), __builtin_amdgcn_readfirstlane(b.y)));
    const uint32_t lb = __builtin_amdgcn_readfirstlane(lds_base);
    // One wait state between the scalar write of M0 and the copy that reads
    // it (the LDS-DMA read-after-SALU-write hazard of this generation).
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(off), "s"(sb), "s"(lb), "i"(IMM)
                 : "memory", "m0", "scc");
}

// LDS byte address of an element of a __shared__ array: the low 32 bits of
// its generic address (no null-pointer test as in a cast to the LDS space).
__device__ __forceinline__ uint32_t lds_addr(const uint32_t *p) { return (uint32_t)(uintptr_t)p; }

// One operand's D x BK chunk (D = rows of op(A) or columns of op(B)) in
// segments of four elements consecutive in memory; T is the operand's
// element type (float or bfloat16 bits).
//
// KCONTIG: a segment is (row o, k quad).  Thread t stages the L rows
// j * L .. j * L + L - 1 of one k quad kq, so that it can write each k of them
// as one L-word LDS store.  Lane 16 * q + i of a wave takes row group
// j = 16 * (wave / (BK / 16)) + i and k quad kq = q + 4 * (wave % (BK / 16)):
// with float32 operands, one copy instruction reads 16 rows x 64 contiguous
// bytes (16 cache lines), and the 16 lanes of each store pass write 16
// consecutive row groups of one k row (no bank conflicts).
//
// Otherwise a segment is (k, column quad); thread t's segment r is number
// t + r * NT, so consecutive lanes hold consecutive column quads of one k.
template <int D, int BK, int NT, bool KCONTIG, typename T>
struct DmaTile {
    static constexpr int SEGS = D * BK / 4;
    static constexpr int L = SEGS / NT;                  // segments per thread
    static constexpr int G = D / L;                      // KCONTIG: row groups
    static constexpr int KS = BK / 16;                   // KCONTIG: waves per 16 row groups
    static constexpr int NW = NT / 64;
    static constexpr bool kWide = sizeof(T) == 4;        // float32 operands; else bfloat16
    static constexpr int EPC = 16 / (int)sizeof(T);      // elements per 16-byte copy
    static constexpr int CL = D * BK / EPC / NT;         // copies per thread
    static_assert(L * NT == SEGS && (L == 2 || L == 4 || (L == 1 && !KCONTIG)),
                  "chunk does not divide over the threads");
    static_assert(CL * EPC * NT == D * BK && CL >= 1, "chunk copies do not divide over the threads");
    static_assert(!KCONTIG || (G % 16 == 0 && BK % 16 == 0 && (G / 16) * KS == NW), "bad K-contiguous segment split");

    uint4 v[L];          // the segments being encoded (live only at the chunk boundary)

    static __device__ __forceinline__ int seg_o(int t, int r) {
        return KCONTIG ? (16 * ((t >> 6) / KS) + (t & 15)) * L + r : ((t + r * NT) % (D / 4)) * 4;
    }
    static __device__ __forceinline__ int seg_k(int t, int r) {
        return KCONTIG ? (((t & 63) >> 4) + 4 * ((t >> 6) % KS)) * 4 : (t + r * NT) / (D / 4);
    }

    // Copies.  A float32 copy is one segment (seg_o / seg_k).  A bfloat16
    // copy is eight elements consecutive in memory, and a wave copies exactly
    // the elements its own lanes stage (so that, after its own wait for the
    // copies, it reads no other wave's): copy r of lane i takes q = i + 64 r
    // of the wave's pieces.  K-contiguous: the wave stages 16 L rows x 16 k
    // (row groups 16 (w / KS) + 0..15, k quads 4 (w % KS) + 0..3), piece q is
    // row q / 2 of them, k octet q % 2.  Otherwise the wave's segments r' =
    // 0..L-1 are 64 consecutive column quads each (from quad 64 w + r' NT of
    // the k-major order), piece q is octet q % 32 of run q / 32.  Either way
    // consecutive lanes read consecutive 16-byte pieces of the operand.
    static __device__ __forceinline__ int copy_o(int t, int r) {
        if constexpr (kWide)
            return seg_o(t, r);
        const int q = (t & 63) + 64 * r;
        if (KCONTIG)
            return 16 * L * ((t >> 6) / KS) + q / 2;
        return (((64 * (t >> 6) + (q / 32) * NT) / 2 + q % 32) % (D / 8)) * 8;
    }
    static __device__ __forceinline__ int copy_k(int t, int r) {
        if constexpr (kWide)
            return seg_k(t, r);
        const int q = (t & 63) + 64 * r;
        if (KCONTIG)
            return 16 * ((t >> 6) % KS) + 8 * (q & 1);
        return ((64 * (t >> 6) + (q / 32) * NT) / 2 + q % 32) / (D / 8);
    }

    // Byte offset of copy r from its chunk's base, for a chunk and tile whose
    // pieces lie inside the operand or wholly past o_lim (those rows and pieces
    // are clamped to the last valid ones: their outputs are discarded).  In builds
    // for three or four waves per SIMD recomputed per chunk from the thread
    // index, so that no per-thread offsets stay live across the K loop.  The
    // leading dimension is below 2^22 elements (the library rejects larger
    // ones), so its bytes and the row or k index fit a 24-bit multiply.
    // CLAMP: pieces may lie past o_lim.
    template <bool CLAMP>
    static __device__ __forceinline__ uint32_t boff(int tid, int r, int64_t ld, int o0, int o_lim) {
        const int o = copy_o(tid, r);
        const int kk = copy_k(tid, r);
        const uint32_t es = (uint32_t)sizeof(T);
        const uint32_t ldb = (uint32_t)ld * es;
        if (KCONTIG)
            return __umul24((uint32_t)min(o, o_lim - 1 - o0), ldb) + (uint32_t)kk * es;
        return __umul24((uint32_t)kk, ldb) + (uint32_t)(CLAMP ? min(o, o_lim - EPC - o0) : o) * es;
    }
    // What a tile's copies have to heed, the same for the whole workgroup:
    // kEdge when a piece of it straddles the last column of an operand that is
    // not K-contiguous; kThin when such an operand has fewer columns than a
    // piece; kShort when a K-contiguous row (up to k = ke) is shorter than a
    // piece, or the whole thin operand.
    static constexpr uint32_t kEdge = 1u, kShort = 2u, kThin = 3u;
    static __device__ __forceinline__ uint32_t kind(int ke, int o0, int o_lim, int64_t ld) {
        if (KCONTIG)
            return ke >= EPC ? 0u : kShort;
        if (o_lim < EPC)
            return (int64_t)(ke - 1) * ld + o_lim >= EPC ? kThin : kShort;
        return o0 + D <= o_lim || o_lim % EPC == 0 ? 0u : kEdge;
    }

    // At the last k steps of a row, or at the last columns, a piece that
    // would pass the end starts earlier, on the last EPC elements: every
    // piece is copied whole and inside the operand, and fetch() picks a
    // segment's elements out of it.  k_rem: valid k steps from the chunk's
    // base.  First element (k or column, relative to the chunk's base) of the
    // piece that would start at x; below zero by at most EPC - 1.
    static __device__ __forceinline__ int piece_k(int kk, int k_rem) { return min(kk, k_rem - EPC); }
    static __device__ __forceinline__ int piece_o(int o, int o0, int o_lim) { return min(o, o_lim - EPC - o0); }
    // kThin: first element, from the chunk's base, of the piece of row kk <
    // k_rem.  It runs on over the gap and the rows after it; at the operand's
    // last element (BK rows on suffices) it starts earlier instead.
    // (Copied element by element such an operand held up every chunk: 4096 x 3 x
    // 4096 74.8 us, now 57.9 us; x 4, whole pieces, 50.6 us.)
    static __device__ __forceinline__ int piece_thin(int kk, int64_t ld, int o_lim, int k_rem) {
        const uint32_t row = __umul24((uint32_t)kk, (uint32_t)ld);
        return min((int)row, (int)__umul24((uint32_t)min(k_rem - 1, BK), (uint32_t)ld) + o_lim - EPC);
    }
    // As boff, from EPC elements before the chunk's base.
    static __device__ __forceinline__ uint32_t boff_edge(int tid, int r, int64_t ld, int o0, int o_lim, int k_rem,
                                                         uint32_t kind) {
        const int o = copy_o(tid, r);
        const int kk = copy_k(tid, r);
        const uint32_t es = (uint32_t)sizeof(T);
        const uint32_t ldb = (uint32_t)ld * es;
        if (!KCONTIG && kind == kThin)
            return (uint32_t)(piece_thin(min(kk, k_rem - 1), ld, o_lim, k_rem) + EPC) * es;
        if (KCONTIG)
            return __umul24((uint32_t)min(o, o_lim - 1 - o0), ldb) + (uint32_t)(piece_k(kk, k_rem) + EPC) * es;
        return __umul24((uint32_t)min(kk, k_rem - 1), ldb) + (uint32_t)(piece_o(o, o0, o_lim) + EPC) * es;
    }

    // Start copying the chunk at `base` into the landing buffer at byte
    // RAW_OFF of the LDS array; lds_w is the LDS byte address of that array
    // plus 1024 per wave index, so that copy r of wave w lands in block
    // (r * NW + w) at lds_w + RAW_OFF + r * NW * 1024 (16 bytes per lane).
    // Pieces may lie at any address: the copy needs no alignment of the
    // operand.  k_rem >= 1.
    // EDGE 0: every chunk and tile of the launch lies inside the operand (but for
    // rows past o_lim); 1: pieces may lie wholly past the last column; 2: chunks
    // may pass the end of K and pieces straddle the last column.  What a launch
    // does not need is not compiled in.
    template <int RAW_OFF, int EDGE>
    static __device__ __forceinline__ void copy(const T *__restrict__ base, uint32_t lds_w, int tid, int64_t ld,
                                                int o0, int o_lim, int k_rem, uint32_t kind) {
        const char *cb = reinterpret_cast<const char *>(base);
        static_assert(CL == 1 || CL == 2 || CL == 4, "copies per thread");
        // In a whole chunk with a whole piece of columns the straddling piece
        // starts where boff clamps it to.  (With this and its short way in fetch(), 64
        // matrices of op T 384 x 139 x 1373 took 520 us, now 497 us.)
        if (EDGE < 2 || (k_rem >= BK && (kind == 0u || (kind == kEdge && o_lim - o0 >= EPC)))) {
            dma_copy16<RAW_OFF>(cb, boff<(EDGE > 0)>(tid, 0, ld, o0, o_lim), lds_w);
            if constexpr (CL >= 2)
                dma_copy16<RAW_OFF + NW * 1024>(cb, boff<(EDGE > 0)>(tid, 1, ld, o0, o_lim), lds_w);
            if constexpr (CL == 4) {
                dma_copy16<RAW_OFF + 2 * NW * 1024>(cb, boff<(EDGE > 0)>(tid, 2, ld, o0, o_lim), lds_w);
                dma_copy16<RAW_OFF + 3 * NW * 1024>(cb, boff<(EDGE > 0)>(tid, 3, ld, o0, o_lim), lds_w);
            }
            return;
        }
        // Edges are rare: their addresses are worked out here, never kept.
        asm volatile("" : "+v"(tid), "+s"(o0), "+s"(o_lim), "+s"(ld));
        cb -= 16;
        if (kind == kShort) {
            // Its elements one by one, those before the row's first as zeros.
            const int before = KCONTIG ? EPC - k_rem : EPC - (o_lim - o0);
#pragma unroll 1
            for (int r = 0; r < CL; ++r) {
                const char *src = cb + boff_edge(tid, r, ld, o0, o_lim, k_rem, kind);
                const uint32_t dst = lds_w + RAW_OFF + (uint32_t)(r * NW) * 1024u + (uint32_t)(tid & 63) * 16u;
#pragma unroll 1
                for (int x = 0; x < EPC; ++x)
                    *(lds_t *)(uintptr_t)(dst + (uint32_t)(x * (int)sizeof(T))) =
                        x >= before ? *reinterpret_cast<const T *>(src + x * (int)sizeof(T)) : (T)0;
            }
            return;
        }
        dma_copy16<RAW_OFF>(cb, boff_edge(tid, 0, ld, o0, o_lim, k_rem, kind), lds_w);
        if constexpr (CL >= 2)
            dma_copy16<RAW_OFF + NW * 1024>(cb, boff_edge(tid, 1, ld, o0, o_lim, k_rem, kind), lds_w);
        if constexpr (CL == 4) {
            dma_copy16<RAW_OFF + 2 * NW * 1024>(cb, boff_edge(tid, 2, ld, o0, o_lim, k_rem, kind), lds_w);
            dma_copy16<RAW_OFF + 3 * NW * 1024>(cb, boff_edge(tid, 3, ld, o0, o_lim, k_rem, kind), lds_w);
        }
    }

    // Where segment r of this thread (wave w, lane) sits in the landing
    // buffer: the word offset of its 16 (float32) or 8 (bfloat16) bytes.  A
    // float32 segment is the lane's own copy r (block r * NW + w); a bfloat16
    // segment is half of the copy of its eight elements, made by a lane of
    // the same wave.
    static __device__ __forceinline__ uint32_t slot_of(int w, int lane, int r) {
        if constexpr (kWide)
            return (uint32_t)((r * NW + w) * 256 + lane * 4);
        const int q = KCONTIG ? ((lane & 15) * L + r) * 2 + (lane >> 5) : r * 32 + lane / 2;
        const int half = KCONTIG ? (lane >> 4) & 1 : lane & 1;
        return (uint32_t)(((q / 64) * NW + w) * 256 + (q % 64) * 4 + half * 2);
    }
    // Reads through an LDS-space pointer: never a generic (flat) load.
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
    typedef __attribute__((address_space(3))) const u32x2 lds_u32x2;
    typedef __attribute__((address_space(3))) T lds_t;
    static __device__ __forceinline__ uint4 read_slot(const uint32_t *raw, uint32_t off) {
        if constexpr (kWide) {
            const u32x4 x = *(lds_u32x4 *)(raw + off);
            return make_uint4(x[0], x[1], x[2], x[3]);
        }
        const u32x2 y = *(lds_u32x2 *)(raw + off);
        const uint2 d = make_uint2(y[0], y[1]);
        // Four bfloat16 elements widened exactly to float32 encodings.
        return make_uint4(d.x << 16, d.x & 0xFFFF0000u, d.y << 16, d.y & 0xFFFF0000u);
    }

    // Segment r's elements from element x of the piece that holds it (0 <= x <
    // EPC; elements past the piece's end are of no meaning).
    static __device__ __forceinline__ uint4 piece_elements(const uint32_t *raw, int w, int lane, int r, uint32_t x) {
        const u32x4 q = *(lds_u32x4 *)(raw + (slot_of(w, lane, r) & ~3u));
        uint32_t q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
        if constexpr (kWide) {
            if (x & 1u) {
                q0 = q1;
                q1 = q2;
                q2 = q3;
            }
            return (x & 2u) ? make_uint4(q2, q3, q3, q3) : make_uint4(q0, q1, q2, q3);
        }
        if (x & 4u) {
            q0 = q2;
            q1 = q3;
        }
        if (x & 2u) {
            q0 = q1;
            q1 = q2;
            q2 = q3;
        }
        if (x & 1u) {
            q0 = __builtin_amdgcn_alignbit(q1, q0, 16);
            q1 = __builtin_amdgcn_alignbit(q2, q1, 16);
        }
        return make_uint4(q0 << 16, q0 & 0xFFFF0000u, q1 << 16, q1 & 0xFFFF0000u);
    }

    // The thread's segments of a chunk with k_rem valid k steps (the elements
    // past them are zero; columns past o_lim repeat the last one, their
    // outputs are discarded) from the landing buffer.
    template <int EDGE>
    __device__ __forceinline__ void fetch(const uint32_t *raw, int w, int64_t ld, int o0, int o_lim, int k_rem,
                                          uint32_t kind, int tid) {
        if (EDGE < 2 || (k_rem >= BK && kind == 0u)) {
            // The common case, one branch for all segments: the reads issue
            // back to back and are waited for once.
#pragma unroll
            for (int r = 0; r < L; ++r)
                v[r] = read_slot(raw, slot_of(w, tid & 63, r));
            if constexpr (EDGE > 0)
                blank(o_lim - o0, tid);
            return;
        }
        asm volatile("" : "+v"(tid), "+s"(o0), "+s"(o_lim), "+s"(ld), "+s"(w));   // as in copy()
        // A segment out of its piece, moved or not: one read, a shift and selects
        // for all lanes.  (Element by element, behind a branch each, a bfloat16
        // 4096 x 9 x 4096 product took 59.5 us, now 56.7 us.)
        auto take = [&](int r) {
            const int o = seg_o(tid, r);
            const int kk = seg_k(tid, r);
            int x;   // the segment's first element in its piece
            if (KCONTIG)
                x = kk - piece_k(kk & -EPC, k_rem);
            else if (kind == kThin)
                x = o + (int)__umul24((uint32_t)kk, (uint32_t)ld) - piece_thin(kk, ld, o_lim, k_rem);
            else
                x = o - piece_o(o & -EPC, o0, o_lim);
            const uint4 q = piece_elements(raw, w, tid & 63, r, (uint32_t)x);
            uint32_t e[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (KCONTIG)
                    e[c] = kk + c < k_rem ? e[c] : 0u;
                else if (c > 0)
                    e[c] = o + c < o_lim - o0 ? e[c] : e[c > 0 ? c - 1 : 0];
            }
            v[r] = make_uint4(e[0], e[1], e[2], e[3]);
        };
        if (!KCONTIG && kWide && k_rem >= BK && kind == kEdge) {
            // A moved float32 piece ends with the last column: shifted, it repeats it.
#pragma unroll
            for (int r = 0; r < L; ++r)
                v[r] = piece_elements(raw, w, tid & 63, r, (uint32_t)max(seg_o(tid, r) - (o_lim - EPC - o0), 0));
        } else if (!KCONTIG && k_rem >= BK) {
#pragma unroll
            for (int r = 0; r < L; ++r)
                take(r);
        } else {
            // Whole waves lie past a short K and skip their segments.
#pragma unroll
            for (int r = 0; r < L; ++r) {
                v[r] = make_uint4(0u, 0u, 0u, 0u);
                if (seg_k(tid, r) < k_rem)
                    take(r);
            }
        }
        blank(o_lim - o0, tid);
    }

    // Segments wholly past the last column hold the clamped pieces' elements,
    // other ones for float32 than for bfloat16; as ones they have no say in
    // the steps' forms and thus in the order of the sums.
    __device__ __forceinline__ void blank(int o_rem, int tid) {
        if constexpr (!KCONTIG) {
            if (o_rem < D) {
                asm volatile("" : "+v"(tid));   // nothing of this is kept across the chunks
#pragma unroll
                for (int r = 0; r < L; ++r)
                    if (seg_o(tid, r) >= o_rem)
                        v[r] = make_uint4(kBias, kBias, kBias, kBias);
            }
        }
    }

    // Round every held element to 23 - drop mantissa bits, nearest even (inf
    // and NaN unchanged).
    __device__ __forceinline__ void round_mantissa(int drop) {
        const uint32_t low = (1u << drop) - 1u;
        const uint32_t half_m1 = low >> 1;
#pragma unroll
        for (int r = 0; r < L; ++r) {
            uint32_t e[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t u = e[c];
                const uint32_t rounded = (u + half_m1 + ((u >> drop) & 1u)) & ~low;
                e[c] = ((u & kExpMask) == kExpMask) ? u : rounded;
            }
            v[r] = make_uint4(e[0], e[1], e[2], e[3]);
        }
    }

    // One pass over the held elements with the exponent field moved to the
    // top byte and the sign dropped (x << 1): per segment r the least such
    // value (below 64 << 24 iff the segment holds an element below the S1
    // range: a zero, denormal or |x| < 2^-63), and the largest over all
    // elements, returned (at least 191 << 24 iff one needs the SPECIAL
    // path: |x| >= 2^64, inf, NaN).
    __device__ __forceinline__ uint32_t scan(uint32_t (&smin)[L]) const {
        uint32_t mx = 0;
#pragma unroll
        for (int r = 0; r < L; ++r) {
            const uint32_t j0 = v[r].x << 1, j1 = v[r].y << 1, j2 = v[r].z << 1, j3 = v[r].w << 1;
            smin[r] = min(min(j0, j1), min(j2, j3));
            mx = max(mx, max(max(j0, j1), max(j2, j3)));
        }
        return mx;
    }
    static __device__ __forceinline__ bool low_seg(uint32_t smin) { return smin < (64u << 24); }

    // A denormal element to its signed zero (multiplying by 1.0 flushes it;
    // NaN stays NaN).  Needed for B only, and only where scan() found an
    // element below the S1 range.
    __device__ __forceinline__ void flush_denormals() {
#pragma unroll
        for (int r = 0; r < L; ++r) {
            uint32_t e[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                asm("v_mul_f32 %0, 1.0, %1" : "=v"(e[c]) : "v"(e[c]));
            v[r] = make_uint4(e[0], e[1], e[2], e[3]);
        }
    }

    // Element encodings: A as it is; B as b' = b - bias (denormals already
    // flushed).
    static __device__ __forceinline__ uint32_t enc(uint32_t u, bool is_b) { return is_b ? u - kBias : u; }

    // Write the encoded chunk k-major into s[k * D + o].
    __device__ __forceinline__ void store_values(uint32_t *s, bool is_b, int tid) const {
        if constexpr (KCONTIG) {
            // One address; the four k rows at constant offsets from it.
            uint32_t *const row0 = s + seg_k(tid, 0) * D + seg_o(tid, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                uint32_t w[L];
#pragma unroll
                for (int r = 0; r < L; ++r) {
                    const uint32_t u = c == 0 ? v[r].x : c == 1 ? v[r].y : c == 2 ? v[r].z : v[r].w;
                    w[r] = enc(u, is_b);
                }
                uint32_t *dst = row0 + c * D;
                if constexpr (L == 2)
                    *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
                else
                    *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < L; ++r) {
                const int o = seg_o(tid, r);
                const int kk = seg_k(tid, r);
                *reinterpret_cast<uint4 *>(s + kk * D + o) =
                    make_uint4(enc(v[r].x, is_b), enc(v[r].y, is_b), enc(v[r].z, is_b), enc(v[r].w, is_b));
            }
        }
    }

    // Mark the step masks: bit k % KPG of the word of k-group k / KPG and of the
    // element's slot when it has exponent field below 64, also bit 16 +
    // k % KPG when it is a normal number.  Eight consecutive lanes hold
    // elements of one slot and of one k quad (K-contiguous) or k row: their
    // words are combined before the LDS atomic.  (One atomic per element
    // cost a chunk of ReLU activations, half of them zeros, as much as its
    // compute steps: 32 lanes a time on one address.)
    template <int KPG, typename SlotOf>
    __device__ __forceinline__ void mark(int tid, const uint32_t (&smin)[L], uint32_t *mask, int slots,
                                         SlotOf slot_of) const {
        // Segments r of one k-group: all, or runs of RUN.
        constexpr int STEP = KCONTIG ? 1 : NT * 4 / D;   // k rows from a thread's segment to its next
        constexpr int RUN = KCONTIG || KPG / STEP >= L ? L : KPG / STEP;
        static_assert(KPG % STEP == 0 && RUN >= 1 && L % RUN == 0, "segments do not divide over the k-groups");
#pragma unroll
        for (int r0 = 0; r0 < L; r0 += RUN) {
            uint32_t least = smin[r0];
#pragma unroll
            for (int r = r0 + 1; r < r0 + RUN; ++r)
                least = min(least, smin[r]);
            if (__builtin_amdgcn_ballot_w64(low_seg(least)) == 0u)
                continue;   // the whole wave: no such element
            const int kk = seg_k(tid, r0);
            uint32_t word = 0u;
            if constexpr (KCONTIG) {
                uint32_t tiny = 0xFFFFFFFFu;   // least exponent field less 1, zero and denormal wrapped to the top
#pragma unroll
                for (int c = 3; c >= 0; --c) {
                    uint32_t ex = 0xFFFFFFFFu;
#pragma unroll
                    for (int r = 0; r < L; ++r) {
                        const uint32_t e = element(r, c) & kExpMask;
                        ex = min(ex, e);
                        tiny = min(tiny, e - kMinNormal);
                    }
                    // word << 1, with the sign of ex - (64 << 23) shifted in
                    word = __builtin_amdgcn_alignbit(word, ex - (64u << 23), 31);
                }
                if (tiny < (63u << 23)) {
#pragma unroll
                    for (int r = 0; r < L; ++r)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            word |= tiny_normal(element(r, c)) ? 0x10000u << c : 0u;
                }
                word <<= kk % KPG;
            } else {
#pragma unroll
                for (int r = r0; r < r0 + RUN; ++r) {
                    const uint32_t bit = 1u << (seg_k(tid, r) % KPG);
                    if (low_seg(smin[r])) {
                        word |= bit;
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            word |= tiny_normal(element(r, c)) ? bit << 16 : 0u;
                    }
                }
            }
            word |= __builtin_amdgcn_update_dpp(0u, word, 0xB1, 0xF, 0xF, true);    // lane ^ 1
            word |= __builtin_amdgcn_update_dpp(0u, word, 0x4E, 0xF, 0xF, true);    // lane ^ 2
            word |= __builtin_amdgcn_update_dpp(0u, word, 0x141, 0xF, 0xF, true);   // mirrored in eight lanes
            if ((tid & 7) == 0 && word != 0u)
                atomicOr(&mask[(kk / KPG) * slots + slot_of(seg_o(tid, 0))], word);
        }
    }

    // Some held element is a tiny normal.
    __device__ __forceinline__ bool any_tiny() const {
        bool any = false;
#pragma unroll
        for (int r = 0; r < L; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                any = any || tiny_normal(element(r, c));
        return any;
    }

    __device__ __forceinline__ uint32_t element(int r, int c) const {
        return c == 0 ? v[r].x : c == 1 ? v[r].y : c == 2 ? v[r].z : v[r].w;
    }
    // A normal number with exponent field below 64.
    static __device__ __forceinline__ bool tiny_normal(uint32_t u) {
        return (u & kExpMask) - kMinNormal < (63u << 23);
    }
};

}  // namespace pamk
