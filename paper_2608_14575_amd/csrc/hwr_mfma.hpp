// MFMA helpers shared by the bf16 kernels of libhwr (gfx950).
//
// Operand layouts (v_mfma_f32_32x32x16_bf16, wave64): A is 32 rows x 16 k, B
// is 16 k x 32 columns; lane l holds 8 consecutive-in-k values of row (A) /
// column (B) l & 31, lane half l >> 5 selecting which 8 of the 16 k.  The
// accumulator holds column l & 31 and rows crow(r, l >> 5), r = 0..15.
#pragma once

#include "hwr_device.hpp"

namespace hwr {

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// v_mfma_f32_16x16x32_bf16: A is 16 rows x 32 k, B 32 k x 16 columns; lane l
// holds 8 consecutive-in-k values of row (A) / column (B) l & 15, k-group
// l >> 4.  The accumulator holds column l & 15, rows 4 * (l >> 4) + 0..3.
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 bias_tile(const f32x4 *p) {
    const f32x4 a = p[0], b = p[1], c = p[2], d = p[3];
    return (f32x16){a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3],
                    c[0], c[1], c[2], c[3], d[0], d[1], d[2], d[3]};
}

// ReLU + bf16 rounding of accumulator elements [base, base + 8), packed as the
// 8 k-values of one B operand.
__device__ __forceinline__ bf16x8 relu_pack8(const f32x16 &c, int base) {
    u32x4 u;
    u[0] = __builtin_bit_cast(uint32_t, relu_bf16x2(c[base + 0], c[base + 1]));
    u[1] = __builtin_bit_cast(uint32_t, relu_bf16x2(c[base + 2], c[base + 3]));
    u[2] = __builtin_bit_cast(uint32_t, relu_bf16x2(c[base + 4], c[base + 5]));
    u[3] = __builtin_bit_cast(uint32_t, relu_bf16x2(c[base + 6], c[base + 7]));
    return __builtin_bit_cast(bf16x8, u);
}

// One wave's 32 queries x 32 (padded) models of the quality GEMM (Sec. 3.2
// item 3), queries q0 .. q0 + 31.  Per 64-wide slice of the embedding, lane
// half h reads 64 contiguous bytes of its query row, as four k-blocks; Wq is
// pre-packed so that each lane's B operand for the same k-block is one
// contiguous 16-byte load.  U slices are loaded before their MFMAs; the chain
// runs over the slices in the same order for every U.
template <int U>
__device__ __forceinline__ void quality_tile(const QualityArgs &a, int q0, int lane) {
    const int row = lane & 31, h = lane >> 5;
    const int qa = q0 + row;
    const bool valid = qa < a.nq;
    const uint16_t *e = static_cast<const uint16_t *>(a.emb) +
                        static_cast<size_t>(valid ? qa : 0) * a.D + 32 * h;
    const bf16x8 *wq = reinterpret_cast<const bf16x8 *>(a.wq_pk) + lane;
    f32x16 acc = {};
    const int S = a.D / 64;
    const bf16x8 zero = {};
    int s = 0;
    for (; s + U <= S; s += U) {
        bf16x8 av[U][4], bv[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                av[u][c] = *reinterpret_cast<const bf16x8 *>(e + 64 * (s + u) + 8 * c);
                bv[u][c] = wq[((s + u) * 4 + c) * 64];
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc = mfma32(valid ? av[u][c] : zero, bv[u][c], acc);
    }
    for (; s < S; ++s) {
        bf16x8 av[4], bv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            av[c] = *reinterpret_cast<const bf16x8 *>(e + 64 * s + 8 * c);
            bv[c] = wq[(s * 4 + c) * 64];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) acc = mfma32(valid ? av[c] : zero, bv[c], acc);
    }
    const int m = lane & 31;
    if (m < a.M) {
        const float bias = a.bq[m];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = q0 + crow(r, h);
            if (q < a.nq) a.qmat[static_cast<size_t>(q) * a.M + m] = acc[r] + bias;
        }
    }
}

// The predictor's weights in LDS: A-operand fragments of W1, W2 and the heads
// (per k-block the 2 * NH data fragments, then one of zeros) and the bias
// tiles (accumulator initial values), laid out as pack_predictor writes them.
template <int H, int NH>
struct PredictorLds {
    static constexpr int MT = H / 32;     // 32-row tiles of a hidden layer
    static constexpr int KB2 = H / 16;    // k-blocks of the second layer
    static constexpr int W3S = 2 * NH + 1;
    bf16x8 w1[MT * 2 * 64];
    bf16x8 w2[MT * KB2 * 64];
    f32x4 b1[MT * 2 * 4];
    f32x4 b2[MT * 2 * 4];
    bf16x8 w3f[KB2 * W3S];
};

// Copy the weights into LDS with T threads (the caller synchronises).
template <int H, int NH, int T>
__device__ __forceinline__ void stage_predictor(const PredictorWeights &w, PredictorLds<H, NH> &s) {
    constexpr int MT = H / 32, KB2 = H / 16;
    const int tid = threadIdx.x;
            // Every load of a staging round is issued before its first LDS
            // store: one memory round trip for W1, the biases and the head
            // fragments, then one per round of up to kStageRound W2 pieces per
            // thread (one round for 512 threads, two for 256).  Indices past an
            // array's end are clamped for the loads and skipped for the stores.
            constexpr int nW1 = MT * 2 * 64, nW2 = MT * KB2 * 64, nB = MT * 2 * 4, nW3 = KB2 * (2 * NH + 1);
            constexpr int pW1 = (nW1 + T - 1) / T;
            constexpr int pW2 = (nW2 + T - 1) / T;
            constexpr int pB = (nB + T - 1) / T;
            constexpr int pW3 = (nW3 + T - 1) / T;
            constexpr int kStageRound = 16;
            constexpr int rW2 = pW2 < kStageRound ? pW2 : kStageRound;
            static_assert(pW2 % rW2 == 0, "whole staging rounds");
            const uint4 *g1 = reinterpret_cast<const uint4 *>(w.w1_pk);
            const uint4 *g2 = reinterpret_cast<const uint4 *>(w.w2_pk);
            const uint4 *gb1 = reinterpret_cast<const uint4 *>(w.b1_pk);
            const uint4 *gb2 = reinterpret_cast<const uint4 *>(w.b2_pk);
            const uint4 *g3 = reinterpret_cast<const uint4 *>(w.w3_frag);
            uint4 v1[pW1], v2[rW2], vb1[pB], vb2[pB], v3[pW3];
            // W1, the biases and the head fragments first (one round trip), so
            // that nothing is held across the W2 rounds: otherwise the compiler
            // keeps W1 in scratch memory meanwhile
#pragma unroll
            for (int i = 0; i < pW1; ++i) {
                const int k = tid + i * T;
                v1[i] = g1[k < nW1 ? k : 0];
            }
#pragma unroll
            for (int i = 0; i < pB; ++i) {
                const int k = tid + i * T;
                vb1[i] = gb1[k < nB ? k : 0];
                vb2[i] = gb2[k < nB ? k : 0];
            }
#pragma unroll
            for (int i = 0; i < pW3; ++i) {
                const int k = tid + i * T;
                v3[i] = g3[k < nW3 ? k : 0];
            }
#pragma unroll
            for (int i = 0; i < pW1; ++i) {
                const int k = tid + i * T;
                if (k < nW1) reinterpret_cast<uint4 *>(s.w1)[k] = v1[i];
            }
#pragma unroll
            for (int i = 0; i < pB; ++i) {
                const int k = tid + i * T;
                if (k < nB) {
                    reinterpret_cast<uint4 *>(s.b1)[k] = vb1[i];
                    reinterpret_cast<uint4 *>(s.b2)[k] = vb2[i];
                }
            }
#pragma unroll
            for (int i = 0; i < pW3; ++i) {
                const int k = tid + i * T;
                if (k < nW3) reinterpret_cast<uint4 *>(s.w3f)[k] = v3[i];
            }
#pragma unroll
            for (int r = 0; r < pW2 / rW2; ++r) {
#pragma unroll
                for (int i = 0; i < rW2; ++i) {
                    const int k = tid + (r * rW2 + i) * T;
                    v2[i] = g2[k < nW2 ? k : 0];
                }
#pragma unroll
                for (int i = 0; i < rW2; ++i) {
                    const int k = tid + (r * rW2 + i) * T;
                    if (k < nW2) reinterpret_cast<uint4 *>(s.w2)[k] = v2[i];
                }
            }
}

// Head-layer A fragment of a lane for column tiles t & 1 == 0, 1 (an index
// into a k-block's fragments): lane 16g + i holds row i, k-group g.  Row
// i = 8(t & 1) + 4s + m is head m of sub-column s; it takes weights only from
// the k-groups whose B lanes carry sub-column s (g & 1 == s), namely the
// hidden-unit half g >> 1.  Every other lane reads the zero fragment.  Tiles
// t and t ^ 1 share one head accumulator, acc3[t >> 1].
template <int NH>
__device__ __forceinline__ void head_fragments(int lane, int (&sel)[2]) {
    const int i = lane & 15, g = lane >> 4, m = i & 3, s = (i >> 2) & 1;
#pragma unroll
    for (int t = 0; t < 2; ++t)
        sel[t] = ((i >> 3) == t && m < NH && (g & 1) == s) ? m * 2 + (g >> 1) : 2 * NH;
}

// Second-layer row tile mo of NT column tiles (NT even), folded into the head
// layer on the matrix pipe: z = W3^T h2^T on 16x16x32 tiles (the heads need few
// rows, and this shape takes the same B operand as the 32x32x16 one in half
// the cycles).  A 16x16x32 B operand reads lanes j, j + 16, j + 32, j + 48 as
// its column j: candidates j and j + 16 of the column tile, each split over two
// lanes (hidden-unit halves).  The A fragments (head_fragments) keep them
// apart: tile t's row 8(t & 1) + 4s + m is head m of candidate 32t + 16s + j,
// so after tiles t and t ^ 1 every lane holds its own candidate's heads in
// accumulator elements 0..NH-1 of acc3[t >> 1].  One fragment read serves the
// tiles of every accumulator.  (Packed bf16 dot products would stall the
// matrix pipe: they do not co-issue with MFMA on gfx950.)
template <int H, int NH, int NT>
__device__ __forceinline__ void head_tile(const PredictorLds<H, NH> &s, int mo, int w3o0, int w3o1,
                                          const f32x16 (&c)[NT], f32x4 (&acc3)[NT / 2]) {
    bf16x8 h2[NT][2];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        h2[t][0] = relu_pack8(c[t], 0);
        h2[t][1] = relu_pack8(c[t], 8);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int kb = 2 * mo + b;
        const bf16x8 f0 = s.w3f[kb * (2 * NH + 1) + w3o0], f1 = s.w3f[kb * (2 * NH + 1) + w3o1];
#pragma unroll
        for (int j = 0; j < NT / 2; ++j) {
            acc3[j] = mfma16(f0, h2[2 * j][b], acc3[j]);
            acc3[j] = mfma16(f1, h2[2 * j + 1][b], acc3[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < NT / 2; ++j) asm volatile("" : "+v"(acc3[j]));
}

// The predictor of two 32-candidate column tiles (feature operands xf) on one
// wave: head sums, before the output bias, of lane (n, h)'s candidate n of tile
// h in acc3[0][0 .. NH-1].  lo, ho, w3o0 and w3o1 are the lane, its half and
// its head fragments; a loop makes them opaque per step: the weight fragments
// are loop-invariant, and hoisting all of them out of the loop would need far
// more registers than a lane has.
//
// Software-pipelined: the VALU epilogue of row tile i-1 (ReLU, bf16 rounding,
// head products) is issued between the first and the remaining MFMAs of row
// tile i, so it runs while those MFMAs occupy the matrix pipe.  The fences
// keep that order (the scheduler would otherwise cluster the epilogues after
// the MFMAs); LDS and global reads may still move across them.  FB: b1 enters
// through the folded-bias feature slots.
template <int H, int NH, bool FB>
__device__ __forceinline__ void predict_two_tiles(const PredictorLds<H, NH> &s, const bf16x8 (&xf)[2][2], int lo, int ho,
                                                  int w3o0, int w3o1, f32x4 (&acc3)[1]) {
    constexpr int NT = 2, MT = H / 32, KB2 = H / 16;
    constexpr int kFence = 0x100 | 0x020;   // DS reads, VMEM reads may cross
    bf16x8 h1[NT][KB2];
    f32x16 acc[2][NT];
    acc3[0] = f32x4{};
    auto l1_mfma = [&](int mt, f32x16 (&c)[NT]) {
        const f32x16 bi = FB ? f32x16{} : bias_tile(s.b1 + (mt * 2 + ho) * 4);
#pragma unroll
        for (int t = 0; t < NT; ++t) c[t] = bi;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const bf16x8 w = s.w1[(mt * 2 + kb) * 64 + lo];
#pragma unroll
            for (int t = 0; t < NT; ++t) c[t] = mfma32(w, xf[t][kb], c[t]);
        }
    };
    // (the empty asm statements pin each epilogue's results at this point:
    // otherwise IR passes sink the pure ReLU / dot-product chains to their
    // last use, past the fences, and the registers overflow)
    auto l1_epi = [&](int mt, const f32x16 (&c)[NT]) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            h1[t][2 * mt] = relu_pack8(c[t], 0);
            h1[t][2 * mt + 1] = relu_pack8(c[t], 8);
            asm volatile("" : "+v"(h1[t][2 * mt]), "+v"(h1[t][2 * mt + 1]));
        }
    };
    auto l2_mfma = [&](int mo, int kb0, int kb1, f32x16 (&c)[NT]) {
        if (kb0 == 0) {
            const f32x16 bi = bias_tile(s.b2 + (mo * 2 + ho) * 4);
#pragma unroll
            for (int t = 0; t < NT; ++t) c[t] = bi;
        }
#pragma unroll
        for (int kb = kb0; kb < kb1; ++kb) {
            const bf16x8 w = s.w2[(mo * KB2 + kb) * 64 + lo];
#pragma unroll
            for (int t = 0; t < NT; ++t) c[t] = mfma32(w, h1[t][kb], c[t]);
        }
    };
    // MFMA k-steps of tile mo issued before the previous epilogue.  For
    // mo = 0 that epilogue produces layer-1 k-blocks KB2-2 and KB2-1, so the
    // head steps must stop short of them.
    constexpr int kHead = KB2 - 2 < 4 ? KB2 - 2 : 4;
    // layer 1: MFMAs of tile mt, then the epilogue of tile mt - 1
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        l1_mfma(mt, acc[mt & 1]);
        if (mt > 0) {
            __builtin_amdgcn_sched_barrier(kFence);
            l1_epi(mt - 1, acc[(mt - 1) & 1]);
            __builtin_amdgcn_sched_barrier(kFence);
        }
    }
    // layer 2: first k-steps of tile mo, epilogue of the previous tile
    // (layer-1 tile MT-1 for mo = 0), then the remaining k-steps
#pragma unroll
    for (int mo = 0; mo < MT; ++mo) {
        const int cur = (MT + mo) & 1, prev = (MT + mo - 1) & 1;
        l2_mfma(mo, 0, kHead, acc[cur]);
        __builtin_amdgcn_sched_barrier(kFence);
        if (mo == 0) l1_epi(MT - 1, acc[prev]);
        else head_tile<H, NH, NT>(s, mo - 1, w3o0, w3o1, acc[prev], acc3);
        __builtin_amdgcn_sched_barrier(kFence);
        l2_mfma(mo, kHead, KB2, acc[cur]);
    }
    head_tile<H, NH, NT>(s, MT - 1, w3o0, w3o1, acc[(2 * MT - 1) & 1], acc3);
}

}  // namespace hwr
