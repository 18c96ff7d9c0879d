// bf16 MFMA kernels of libhwr (gfx950): the quality GEMM and the staged cost
// predictor (the fused pipeline's predictor table is in k_table.hip).
//
// The predictor computes every layer transposed, h^T = W^T x^T: rows are
// hidden units, columns are candidates.  An accumulator tile then holds, per
// lane, 16 hidden units of one candidate -- exactly the per-lane shape of the
// next layer's B operand -- so activations stay in registers from layer to
// layer; the weights (A operands) are re-laid-out on the host so that their k
// order matches the accumulator row order (see hwr_api.hip, pack_predictor).
#include <type_traits>

#include "hwr_mfma.hpp"

namespace hwr {

// ------------------------------------------------------------ quality GEMM
// Q[q][m] = e_q . Wq[:, m] + bq[m] (Sec. 3.2 item 3), bf16 in, fp32 out.
// Each wave: 32 queries x 32 (padded) models (quality_tile).  The embedding
// stream dominates the traffic (HBM-bound, arithmetic intensity ~M flop/byte).
// U slices are loaded before their MFMAs.  Large batches: four waves per
// workgroup and U = 1, which streams best.  Batches with fewer four-wave
// workgroups than compute units: one wave per workgroup (four times the
// compute units busy) and U = 4 (a quarter of the dependent memory round
// trips).  The MFMA chain runs over the slices in the same order either way:
// identical results.
template <int U>
__global__ __launch_bounds__(256) void k_quality_bf16(QualityArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    quality_tile<U>(a, (blockIdx.x * (blockDim.x >> 6) + wave) * 32, lane);
}

// Large batches with D a multiple of 256: the workgroup (four waves, 64
// queries) streams its rows through LDS in slabs of 256 k (512 bytes per row),
// all four waves loading coalesced with the next slab prefetched in
// registers; waves 0 and 1 run the MFMA chains of the two 32-query tiles from
// LDS in the same k order as k_quality_bf16, so the results are identical.
// Each load instruction then covers two rows' 512 contiguous bytes instead of
// 16 bytes of 32 rows (3.6% faster on HBM-resident chunks).
constexpr int kQSlab = 256;                       // k per slab
constexpr int kQRows = 64;                        // queries per workgroup
__global__ __launch_bounds__(256) void k_quality_bf16_lds(QualityArgs a) {
    constexpr int RB = 2 * kQSlab + 16;           // LDS row stride in bytes (16-byte pad)
    constexpr int PPR = 2 * kQSlab / 16;          // 16-byte pieces per row per slab
    constexpr int PT = kQRows * PPR / 256;        // pieces per thread per slab
    __shared__ __attribute__((aligned(16))) unsigned char s_slab[kQRows * RB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = blockIdx.x * kQRows;
    const int nslab = a.D / kQSlab;
    const uint16_t *emb = static_cast<const uint16_t *>(a.emb);
    u32x4 pre[PT];
    auto load = [&](int j) {
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int p = tid + 256 * i, row = p / PPR, col = p % PPR;
            const int q = r0 + row < a.nq ? r0 + row : a.nq - 1;
            // plain loads: a chunk that is still in the last-level cache
            // (embeddings written just before routing) is read from there;
            // non-temporal loads would bypass it
            pre[i] = *reinterpret_cast<const u32x4 *>(emb + static_cast<size_t>(q) * a.D + j * kQSlab + col * 8);
        }
    };
    const int row = lane & 31, h = lane >> 5;
    const bf16x8 *wq = reinterpret_cast<const bf16x8 *>(a.wq_pk) + lane;
    f32x16 acc = {};
    load(0);
    for (int j = 0; j < nslab; ++j) {
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int p = tid + 256 * i, rw = p / PPR, col = p % PPR;
            *reinterpret_cast<u32x4 *>(s_slab + rw * RB + col * 16) = pre[i];
        }
        __syncthreads();
        if (j + 1 < nslab) load(j + 1);
        if (wave < 2) {
            const unsigned char *base = s_slab + (32 * wave + row) * RB + 64 * h;
#pragma unroll
            for (int sl = 0; sl < kQSlab / 64; ++sl) {
                const int sg = j * (kQSlab / 64) + sl;
                bf16x8 av[4], bv[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    av[c] = *reinterpret_cast<const bf16x8 *>(base + sl * 128 + 16 * c);
                    bv[c] = wq[(sg * 4 + c) * 64];
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) acc = mfma32(av[c], bv[c], acc);
            }
        }
        __syncthreads();
    }
    if (wave < 2) {
        const int m = lane & 31;
        if (m < a.M) {
            const float bias = a.bq[m];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int q = r0 + 32 * wave + crow(r, h);
                if (q < a.nq) a.qmat[static_cast<size_t>(q) * a.M + m] = acc[r] + bias;
            }
        }
    }
}

hipError_t launch_quality_bf16(const QualityArgs &a, int cus, hipStream_t s) {
    const int grid = (a.nq + 127) / 128;
    if (grid < cus) return launch_kernel(k_quality_bf16<4>, dim3((a.nq + 31) / 32), dim3(64), 0, s, a);
    if (a.D % kQSlab == 0)
        return launch_kernel(k_quality_bf16_lds, dim3((a.nq + kQRows - 1) / kQRows), dim3(256), 0, s, a);
    return launch_kernel(k_quality_bf16<1>, dim3(grid), dim3(256), 0, s, a);
}


// ------------------------------------------------------------ predictor
// Eq. 1 cost predictor on MFMA tiles over the staged feature rows, for all
// (query, pair) candidates of a chunk.  A workgroup covers kQPerBlock queries;
// its waves form query groups of 32 * NT queries, two waves per group, and the
// two waves of a group split the pairs in halves.  NT = 2: 8 waves, two per
// SIMD, so that one wave's VALU epilogue overlaps the other's MFMAs.  NT = 4:
// 4 waves, one per SIMD, each holding twice the candidates, so that every
// weight fragment read from LDS feeds four MFMAs instead of two (half the LDS
// traffic per candidate); the first layer's activations then sit in the
// accumulation registers (AGPRs), which the MFMA reads directly.  Each wave
// steps through its pairs, evaluating NT x 32 candidates (one pair, 32 * NT
// queries) per step:
//   X^T  (32 features x 32 candidates, bf16)   read from HBM;
//   h1^T = ReLU(W1^T X^T + b1)  -> bf16, registers;
//   h2^T = ReLU(W2^T h1^T + b2) -> bf16, per 32-row tile, each tile folded at
//   once into the head layer z = W3^T h2^T + b3, itself a chain of 16x16x32
//   MFMAs that leaves each candidate's heads in one lane;
//   TTFT = softplus(z0), TPOT = softplus(z1).
// The layers are software-pipelined: a tile's MFMAs are issued before the
// previous tile's VALU epilogue (bias, ReLU, bf16 packing), so the matrix
// pipe and the vector ALU overlap.  W1, W2 and W3 (A operands) and the biases
// (accumulator initial values) live in LDS.  After the heads, lane half h
// carries column tiles h, h + 2, ... (one query per lane and tile pair) and
// writes their TTFT/TPOT.  X and the outputs are pair-major (candidate (q, d)
// at d * ldq + q): the 64 lanes of a wave, 64 consecutive queries, read whole
// rows and write 256 contiguous bytes.
template <int NT>
struct MlpShape {
    static constexpr int kWaves = NT == 4 ? 4 : 8;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kQPW = 32 * NT;                 // queries per wave
    static constexpr int kQG = kQPerBlock / kQPW;        // query groups per workgroup
    static_assert(kWaves == 2 * kQG, "two waves (pair halves) per query group");
};

template <int H, int NH, bool FB, int NT>
__global__ __launch_bounds__(MlpShape<NT>::kThreads, 1) void k_mlp_bf16(MlpArgs a) {
    constexpr int MT = H / 32;     // 32-row tiles of a hidden layer
    constexpr int KB2 = H / 16;    // k-blocks of the second layer
    constexpr int NO = NT / 2;     // queries each lane completes (tiles h, h + 2, ...)
    constexpr int kThreads = MlpShape<NT>::kThreads;
    constexpr int kQPW = MlpShape<NT>::kQPW;
    constexpr int kQG = MlpShape<NT>::kQG;
    static_assert(NT == 2 || NT == 4, "two or four column tiles per wave");
    __shared__ PredictorLds<H, NH> s;
    stage_predictor<H, NH, kThreads>(a.w, s);
    const int tid = threadIdx.x;
    bf16x8 *const s_w1 = s.w1, *const s_w2 = s.w2, *const s_w3f = s.w3f;
    f32x4 *const s_b1 = s.b1, *const s_b2 = s.b2;
    constexpr int W3S = 2 * NH + 1;
    __syncthreads();

    // (the wave index is uniform: kept in scalar registers, so are the
    // pair loop and the per-pair table reads)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 31, h = lane >> 5;
    const int qw = wave % kQG, grp = wave / kQG;
    const int nq = a.nq;
    const int qbase = blockIdx.x * kQPerBlock + qw * kQPW;
    // every lane reads the feature rows of all column tiles ...
    int qc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int q = qbase + 32 * t + n;
        qc[t] = q < nq ? q : 0;
    }
    // ... and completes column tiles h, h + 2, ... only (queries qme[j])
    int qme[NO];
    bool vme[NO];
#pragma unroll
    for (int j = 0; j < NO; ++j) {
        qme[j] = qbase + 32 * (2 * j + h) + n;
        vme[j] = qme[j] < nq;
    }
    const int d0 = a.N * grp / 2;
    const int d1 = a.N * (grp + 1) / 2;

    int w3_sel[2];
    head_fragments<NH>(lane, w3_sel);

    // The candidates' feature rows are loaded one step ahead; in the four-tile
    // form once the first layer has consumed this step's (they share
    // registers), in the second layer's shadow.
    constexpr bool kLateX = NT == 4;
    bf16x8 nr[NT][2];
    auto load_x = [&](int dn) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const bf16x8 *xr = reinterpret_cast<const bf16x8 *>(
                a.X + (static_cast<size_t>(dn) * a.ldq + qc[t]) * kFeatPad);
            nr[t][0] = xr[h];
            nr[t][1] = xr[2 + h];
        }
    };
    load_x(d0 < d1 ? d0 : 0);

    for (int d = d0; d < d1; ++d) {
        bf16x8 xf[NT][2];              // B operand of layer 1 (Eq. 1 features)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            xf[t][0] = nr[t][0];
            xf[t][1] = nr[t][1];
        }
        if constexpr (!kLateX) load_x(d + 1 < d1 ? d + 1 : d);
        // LDS offsets made opaque per step: the weight fragments are
        // loop-invariant, and hoisting all of them out of the pair loop would
        // need far more registers than a lane has.
        int lo = lane, ho = h, w3o0 = w3_sel[0], w3o1 = w3_sel[1];
        asm volatile("" : "+v"(lo), "+v"(ho), "+v"(w3o0), "+v"(w3o1));
        f32x4 acc3[NO];
#pragma unroll
        for (int j = 0; j < NO; ++j) acc3[j] = f32x4{};
        if constexpr (NT == 4) {
            // One wave per SIMD: the matrix pipe and the vector ALU overlap
            // only where this wave's own instruction stream interleaves them,
            // and LDS latency is hidden only by loading fragments ahead, so
            // both phases below are scheduled by hand (a fence after every
            // MFMA slot).  Phase A runs the first layer together with the
            // second layer's row tile 0, whose k-blocks become available two
            // at a time.  Phase B runs the second layer's other row tiles,
            // each with the previous tile's epilogue interleaved, its weight
            // fragments streamed through a ring of kRing fragments loaded
            // kRing k-steps ahead.  Measured on one wave per SIMD: an MFMA
            // 32x32x16 issues every ~34 cycles with four independent
            // accumulators; v_cvt_pk_bf16_f32 costs ~7 issue cycles,
            // v_pk_max_i16 ~5 and v_accvgpr_write ~6, so phase A is bound by
            // its epilogue's vector work and phase B by the MFMA issue rate.
            constexpr int kRing = 3;
            constexpr int kFull = 0;             // nothing crosses
            bf16x8 h1[NT][KB2];                  // first-layer activations (accumulation registers)
            f32x16 acc[2][NT];
            f32x16 a1[NT];                       // first-layer row tile in flight
            bf16x8 w1c0[2];                      // its W1 fragments
            auto l1_tile = [&](int mt, int t, const bf16x8 (&w)[2]) {
                a1[t] = FB ? f32x16{} : bias_tile(s_b1 + (mt * 2 + ho) * 4);
                a1[t] = mfma32(w[0], xf[t][0], a1[t]);
                a1[t] = mfma32(w[1], xf[t][1], a1[t]);
            };
            // Phase A, scheduled by hand, one iteration per first-layer row
            // tile mt, 16 MFMA slots each with one sixth of the epilogue of
            // row tile mt (per tile t: four slots, two ReLU + bf16 pairs
            // each, and the move of every finished fragment into the
            // accumulation registers).  The MFMAs of a slot: tile 3 of row
            // tile mt (held back from the previous iteration), tiles 0-2 of
            // row tile mt + 1 (each after its tile's epilogue has read the
            // accumulator), and the second layer's row tile 0 over the
            // k-blocks of row tile mt - 1.  Weight fragments are loaded one
            // iteration ahead; a fence after every slot keeps the order.
            bf16x8 w1n[2], w2n[2];
            {
                const bf16x8 w[2] = {s_w1[0 * 64 + lo], s_w1[1 * 64 + lo]};
                w1n[0] = s_w1[2 * 64 + lo];
                w1n[1] = s_w1[3 * 64 + lo];
                w2n[0] = s_w2[0 * 64 + lo];
                w2n[1] = s_w2[1 * 64 + lo];
                const f32x16 bi = bias_tile(s_b2 + (0 * 2 + ho) * 4);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[0][t] = bi;
                w1c0[0] = w[0];
                w1c0[1] = w[1];
#pragma unroll
                for (int t = 0; t < NT - 1; ++t) l1_tile(0, t, w);
            }
            __builtin_amdgcn_sched_barrier(kFull);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const bf16x8 w1c[2] = {w1n[0], w1n[1]};      // row tile mt + 1
                const bf16x8 w2c[2] = {w2n[0], w2n[1]};      // row tile 0, k-blocks 2mt - 2, 2mt - 1
                const bf16x8 w1m[2] = {w1c0[0], w1c0[1]};    // row tile mt (its tile 3)
                if (mt + 2 < MT) {
                    w1n[0] = s_w1[((mt + 2) * 2 + 0) * 64 + lo];
                    w1n[1] = s_w1[((mt + 2) * 2 + 1) * 64 + lo];
                }
                if (mt >= 1) {                   // row tile 0, k-blocks 2mt, 2mt + 1 next
                    w2n[0] = s_w2[(2 * mt + 0) * 64 + lo];
                    w2n[1] = s_w2[(2 * mt + 1) * 64 + lo];
                }
                w1c0[0] = w1c[0];
                w1c0[1] = w1c[1];
                u32x4 hv[2];
#pragma unroll
                for (int sl = 0; sl < 16; ++sl) {
                    const int t = sl / 4, part = sl % 4;
                    // MFMA of this slot
                    if (sl == 0 || sl == 1) {
                        const int kb = sl;
                        if (kb == 0) a1[NT - 1] = FB ? f32x16{} : bias_tile(s_b1 + (mt * 2 + ho) * 4);
                        a1[NT - 1] = mfma32(w1m[kb], xf[NT - 1][kb], a1[NT - 1]);
                    } else if (part >= 2) {
                        if (mt > 0) {
                            const int b = sl >= 8 ? 1 : 0;
                            const int tt = (sl % 8 < 4 ? 0 : 2) + (part - 2);
                            acc[0][tt] = mfma32(w2c[b], h1[tt][2 * mt - 2 + b], acc[0][tt]);
                        }
                    } else if (mt + 1 < MT) {        // part 0 or 1, slots 4.. : row tile mt + 1, tile t - 1
                        const int tt = t - 1, kb = part;
                        if (kb == 0) a1[tt] = FB ? f32x16{} : bias_tile(s_b1 + ((mt + 1) * 2 + ho) * 4);
                        a1[tt] = mfma32(w1c[kb], xf[tt][kb], a1[tt]);
                    }
                    __builtin_amdgcn_sched_barrier(kFull);
                    // epilogue of row tile mt, tile t: fragment part / 2,
                    // pairs 2 (part % 2) .. + 1
                    {
                        const int fr = part / 2, p0 = 2 * (part % 2);
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const int e = 4 * fr + p0 + q;
                            hv[fr][p0 + q] = __builtin_bit_cast(uint32_t, relu_bf16x2(a1[t][2 * e], a1[t][2 * e + 1]));
                        }
                        if (part % 2 == 1) {
                            h1[t][2 * mt + fr] = __builtin_bit_cast(bf16x8, hv[fr]);
                            asm volatile("" : "+a"(h1[t][2 * mt + fr]));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(kFull);
                }
            }
            // the last two k-blocks of row tile 0; the phase-B ring and the
            // bias of row tile 1 are loaded first
            if constexpr (kLateX) load_x(d + 1 < d1 ? d + 1 : d);
            bf16x8 ring[kRing];
            auto w2idx = [&](int i) { return s_w2[(KB2 + i) * 64 + lo]; };   // row tiles 1.. in order
#pragma unroll
            for (int i = 0; i < kRing; ++i) ring[i] = w2idx(i);
            f32x16 bnext = bias_tile(s_b2 + (1 * 2 + ho) * 4);
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[0][t] = mfma32(w2n[b], h1[t][KB2 - 2 + b], acc[0][t]);
            __builtin_amdgcn_sched_barrier(kFull);
            // Phase B, scheduled by hand: every MFMA of row tile mo is
            // followed by one slot of work on row tile mo - 1 (slot
            // s = 4 kb + t): slots 0-31 take the ReLU and bf16 rounding of
            // one element pair each (tile s / 8, pair s % 8), slots 8-11 load
            // the head fragments, and the head MFMAs follow once their tiles'
            // activations are complete.  With 64 slots per row tile (H = 256)
            // they take slots 32-39; with 32 (H = 128) the head MFMAs of tiles
            // 0-1 take slots 16-19 and those of tiles 2-3, whose activations
            // complete at the row tile's last slot, slots 0-3 of the next row
            // tile (their activations and fragments carried over).  Either
            // way each head accumulator takes its contributions in the order
            // of the other form.  The next row tile's bias is loaded at
            // k-step 1.  A scheduling fence after every slot keeps this order.
            constexpr int kSteps = (MT - 1) * KB2;
            constexpr int kSlots = KB2 * NT;
            constexpr bool kWide = kSlots >= 40 + 8 * NO;
            static_assert(kWide || kSlots == 32, "four-tile slot maps: H = 256 or H = 128");
            u32x4 h2c[2][2];                     // narrow: tiles 2-3 of the previous row tile [par][b]
            bf16x8 f3c[2][2];                    // narrow: their head fragments [b][par]
            auto epi_pair = [&](const f32x16 &v, int e) {
                return __builtin_bit_cast(uint32_t, relu_bf16x2(v[2 * e], v[2 * e + 1]));
            };
            // row tile mo of phase B
            auto row_tile = [&](auto mo_c) {
                constexpr int mo = decltype(mo_c)::value;
                f32x16 (&c)[NT] = acc[mo & 1];
                const f32x16 (&pv)[NT] = acc[(mo - 1) & 1];
                const f32x16 bi = bnext;
                u32x4 h2u[NT][2];
                bf16x8 f3[2][2];                 // head fragments [k-block half b][tile parity]
#pragma unroll
                for (int kb = 0; kb < KB2; ++kb) {
                    const int i = (mo - 1) * KB2 + kb;
                    const bf16x8 w = ring[i % kRing];
                    if (i + kRing < kSteps) ring[i % kRing] = w2idx(i + kRing);
                    if (kb == 1 && mo + 1 < MT) bnext = bias_tile(s_b2 + ((mo + 1) * 2 + ho) * 4);
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        c[t] = mfma32(w, h1[t][kb], kb == 0 ? bi : c[t]);
                        __builtin_amdgcn_sched_barrier(kFull);
                        const int sl = 4 * kb + t;
                        if (sl < 32) {
                            const int tt = sl / 8, e = sl % 8;
                            h2u[tt][e / 4][e % 4] = epi_pair(pv[tt], e);
                        }
                        if (sl >= 8 && sl < 12) {
                            const int b = (sl - 8) / 2, par = (sl - 8) % 2;
                            const int kh = 2 * (mo - 1) + b;
                            f3[b][par] = s_w3f[kh * W3S + (par ? w3o1 : w3o0)];
                        }
                        // acc3[j]: (b 0, tile 2j), (b 0, tile 2j + 1), (b 1, 2j), (b 1, 2j + 1)
                        if (kWide && sl >= 32 && sl < 40) {
                            const int j = (sl - 32) / 4, r = (sl - 32) % 4, b = r / 2, par = r % 2;
                            acc3[j] = mfma16(f3[b][par], __builtin_bit_cast(bf16x8, h2u[2 * j + par][b]), acc3[j]);
                        }
                        if (!kWide && sl >= 16 && sl < 20) {
                            const int r = sl - 16, b = r / 2, par = r % 2;
                            acc3[0] = mfma16(f3[b][par], __builtin_bit_cast(bf16x8, h2u[par][b]), acc3[0]);
                        }
                        if (!kWide && mo >= 2 && sl < 4) {
                            const int b = sl / 2, par = sl % 2;
                            acc3[1] = mfma16(f3c[b][par], __builtin_bit_cast(bf16x8, h2c[par][b]), acc3[1]);
                        }
                        __builtin_amdgcn_sched_barrier(kFull);
                    }
                }
                if constexpr (!kWide) {
#pragma unroll
                    for (int par = 0; par < 2; ++par)
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            h2c[par][b] = h2u[2 + par][b];
                            f3c[b][par] = f3[b][par];
                        }
                }
            };
            // row tiles 1 .. MT - 1 (compile-time indices)
            auto run_tiles = [&](auto self, auto mo_c) {
                constexpr int mo = decltype(mo_c)::value;
                if constexpr (mo < MT) {
                    row_tile(mo_c);
                    self(self, std::integral_constant<int, mo + 1>{});
                }
            };
            run_tiles(run_tiles, std::integral_constant<int, 1>{});
            if constexpr (!kWide) {
                // tiles 2-3 of row tile MT - 2, before row tile MT - 1's heads
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int b = r / 2, par = r % 2;
                    acc3[1] = mfma16(f3c[b][par], __builtin_bit_cast(bf16x8, h2c[par][b]), acc3[1]);
                }
            }
            head_tile<H, NH, NT>(s, MT - 1, w3o0, w3o1, acc[(MT - 1) & 1], acc3);
        } else {
            predict_two_tiles<H, NH, FB>(s, xf, lo, ho, w3o0, w3o1, acc3);
        }
        // ---- heads: lane half h completes column tiles h, h + 2, ... (its
        // partner lane holds the other half of the same candidates' hidden
        // units)
#pragma unroll
        for (int j = 0; j < NO; ++j) {
            if (vme[j]) {
                const size_t ci = static_cast<size_t>(d) * a.ldq + qme[j];   // pair-major
                a.cand_ttft[ci] = softplus_fast(acc3[j][0] + a.w.b3_0);
                a.cand_tpot[ci] = softplus_fast(acc3[j][1] + a.w.b3_1);
                if constexpr (NH == 3) a.cand_nout[ci] = softplus_fast(acc3[j][2] + a.w.b3_2);
            }
        }
    }
}

// Column tiles per wave: four at H = 256 and H = 128 (one wave per SIMD, the
// hand-scheduled form) for batches that give every compute unit a workgroup;
// two otherwise (two waves per SIMD: smaller batches start and drain faster).
// The two forms give bit-identical results.
template <int H, int NH, bool FB>
static hipError_t launch_mlp_t(const MlpArgs &a, dim3 grid, hipStream_t s) {
    if constexpr (H == 256 || H == 128) {
        if (a.four_tiles) return launch_kernel(k_mlp_bf16<H, NH, FB, 4>, grid, dim3(MlpShape<4>::kThreads), 0, s, a);
    }
    return launch_kernel(k_mlp_bf16<H, NH, FB, 2>, grid, dim3(MlpShape<2>::kThreads), 0, s, a);
}

template <int H>
static hipError_t launch_mlp_h(const MlpArgs &a, hipStream_t s) {
    const dim3 grid((a.nq + kQPerBlock - 1) / kQPerBlock);
    if (a.fold_b1) return a.nheads == 3 ? launch_mlp_t<H, 3, true>(a, grid, s) : launch_mlp_t<H, 2, true>(a, grid, s);
    return a.nheads == 3 ? launch_mlp_t<H, 3, false>(a, grid, s) : launch_mlp_t<H, 2, false>(a, grid, s);
}

hipError_t launch_mlp_bf16(int H, const MlpArgs &a, hipStream_t s) {
    switch (H) {
        case 64: return launch_mlp_h<64>(a, s);
        case 128: return launch_mlp_h<128>(a, s);
        case 256: return launch_mlp_h<256>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace hwr
