// Decisions of the fused pipeline (gfx950): per query, cost (Eq. 2), bound test
// and utility of every pair from the query's row of the predictor table, then
// the Eq. 3 argmax, once per cost weight.
#include <algorithm>

#include "hwr_mfma.hpp"

namespace hwr {

constexpr int kRouteThreads = 256;
constexpr int kRouteLanes = 8;                    // lanes per query in the decision
constexpr int kRoutePass = kRouteThreads / kRouteLanes;   // queries decided at once
constexpr int kRouteSlab = 256;                   // k per slab of the quality GEMM
constexpr int kQStride = kMaxModels + 1;          // LDS quality row (odd: rows in different banks)

// Running bests of one lane and one cost weight, over its pairs in increasing
// order: the best among the feasible pairs and the best over all, each
// replaced only by a strictly larger utility (so ties keep the lower pair, and
// a NaN or -inf utility is never taken).  lane_key turns them into the lane's
// decision key.
struct LaneBest {
    float uf, ua;
    int df, da;                   // -1: none
};

// The lane's decision key.  When nothing feasible was taken but a feasible
// pair exists (its utility is -inf or NaN, which ranks as -inf), that pair,
// the lane's first feasible one (ff), is its best; when nothing at all was
// taken, the lane's first pair (d0; none: 0).
__device__ __forceinline__ uint64_t lane_key(const LaneBest &b, int ff, int d0, int N) {
    if (b.df >= 0) return decision_key(true, b.uf, b.df);
    if (ff >= 0) return decision_key(true, -__builtin_huge_valf(), ff);
    if (b.da >= 0) return decision_key(false, b.ua, b.da);
    return d0 < N ? decision_key(false, -__builtin_huge_valf(), d0) : 0;
}

// Utility of a decision key (the inverse of ord_u32).
__device__ __forceinline__ float key_utility(uint64_t k) {
    const uint32_t o = static_cast<uint32_t>(k >> 31);
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

// QUAL: the workgroup first computes its 64 queries' qualities (the MFMA chain
// of quality_tile, the rows streamed through LDS in slabs of 256 k with the
// next slab prefetched in registers) and keeps them in LDS; otherwise it takes
// 32 queries' from a.quality.qmat.  Then eight lanes decide each query: they
// read its table row 128 bytes at a time (16 pairs), each lane two pairs of
// it, in increasing order, and compare packed decision keys (unique: they hold
// the pair index) with DPP steps.  One thread per query and weight then reads
// the chosen pair's predictions again and writes the outputs.
// PN: N_out predicted per candidate; GEN: the paper's score or bound; DBG:
// per-candidate outputs.
template <bool QUAL, bool PN, bool MULTI, bool GEN, bool DBG>
__global__ __launch_bounds__(kRouteThreads) void k_route(RouteArgs a) {
    constexpr int QB = QUAL ? 64 : kRoutePass;    // queries per workgroup
    constexpr int NW = MULTI ? kMaxWeights : 1;
    constexpr int RB = 2 * kRouteSlab + 16;       // LDS slab row in bytes (16-byte pad)
    constexpr int kSlabBytes = QUAL ? QB * RB : 0, kQualBytes = QB * kQStride * 4;
    __shared__ __attribute__((aligned(16))) unsigned char s_buf[kSlabBytes > kQualBytes ? kSlabBytes : kQualBytes];
    __shared__ uint8_t s_model[kMaxPairs];
    __shared__ int s_row[QB], s_len[QB];
    __shared__ float s_nout[QB], s_slo[QB];
    __shared__ uint64_t s_key[QB * NW];
    float *s_q = reinterpret_cast<float *>(s_buf);   // [QB][kQStride]
    Rule rule = a.rule;
    if constexpr (!GEN) rule = Rule{};
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nq = a.q.nq, N = a.N, M = a.M;
    const int q0 = blockIdx.x * QB;
    const int nqb = min(QB, nq - q0);

    auto query_inputs = [&] {
        if (tid < QB) {
            const int q = tid < nqb ? q0 + tid : nq - 1;
            const int32_t len = a.q.input_len[q];
            const int32_t no = PN ? 0 : a.q.nout[q];
            s_len[tid] = len;
            s_nout[tid] = static_cast<float>(no < 0 ? 0 : no);
            s_slo[tid] = a.q.slo ? a.q.slo[q] : a.q.default_slo;
            if (a.len_row) s_row[tid] = a.len_row[len_index(bf16_bits(len_feature(len)))];
            else s_row[tid] = a.owner && static_cast<uint32_t>(len) < static_cast<uint32_t>(kOwnLens) ? a.owner[len] : q;
        }
        for (int i = tid; i < N; i += kRouteThreads) s_model[i] = static_cast<uint8_t>(a.dep_model[i]);
    };

    if constexpr (QUAL) {
        const QualityArgs &qa = a.quality;
        constexpr int PPR = 2 * kRouteSlab / 16;      // 16-byte pieces per row per slab
        constexpr int PT = QB * PPR / kRouteThreads;  // pieces per thread per slab
        const int nslab = (qa.D + kRouteSlab - 1) / kRouteSlab;
        const uint16_t *emb = static_cast<const uint16_t *>(qa.emb);
        u32x4 pre[PT];
        auto load = [&](int j) {
#pragma unroll
            for (int i = 0; i < PT; ++i) {
                const int p = tid + kRouteThreads * i, row = p / PPR, col = p % PPR;
                const int q = row < nqb ? q0 + row : nq - 1;
                // past the row's end (D not a multiple of the slab): its last piece, never used
                const int k = min(j * kRouteSlab + col * 8, qa.D - 8);
                // plain loads: a chunk still in the last-level cache (embeddings
                // written just before routing) is read from there
                pre[i] = *reinterpret_cast<const u32x4 *>(emb + static_cast<size_t>(q) * qa.D + k);
            }
        };
        const int row = lane & 31, h = lane >> 5;
        const bf16x8 *wq = reinterpret_cast<const bf16x8 *>(qa.wq_pk) + lane;
        f32x16 acc = {};
        load(0);
        query_inputs();
        for (int j = 0; j < nslab; ++j) {
#pragma unroll
            for (int i = 0; i < PT; ++i) {
                const int p = tid + kRouteThreads * i, rw = p / PPR, col = p % PPR;
                *reinterpret_cast<u32x4 *>(s_buf + rw * RB + col * 16) = pre[i];
            }
            __syncthreads();
            if (j + 1 < nslab) load(j + 1);
            if (wave < 2) {
                const unsigned char *base = s_buf + (32 * wave + row) * RB + 64 * h;
                const int slices = min(kRouteSlab / 64, qa.D / 64 - j * (kRouteSlab / 64));
                for (int sl = 0; sl < slices; ++sl) {
                    const int sg = j * (kRouteSlab / 64) + sl;
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
        if (wave < 2 && row < M) {
            const int m = row;
            const float bias = qa.bq[m];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int ql = 32 * wave + crow(r, h);
                s_q[ql * kQStride + m] = acc[r] + bias;
                if (DBG && qa.qmat && ql < nqb) qa.qmat[static_cast<size_t>(q0 + ql) * M + m] = acc[r] + bias;
            }
        }
    } else {
        query_inputs();
        for (int i = tid; i < nqb * M; i += kRouteThreads) {
            const int r = i / M, m = i - r * M;
            s_q[r * kQStride + m] = a.quality.qmat[static_cast<size_t>(q0) * M + i];
        }
    }
    __syncthreads();

    const int nw = MULTI ? a.nw : 1;
    const int l8 = lane & (kRouteLanes - 1);
#pragma unroll 1
    for (int pass = 0; pass < QB / kRoutePass; ++pass) {
        const int ql = pass * kRoutePass + tid / kRouteLanes;   // queries past nqb repeat the last: never written
        const bool live = ql < nqb;
        const f32x4 *row = reinterpret_cast<const f32x4 *>(a.tab + static_cast<size_t>(s_row[ql]) * a.ldn * 2) + l8;
        const f32x2 *rown = PN ? reinterpret_cast<const f32x2 *>(a.tab_nout + static_cast<size_t>(s_row[ql]) * a.ldn) + l8 : nullptr;
        const float *sq = s_q + ql * kQStride;
        const float nout = s_nout[ql];
        const QueryRule qr = query_rule(rule, s_slo[ql], s_len[ql], nout, a.w[0]);
        LaneBest best[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) best[k] = LaneBest{-__builtin_huge_valf(), -__builtin_huge_valf(), -1, -1};
        int ff = -1;                               // the lane's first feasible pair
        auto take = [&](int d, float tt, float tp, float no) {
            const float e2e = __fmaf_rn(tp, no, tt);
            const float B = rule.per_cand ? __fmaf_rn(no, rule.tpot_slo, qr.base) : qr.bound.slo;
            const bool feasible = e2e <= B;
            const float Q = sq[s_model[d]];
            float t = 0.0f;
            if (!rule.score_paper) {
                if (rule.per_cand) {
                    asm volatile("");     // a real branch: the division stays off the other paths
                    t = __fdiv_rn(e2e, B);
                } else {
                    t = div_bound(e2e, qr.bound);
                }
            }
            ff = (feasible & (ff < 0)) ? d : ff;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                if (MULTI && k >= nw) break;
                const float w = a.w[k];
                const float u = rule.score_paper ? __fsub_rn(__fmul_rn(__fsub_rn(1.0f, w), Q), __fmul_rn(w, e2e))
                                                 : __fsub_rn(Q, __fmul_rn(w, t));
                LaneBest &b = best[k];
                const bool ta = u > b.ua, tf = feasible & (u > b.uf);
                b.ua = ta ? u : b.ua;
                b.da = ta ? d : b.da;
                b.uf = tf ? u : b.uf;
                b.df = tf ? d : b.df;
            }
            if (DBG && live) {
                const size_t co = static_cast<size_t>(q0 + ql) * N + d;
                if (a.dbg_ttft) a.dbg_ttft[co] = tt;
                if (a.dbg_tpot) a.dbg_tpot[co] = tp;
                if (PN && a.dbg_nout) a.dbg_nout[co] = no;
            }
        };
        // four steps of 16 pairs are loaded before the first is decided
        constexpr int kAhead = 4;
        const int steps = (N + 15) / 16;
        for (int i0 = 0; i0 < steps; i0 += kAhead) {
            f32x4 v[kAhead];
            f32x2 vn[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                // a step past the row's end reads the row's start
                const bool in = 16 * (i0 + i) + 2 * l8 < N;
                const int at = in ? 8 * (i0 + i) : -l8;
                v[i] = row[at];
                if constexpr (PN) vn[i] = rown[at];
            }
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                const int d = 16 * (i0 + i) + 2 * l8;
                if (d < N) take(d, v[i][0], v[i][1], PN ? vn[i][0] : nout);
                if (d + 1 < N) take(d + 1, v[i][2], v[i][3], PN ? vn[i][1] : nout);
            }
        }
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (MULTI && k >= nw) break;
            const uint64_t key = group_max_u64(lane_key(best[k], ff, 2 * l8, N), kRouteLanes);
            if (l8 == 0) s_key[ql * nw + k] = key;
        }
    }
    __syncthreads();
    for (int i = tid; i < nqb * nw; i += kRouteThreads) {
        const int ql = MULTI ? i / nw : i;
        const uint64_t key = s_key[i];
        const int d = key_pair(key);
        const size_t at = static_cast<size_t>(s_row[ql]) * a.ldn + d;
        const f32x2 p = *reinterpret_cast<const f32x2 *>(a.tab + 2 * at);
        const float no = PN ? a.tab_nout[at] : s_nout[ql];
        write_outputs(a.out, q0 * nw + i, key, key_utility(key), __fmaf_rn(p[1], no, p[0]), p[0], p[1], no);
    }
}

template <bool QUAL, bool PN, bool MULTI, bool GEN>
static hipError_t launch_route_t(const RouteArgs &a, bool dbg, hipStream_t s) {
    constexpr int QB = QUAL ? 64 : kRoutePass;
    const dim3 grid(static_cast<unsigned>((a.q.nq + QB - 1) / QB)), block(kRouteThreads);
    return dbg ? launch_kernel(k_route<QUAL, PN, MULTI, GEN, true>, grid, block, 0, s, a)
               : launch_kernel(k_route<QUAL, PN, MULTI, GEN, false>, grid, block, 0, s, a);
}

template <bool QUAL>
static hipError_t launch_route_q(const RouteArgs &a, bool dbg, hipStream_t s) {
    const bool gen = a.rule.score_paper || a.rule.bound_paper;
    const int idx = (a.tab_nout ? 4 : 0) + (a.nw > 1 ? 2 : 0) + (gen ? 1 : 0);
    switch (idx) {
        case 0: return launch_route_t<QUAL, false, false, false>(a, dbg, s);
        case 1: return launch_route_t<QUAL, false, false, true>(a, dbg, s);
        case 2: return launch_route_t<QUAL, false, true, false>(a, dbg, s);
        case 3: return launch_route_t<QUAL, false, true, true>(a, dbg, s);
        case 4: return launch_route_t<QUAL, true, false, false>(a, dbg, s);
        case 5: return launch_route_t<QUAL, true, false, true>(a, dbg, s);
        case 6: return launch_route_t<QUAL, true, true, false>(a, dbg, s);
        default: return launch_route_t<QUAL, true, true, true>(a, dbg, s);
    }
}

hipError_t launch_route(const RouteArgs &a, bool with_quality, hipStream_t s) {
    const bool dbg = a.dbg_ttft || a.dbg_tpot || a.dbg_nout || (with_quality && a.quality.qmat);
    return with_quality ? launch_route_q<true>(a, dbg, s) : launch_route_q<false>(a, dbg, s);
}

}  // namespace hwr
