// Decisions of the fused pipeline and of the fp32 path (gfx950): per query, cost (Eq. 2), bound test
// and utility of every pair from the query's row of the predictor table, then
// the Eq. 3 argmax, once per cost weight.
#include <algorithm>

#include "hwr_mfma.hpp"

namespace hwr {

constexpr int kRouteThreads = 256;
constexpr int kRouteLanes = 8;                    // lanes per query in the decision
constexpr int kRoutePass = kRouteThreads / kRouteLanes;   // queries decided at once
constexpr int kQStride = kMaxModels + 1;          // LDS quality row (odd: rows in different banks)

// Utility of a decision key (the inverse of ord_u32).
__device__ __forceinline__ float key_utility(uint64_t k) {
    const uint32_t o = static_cast<uint32_t>(k >> 31);
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

// Outputs of decision key: the chosen pair's predictions are read again.
template <bool PN>
__device__ __forceinline__ void write_decision(const RouteArgs &a, int out, uint64_t key, int row, float nout) {
    const size_t at = static_cast<size_t>(row) * a.ldn + key_pair(key);
    const f32x2 p = *reinterpret_cast<const f32x2 *>(a.tab + 2 * at);
    const float no = PN ? a.tab_nout[at] : nout;
    write_outputs(a.out, out, key, key_utility(key), __fmaf_rn(p[1], no, p[0]), p[0], p[1], no);
}

// The queries' inputs and qualities in LDS, as decide_queries reads them.
struct DecideLds {
    const int *row, *len;         // table row, input length
    const float *nout, *slo;
    const float *q;               // [query][kQStride]
    const uint8_t *model;         // stage_models
    uint64_t *key;                // out: [query][weights]
};

// The pairs' models for decide_queries, as byte offsets into a quality row, up
// to the next multiple of 64 pairs; entries past the last pair are those of the
// pair that decide_queries takes in their place.
__device__ __forceinline__ void stage_models(uint8_t *s_model, const int32_t *dep_model, int N, int tid) {
    for (int i = tid; i < (N + 63) / 64 * 64; i += kRouteThreads) {
        int d = i;
        if (d >= N) d = (d == N && (N & 1)) ? N - 1 : min(d & 15, N - 1);
        s_model[i] = static_cast<uint8_t>(4 * dep_model[d]);
    }
}

// Eight lanes decide each of the queries ql0, ql0 + step, ... (passes of them;
// l8: the lane of the eight): they read the query's table row 128 bytes at a
// time (16 pairs), each lane two pairs of it, in increasing order, and compare
// packed decision keys (unique: they hold the pair index) with DPP steps; lane
// 0 of the eight stores them, one per cost weight.  The loads run one group of
// four steps (64 pairs) ahead, across queries.
//
// Vector instructions bound the decision (about 14 per candidate).  A lane
// keeps one running best, which starts as its first pair at -inf, infeasible; a
// candidate replaces it when it is the first feasible one, or has the same
// feasibility and a strictly larger utility (ties keep the lower pair; a NaN
// utility ranks as -inf).  Feasibility is a wave mask in scalar registers, the
// same for every weight.  Candidates past the last pair repeat one that the
// lane has taken already (its first pair, or the other of the same step), which
// never replaces anything, so none is masked.  The range check of the division
// is made once per eight candidates.  Every lane of the wave takes part.
template <bool PN, bool MULTI, bool GEN, bool DBG>
__device__ __forceinline__ void decide_queries(const RouteArgs &a, const Rule &rule, const DecideLds &s, int q0, int nqb,
                                               int ql0, int step, int passes, int l8) {
    constexpr int NW = MULTI ? kMaxWeights : 1;
    constexpr int kSteps = 4, kCand = 2 * kSteps;
    constexpr float kInf = __builtin_huge_valf();
    const int nw = MULTI ? a.nw : 1, N = a.N;
    const int groups = (N + 16 * kSteps - 1) / (16 * kSteps), total = passes * groups;
    struct Group {
        f32x4 v[kSteps];
        f32x2 n[kSteps];
    };
    int lpass = 0, lgroup = 0;                     // the group to load next
    auto load = [&](Group &g) {
        const size_t base = static_cast<size_t>(s.row[ql0 + lpass * step]) * a.ldn;
        const f32x4 *row = reinterpret_cast<const f32x4 *>(a.tab + 2 * base);
        const f32x2 *rown = PN ? reinterpret_cast<const f32x2 *>(a.tab_nout + base) : nullptr;
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            // past the last pair: the lane's first (none: the row's start)
            int at = 8 * (kSteps * lgroup + i) + l8;
            at = 2 * at < N ? at : 2 * l8 < N ? l8 : 0;
            g.v[i] = row[at];
            if constexpr (PN) g.n[i] = rown[at];
        }
        if (++lgroup == groups) {
            lgroup = 0;
            if (lpass + 1 < passes) ++lpass;       // past the last query: loaded again, unused
        }
    };
    int ql = ql0, group = 0;
    float nout = 0.0f;
    QueryRule qr{};
    float bu[NW];
    int bd[NW];
    uint64_t bf = 0;                               // lanes whose best is feasible
    auto take = [&](Group &g) {
        if (group == 0) {
            nout = s.nout[ql];
            qr = query_rule(rule, s.slo[ql], s.len[ql], nout, a.w[0]);
            bf = 0;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                bu[k] = -kInf;
                bd[k] = 2 * l8;
            }
        }
        const unsigned char *sq = reinterpret_cast<const unsigned char *>(s.q + ql * kQStride);
        const int d0 = 16 * kSteps * group + 2 * l8;
        if (N & 1) {
            // the last pair's neighbour in the row is padding
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                const int at = 2 * (d0 / 2 + 8 * i) < N ? d0 / 2 + 8 * i : l8;
                if (2 * at + 1 == N) {
                    g.v[i][2] = g.v[i][0];
                    g.v[i][3] = g.v[i][1];
                    if constexpr (PN) g.n[i][1] = g.n[i][0];
                }
            }
        }
        float e[kCand], t[kCand], Q[kCand], no[kCand];
#pragma unroll
        for (int i = 0; i < kCand; ++i) {
            no[i] = PN ? g.n[i >> 1][i & 1] : nout;
            e[i] = __fmaf_rn(g.v[i >> 1][2 * (i & 1) + 1], no[i], g.v[i >> 1][2 * (i & 1)]);
            Q[i] = *reinterpret_cast<const float *>(sq + s.model[d0 + 16 * (i >> 1) + (i & 1)]);
        }
        if (!rule.score_paper) {
            if (rule.per_cand) {
                asm volatile("");     // a real branch: the division stays off the other paths
#pragma unroll
                for (int i = 0; i < kCand; ++i) t[i] = __fdiv_rn(e[i], __fmaf_rn(no[i], rule.tpot_slo, qr.base));
            } else {
                float lo = e[0], hi = e[0];        // (a NaN leaves both as they are, and either division gives NaN)
#pragma unroll
                for (int i = 0; i < kCand; ++i) {
                    lo = fminf(lo, e[i]);
                    hi = fmaxf(hi, e[i]);
                    t[i] = div_bound_fast(e[i], qr.bound);
                }
                if (!div_in_range(lo, hi, qr.bound)) {
                    asm volatile("");
#pragma unroll
                    for (int i = 0; i < kCand; ++i) t[i] = __fdiv_rn(e[i], qr.bound.slo);
                }
            }
        }
        int bi[NW];                                // the group's last replacement
#pragma unroll
        for (int k = 0; k < NW; ++k) bi[k] = -1;
#pragma unroll
        for (int i = 0; i < kCand; ++i) {
            const int di = 16 * (i >> 1) + (i & 1);
            const float B = rule.per_cand ? __fmaf_rn(no[i], rule.tpot_slo, qr.base) : qr.bound.slo;
            const uint64_t feasible = __builtin_amdgcn_ballot_w64(e[i] <= B);
            const uint64_t first = feasible & ~bf, same = ~(feasible ^ bf);
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                if (MULTI && k >= nw) break;
                const float w = a.w[k];
                const float u = rule.score_paper ? __fsub_rn(__fmul_rn(__fsub_rn(1.0f, w), Q[i]), __fmul_rn(w, e[i]))
                                                 : __fsub_rn(Q[i], __fmul_rn(w, t[i]));
                const uint64_t m = first | (same & __builtin_amdgcn_ballot_w64(u > bu[k]));
                const bool r = __builtin_amdgcn_inverse_ballot_w64(m);
                bu[k] = r ? fmaxf(u, -kInf) : bu[k];
                bi[k] = r ? di : bi[k];
            }
            bf |= feasible;
            if (DBG && d0 + di < N && ql < nqb) {
                const size_t co = static_cast<size_t>(q0 + ql) * N + d0 + di;
                if (a.dbg_ttft) a.dbg_ttft[co] = g.v[i >> 1][2 * (i & 1)];
                if (a.dbg_tpot) a.dbg_tpot[co] = g.v[i >> 1][2 * (i & 1) + 1];
                if (PN && a.dbg_nout) a.dbg_nout[co] = no[i];
            }
        }
#pragma unroll
        for (int k = 0; k < NW; ++k) bd[k] = bi[k] >= 0 ? d0 + bi[k] : bd[k];
        if (++group == groups) {
            const bool f = __builtin_amdgcn_inverse_ballot_w64(bf);
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                if (MULTI && k >= nw) break;
                const uint64_t key = group_max_u64(2 * l8 < N ? decision_key(f, bu[k], bd[k]) : 0, kRouteLanes);
                if (l8 == 0) s.key[ql * nw + k] = key;
            }
            group = 0;
            ql += step;
        }
    };
    Group g0, g1;
    load(g0);
#pragma unroll 1
    for (int it = 0; it < total; it += 2) {
        load(g1);
        take(g0);
        if (it + 1 == total) break;
        load(g0);
        take(g1);
    }
}

// Decisions of 32 queries from their qualities (a.quality.qmat).
// PN: N_out predicted per candidate; GEN: the paper's score or bound; DBG:
// per-candidate outputs.
template <bool PN, bool MULTI, bool GEN, bool DBG>
__global__ __launch_bounds__(kRouteThreads) void k_route(RouteArgs a) {
    constexpr int QB = kRoutePass;                // queries per workgroup
    constexpr int NW = MULTI ? kMaxWeights : 1;
    __shared__ float s_q[QB * kQStride];
    __shared__ uint8_t s_model[kMaxPairs];
    __shared__ int s_row[QB], s_len[QB];
    __shared__ float s_nout[QB], s_slo[QB];
    __shared__ uint64_t s_key[QB * NW];
    Rule rule = a.rule;
    if constexpr (!GEN) rule = Rule{};
    const int tid = threadIdx.x;
    const int nq = a.q.nq, M = a.M, nw = MULTI ? a.nw : 1;
    const int q0 = blockIdx.x * QB;
    const int nqb = min(QB, nq - q0);
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
    stage_models(s_model, a.dep_model, a.N, tid);
    for (int i = tid; i < nqb * M; i += kRouteThreads) {
        const int r = i / M, m = i - r * M;
        s_q[r * kQStride + m] = a.quality.qmat[static_cast<size_t>(q0) * M + i];
    }
    __syncthreads();
    // queries past nqb repeat the last: never written
    decide_queries<PN, MULTI, GEN, DBG>(a, rule, DecideLds{s_row, s_len, s_nout, s_slo, s_q, s_model, s_key}, q0, nqb,
                                        tid / kRouteLanes, kRoutePass, 1, tid & (kRouteLanes - 1));
    __syncthreads();
    for (int i = tid; i < nqb * nw; i += kRouteThreads)
        write_decision<PN>(a, q0 * nw + i, s_key[i], s_row[MULTI ? i / nw : i], s_nout[MULTI ? i / nw : i]);
}

// LDS of one wave of k_route_stream: the stage being multiplied (128 k of its 32
// queries) and, once the qualities are done, the qualities; then the queries'
// inputs and decision keys.
constexpr int kStreamSlices = 2;                  // 64-wide slices of k per stage
constexpr int kStreamRow = kStreamSlices * 128 + 16;   // bytes of a stage's row (16-byte pad: rows in different banks)
template <int NW>
struct StreamLds {
    union {
        unsigned char stage[32 * kStreamRow];
        float q[32 * kQStride];
    };
    uint64_t key[32 * NW];
    int row[32], len[32];
    float nout[32], slo[32];
};

// Orders a wave's LDS accesses for the compiler (the hardware keeps them in
// order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kStreamWaves = kRouteThreads / 64;
constexpr int kStreamBlocks = 3;                  // workgroups per compute unit

// Qualities and decisions of a large batch.  Every wave takes 32 queries at a time
// by itself, no workgroup barrier: it streams their embeddings through its own LDS
// in stages of 128 k (the next stage's loads in registers), multiplies them as
// quality_tile does (same bits), and decides them while the other waves of its
// SIMD keep loads in flight (at 256 compute units a SIMD has one wave up to 32,768
// queries and three from 98,304 on).  The quality weights come from L2 one stage
// ahead too: loads return in order, so weights requested behind the next stage's
// embeddings would wait for memory.
//
// Bound by HBM with the decisions' vector instructions beside it, and by the
// weights' way from L2, which every wave asks for again (2.9 GB at 1M x 256 beside
// 3.2 GB of embeddings).  Calls at 1,048,576 x 256, D = 1,536 (3.25 GB, table
// included): 704 us; without the decisions 602, the decisions alone about 200.
// Workgroups of four waves on 64 queries in 65,536-query launches, with barriers
// per 256 k, took 884 us (712 in one launch with the present decisions); at 65,536
// x 64, D = 1,024, 38 against 46 us.  Other shapes, in us for 1M x 256: stages of
// 64 k with two ahead 739, of 256 k at two waves per SIMD 706, four waves per SIMD
// 739; the next tile's first stage requested before the decisions: no gain.
// Non-temporal embedding loads (each byte is read once, and the table stays in L2)
// took 65,536 x 64 from 43.9 to 39.4 us.
template <bool PN, bool MULTI, bool GEN, bool DBG>
__global__ __launch_bounds__(kRouteThreads, kStreamBlocks) void k_route_stream(RouteArgs a) {
    constexpr int NW = MULTI ? kMaxWeights : 1;
    constexpr int KS = kStreamSlices;
    __shared__ __attribute__((aligned(16))) StreamLds<NW> s_wave[kStreamWaves];
    __shared__ uint8_t s_model[kMaxPairs];
    Rule rule = a.rule;
    if constexpr (!GEN) rule = Rule{};
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const QualityArgs &qa = a.quality;
    const int nq = a.q.nq, M = a.M, nw = MULTI ? a.nw : 1;
    StreamLds<NW> &s = s_wave[wave];
    stage_models(s_model, a.dep_model, a.N, tid);
    __syncthreads();
    const int n = lane & 31, h = lane >> 5, l8 = lane & (kRouteLanes - 1);
    // columns past the models repeat the first one's weights (never used)
    const bf16x8 *wq = reinterpret_cast<const bf16x8 *>(qa.wq_pk) + (n < M ? lane : 32 * h);
    const int S = qa.D / 64;
    // 16-byte pieces of a stage: lane l takes rows l / PPR + RPL i, piece l % PPR
    constexpr int PPR = 8 * KS, RPL = 64 / PPR, NL = 4 * KS;
    const int prow = lane / PPR, pcol = lane % PPR;
    const uint32_t rb = static_cast<uint32_t>(qa.D) * 2;
    const int T = (S + KS - 1) / KS;
    const int tiles = (nq + 31) / 32, stride = static_cast<int>(gridDim.x) * kStreamWaves;
#pragma unroll 1
    for (int tile = static_cast<int>(blockIdx.x) * kStreamWaves + wave; tile < tiles; tile += stride) {
        const int q0 = tile * 32, nqb = min(32, nq - q0);
        const unsigned char *emb = static_cast<const unsigned char *>(qa.emb) + static_cast<size_t>(q0) * rb;
        uint32_t off[NL];                          // rows past the queries repeat the last one
#pragma unroll
        for (int i = 0; i < NL; ++i) off[i] = static_cast<uint32_t>(min(prow + RPL * i, nqb - 1)) * rb;
        u32x4 e[NL];
        bf16x8 w[NL];
        auto load_e = [&](int st) {
            // past the row's end (an odd number of slices): its last piece, never used
            const uint32_t col = min(static_cast<uint32_t>(st * PPR + pcol) * 16, rb - 16);
#pragma unroll
            for (int i = 0; i < NL; ++i)
                e[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(emb + (off[i] + col)));
        };
        auto load_w = [&](int st) {
#pragma unroll
            for (int c = 0; c < NL; ++c) w[c] = wq[min(st * NL + c, 4 * S - 1) * 64];
        };
        const int qi = q0 + min(n, nqb - 1);
        const int32_t len = a.q.input_len[qi];
        const int32_t no = PN ? 0 : a.q.nout[qi];
        const float slo = a.q.slo ? a.q.slo[qi] : a.q.default_slo;
        load_e(0);
        load_w(0);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc = {};
#pragma unroll 1
        for (int st = 0; st < T; ++st) {
#pragma unroll
            for (int i = 0; i < NL; ++i)
                *reinterpret_cast<u32x4 *>(s.stage + (prow + RPL * i) * kStreamRow + 16 * pcol) = e[i];
            if (st + 1 < T) load_e(st + 1);
            wave_sync();
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                if (k == 0 || st * KS + k < S) {
                    bf16x8 av[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        av[c] = *reinterpret_cast<const bf16x8 *>(s.stage + n * kStreamRow + 128 * k + 64 * h + 16 * c);
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc = mfma32(av[c], w[4 * k + c], acc);
                }
            }
            if (st + 1 < T) load_w(st + 1);
            wave_sync();
            __builtin_amdgcn_sched_barrier(0);
        }
        if (n < M) {
            const float bias = qa.bq[n];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int ql = crow(r, h);
                s.q[ql * kQStride + n] = acc[r] + bias;
                if (DBG && qa.qmat && ql < nqb) qa.qmat[static_cast<size_t>(q0 + ql) * M + n] = acc[r] + bias;
            }
        }
        if (lane < 32) {
            s.len[n] = len;
            s.nout[n] = static_cast<float>(no < 0 ? 0 : no);
            s.slo[n] = slo;
            s.row[n] = a.len_row[len_index(bf16_bits(len_feature(len)))];
        }
        wave_sync();
        decide_queries<PN, MULTI, GEN, DBG>(a, rule, DecideLds{s.row, s.len, s.nout, s.slo, s.q, s_model, s.key}, q0, nqb,
                                            lane / kRouteLanes, 64 / kRouteLanes, 32 * kRouteLanes / 64, l8);
        wave_sync();
        for (int i = lane; i < nqb * nw; i += 64)
            write_decision<PN>(a, q0 * nw + i, s.key[i], s.row[MULTI ? i / nw : i], s.nout[MULTI ? i / nw : i]);
        wave_sync();                               // the next tile reuses the wave's LDS
    }
}

template <bool PN, bool MULTI, bool GEN>
static hipError_t launch_route_t(const RouteArgs &a, bool with_quality, bool dbg, int cus, hipStream_t s) {
    const dim3 block(kRouteThreads);
    if (with_quality) {
        const int blocks = ((a.q.nq + 31) / 32 + kStreamWaves - 1) / kStreamWaves;
        const dim3 grid(static_cast<unsigned>(std::min(blocks, cus * kStreamBlocks)));
        return dbg ? launch_kernel(k_route_stream<PN, MULTI, GEN, true>, grid, block, 0, s, a)
                   : launch_kernel(k_route_stream<PN, MULTI, GEN, false>, grid, block, 0, s, a);
    }
    const dim3 grid(static_cast<unsigned>((a.q.nq + kRoutePass - 1) / kRoutePass));
    return dbg ? launch_kernel(k_route<PN, MULTI, GEN, true>, grid, block, 0, s, a)
               : launch_kernel(k_route<PN, MULTI, GEN, false>, grid, block, 0, s, a);
}

hipError_t launch_route(const RouteArgs &a, bool with_quality, int cus, hipStream_t s) {
    const bool dbg = a.dbg_ttft || a.dbg_tpot || a.dbg_nout || (with_quality && a.quality.qmat);
    const bool gen = a.rule.score_paper || a.rule.bound_paper;
    const int idx = (a.tab_nout ? 4 : 0) + (a.nw > 1 ? 2 : 0) + (gen ? 1 : 0);
    switch (idx) {
        case 0: return launch_route_t<false, false, false>(a, with_quality, dbg, cus, s);
        case 1: return launch_route_t<false, false, true>(a, with_quality, dbg, cus, s);
        case 2: return launch_route_t<false, true, false>(a, with_quality, dbg, cus, s);
        case 3: return launch_route_t<false, true, true>(a, with_quality, dbg, cus, s);
        case 4: return launch_route_t<true, false, false>(a, with_quality, dbg, cus, s);
        case 5: return launch_route_t<true, false, true>(a, with_quality, dbg, cus, s);
        case 6: return launch_route_t<true, true, false>(a, with_quality, dbg, cus, s);
        default: return launch_route_t<true, true, true>(a, with_quality, dbg, cus, s);
    }
}

}  // namespace hwr
