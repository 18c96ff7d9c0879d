// Predictor table of the fused pipeline (gfx950, bf16).
//
// The predictor's input (Eq. 1) holds the pair's attributes and signals and a
// single query feature, bf16(ln(input_len) / 8).  That feature takes at most a
// few hundred values over every int32 length, so a batch of many queries holds
// the same (feature, pair) inputs again and again.  The table holds the
// predictions of each (row, pair), a row being one feature value, or, for
// batches of fewer queries than feature values, one query; the decision kernel
// (k_route.hip) reads the row of each query.  Each entry is computed exactly as
// a candidate of the staged predictor is: the same bits.  Against the predictor
// on every candidate (same box, whole calls, same outputs bit for bit):
// 1,048,576 x 256, H = 256: 23,250 -> 882 us; 65,536 x 64, H = 256: 386 -> 48 us;
// 4,096 x 16, H = 128: 18.2 -> 10.6 us; 8,192 x 48 with eight cost weights: 132 ->
// 16.8 us.
#include <algorithm>

#include "hwr_mfma.hpp"

namespace hwr {

constexpr int kTableWaves = 8;                    // two per SIMD
constexpr int kTableThreads = 64 * kTableWaves;

// Quality tiles of a workgroup of their own, RT of them (32 queries each): all
// eight waves fetch the rows and the weights of 512 k into LDS, with the next 512
// k already requested, so that one trip to memory covers D <= 1,024; wave i < RT
// multiplies tile i (quality_tile's chain: same bits).  A lone wave per tile
// (quality_tile) waits for memory once per 256 k: the
// call at 4,096 x 16, D = 768 11.15 -> 10.42 us, at 8,192 x 48 15.9 -> 15.2, at 1,003
// x 91 10.87 -> 10.62.  More tiles to a workgroup keep a wave each: their loads
// already overlap, and one or two waves multiplying for all would be the longer
// chain.
constexpr int kCoopK = 512, kCoopRow = 2 * kCoopK + 16;    // 16-byte pad: rows in different banks
constexpr int kCoopTiles = 2;                              // at most: the loads held per thread
constexpr int kCoopBytes = 32 * kCoopTiles * kCoopRow + kCoopK * 64;
template <int RT>
__device__ __forceinline__ void quality_tiles_coop(const QualityArgs &a, int q0, unsigned char *lds) {
    constexpr int T = kTableThreads, PPR = 2 * kCoopK / 16;
    constexpr int NE = 32 * RT * PPR / T, NQ = kCoopK * 4 / T;   // 16-byte pieces per thread: rows, weights
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 31, h = lane >> 5, S = a.D / 64, chunks = (a.D + kCoopK - 1) / kCoopK;
    const uint16_t *emb = static_cast<const uint16_t *>(a.emb);
    const u32x4 *wq = reinterpret_cast<const u32x4 *>(a.wq_pk);
    unsigned char *lds_w = lds + 32 * RT * kCoopRow;
    u32x4 e[NE], w[NQ];
    // past the queries, a row's end or the weights: the last piece, never used
    auto load = [&](int j) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int p = tid + T * i, q = min(q0 + p / PPR, a.nq - 1), k = min(j * kCoopK + p % PPR * 8, a.D - 8);
            e[i] = *reinterpret_cast<const u32x4 *>(emb + static_cast<size_t>(q) * a.D + k);
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) w[i] = wq[min(j * kCoopK * 4 + tid + T * i, a.D * 4 - 1)];
    };
    f32x16 acc = {};
    load(0);
    for (int j = 0; j < chunks; ++j) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int p = tid + T * i;
            *reinterpret_cast<u32x4 *>(lds + p / PPR * kCoopRow + p % PPR * 16) = e[i];
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) *reinterpret_cast<u32x4 *>(lds_w + (tid + T * i) * 16) = w[i];
        if (j + 1 < chunks) load(j + 1);
        __syncthreads();
        if (wave < RT) {
            const unsigned char *base = lds + (32 * wave + row) * kCoopRow + 64 * h;
            const int slices = min(kCoopK / 64, S - j * (kCoopK / 64));
            for (int sl = 0; sl < slices; ++sl)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc = mfma32(*reinterpret_cast<const bf16x8 *>(base + 128 * sl + 16 * c),
                                 *reinterpret_cast<const bf16x8 *>(lds_w + ((sl * 4 + c) * 64 + lane) * 16), acc);
        }
        __syncthreads();
    }
    if (wave < RT && row < a.M) {
        const float bias = a.bq[row];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = q0 + 32 * wave + crow(r, h);
            if (q < a.nq) a.qmat[static_cast<size_t>(q) * a.M + row] = acc[r] + bias;
        }
    }
}

// A wave evaluates 64 consecutive (row, pair) entries per step, two 32-column
// tiles whose columns may lie in any rows: no padding but the last step's.  A
// step's cost is its MFMA chain (H = 256: 288 32x32x16 MFMAs, about 9,300
// cycles for one wave on a SIMD), so the steps are dealt out over the
// workgroups first and over a workgroup's waves last: few steps run one wave
// per SIMD or less.  Workgroups past a.blocks run quality tiles of the batch
// (HBM-bound, and independent of the table) at the same time.
template <int H, int NH, bool FB>
__global__ __launch_bounds__(kTableThreads, 1) void k_table(TableArgs a) {
    constexpr int kLds = sizeof(PredictorLds<H, NH>) > kCoopBytes ? sizeof(PredictorLds<H, NH>) : kCoopBytes;
    __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
    PredictorLds<H, NH> &s = *reinterpret_cast<PredictorLds<H, NH> *>(lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (static_cast<int>(blockIdx.x) >= a.blocks) {
        const int first = (blockIdx.x - a.blocks) * a.qual_waves * 32;
        if (a.qual_waves == 1) return quality_tiles_coop<1>(a.quality, first, lds);
        if (a.qual_waves == kCoopTiles) return quality_tiles_coop<kCoopTiles>(a.quality, first, lds);
        const int q0 = first + wave * 32;
        if (wave < a.qual_waves && q0 < a.quality.nq) quality_tile<4>(a.quality, q0, lane);
        return;
    }
    const int n = lane & 31, h = lane >> 5;
    const int total = a.rows * a.N;
    const int units = (total + 63) / 64;
    const bf16x8 *dep = reinterpret_cast<const bf16x8 *>(a.dep_bf16);
    // the input-length slot: k-block, lane half and element holding it
    const int ls_kb = a.len_slot >> 4, ls_h = (a.len_slot >> 3) & 1, ls_e = a.len_slot & 7;
    const bool patch = (h == ls_h);
    bf16x8 nf[2][2];
    uint32_t nx[2];
    auto load = [&](int unit) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int c = unit * 64 + 32 * t + n;
            const int cc = c < total ? c : 0;
            const int r = cc / a.N, d = cc - r * a.N;
            nf[t][0] = dep[d * 4 + h];
            nf[t][1] = dep[d * 4 + 2 + h];
            nx[t] = a.row_bits ? a.row_bits[r] : bf16_bits(len_feature(a.input_len[r]));
        }
    };
    int unit = wave * a.blocks + blockIdx.x;
    const int step = kTableWaves * a.blocks;
    load(unit < units ? unit : 0);
    stage_predictor<H, NH, kTableThreads>(a.w, s);
    __syncthreads();
    int w3_sel[2];
    head_fragments<NH>(lane, w3_sel);
    for (; unit < units; unit += step) {
        bf16x8 xf[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            xf[t][0] = (patch && ls_kb == 0) ? put_elem(nf[t][0], ls_e, nx[t]) : nf[t][0];
            xf[t][1] = (patch && ls_kb == 1) ? put_elem(nf[t][1], ls_e, nx[t]) : nf[t][1];
        }
        load(unit + step < units ? unit + step : unit);
        int lo = lane, ho = h, w3o0 = w3_sel[0], w3o1 = w3_sel[1];
        asm volatile("" : "+v"(lo), "+v"(ho), "+v"(w3o0), "+v"(w3o1));
        f32x4 z[1];
        predict_two_tiles<H, NH, FB>(s, xf, lo, ho, w3o0, w3o1, z);
        const int c = unit * 64 + lane;            // lane (n, h) completes column n of tile h
        if (c < total) {
            const int r = c / a.N, d = c - r * a.N;
            const size_t at = static_cast<size_t>(r) * a.ldn + d;
            const f32x2 v = {softplus_fast(z[0][0] + a.w.b3_0), softplus_fast(z[0][1] + a.w.b3_1)};
            *reinterpret_cast<f32x2 *>(a.tab + 2 * at) = v;
            if constexpr (NH == 3) a.tab_nout[at] = softplus_fast(z[0][2] + a.w.b3_2);
        }
    }
}

template <int H>
static hipError_t launch_table_h(const TableArgs &a, dim3 grid, hipStream_t s) {
    const dim3 block(kTableThreads);
    if (a.fold_b1)
        return a.nheads == 3 ? launch_kernel(k_table<H, 3, true>, grid, block, 0, s, a)
                             : launch_kernel(k_table<H, 2, true>, grid, block, 0, s, a);
    return a.nheads == 3 ? launch_kernel(k_table<H, 3, false>, grid, block, 0, s, a)
                         : launch_kernel(k_table<H, 2, false>, grid, block, 0, s, a);
}

// One workgroup per compute unit at most (at H = 256 no more fit): the table's
// steps one to a workgroup as far as they go, or half the device when the
// quality tiles want the rest, which take what is left one wave to a workgroup
// as far as that goes.
hipError_t launch_table(int H, const TableArgs &args, int cus, hipStream_t s) {
    TableArgs a = args;
    const int units = (a.rows * a.N + 63) / 64;
    const int tiles = (a.quality.nq + 31) / 32;
    a.blocks = std::min(units, std::max(cus / 2, cus - tiles));
    int qblocks = 0;
    if (tiles > 0) {
        qblocks = std::max(std::min(tiles, cus - a.blocks), (tiles + kTableWaves - 1) / kTableWaves);
        a.qual_waves = (tiles + qblocks - 1) / qblocks;
    }
    const dim3 grid(static_cast<unsigned>(a.blocks + qblocks));
    switch (H) {
        case 64: return launch_table_h<64>(a, grid, s);
        case 128: return launch_table_h<128>(a, grid, s);
        case 256: return launch_table_h<256>(a, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace hwr
