// fp32 quality and predictor of libhwr (gfx950), on fp32 MFMA.
//
// v_mfma_f32_16x16x4_f32: A is 16 rows x 4 k, B is 4 k x 16 columns; lane l
// holds one value, row (A) / column (B) l & 15 of k-group g = l >> 4.  The
// accumulator holds column l & 15, rows 4 g + 0..3.  Products and sums are fp32.
// Every accumulator takes its k-steps in one fixed order in every form of these
// kernels, so chunking and launch shape never change a result.
#include <algorithm>

#include "hwr_device.hpp"

namespace hwr {

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// four floats of a caller's buffer: 4-byte alignment is all it promises
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// ------------------------------------------------------------ quality
// Hardware-independent quality (Sec. 3.2 item 3): Q[q][m] = e_q . Wq[:, m] + bq[m].
// A workgroup's first four waves take 16 queries x 32 (padded) models; wave w
// the 64-wide slices w, w + 4, ... of the embedding.  Lane group g reads 16
// consecutive floats of its row per slice (a slice of a row is 256 contiguous
// bytes) as the A operands of 16 k-steps, Wq is packed so that a lane's four B
// operands are one 16-byte load.  Every k-step of a slice has its own
// accumulator, added in a tree at the end, and the four waves' sums are added
// pairwise through LDS: chains of D / 64 products, which round no more than a
// lane's chain and a sum over 64 lanes.
// 8,192 x 384, 8 models: 48 us (one wave per query, lanes over k, a DPP sum per
// model) -> 4.5 us.
constexpr int kQualF32Q = 16;                     // queries per workgroup
struct QualF32Lds {
    f32x4 part[4][2][64];
};

template <int NT>                                 // 16-model column tiles
__device__ __forceinline__ void quality_f32_tiles(const QualityArgs &a, int q0, int wave, int lane, QualF32Lds &s) {
    const int n = lane & 15, g = lane >> 4;
    if (wave < 4) {
        const int q = q0 + n < a.nq ? q0 + n : a.nq - 1;
        const float *e = static_cast<const float *>(a.emb) + static_cast<size_t>(q) * a.D + 16 * g;
        const f32x4 *wq = reinterpret_cast<const f32x4 *>(a.wq) + lane;
        f32x4 acc[NT][16] = {};
        for (int sl = wave; sl < a.D / 64; sl += 4) {
            f32x4 av[4], bv[NT][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                av[j] = *reinterpret_cast<const f32x4_any *>(e + 64 * sl + 4 * j);
#pragma unroll
                for (int t = 0; t < NT; ++t) bv[t][j] = wq[((sl * 4 + j) * 2 + t) * 64];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t][4 * j + i] = mfma_f32(av[j][i], bv[t][j][i], acc[t][4 * j + i]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int w = 8; w >= 1; w /= 2)
#pragma unroll
                for (int i = 0; i < w; ++i) acc[t][i] += acc[t][i + w];
            s.part[wave][t][lane] = acc[t][0];
        }
    }
    __syncthreads();
    if (wave < NT) {
        const int m = 16 * wave + n;
        const f32x4 v = (s.part[0][wave][lane] + s.part[1][wave][lane]) + (s.part[2][wave][lane] + s.part[3][wave][lane]);
        if (m < a.M) {
            const float bias = a.bq[m];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = q0 + 4 * g + i;
                if (q < a.nq) a.qmat[static_cast<size_t>(q) * a.M + m] = v[i] + bias;
            }
        }
    }
}

__device__ __forceinline__ void quality_f32(const QualityArgs &a, int q0, int wave, int lane, QualF32Lds &s) {
    if (a.M <= 16) quality_f32_tiles<1>(a, q0, wave, lane, s);
    else quality_f32_tiles<2>(a, q0, wave, lane, s);
}

// With `owner`, each query also claims its length (< kOwnLens): whichever of
// the chunk's queries of that length is stored last owns it.  Many workgroups
// store to one entry: whole-word (atomic) stores, any of which will do, read by
// later kernels only.  That they all read the same one is the kernel boundary's
// doing: at this kernel's end the L2 of every XCD has written its words back, one
// of them last, and at the next one's start no L2 holds an older copy.  So the
// stores need no scope beyond the workgroup's; at agent scope they write through
// to memory, where the few lines of the common lengths queue up (8,192 queries:
// 44.9 us a call against 36.0).  No entry is cleared: a length the chunk holds has
// been written by it.
__global__ __launch_bounds__(256) void k_quality_f32(QualityArgs a, const int32_t *input_len, int32_t *owner) {
    __shared__ QualF32Lds s;
    const int q0 = blockIdx.x * kQualF32Q;
    const int q = q0 + static_cast<int>(threadIdx.x);
    if (owner && threadIdx.x < kQualF32Q && q < a.nq) {
        const uint32_t len = static_cast<uint32_t>(input_len[q]);
        if (len < static_cast<uint32_t>(kOwnLens))
            __hip_atomic_store(owner + len, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    quality_f32(a, q0, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63, s);
}

hipError_t launch_quality_f32(const QualityArgs &a, const int32_t *input_len, int32_t *owner, hipStream_t s) {
    return launch_kernel(k_quality_f32, dim3((a.nq + kQualF32Q - 1) / kQualF32Q), dim3(256), 0, s, a, input_len, owner);
}

// ------------------------------------------------------------ predictor
// Eq. 1 predictor in fp32, computed transposed (h^T = W^T x^T): rows are hidden
// units, columns candidates.  An accumulator tile (16 units) leaves lane group
// g with units 4 g + 0..3 of its candidate; k-step (t, i) of the next layer
// takes register i of tile t as its B operand, units 16 t + 4 g + i over the
// groups, so activations pass from layer to layer in registers and the packed
// W2 (A operands, four k-steps to a 16-byte LDS read) has its k in that order.
// A second-layer accumulator is two chains, the even and the odd k tiles.  The
// heads are fused multiply-adds per row tile, the tiles' parts added pairwise,
// then the four groups' by two lane exchanges.
template <int H>
struct F32Weights {
    static constexpr int RT = H / 16;             // row tiles
    f32x4 w1[RT * 2 * 64];                        // [tile][k-steps / 4][lane]
    f32x4 w2[RT * RT * 64];                       // [tile][k tile][lane]
    f32x4 w3[RT * kMaxHeads * 4];                 // [tile][head][group]
    f32x4 b1[RT * 4], b2[RT * 4];                 // [tile][group]
};

template <int H, int T>
__device__ __forceinline__ void stage_f32(const F32Predictor &p, F32Weights<H> &s) {
    constexpr int RT = H / 16, n1 = RT * 2 * 64, n2 = RT * RT * 64, n3 = RT * kMaxHeads * 4, nb = RT * 4;
    const f32x4 *g = reinterpret_cast<const f32x4 *>(p.packed);   // w1, w2, w3, b1, b2 as in F32Weights
    f32x4 *d = reinterpret_cast<f32x4 *>(&s);
    constexpr int total = n1 + n2 + n3 + 2 * nb;
    static_assert(sizeof(F32Weights<H>) == total * 16, "packed layout");
    constexpr int kRound = 8;
#pragma unroll
    for (int r = 0; r < (total + T * kRound - 1) / (T * kRound); ++r) {
        f32x4 v[kRound];
#pragma unroll
        for (int i = 0; i < kRound; ++i) {
            const int k = threadIdx.x + (r * kRound + i) * T;
            v[i] = g[k < total ? k : 0];
        }
#pragma unroll
        for (int i = 0; i < kRound; ++i) {
            const int k = threadIdx.x + (r * kRound + i) * T;
            if (k < total) d[k] = v[i];
        }
    }
}

// The candidate features of one lane: k-steps s = 0 .. 4 kq - 1 take feature
// 4 kq g + s of its candidate (kq = 1: the slots past 15 are zero and their
// weights finite).
struct F32Features {
    f32x4 x[2];
};
template <int KQ>
__device__ __forceinline__ F32Features features_f32(const MlpF32Args &a, int q, int d, int g) {
    F32Features f;
    const float xl = len_feature(a.q.input_len[q]);
    const f32x4 *row = reinterpret_cast<const f32x4 *>(a.dep_f32 + static_cast<size_t>(d) * kFeatPad) + KQ * g;
    f.x[0] = row[0];
    f.x[1] = KQ == 2 ? row[1] : f32x4{};
    const int e = a.len_slot - 4 * KQ * g;       // the query's slot, when this lane holds it
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f.x[0][i] = e == i ? xl : f.x[0][i];
        f.x[1][i] = e == 4 + i ? xl : f.x[1][i];
    }
    return f;
}

template <int H, int KQ>
__device__ __forceinline__ f32x4 layer1_tile(const F32Weights<H> &s, int rt, int lane, const F32Features &f) {
    f32x4 c = s.b1[rt * 4 + (lane >> 4)];
    const f32x4 w = s.w1[(rt * 2 + 0) * 64 + lane];
#pragma unroll
    for (int i = 0; i < 4; ++i) c = mfma_f32(w[i], f.x[0][i], c);
    if constexpr (KQ == 2) {
        const f32x4 v = s.w1[(rt * 2 + 1) * 64 + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) c = mfma_f32(v[i], f.x[1][i], c);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = fmaxf(c[i], 0.0f);
    return c;
}

template <int H>
__device__ __forceinline__ float head_part(const F32Weights<H> &s, int rt, int m, int g, const f32x4 &h2) {
    const f32x4 w = s.w3[(rt * kMaxHeads + m) * 4 + g];
    float p = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) p = fmaf(w[i], fmaxf(h2[i], 0.0f), p);
    return p;
}

// Sum of a power of two of values, pairwise.
template <int N>
__device__ __forceinline__ float tree_sum(float (&v)[N]) {
#pragma unroll
    for (int w = N / 2; w >= 1; w /= 2)
#pragma unroll
        for (int i = 0; i < w; ++i) v[i] += v[i + w];
    return v[0];
}

// Head sums of the four lane groups, then softplus: every lane of the
// candidate gets its values.
__device__ __forceinline__ float head_value(float z, float b3) {
    z += __shfl_xor(z, 16);
    z += __shfl_xor(z, 32);
    return softplus_f32(z + b3);
}

__device__ __forceinline__ void write_f32(const MlpF32Args &a, int q, int d, const float (&z)[kMaxHeads], bool live) {
    const float tt = head_value(z[0], a.p.b3_0), tp = head_value(z[1], a.p.b3_1);
    const float nc = a.nheads == 3 ? head_value(z[2], a.p.b3_2) : 0.0f;
    if (!live) return;
    const size_t at = static_cast<size_t>(q) * a.ldn + d;
    *reinterpret_cast<f32x2 *>(a.tab + 2 * at) = (f32x2){tt, tp};
    if (a.nheads == 3) a.tab_nout[at] = nc;
}

// Small batches: the four waves of a workgroup share 16 candidates, wave w
// computing row tiles w, w + 4, ... (a candidate's chain of MFMAs is the call's
// latency, and there are more SIMDs than candidate tiles).  Activations and
// head parts cross through LDS.  Workgroups past mlp_blocks run the chunk's
// quality, at the same time.
template <int H, int KQ>
__global__ __launch_bounds__(256) void k_mlp_f32_small(MlpF32Args a) {
    constexpr int RT = H / 16;
    __shared__ union {
        F32Weights<H> w;
        QualF32Lds q;
    } s;
    __shared__ f32x4 s_h1[RT * 64];
    __shared__ float s_z[RT * kMaxHeads * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (static_cast<int>(blockIdx.x) >= a.mlp_blocks) {
        quality_f32(a.quality, (blockIdx.x - a.mlp_blocks) * kQualF32Q, wave, lane, s.q);
        return;
    }
    const int n = lane & 15, g = lane >> 4;
    const int total = a.q.nq * a.N;
    const int c = blockIdx.x * 16 + n;
    const int cc = c < total ? c : 0;
    const int q = cc / a.N, d = cc - q * a.N;
    const F32Features f = features_f32<KQ>(a, q, d, g);
    stage_f32<H, 256>(a.p, s.w);
    __syncthreads();
#pragma unroll
    for (int rt = wave; rt < RT; rt += 4) s_h1[rt * 64 + lane] = layer1_tile<H, KQ>(s.w, rt, lane, f);
    __syncthreads();
    f32x4 h1[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) h1[t] = s_h1[t * 64 + lane];
#pragma unroll
    for (int rt = wave; rt < RT; rt += 4) {
        f32x4 c[2] = {s.w.b2[rt * 4 + g], f32x4{}};
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const f32x4 w = s.w.w2[(rt * RT + t) * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) c[t & 1] = mfma_f32(w[i], h1[t][i], c[t & 1]);
        }
        const f32x4 acc = c[0] + c[1];
#pragma unroll
        for (int m = 0; m < kMaxHeads; ++m)
            if (m < a.nheads) s_z[(m * RT + rt) * 64 + lane] = head_part<H>(s.w, rt, m, g, acc);
    }
    __syncthreads();
    if (wave == 0) {
        float z[kMaxHeads] = {};
#pragma unroll
        for (int m = 0; m < kMaxHeads; ++m)
            if (m < a.nheads) {
                float part[RT];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) part[rt] = s_z[(m * RT + rt) * 64 + lane];
                z[m] = tree_sum(part);
            }
        write_f32(a, q, d, z, c < total && g == 0);
    }
}

// Larger batches.  The prediction of a pair depends on the query by its length
// alone, so only the queries that own their length (k_quality_f32) are
// evaluated, and every other query reads its owner's row.  A workgroup lists
// the owners among up to kF32List queries; the workgroups of one range (grid y)
// share its (owner, pair) candidates, 32 at a time to a wave, in two 16-column
// tiles.  Two column tiles x two k halves give four independent MFMA chains.
// 8,192 x 24, H = 128 (1,933 lengths): 597 us (one wave per candidate, hidden
// units broadcast with readlane) -> 26.5 us, two steps of 576 MFMAs per SIMD.
// Nothing evens out the owners per range: 99 to 144 at 8,192 queries, 4 to 201,
// 30 on average, at 65,536 (3,877 lengths, two workgroups to a range), where the
// fullest range sets the time.
constexpr int kF32Waves = 8;
constexpr int kF32List = 512;                     // queries looked through at once
template <int H, int KQ>
__global__ __launch_bounds__(64 * kF32Waves) void k_mlp_f32(MlpF32Args a) {
    constexpr int RT = H / 16, T = 64 * kF32Waves;
    static_assert(kF32List == T, "one listed query per thread");
    __shared__ F32Weights<H> s;
    __shared__ int s_list[kF32List];
    __shared__ int s_owns[kF32Waves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int own = blockIdx.x * kF32List + tid;
    bool owns = false;
    if (own < a.q.nq) {
        const uint32_t len = static_cast<uint32_t>(a.q.input_len[own]);
        owns = len >= static_cast<uint32_t>(kOwnLens) || a.owner[len] == own;
    }
    const uint64_t mask = __ballot(owns);
    if (lane == 0) s_owns[wave] = static_cast<int>(__popcll(mask));
    stage_f32<H, T>(a.p, s);
    __syncthreads();
    // in query order: every workgroup of the range makes the same list
    int at = __popcll(mask & ((uint64_t{1} << lane) - 1)), count = 0;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
        at += w < wave ? s_owns[w] : 0;
        count += s_owns[w];
    }
    if (owns) s_list[at] = own;
    __syncthreads();
    const int total = count * a.N;
    for (int u = wave * gridDim.y + blockIdx.y; u * 32 < total; u += kF32Waves * gridDim.y) {
        int lo = lane;
        asm volatile("" : "+v"(lo));              // weight fragments are read per step, not held
        int q[2], d[2];
        bool live[2];
        f32x4 h1[2][RT];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int c = u * 32 + 16 * t + n;
            live[t] = c < total;
            const int cc = live[t] ? c : 0;
            q[t] = s_list[cc / a.N];
            d[t] = cc % a.N;
        }
        const F32Features f[2] = {features_f32<KQ>(a, q[0], d[0], g), features_f32<KQ>(a, q[1], d[1], g)};
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int t = 0; t < 2; ++t) h1[t][rt] = layer1_tile<H, KQ>(s, rt, lo, f[t]);
        float part[2][kMaxHeads][RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            f32x4 c[2][2];                        // [column tile][k tiles' parity]
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                c[t][0] = s.b2[rt * 4 + g];
                c[t][1] = f32x4{};
            }
#pragma unroll
            for (int k = 0; k < RT; k += 2) {
                const f32x4 w[2] = {s.w2[(rt * RT + k) * 64 + lo], s.w2[(rt * RT + k + 1) * 64 + lo]};
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int t = 0; t < 2; ++t) c[t][b] = mfma_f32(w[b][i], h1[t][k + b][i], c[t][b]);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int m = 0; m < kMaxHeads; ++m)
                    if (m < a.nheads) part[t][m][rt] = head_part<H>(s, rt, m, g, c[t][0] + c[t][1]);
        }
        float z[2][kMaxHeads] = {};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int m = 0; m < kMaxHeads; ++m)
                if (m < a.nheads) z[t][m] = tree_sum(part[t][m]);
#pragma unroll
        for (int t = 0; t < 2; ++t) write_f32(a, q[t], d[t], z[t], live[t] && g == 0);
    }
}

int mlp_f32_small_blocks(int nq, int N) { return static_cast<int>((static_cast<long>(nq) * N + 15) / 16); }
int quality_f32_blocks(int nq) { return (nq + kQualF32Q - 1) / kQualF32Q; }

hipError_t launch_mlp_f32_small(int H, const MlpF32Args &args, hipStream_t s) {
    MlpF32Args a = args;
    a.mlp_blocks = mlp_f32_small_blocks(a.q.nq, a.N);
    const dim3 grid(static_cast<unsigned>(a.mlp_blocks + quality_f32_blocks(a.q.nq)));
    const dim3 block(256);
    if (H == 64)
        return a.kq == 1 ? launch_kernel(k_mlp_f32_small<64, 1>, grid, block, 0, s, a)
                         : launch_kernel(k_mlp_f32_small<64, 2>, grid, block, 0, s, a);
    if (H == 128)
        return a.kq == 1 ? launch_kernel(k_mlp_f32_small<128, 1>, grid, block, 0, s, a)
                         : launch_kernel(k_mlp_f32_small<128, 2>, grid, block, 0, s, a);
    return hipErrorInvalidValue;
}

// A workgroup per compute unit (H = 128: no second one fits its LDS), several to
// a range of queries where there are fewer ranges.
hipError_t launch_mlp_f32(int H, const MlpF32Args &a, int cus, hipStream_t s) {
    const int ranges = (a.q.nq + kF32List - 1) / kF32List;
    const dim3 grid(static_cast<unsigned>(ranges), static_cast<unsigned>(std::max(1, cus / ranges)));
    const dim3 block(64 * kF32Waves);
    if (H == 64)
        return a.kq == 1 ? launch_kernel(k_mlp_f32<64, 1>, grid, block, 0, s, a)
                         : launch_kernel(k_mlp_f32<64, 2>, grid, block, 0, s, a);
    if (H == 128)
        return a.kq == 1 ? launch_kernel(k_mlp_f32<128, 1>, grid, block, 0, s, a)
                         : launch_kernel(k_mlp_f32<128, 2>, grid, block, 0, s, a);
    return hipErrorInvalidValue;
}

}  // namespace hwr
