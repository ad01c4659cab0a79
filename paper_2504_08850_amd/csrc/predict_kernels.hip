// Fused per-layer predictor kernel (paper Sec. 4.3.1 features + Sec. 4.3.2
// judgment): one workgroup scores one (layer, token) pair.
//
// Why one workgroup per token: a call moves (K+2) rows of d halves plus ~13 KB
// of predictor weights -- far below the bandwidth-delay product of the memory
// system -- so what matters is the number of dependent memory round trips, not
// bytes per second.  Everything that does not depend on the speculative ids
// (hidden state, RMSNorm weight, the thread's MLP row) is requested first, the
// K LM-head rows follow as soon as the ids arrive, and because the RMSNorm
// scale is a scalar factor of every logit, sum(h^2) and the K dot products run
// in the same pass: the kernel makes exactly two dependent trips to memory.
// All loads are 16 bytes per lane; reductions are DPP within a wavefront and a
// fixed-order LDS exchange across the eight wavefronts.
#include <algorithm>

#include "device_utils.h"
#include "kernels.h"
#include "merge_block.h"
#include "predictor_tail.h"
#include "tree_finish.h"

namespace specee {

constexpr int kPredictThreads = 512;

// The merge of one tree's ids, by a workgroup of its own of the launch that scores the trees' nodes (TREE below):
// the nodes read their rows by id and need nothing of it, so it is off their path.
template <int T>
__device__ __forceinline__ void merge_one_tree(const TreeMergeParams &m, int g) {
    extern __shared__ __attribute__((aligned(16))) int32_t tree_merge_lds[];
    int32_t *uniq;
    int col_of[kMergePerThread];
    const int M = merge_block<T>(m.ids + (size_t)g * m.n, m.n, tree_merge_lds, uniq, col_of);
    if (threadIdx.x == 0) m.M_out[g] = M;
    for (int i = threadIdx.x; i < m.Mcap; i += T) m.merged[(size_t)g * m.Mcap + i] = i < M ? uniq[i] : -1;
#pragma unroll
    for (int e = 0; e < kMergePerThread; ++e) {
        const int i = threadIdx.x + e * T;
        if (i < m.n) m.cols[(size_t)g * m.n + i] = col_of[e];
    }
}

// Workgroups are dealt to the eight XCDs in turn, by their number in the launch.  The nodes of a launch of trees are
// numbered so that each XCD gets one consecutive eighth of them: the nodes of a tree then share an L2, and a row that
// several of them name is fetched into it once, instead of into up to eight of them (64 nodes, d = 4096, K = 4: 32 trees
// 14.6 -> 12.2 us, 64 24.8 -> 21.8; K = 8, d = 8192, 64 trees 59.9 -> 53.2; quantised rows, 64 trees 19.2 -> 18.6).  The
// merge workgroups come first, padded to a multiple of eight.  Returns this workgroup's node, or -1 if it has none.
constexpr int kXcds = 8;
__host__ __device__ __forceinline__ int tree_merge_wgs(int G) {
    return (G + kXcds - 1) / kXcds * kXcds;
}
__device__ __forceinline__ int tree_node(int G, int nodes) {
    const int j = (int)blockIdx.x - tree_merge_wgs(G);
    const int per = (nodes + kXcds - 1) / kXcds;
    const int b = (j % kXcds) * per + j / kXcds;
    return b < nodes ? b : -1;
}

// The layer before l whose predictor is active (-1: none).  The mask is read 64 layers at a time: one by one, every
// inactive layer on the way would cost a trip to memory of its own.
__device__ __forceinline__ int previous_active(const int32_t *active, int l) {
    if (!active) return l - 1;
    const int lane = threadIdx.x & (kWave - 1);
    for (int hi = l; hi > 0; hi -= kWave) {  // layers [hi - 64, hi)
        const int q = hi - 1 - lane;         // lane 0: the nearest
        const unsigned long long m = __ballot(q >= 0 && active[q < 0 ? 0 : q] != 0);
        if (m) return hi - 1 - (int)__builtin_ctzll(m);
    }
    return -1;
}

// What the scoring launch of a layer loop does beside it: nothing is verified yet, and the verifications' counters,
// arg-max slots and notes are cleared (a kernel of its own would be a launch more).
__device__ __forceinline__ void loop_begin(const PredictParams &p, size_t tok) {
    if (threadIdx.x == 0) {
        p.loop.ver_token[tok] = -1;
        p.loop.hit[tok] = 0;
    }
    if (tok == 0) {
        if (threadIdx.x == 0) *p.loop.arrive = *p.loop.abort = 0;
        for (int i = threadIdx.x; i < kLoopKeys + kLoopNotes; i += blockDim.x) p.loop.lines[i * kLoopLine] = 0;
    }
}

// KC: speculative rows held in flight (K <= KC).  VPT: 16-byte vectors per
// thread per row (d/8 <= VPT * 512 * tiles).  SWEEP: the previous layer's local
// probabilities are recomputed from that layer's hidden state instead of read,
// which makes every (layer, token) workgroup independent.
// EXACT: K == KC is known at compile time (K <= 8): every `k < K` predicate and
// the generic MLP path fold away, which shortens the serial instruction stream of this latency-bound
// kernel.
// T: threads per workgroup.  512 gives the shortest single call (one vector of a 4096-wide row and one
// hidden unit per thread).  With thousands of tokens per launch 256 is faster: twice as many
// workgroups fit on a CU, so more independent chains of the two memory trips are in flight, and the
// redundant feature arithmetic and the barriers halve; a thread then owns MU = 2 hidden units, both
// requested up front.
// TREE: the tokens are the nodes of p.tree.G trees; the first p.tree.G workgroups merge the trees' ids.
template <int KC, int VPT, bool SWEEP, bool EXACT, int T = kPredictThreads, int MU = 1, bool TREE = false>
__global__ __launch_bounds__(T) void predict_kernel(PredictParams p) {
    if (TREE && (int)blockIdx.x < tree_merge_wgs(p.tree.G)) {
        if ((int)blockIdx.x < p.tree.G) merge_one_tree<T>(p.tree, blockIdx.x);
        return;
    }
    const int b = TREE ? tree_node(p.tree.G, p.B) : (int)blockIdx.x;
    if (TREE && b < 0) return;
    constexpr int kWaves = T / kWave;
    // throughput shape: hidden states pass through once, so they are read with the non-temporal hint; the
    // LM-head rows are not -- tokens of a batch share rows, and the hint costs those re-reads their cache
    // hits (16384 tokens with repeating ids: 91 -> 104 us with it, though 8000 tokens with distinct ids
    // gain 10 %)
    constexpr bool kStream = T != kPredictThreads;
    __shared__ float red[kWaves][2 * KC + 2];
    __shared__ float red_u[kWaves];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid >> 6;
    const int l = blockIdx.y;
    const int K = EXACT ? KC : p.K, H = p.H, d = p.d;
    const int nv = d >> 3;
    const size_t tok = (size_t)l * p.B + b;

    // ---- which layer supplies the previous probabilities (sweep only)
    int lprev = -1;
    if (SWEEP) {
        if (p.loop.ver_token) loop_begin(p, tok);
        if (p.active && p.active[l] == 0) {
            if (tid < K) {
                p.logits[tok * K + tid] = 0.f;
                p.probs[tok * K + tid] = 0.f;
            }
            if (tid == 0) {
                p.scores[tok] = 0.f;
                p.exit_flags[tok] = 0;
            }
            return;
        }
        lprev = previous_active(p.active, l);
    }

    // ---- the ids (and the token's done flag) are requested before anything else: the LM-head rows, the
    // longest chain of the kernel, hang on them
    // (single layer only: in the sweep the compiler would wait for them before requesting anything else)
    int idv[KC];
    if (!SWEEP) {
#pragma unroll
        for (int k = 0; k < KC; ++k) idv[k] = (k < K) ? p.ids[(size_t)tok * K + k] : 0;
    }

    // ---- requests that do not depend on the ids
    const half_t *W1 = p.W1 + (size_t)l * H * 3 * K;
    const half_t *w2 = p.w2 + (size_t)l * H;
    const half_t *b1 = p.b1 ? p.b1 + (size_t)l * H : nullptr;
    MlpRow<KC> rowm[MU];
#pragma unroll
    for (int m = 0; m < MU; ++m) mlp_row_load<KC>(rowm[m], W1, b1, w2, K, H, tid + m * T);

    const half_t *hrow = p.hidden + tok * d;
    const half_t *hprow = (SWEEP && lprev >= 0) ? p.hidden + ((size_t)lprev * p.B + b) * d : nullptr;
    half8 hv[VPT], gv[VPT], hp[VPT];
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        int v = tid + u * T;
        bool in = v < nv;
        hv[u] = in ? (kStream ? load_half8_stream(hrow + v * 8) : load_half8(hrow + v * 8)) : zero_half8();
        gv[u] = in ? load_half8(p.gamma + v * 8) : zero_half8();
        hp[u] = (SWEEP && in && hprow) ? load_half8(hprow + v * 8) : zero_half8();
    }
    float prev[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) prev[k] = 0.f;
    const float *prev_src = SWEEP ? (lprev < 0 ? p.prev : nullptr) : p.prev;
    if (prev_src) {
#pragma unroll
        for (int k = 0; k < KC; ++k)
            if (k < K) prev[k] = prev_src[(size_t)b * K + k];
    }

    // ---- the K speculative LM-head rows
    // The token's done flag travels with the ids, so looking at it costs the live tokens nothing; a
    // token that already left the model stops here, before the rows are read.
    const int dn = (!SWEEP && p.done) ? p.done[b] : 0;
    const half_t *rows[KC];
    bool bad_id = false;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        int id = SWEEP ? ((k < K) ? p.ids[(size_t)b * K + k] : 0) : idv[k];
        bool ok = id >= 0 && id < p.V;
        if (k < K && !ok) bad_id = true;
        rows[k] = p.lm_head + (size_t)(ok ? id : 0) * d;
    }
    if (!SWEEP && dn != 0) {  // uniform over the workgroup
        if (tid < K) {
            p.logits[tok * K + tid] = 0.f;
            p.probs[tok * K + tid] = p.prev[(size_t)b * K + tid];
        }
        if (tid == 0) {
            p.scores[tok] = 0.f;
            p.exit_flags[tok] = 0;
        }
        return;
    }
    half8 wv[KC][VPT];
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            int v = tid + u * T;
            wv[k][u] = (k < K && v < nv) ? load_half8(rows[k] + v * 8) : zero_half8();
        }

    // ---- one pass: sum of squares and the K dot products (and the previous layer's)
    float ssq = 0.f, ssq_p = 0.f, acc[KC], acc_p[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = acc_p[k] = 0.f;
#pragma unroll
    for (int u = 0; u < VPT; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float g = (float)gv[u][e];
            float hf = (float)hv[u][e];
            float x = hf * g;
            ssq += hf * hf;
            float xp = 0.f;
            if (SWEEP) {
                float hpf = (float)hp[u][e];
                xp = hpf * g;
                ssq_p += hpf * hpf;
            }
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                float w = (float)wv[k][u][e];
                acc[k] += x * w;
                if (SWEEP) acc_p[k] += xp * w;
            }
        }
    // d larger than VPT * 512 vectors: remaining tiles, same arithmetic
    for (int v = tid + VPT * T; v < nv; v += T) {
        half8 h8 = load_half8(hrow + v * 8), g8 = load_half8(p.gamma + v * 8);
        half8 hp8 = (SWEEP && hprow) ? load_half8(hprow + v * 8) : zero_half8();
        half8 w8[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) w8[k] = (k < K) ? load_half8(rows[k] + v * 8) : zero_half8();
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float g = (float)g8[e], hf = (float)h8[e], hpf = (float)hp8[e];
            float x = hf * g, xp = hpf * g;
            ssq += hf * hf;
            ssq_p += hpf * hpf;
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                float w = (float)w8[k][e];
                acc[k] += x * w;
                acc_p[k] += xp * w;
            }
        }
    }

    // ---- wavefront reduction, then fixed-order combination of the eight wave partials
    ssq = wave_sum_to_last_row(ssq);
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = wave_sum_to_last_row(acc[k]);
    if (SWEEP) {
        ssq_p = wave_sum_to_last_row(ssq_p);
#pragma unroll
        for (int k = 0; k < KC; ++k) acc_p[k] = wave_sum_to_last_row(acc_p[k]);
    }
    if (lane == kWave - 1) {
        red[wave][0] = ssq;
        red[wave][1] = ssq_p;
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            red[wave][2 + k] = acc[k];
            red[wave][2 + KC + k] = acc_p[k];
        }
    }
    __syncthreads();
    ssq = ssq_p = 0.f;
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = acc_p[k] = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        ssq += red[w][0];
        if (SWEEP) ssq_p += red[w][1];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            acc[k] += red[w][2 + k];
            if (SWEEP) acc_p[k] += red[w][2 + KC + k];
        }
    }

    // ---- features (every thread computes them redundantly: no second exchange)
    const float inv_d = 1.0f / (float)d;
    float z[KC], pr[KC];
    {
        float r = 1.0f / sqrtf(ssq * inv_d + p.eps);
#pragma unroll
        for (int k = 0; k < KC; ++k) z[k] = bad_id ? quiet_nan() : acc[k] * r;
        local_softmax<KC>(z, K, pr);
    }
    if (SWEEP && lprev >= 0) {
        float zp[KC];
        float rp = 1.0f / sqrtf(ssq_p * inv_d + p.eps);
#pragma unroll
        for (int k = 0; k < KC; ++k) zp[k] = bad_id ? quiet_nan() : acc_p[k] * rp;
        local_softmax<KC>(zp, K, prev);
    }

    // ---- MLP: thread j owns hidden unit j (+512, ...); f = [z | p | p - prev]
    float part = mlp_partial<KC, T, MU>(rowm, W1, b1, w2, K, H, tid, z, pr, prev);
    part = wave_sum_to_last_row(part);
    if (lane == kWave - 1) red_u[wave] = part;
    __syncthreads();

    if (tid == 0) {
        float u = p.b2 ? (float)p.b2[l] : 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) u += red_u[w];
        float s = sigmoidf(u);
        p.scores[tok] = s;
        p.exit_flags[tok] = (s > p.threshold) ? 1 : 0;
#pragma unroll
        for (int k = 0; k < KC; ++k)
            if (k < K) {
                p.logits[tok * K + k] = z[k];
                p.probs[tok * K + k] = pr[k];
            }
    }
}

// Shared tail of the quantised-row kernels: wavefront and workgroup sums (fixed order), RMSNorm scale,
// features, MLP, sigmoid, threshold, outputs.  All threads of the workgroup must call.
template <int KC, int T, int MU>
__device__ __forceinline__ void q4_tail(const PredictParams &p, int b, int K, float ssq, float (&acc)[KC], bool bad_id,
                                        const MlpRow<KC> (&rowm)[MU], const float (&prev)[KC],
                                        float (*red)[KC + 1], float *red_u) {
    constexpr int kWaves = T / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int H = p.H, d = p.d;
    // ---- wavefront reduction, then fixed-order combination of the eight wave partials
    ssq = wave_sum_to_last_row(ssq);
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = wave_sum_to_last_row(acc[k]);
    if (lane == kWave - 1) {
        red[wave][0] = ssq;
#pragma unroll
        for (int k = 0; k < KC; ++k) red[wave][1 + k] = acc[k];
    }
    __syncthreads();
    ssq = 0.f;
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        ssq += red[w][0];
#pragma unroll
        for (int k = 0; k < KC; ++k) acc[k] += red[w][1 + k];
    }
    float z[KC], pr[KC];
    const float r = 1.0f / sqrtf(ssq * (1.0f / (float)d) + p.eps);
#pragma unroll
    for (int k = 0; k < KC; ++k) z[k] = bad_id ? quiet_nan() : acc[k] * r;
    local_softmax<KC>(z, K, pr);
    float part = mlp_partial<KC, T, MU>(rowm, p.W1, p.b1, p.w2, K, H, tid, z, pr, prev);
    part = wave_sum_to_last_row(part);
    if (lane == kWave - 1) red_u[wave] = part;
    __syncthreads();
    if (tid == 0) {
        float u = p.b2 ? (float)p.b2[0] : 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) u += red_u[w];
        const float sc = sigmoidf(u);
        p.scores[b] = sc;
        p.exit_flags[b] = (sc > p.threshold) ? 1 : 0;
#pragma unroll
        for (int k = 0; k < KC; ++k)
            if (k < K) {
                p.logits[(size_t)b * K + k] = z[k];
                p.probs[(size_t)b * K + k] = pr[k];
            }
    }
}

// The predictor on a 4-bit group-quantised LM head (the quantised setting of the paper's cloud
// evaluation, Sec. 7.1 / 7.3; the storage format is this library's reading): element i of a row is a
// code c in 0..15 in bits 4*(i%8).. of 32-bit word i/8 and stands for scale[g] * (c - zero[g]),
// g = i / group.  A speculative row is then d/2 bytes instead of 2d, and the dequantisation never
// materialises: a thread owns eight consecutive elements (one word per row, all in one group), forms
//     sum_e x_e * c_e   and   sum_e x_e          (x = h * gamma, fp32)
// and adds scale * (first - zero * second) to the row's dot product -- one multiply-add per element
// plus three per word.  Same two dependent trips to memory and the same reductions and tail as
// predict_kernel; one workgroup per token.
// EXACT: K == KC at compile time (see predict_kernel).  Every load is unconditional on a clamped, valid
// address -- a load under a branch would make the compiler wait for all outstanding loads at the join
// and turn the K rows into K serial trips to memory; unused data is zeroed by selects instead.
// SWEEP: one workgroup per (layer, token), the previous active layer's probabilities from its hidden state, as in
// predict_kernel.
template <int KC, int VPT, bool EXACT, int T = kPredictThreads, int MU = 1, bool TREE = false, bool SWEEP = false>
__global__ __launch_bounds__(T) void predict_q4_kernel(PredictParams p) {
    if (TREE && (int)blockIdx.x < tree_merge_wgs(p.tree.G)) {
        if ((int)blockIdx.x < p.tree.G) merge_one_tree<T>(p.tree, blockIdx.x);
        return;
    }
    const int b = TREE ? tree_node(p.tree.G, p.B) : (int)blockIdx.x;
    if (TREE && b < 0) return;
    constexpr int kWaves = T / kWave;
    __shared__ float red[kWaves][KC + 1];
    __shared__ float red_u[kWaves];
    const int tid = threadIdx.x;
    const int K = EXACT ? KC : p.K, H = p.H, d = p.d;
    const int nv = d >> 3, ng = d / p.group;
    int lprev = -1;
    if (SWEEP) {  // p becomes this layer's call
        const int l = blockIdx.y;
        const size_t tok = (size_t)l * p.B + b;
        if (p.loop.ver_token) loop_begin(p, tok);
        if (p.active && p.active[l] == 0) {
            if (tid < K) {
                p.logits[tok * K + tid] = 0.f;
                p.probs[tok * K + tid] = 0.f;
            }
            if (tid == 0) {
                p.scores[tok] = 0.f;
                p.exit_flags[tok] = 0;
            }
            return;
        }
        lprev = previous_active(p.active, l);
        const size_t first = (size_t)l * p.B;
        p.W1 += (size_t)l * H * 3 * K;
        p.w2 += (size_t)l * H;
        if (p.b1) p.b1 += (size_t)l * H;
        if (p.b2) p.b2 += l;
        p.logits += first * K;
        p.probs += first * K;
        p.scores += first;
        p.exit_flags += first;
    }

    // ---- requests that do not depend on the ids
    MlpRow<KC> rowm[MU];
#pragma unroll
    for (int m = 0; m < MU; ++m) mlp_row_load<KC>(rowm[m], p.W1, p.b1, p.w2, K, H, tid + m * T);
    const half_t *hrow = p.hidden + ((SWEEP ? (size_t)blockIdx.y * p.B : 0) + b) * d;
    const half_t *hprow = SWEEP && lprev >= 0 ? p.hidden + ((size_t)lprev * p.B + b) * d : hrow;  // always valid
    half8 hv[VPT], gv[VPT], hp[VPT];
    int vc[VPT];
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int v = tid + u * T;
        vc[u] = min(v, nv - 1);
        const half8 h8 = load_half8(hrow + vc[u] * 8), g8 = load_half8(p.gamma + vc[u] * 8);
        hv[u] = v < nv ? h8 : zero_half8();  // a zero hidden state silences the clamped duplicate
        gv[u] = g8;
        if (SWEEP) {
            const half8 p8 = load_half8(hprow + vc[u] * 8);
            hp[u] = v < nv ? p8 : zero_half8();
        }
    }
    float prev[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) prev[k] = 0.f;
    if (!SWEEP || p.prev) {
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const float pv = p.prev[(size_t)b * K + min(k, K - 1)];
            prev[k] = (k < K) ? pv : 0.f;
        }
    }
    const int32_t *donep = p.done ? p.done + b : p.ids;  // always a valid address
    const int dn_raw = *donep;
    const int dn = p.done ? dn_raw : 0;

    // ---- the K speculative rows: one word of codes per row and vector, with its group's scale and zero-point
    int rowi[KC];
    bool bad_id = false;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int id = p.ids[(size_t)b * K + min(k, K - 1)];
        const bool ok = id >= 0 && id < p.V;
        if (k < K && !ok) bad_id = true;
        rowi[k] = ok ? id : 0;
    }
    if (dn != 0) {  // uniform over the workgroup: the token already left the model
        if (tid < K) {
            p.logits[(size_t)b * K + tid] = 0.f;
            p.probs[(size_t)b * K + tid] = p.prev[(size_t)b * K + tid];
        }
        if (tid == 0) {
            p.scores[b] = 0.f;
            p.exit_flags[b] = 0;
        }
        return;
    }
    uint32_t qw[KC][VPT];
    half_t qs[KC][VPT], qz[KC][VPT];
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const size_t gi = (size_t)rowi[k] * ng + (vc[u] * 8) / p.group;
            qw[k][u] = p.qweight[(size_t)rowi[k] * nv + vc[u]];
            qs[k][u] = p.qscales[gi];
            qz[k][u] = p.qzeros[gi];
        }

    float ssq = 0.f, ssq_p = 0.f, acc[KC], acc_p[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = acc_p[k] = 0.f;
    auto dot8 = [&](const half8 &h8, const half8 &g8, const uint32_t (&w)[KC], const half_t (&sc)[KC],
                    const half_t (&zp)[KC], float &ssq, float (&acc)[KC]) {
        float x[8], xs = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float hf = (float)h8[e];
            x[e] = hf * (float)g8[e];
            ssq += hf * hf;
            xs += x[e];
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const uint32_t even = w[k] & 0x0f0f0f0fu, odd = (w[k] >> 4) & 0x0f0f0f0fu;  // elements 0,2,4,6 / 1,3,5,7
            if constexpr (SWEEP) {
                // weight by weight, as in the layer loop's other kernel: the difference of two sums below is off by half
                // as much again (error of the loop's logits against float64 1.6e-7 / 1.1e-7), and few workgroups wait for
                // memory here, not for arithmetic
                const float s = (float)sc[k], z = (float)zp[k];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[k] += x[2 * j] * (s * ((float)((even >> (8 * j)) & 0xffu) - z));
                    acc[k] += x[2 * j + 1] * (s * ((float)((odd >> (8 * j)) & 0xffu) - z));
                }
            } else {
                float pd = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    pd += x[2 * j] * (float)((even >> (8 * j)) & 0xffu);
                    pd += x[2 * j + 1] * (float)((odd >> (8 * j)) & 0xffu);
                }
                acc[k] += (float)sc[k] * (pd - (float)zp[k] * xs);
            }
        }
    };
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        uint32_t w[KC];
        half_t sc[KC], zp[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            w[k] = qw[k][u];
            sc[k] = qs[k][u];
            zp[k] = qz[k][u];
        }
        dot8(hv[u], gv[u], w, sc, zp, ssq, acc);
        if (SWEEP) dot8(hp[u], gv[u], w, sc, zp, ssq_p, acc_p);
    }
    // d larger than VPT * 512 vectors: remaining tiles, same arithmetic
    for (int v = tid + VPT * T; v < nv; v += T) {
        const half8 h8 = load_half8(hrow + v * 8), g8 = load_half8(p.gamma + v * 8);
        uint32_t w[KC];
        half_t sc[KC], zp[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const size_t gi = (size_t)rowi[k] * ng + (v * 8) / p.group;
            w[k] = p.qweight[(size_t)rowi[k] * nv + v];
            sc[k] = p.qscales[gi];
            zp[k] = p.qzeros[gi];
        }
        dot8(h8, g8, w, sc, zp, ssq, acc);
        if (SWEEP) dot8(load_half8(hprow + v * 8), g8, w, sc, zp, ssq_p, acc_p);
    }

    if (SWEEP && lprev >= 0) {  // uniform over the workgroup
        __shared__ float red_p[kWaves][KC + 1];
        const int lane = tid & (kWave - 1), wave = tid >> 6;
        ssq_p = wave_sum_to_last_row(ssq_p);
#pragma unroll
        for (int k = 0; k < KC; ++k) acc_p[k] = wave_sum_to_last_row(acc_p[k]);
        if (lane == kWave - 1) {
            red_p[wave][0] = ssq_p;
#pragma unroll
            for (int k = 0; k < KC; ++k) red_p[wave][1 + k] = acc_p[k];
        }
        __syncthreads();
        ssq_p = 0.f;
        float zp[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) zp[k] = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            ssq_p += red_p[w][0];
#pragma unroll
            for (int k = 0; k < KC; ++k) zp[k] += red_p[w][1 + k];
        }
        const float rp = 1.0f / sqrtf(ssq_p * (1.0f / (float)d) + p.eps);
#pragma unroll
        for (int k = 0; k < KC; ++k) zp[k] = bad_id ? quiet_nan() : zp[k] * rp;
        local_softmax<KC>(zp, K, prev);
    }
    q4_tail<KC, T, MU>(p, b, K, ssq, acc, bad_id, rowm, prev, red, red_u);
}

// Throughput shape of predict_q4_kernel (thousands of tokens per launch).  A thread owns chunks of 32
// consecutive elements = four consecutive words of codes: one 16-byte load per row brings its codes, and
// because a chunk lies inside one quantisation group (group % 32 == 0) one scale and one zero-point per
// row serve all 32 elements.  Per token that is a third of the load instructions of the word-per-thread
// layout (the small scale / zero-point loads dominate there), and the vector memory path, not HBM, is
// what a CU runs out of first with rows this short.  CPT: chunks per thread (d <= 32 * T * CPT).
template <int KC, int T, int CPT, int MU, bool TREE = false>
__global__ __launch_bounds__(T) void predict_q4_wide_kernel(PredictParams p) {
    if (TREE && (int)blockIdx.x < tree_merge_wgs(p.tree.G)) {
        if ((int)blockIdx.x < p.tree.G) merge_one_tree<T>(p.tree, blockIdx.x);
        return;
    }
    const int b = TREE ? tree_node(p.tree.G, p.B) : (int)blockIdx.x;
    if (TREE && b < 0) return;
    constexpr int kWaves = T / kWave;
    constexpr int K = KC;
    __shared__ float red[kWaves][KC + 1];
    __shared__ float red_u[kWaves];
    const int tid = threadIdx.x;
    const int H = p.H, d = p.d;
    const int nc = d >> 5, nv = d >> 3, ng = d / p.group;

    // ---- requests that do not depend on the ids
    MlpRow<KC> rowm[MU];
#pragma unroll
    for (int m = 0; m < MU; ++m) mlp_row_load<KC>(rowm[m], p.W1, p.b1, p.w2, K, H, tid + m * T);
    const half_t *hrow = p.hidden + (size_t)b * d;
    half8 hv[CPT][4], gv[CPT][4];
    int cc[CPT], gofs[CPT];
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        const int c = tid + u * T;
        cc[u] = min(c, nc - 1);
        gofs[u] = (cc[u] * 32) / p.group;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const half8 h8 = load_half8(hrow + cc[u] * 32 + i * 8);
            hv[u][i] = c < nc ? h8 : zero_half8();  // a zero hidden state silences the clamped duplicate
            gv[u][i] = load_half8(p.gamma + cc[u] * 32 + i * 8);
        }
    }
    float prev[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) prev[k] = p.prev[(size_t)b * K + k];
    const int32_t *donep = p.done ? p.done + b : p.ids;  // always a valid address
    const int dn_raw = *donep;
    const int dn = p.done ? dn_raw : 0;

    // ---- the K speculative rows
    int rowi[KC];
    bool bad_id = false;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int id = p.ids[(size_t)b * K + k];
        const bool ok = id >= 0 && id < p.V;
        if (!ok) bad_id = true;
        rowi[k] = ok ? id : 0;
    }
    if (dn != 0) {  // uniform over the workgroup: the token already left the model
        if (tid < K) {
            p.logits[(size_t)b * K + tid] = 0.f;
            p.probs[(size_t)b * K + tid] = p.prev[(size_t)b * K + tid];
        }
        if (tid == 0) {
            p.scores[b] = 0.f;
            p.exit_flags[b] = 0;
        }
        return;
    }
    uintx4 qw[KC][CPT];
    half_t qs[KC][CPT], qz[KC][CPT];
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const size_t gi = (size_t)rowi[k] * ng + gofs[u];
            qw[k][u] = *reinterpret_cast<const uintx4 *>(p.qweight + (size_t)rowi[k] * nv + cc[u] * 4);
            qs[k][u] = p.qscales[gi];
            qz[k][u] = p.qzeros[gi];
        }

    float ssq = 0.f, acc[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = 0.f;
    // Byte j of a word holds elements 2j (low nibble) and 2j+1 (high nibble).  With a = x[2j] - x[2j+1]/16
    // and bq = x[2j+1]/16 (computed once, shared by the K rows),
    //     x[2j]*lo + x[2j+1]*hi = a*lo + bq*(lo + 16*hi) = a*lo + bq*byte,
    // so a row costs one mask per word and one byte-to-float conversion plus one FMA per nibble; the
    // high nibbles are never extracted.  This arithmetic, not memory, bounds the kernel.
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        float xs = 0.f, pd[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) pd[k] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float a[4], bq[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const half2_t hh = {hv[u][i][2 * j], hv[u][i][2 * j + 1]};
                ssq = __builtin_amdgcn_fdot2(hh, hh, ssq, false);
                const float x0 = (float)hh[0] * (float)gv[u][i][2 * j];
                const float x1 = (float)hh[1] * (float)gv[u][i][2 * j + 1];
                xs += x0 + x1;
                bq[j] = x1 * 0.0625f;
                a[j] = x0 - bq[j];
            }
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                const uint32_t w = qw[k][u][i];
                uint32_t lo = w & 0x0f0f0f0fu;
                asm("" : "+v"(lo));  // keeps the mask a mask: the byte selects below then fold into the conversions
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    pd[k] += a[j] * (float)((lo >> (8 * j)) & 0xffu);
                    pd[k] += bq[j] * (float)((w >> (8 * j)) & 0xffu);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) acc[k] += (float)qs[k][u] * (pd[k] - (float)qz[k][u] * xs);
    }
    q4_tail<KC, T, MU>(p, b, K, ssq, acc, bad_id, rowm, prev, red, red_u);
}

// first_exit[b] = first layer with exit flag 1 (inactive layers carry 0), else -1
__global__ void first_exit_kernel(const int32_t *exit_flags, int L, int B, int32_t *first_exit) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    int f = -1;
    for (int l = 0; l < L; ++l)
        if (exit_flags[(size_t)l * B + b] != 0) {
            f = l;
            break;
        }
    first_exit[b] = f;
}

constexpr int kBatchMinTokens = 1024;  // tokens per launch from which the throughput shapes are used
// The same on quantised rows, whose small workgroups pay earlier.  In chunks of 32 elements, K >= 3 (d = 4096, K = 4: 128
// tokens 4.2 us either way, 512 tokens 5.9 -> 5.5, 900 tokens 8.4 -> 5.8 us; d = 5120: 128 tokens 5.0 -> 4.5, 900 tokens
// 10.8 -> 8.2 us); K <= 2, with fewer rows to unpack (K = 2: 128 tokens 3.7 -> 3.9, 400 tokens 4.8 either way, 900 tokens
// 6.7 -> 5.2 us); word by word (d = 4104, K = 4 / 8: 128 tokens 5.0 -> 5.3 / 6.6 -> 6.9, 512 tokens 7.1 -> 7.0 / 10.2 ->
// 9.7 us).
constexpr int q4_batch_min_tokens(int K, bool wide) {
    return !wide ? 512 : K <= 2 ? 400 : 128;
}

// Workgroups of a launch of trees: the merges, and eight equal shares of the nodes.
static int tree_wgs(const PredictParams &p) {
    return tree_merge_wgs(p.tree.G) + (p.B + kXcds - 1) / kXcds * kXcds;
}

// A tree's ids are merged by one workgroup of the launch, at most kMergePerThread of them per thread.
template <bool TREE>
static bool merge_fits(const PredictParams &p, int threads) {
    return !TREE || p.tree.n <= kMergePerThread * threads;
}

template <int KC, bool SWEEP, bool EXACT, bool TREE>
static hipError_t launch_vpt(const PredictParams &p, hipStream_t s) {
    dim3 grid(TREE ? tree_wgs(p) : p.B, p.L), block(kPredictThreads);
    const size_t lds = TREE ? (size_t)merge_lds_ints(p.tree.n) * sizeof(int32_t) : 0;
    const int nv = p.d >> 3;
    if constexpr (!SWEEP && EXACT && KC <= 8) {
        // throughput shape: K known at compile time, many tokens, rows of at most 4 * 256 vectors (d <= 8192)
        // (also for a few tokens when a row is exactly two vectors per thread, d = 4096: four wavefronts
        // instead of eight start and meet sooner -- 3.36 -> 3.32 us per call, 3.89 -> 3.47 us with the rows in HBM;
        // at d = 5120, where the last vectors are masked, the 512-thread shape stays ahead)
        if constexpr (KC <= 5) {
            // rows of at most two vectors per thread of 128 (d = 2048, K = 4: B=2000 9.9 -> 8.2 us, B=8000 29.3 -> 26.6)
            if (p.B >= kBatchMinTokens && nv <= 2 * 128 && merge_fits<TREE>(p, 128)) {
                hipLaunchKernelGGL((predict_kernel<KC, 2, false, true, 128, 4, TREE>), grid, dim3(128), lds, s, p);
                return hipGetLastError();
            }
        }
        const bool small_fit = KC == 4 && nv == 2 * 256;
        if ((p.B >= kBatchMinTokens || small_fit) && nv <= 2 * 256 * (KC <= 4 ? 2 : 1)) {
            const dim3 blk(256);
            if (nv <= 2 * 256)
                hipLaunchKernelGGL((predict_kernel<KC, 2, false, true, 256, 2, TREE>), grid, blk, lds, s, p);
            else
                hipLaunchKernelGGL((predict_kernel<KC, 4, false, true, 256, 2, TREE>), grid, blk, lds, s, p);
            return hipGetLastError();
        }
    }
    const int vpt = (nv + kPredictThreads - 1) / kPredictThreads;
    if (vpt <= 1)
        hipLaunchKernelGGL((predict_kernel<KC, 1, SWEEP, EXACT, kPredictThreads, 1, TREE>), grid, block, lds, s, p);
    else if (vpt <= 2 || KC > 8)
        hipLaunchKernelGGL((predict_kernel<KC, 2, SWEEP, EXACT, kPredictThreads, 1, TREE>), grid, block, lds, s, p);
    else if constexpr (KC <= 8)
        hipLaunchKernelGGL((predict_kernel<KC, 4, SWEEP, EXACT, kPredictThreads, 1, TREE>), grid, block, lds, s, p);
    return hipGetLastError();
}

// K values that are compiled in: up to 8, where the rows of every shape fit in registers.  Against the generic form, which
// larger K take (rows of W1 read where they are used, tests of k < K), at d = 4096: one token K = 1 3.7 -> 2.9 us, 2
// 3.9 -> 3.0, 3 4.3 -> 3.3, 5 5.9 -> 3.8, 6 6.3 -> 3.8, 7 6.8 -> 4.9; 8000 tokens 39 -> 23, 45 -> 30, 51 -> 38, 103 -> 55,
// 118 -> 65, 134 -> 77 us; the same on quantised rows, 8000 tokens 54 -> 20, 58 -> 23, 60 -> 27, 124 -> 35, 133 -> 34,
// 143 -> 57, and K = 8, which has their throughput shapes too, 78 -> 42 us.
template <bool SWEEP, bool TREE>
static hipError_t launch_kc(const PredictParams &p, hipStream_t s) {
    switch (p.K) {
        case 1: return launch_vpt<1, SWEEP, true, TREE>(p, s);
        case 2: return launch_vpt<2, SWEEP, true, TREE>(p, s);
        case 3: return launch_vpt<3, SWEEP, true, TREE>(p, s);
        case 4: return launch_vpt<4, SWEEP, true, TREE>(p, s);
        case 5: return launch_vpt<5, SWEEP, true, TREE>(p, s);
        case 6: return launch_vpt<6, SWEEP, true, TREE>(p, s);
        case 7: return launch_vpt<7, SWEEP, true, TREE>(p, s);
        case 8: return launch_vpt<8, SWEEP, true, TREE>(p, s);
        default: return launch_vpt<16, SWEEP, false, TREE>(p, s);
    }
}

hipError_t launch_predict(const PredictParams &p, hipStream_t s) {
    return launch_kc<false, false>(p, s);
}

template <int KC, bool EXACT, bool TREE>
static hipError_t launch_q4_kc(const PredictParams &p, hipStream_t s) {
    const dim3 grid(TREE ? tree_wgs(p) : p.B), block(kPredictThreads);
    const size_t lds = TREE ? (size_t)merge_lds_ints(p.tree.n) * sizeof(int32_t) : 0;
    const int nv = p.d >> 3;
    if constexpr (EXACT && KC <= 8) {
        // throughput shape (see predict_kernel): a quantised row is a quarter of the bytes, so the fixed
        // cost per workgroup weighs more and small workgroups pay: 128 threads per token, four words per
        // row and thread, four hidden units per thread (B=8000 at d=4096: 51 -> 37 us)
        // chunks of 32 elements per thread when the format allows it (group % 32 == 0, rows 16-byte aligned):
        // B=8000 at d=4096: 37 -> 29 us, at d=8192: 71 -> 58 us
        const bool wide_ok = p.group % 32 == 0 && p.d % 32 == 0 && (reinterpret_cast<uintptr_t>(p.qweight) & 15) == 0;
        const bool batch = p.B >= q4_batch_min_tokens(KC, wide_ok);
        if (wide_ok && batch && p.d <= 32 * 128 && merge_fits<TREE>(p, 128)) {
            hipLaunchKernelGGL((predict_q4_wide_kernel<KC, 128, 1, 4, TREE>), grid, dim3(128), lds, s, p);
            return hipGetLastError();
        }
        if (wide_ok && batch && p.d <= 32 * 256) {
            hipLaunchKernelGGL((predict_q4_wide_kernel<KC, 256, 1, 2, TREE>), grid, dim3(256), lds, s, p);
            return hipGetLastError();
        }
        if (batch && nv <= 4 * 128 && merge_fits<TREE>(p, 128)) {
            hipLaunchKernelGGL((predict_q4_kernel<KC, 4, true, 128, 4, TREE>), grid, dim3(128), lds, s, p);
            return hipGetLastError();
        }
        if (batch && nv <= 4 * 256) {
            hipLaunchKernelGGL((predict_q4_kernel<KC, 4, true, 256, 2, TREE>), grid, dim3(256), lds, s, p);
            return hipGetLastError();
        }
    }
    if (nv <= kPredictThreads)
        hipLaunchKernelGGL((predict_q4_kernel<KC, 1, EXACT, kPredictThreads, 1, TREE>), grid, block, lds, s, p);
    else
        hipLaunchKernelGGL((predict_q4_kernel<KC, 2, EXACT, kPredictThreads, 1, TREE>), grid, block, lds, s, p);
    return hipGetLastError();
}

template <bool TREE>
static hipError_t launch_q4_any(const PredictParams &p, hipStream_t s) {
    switch (p.K) {
        case 1: return launch_q4_kc<1, true, TREE>(p, s);
        case 2: return launch_q4_kc<2, true, TREE>(p, s);
        case 3: return launch_q4_kc<3, true, TREE>(p, s);
        case 4: return launch_q4_kc<4, true, TREE>(p, s);
        case 5: return launch_q4_kc<5, true, TREE>(p, s);
        case 6: return launch_q4_kc<6, true, TREE>(p, s);
        case 7: return launch_q4_kc<7, true, TREE>(p, s);
        case 8: return launch_q4_kc<8, true, TREE>(p, s);
        default: return launch_q4_kc<16, false, TREE>(p, s);
    }
}

hipError_t launch_predict_q4(const PredictParams &p, hipStream_t s) {
    return launch_q4_any<false>(p, s);
}

// Second half of the node-by-node tree call: a tree whose merged set did not fit is refused as a whole (NaN, no
// exit), otherwise the path rule on the exit flags.  One workgroup per tree.
constexpr int kTreeTailThreads = 256;
__global__ __launch_bounds__(kTreeTailThreads) void tree_tail_kernel(PredictParams p, int N, const int32_t *parent,
                                                                     int32_t *path_exit) {
    extern __shared__ __attribute__((aligned(16))) int32_t tree_tail_lds[];  // exit flags [N], parents [N]
    int32_t *ex = tree_tail_lds, *par = tree_tail_lds + N;
    const int g = blockIdx.x, tid = threadIdx.x;
    const size_t base = (size_t)g * N;
    for (int n = tid; n < N; n += kTreeTailThreads) {
        ex[n] = p.exit_flags[base + n];
        par[n] = path_exit ? parent[base + n] : -1;
    }
    if (p.tree.M_out[g] > p.tree.Mcap) {  // uniform over the workgroup
        for (int n = tid; n < N; n += kTreeTailThreads) {
            ex[n] = 0;  // (each thread its own entries)
            p.exit_flags[base + n] = 0;
            p.scores[base + n] = quiet_nan();
        }
        for (int i = tid; i < N * p.K; i += kTreeTailThreads) {
            p.logits[base * p.K + i] = quiet_nan();
            p.probs[base * p.K + i] = quiet_nan();
        }
    }
    if (!path_exit) return;
    __syncthreads();
    finish_paths(ex, par, N, tid, kTreeTailThreads, path_exit + base);
}

// Trees scored node by node: every node is a token of its own that gathers its K rows, while one workgroup per tree
// merges the ids beside them.  Against one workgroup per tree (or the split contraction of a few trees) this gives up
// reading a shared row once per tree -- the caches serve the repeats -- and gains a chain of two memory trips per
// node on every CU instead of merge -> contraction -> scoring in series.
// The line between them lies where the times below, in microseconds, cross.  They are fitted to 2958 pairs of
// measurements (K = 1 ... 16, d = 256 ... 8192, 1 ... 1024 nodes per tree, 1 ... 4096 trees, H = 100 ... 2048, merged
// sets of 64 ... 400 rows, groups of 32, 64 and 128, rows in the last-level cache or from HBM); the slower side is chosen
// by more than 6 % in 69 of them, by 0.4 % on average.
// Node by node / tree kernels at d = 4096, K = 4, H = 512, trees of 64 nodes with 64 merged rows: 4 trees 6.4 / 15.3, 16
// 8.9 / 20.2, 48 16.9 / 23.2, 64 21.8 / 23.9, 80 25.7 / 26.0, 128 37.6 / 34.2; merged rows for 256: 64 trees 22.7 / 39.9,
// 192 53.5 / 65.6, 256 69.1 / 76.3.  d = 2048: 80 trees 16.3 / 20.8, 128 24.6 / 24.0; d = 8192: 32 trees 19.4 / 24.9, 48
// 27.1 / 28.8, 64 34.4 / 34.3.  K = 8: 48 trees 23.8 / 27.9, 64 30.3 / 28.8.  K = 8, H = 2048: 48 trees 32.1 / 39.2.
// K = 3, an MLP without the matrix cores: 64 trees 21.0 / 81.5, 256 65.5 / 98.5; H = 128, 192 trees 47.9 / 53.8, 256
// 62.0 / 59.3.  K = 16, not compiled in: 8 trees 20.5 / 22.9, 16 33.0 / 24.5, 20 39.3 / 64.6, 48 83.1 / 66.5.  Trees of
// 256 nodes: 32 trees 37.0 / 68.5, 128 120 / 129.  Quantised rows: K = 4, 16 trees 8.7 / 44.7, 192 41.9 / 48.7, 256
// 52.5 / 51.2; K = 8, 128 trees 44.6 / 48.3, 192 61.0 / 49.6; d = 512, 64 trees 16.9 / 18.8, 128 26.5 / 19.2.
static float tree_nodes_us(int G, int N, int d, int K, int H, bool q4) {
    const float elems = 1e-3f * (K + 1) * d;  // gathered per node, in thousands
    float ns;                                 // per node, the chip filled
    if (K > 8) {  // not compiled in; K = 16 has whole vectors of W1
        ns = (K == 16 ? 22.f : 18.f + 1.3f * K) + 0.11f * elems;
        return 9.f + 1e-3f * ns * G * N;
    }
    const float mlp = (K & 1 ? 0.45e-3f : 0.27e-3f) * K * std::max(H, 256);  // odd K: W1 by single halves
    if (q4) {
        ns = std::max(0.9f + 0.34f * K, 0.7f + mlp + (d <= 4096 ? 0.08f : 0.11f) * elems);
    } else {
        // the least a workgroup of 128 threads (of 256 or 512) takes, and the bytes
        const float least = K <= 5 && d <= 2048 && N * K <= kMergePerThread * 128 ? 1.4f : 1.f + 0.35f * K;
        ns = std::max(least, 0.3f + mlp + (K > 5 && d > 4096 ? 0.16f : 0.13f) * elems);
    }
    return 7.5f + 1e-3f * ns * G * N;
}

static float tree_kernels_us(int G, int N, int d, int K, int H, int Mcap, int group, bool whole) {
    const int rounds = (G + 255) / 256;
    const bool mfma = mlp_mfma_ok(K, H), vec = K == 4 || K == 8 || K == 16;  // vec: whole vectors of W1
    const float wide = 1e-3f * std::max(0, H - 512);
    const float mlp = mfma ? 8.f * wide : 4.f + 1e-3f * (vec ? 3.6f * K : 35.f + 36.f * K) * H * N / 64;
    if (group > 0)  // quantised rows: a fixed time per tree, one tree per CU and round
        return rounds * ((group >= 128 ? 16.f : 20.f) + 7e-3f * d * (Mcap <= 64 ? 1.f : 2.2f) + mlp);
    const float rows = std::min((float)Mcap, 0.3f * N * K);  // merged rows, as overlapping ids leave them
    if (whole) {
        const float mb = 2e-6f * G * (N + rows) * d;
        float t = (Mcap <= 64 ? 17.f : Mcap <= 128 ? 25.f : 31.f) + (K <= 4 ? 0.f : 3.5f) +
                  mb / (Mcap <= 64 ? 9.f : 7.5f) + std::max(0.f, mb - 250.f) / 10;  // beyond the last-level cache
        if (rounds > 1) t = std::max(t + 10.f, rounds * (10.f + 3.4e-3f * d));
        return t + rounds * mlp;
    }
    // split contraction, one wavefront per node behind it (a workgroup per tree from 32 trees on)
    const float tail = mfma ? 9.f * wide : vec ? 6e-3f * H : 2.f + (K <= 8 ? 12e-3f : 40e-3f) * H;
    if (G < 20 && N <= 64 && Mcap <= 256)
        return 15.5f + tail + (Mcap > 64 ? 2.f : 0.f) + std::min(9.f, 0.67e-6f * G * (N + rows) * d);
    const float gmac = 1e-9f * G * N * rows * d;
    return 15.5f + tail + 0.4e-3f * G * N + 8.5f * gmac + 10.f * std::min(1.f, gmac) + (G < 32 ? 0.f : 15.f + mlp);
}

bool tree_nodes_preferred(int G, int N, int d, int K, int H, int Mcap, int group, bool whole) {
    if (N * K > kMergePerThread * 256) return false;  // one workgroup of 256 threads merges a tree's ids
    return tree_nodes_us(G, N, d, K, H, group > 0) < tree_kernels_us(G, N, d, K, H, Mcap, group, whole);
}

hipError_t launch_tree_nodes(const PredictParams &p, int N, const int32_t *parent, int32_t *path_exit, hipStream_t s) {
    const hipError_t e = p.qweight ? launch_q4_any<true>(p, s) : launch_kc<false, true>(p, s);
    if (e != hipSuccess) return e;
    if (!path_exit && p.tree.n <= p.tree.Mcap) return hipSuccess;  // no path rule, and the set always fits
    hipLaunchKernelGGL(tree_tail_kernel, dim3(p.tree.G), dim3(kTreeTailThreads), (size_t)2 * N * sizeof(int32_t), s, p,
                       N, parent, path_exit);
    return hipGetLastError();
}

// Every (layer, token) pair of a layer loop, fp16 or quantised head (K <= 8 there, d <= 8192)
template <int KC>
static hipError_t launch_q4_sweep(const PredictParams &p, hipStream_t s) {
    const dim3 grid(p.B, p.L), block(kPredictThreads);
    if ((p.d >> 3) <= kPredictThreads)
        hipLaunchKernelGGL((predict_q4_kernel<KC, 1, true, kPredictThreads, 1, false, true>), grid, block, 0, s, p);
    else
        hipLaunchKernelGGL((predict_q4_kernel<KC, 2, true, kPredictThreads, 1, false, true>), grid, block, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_loop_scores(const LoopParams &lp, hipStream_t s) {
    PredictParams p{};
    p.d = lp.d; p.V = lp.V; p.K = lp.K; p.H = lp.H; p.eps = lp.eps; p.threshold = lp.threshold;
    p.B = lp.B; p.L = lp.L;
    p.hidden = lp.hidden; p.gamma = lp.gamma; p.lm_head = lp.lm_head; p.ids = lp.ids; p.prev = lp.prev0;
    p.W1 = lp.W1; p.b1 = lp.b1; p.w2 = lp.w2; p.b2 = lp.b2;
    p.active = lp.active;
    p.qweight = lp.qweight; p.qscales = lp.qscales; p.qzeros = lp.qzeros; p.group = lp.group;
    p.logits = lp.logits; p.probs = lp.probs; p.scores = lp.scores; p.exit_flags = lp.exit_flags;
    p.loop.ver_token = lp.ver_token; p.loop.hit = lp.hit; p.loop.arrive = lp.arrive; p.loop.abort = lp.abort;
    p.loop.lines = lp.lines;
    if (!p.qweight) return launch_kc<true, false>(p, s);
    switch (p.K) {
        case 1: return launch_q4_sweep<1>(p, s);
        case 2: return launch_q4_sweep<2>(p, s);
        case 3: return launch_q4_sweep<3>(p, s);
        case 4: return launch_q4_sweep<4>(p, s);
        case 5: return launch_q4_sweep<5>(p, s);
        case 6: return launch_q4_sweep<6>(p, s);
        case 7: return launch_q4_sweep<7>(p, s);
        case 8: return launch_q4_sweep<8>(p, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_predict_sweep(const PredictParams &p, int32_t *first_exit, hipStream_t s) {
    if (p.L > 0) {
        hipError_t e = launch_kc<true, false>(p, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(first_exit_kernel, dim3((p.B + 255) / 256), dim3(256), 0, s, p.exit_flags, p.L, p.B,
                       first_exit);
    return hipGetLastError();
}

}  // namespace specee
