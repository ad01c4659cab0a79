// Full LM head for up to 16 hidden states per pass over the head: the stand-alone kernels (logits, or arg-max candidates
// for a verification) on the fp16 and on the 4-bit group-quantised head.  The stream itself: head_states.h.
#include <algorithm>

#include "head_states.h"
#include "kernels.h"

namespace specee {

struct HeadStatesParams {
    HsParams hs;
    int N;
    int tiles_per_wg, tiles_over;  // the first `tiles_over` workgroups take one tile more
    const half_t *hidden;
    float *out;
    float *best_val;
    int32_t *best_idx;
    const int32_t *gate, *done;
};

template <int LW, int CPW, bool RAGGED, bool NT, bool ARGMAX>
__global__ __launch_bounds__(hs_max_waves(CPW) * kWave) void head_states_kernel(HeadStatesParams p) {
    constexpr int kHsBlock = hs_block(CPW);
    extern __shared__ __attribute__((aligned(16))) unsigned char hs_smem[];
    __shared__ float cand_v[kHsBlock][kHsStates];
    __shared__ int cand_i[kHsBlock][kHsStates];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int c = lane & 15, q = lane >> 4;
    const int n0 = blockIdx.y * kHsStates, V = p.hs.V, wg = blockIdx.x;
    if (ARGMAX && (p.gate || p.done)) {
        // none of this workgroup's states is to be verified: no pass (the tail kernel fills in the outputs)
        int any = 0;
        if (tid < kHsStates && n0 + tid < p.N)
            any = (!p.gate || p.gate[n0 + tid] != 0) && (!p.done || p.done[n0 + tid] == 0);
        if (__syncthreads_or(any) == 0) return;
    }
    const int t0 = wg * p.tiles_per_wg + min(wg, p.tiles_over);
    const int t1 = t0 + p.tiles_per_wg + (wg < p.tiles_over ? 1 : 0);
    float bv[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    int bi[4] = {0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff};
    // (several passes over the rows: the sums of as many tiles wait in LDS as there is room for)
    const int most = p.hs.passes > 1 ? kHsMaxTiles : t1 - t0;
    for (int t = t0; t < t1; t += most)
        head_states_rows<LW, CPW, RAGGED, NT>(
            p.hs, hs_smem, 1, t, min(t1, t + most), [&](int n) { return p.hidden + (size_t)min(n0 + n, p.N - 1) * p.hs.d; },
            [&](int row, int n, floatx4 y) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (ARGMAX) {
                        if (row < V && y[r] > bv[r]) {  // rows ascend: strict '>' keeps the lowest row on ties
                            bv[r] = y[r];
                            bi[r] = row;
                        }
                    } else if (row < V && n0 + n + r < p.N) {
                        p.out[(size_t)(n0 + n + r) * V + row] = y[r];
                    }
                }
            });
    if (ARGMAX) {
        const int ncand = min(kHsBlock, (int)blockDim.x >> 6);
        if (wave < ncand) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // the sixteen rows of a tile: lanes of one DPP row
                row16_argmax(bv[r], bi[r]);
                if (c == 0) {
                    cand_v[wave][4 * q + r] = bv[r];
                    cand_i[wave][4 * q + r] = bi[r];
                }
            }
        }
        __syncthreads();
        if (tid < kHsStates && n0 + tid < p.N) {
            float v = cand_v[0][tid];
            int i = cand_i[0][tid];
            for (int w = 1; w < ncand; ++w)
                if (cand_v[w][tid] > v || (cand_v[w][tid] == v && cand_i[w][tid] < i)) {
                    v = cand_v[w][tid];
                    i = cand_i[w][tid];
                }
            p.best_val[(size_t)(n0 + tid) * gridDim.x + wg] = v;
            p.best_idx[(size_t)(n0 + tid) * gridDim.x + wg] = i;
        }
    }
}

// Workgroups of a pass, each with its share of the tiles; never more than `limit` (the arg-max candidates that the caller's
// workspace holds).  One per CU; where two fit, two of them if the tiles go round: with one or two each, the second one's
// operands cost more than it brings (16 states, 512 / 256 workgroups, us, 2048 columns: fp16 8000 rows 13.0 / 10.1, 20011 20.0
// / 18.3, 32000 27.4 / 26.2, 50280 39.5 / 39.1; codes in groups of 128 11.0 / 8.6, 13.3 / 11.7, 15.8 / 15.0, 19.4 / 20.6;
// 1024 columns, codes, 24000 rows 8.9 / 8.6, 32000 9.7 / 10.6), but not fp16 rows of a single wavefront (512 columns,
// 8000 rows 5.7 / 6.2, 32000 9.9 / 13.2).
int head_states_workgroups(int d, int V, int group, int limit) {
    const int tiles = (V + kHsTile - 1) / kHsTile, lw = hs_words(group);
    const HsShape sh = hs_shape(d, lw, hs_chunks_per_wave(d, lw));
    const bool two = 2 * sh.waves <= hs_max_waves(sh.cpw) && (tiles >= 1800 || (lw == 0 && sh.waves == 1));
    return std::min({two ? 512 : 256, tiles, limit});
}

template <int LW, int CPW, bool RAGGED, bool NT, bool ARGMAX>
static hipError_t launch_hs(HeadStatesParams &p, const HsShape &sh, int wgs, hipStream_t s) {
    const int tiles = (p.hs.V + kHsTile - 1) / kHsTile;
    p.tiles_per_wg = tiles / wgs;
    p.tiles_over = tiles % wgs;
    p.hs.passes = sh.passes; p.hs.chunks = sh.chunks; p.hs.subs = sh.subs; p.hs.buffers = sh.buffers;
    auto kern = head_states_kernel<LW, CPW, RAGGED, NT, ARGMAX>;
    // per launch: the library keeps no state; a refusal shows as the launch error
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh.lds);
    hipLaunchKernelGGL(kern, dim3(wgs, (p.N + kHsStates - 1) / kHsStates), dim3(sh.waves * kWave), sh.lds, s, p);
    return hipGetLastError();
}

template <bool ARGMAX>
static hipError_t launch_hs_format(HeadStatesParams &p, int wgs, hipStream_t s) {
    return hs_dispatch(p.hs.d, p.hs.V, p.hs.qweight ? p.hs.group : 0, [&](auto lw, auto cpw, auto ragged, auto nt, const HsShape &sh) {
        return launch_hs<decltype(lw)::value, decltype(cpw)::value, decltype(ragged)::value, decltype(nt)::value, ARGMAX>(p, sh, wgs, s);
    });
}

static HeadStatesParams hs_params(int d, int V, float eps, int N, const half_t *hidden, const half_t *gamma,
                                  const half_t *lm_head, const HeadQ4 &q4) {
    HeadStatesParams p{};
    p.hs.d = d; p.hs.V = V; p.hs.eps = eps; p.hs.gamma = gamma; p.hs.lm_head = lm_head;
    p.hs.qweight = q4.qweight; p.hs.scales = q4.scales; p.hs.zeros = q4.zeros; p.hs.group = q4.group;
    p.N = N; p.hidden = hidden;
    return p;
}

bool head_states_q4_ok(int group) {
    return hs_words(group) > 0;
}

// A pass here costs the same for one state as for sixteen, and at least some 5 us + 1.2 us per 1024 columns; the vector
// kernel's time is that of all its rows, N * V.  Vector kernel against this one, logits, us, 4096 columns: groups of 128:
// 32000 rows, 2 states 32.5 / 21.2, 16 states 201 / 23.8; 8000 rows, 2 states 12.5 / 10.7; 2000 rows, 8 states 12.6 / 9.1;
// 500 rows, 16 states 7.8 / 10.5; groups of 64: 32000 rows, 2 states 32.5 / 22.8; 8000 rows, 2 states 12.0 / 12.0, 4
// states 20.1 / 12.0; 4096 rows, 4 states 9.8 / 10.5.  4608 and 5120 columns, whose last wavefronts are idle in part, are
// the latest to gain (8000 rows, 2 states, groups of 128: 14.9 / 15.7, of 64: 15.2 / 18.4).  One state stays on the
// vector units (32000 rows 18.2 / 21.2).
// Which states a gate lets through is known on the device only, and a state's logits are the same whoever else is let
// through, so the line is that of all N.  The vector kernel skips the others one by one and is the faster one, on small
// heads, while few are let through (verification, 8000 rows, groups of 128, 1 of 4 states 11.1 / 16.1, 2 of 4 14.0 / 16.3,
// all 23.4 / 16.3; 2000 rows, 1 of 16 10.2 / 15.7, all 22.4 / 15.8; 32000 rows, groups of 64, 1 of 2 20.0 / 27.2, both 33.5 /
// 27.2), and none at all costs 4 us with both.
bool head_states_q4_preferred(int d, int V, int N, int group) {
    return N >= 2 && head_states_q4_ok(group) && (long long)N * V >= (group == 128 ? 16000 : 24000);
}

// Against the tiles of up to 64 states (gemm_kernels.hip), whose 128 rows per workgroup leave most of the chip idle on a small
// head, us: 32000 x 4096, 16 states 65.7 / 49.0, 32 states, a pass per 16, 64 / 93; 6000 x 4096, 16 states 39.4 / 16.8, 32
// states 38.5 / 27.7, 64 states, 4000 rows 49.0 / 48.2; 2000 x 4096, 64 states 48.6 / 24.6; 300 x 1024, 3 states 11.8 / 4.7;
// 16000 x 1024, 32 states 14.2 / 16.5; 128256 x 8192, 16 states 397 / 390; verification of 16 states, 8000 x 4096 41.9 /
// 22.6, 20011 x 4104 42.6 / 43.8 (from memory 72 / 62).
// Rows that leave wavefronts idle are not faster everywhere (16 states, 32000 x 256 6.5 / 11.8, 32000 x 768 12.1 / 16.5, from
// memory 15.7 / 18.4; 32 states, 10000 x 768 10.3 / 15.7; 64 states, 4000 x 4104 54.5 / 71.8); they are here for the sums,
// 1.0e-7 to 1.35e-7 off float64 instead of 4e-7 to 9e-7.  Two states would gain too (32000 x 4096 87.3 / 47), but have those
// of the vector kernel, which are as exact.
bool head_states_preferred(int d, int V, int N) {
    const int passes = (N + kHsStates - 1) / kHsStates;
    return N > 2 && (passes == 1 || (N <= 64 && (long long)passes * V <= 20000));
}

hipError_t launch_head_states(int d, int V, float eps, int N, const half_t *hidden, const half_t *gamma,
                              const half_t *lm_head, const HeadQ4 &q4, float *out, hipStream_t s) {
    HeadStatesParams p = hs_params(d, V, eps, N, hidden, gamma, lm_head, q4);
    p.out = out;
    return launch_hs_format<false>(p, head_states_workgroups(d, V, q4.group, 1 << 30), s);
}

hipError_t launch_head_states_argmax(int d, int V, float eps, int N, const half_t *hidden, const half_t *gamma,
                                     const half_t *lm_head, const HeadQ4 &q4, int workgroups, float *best_val,
                                     int32_t *best_idx, const int32_t *gate, const int32_t *done, hipStream_t s) {
    HeadStatesParams p = hs_params(d, V, eps, N, hidden, gamma, lm_head, q4);
    p.best_val = best_val; p.best_idx = best_idx; p.gate = gate; p.done = done;
    return launch_hs_format<true>(p, workgroups, s);
}

}  // namespace specee
