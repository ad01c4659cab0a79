// Full-vocabulary LM head on a 4-bit group-quantised head for several hidden states at once, on the matrix cores
// (paper Sec. 4.1 and Sec. 4.3.3 in the weight-quantised setting of Sec. 7.1 / 7.3; format as in
// lm_head_q4_kernels.hip).  The vector kernel there makes one pass over the codes per hidden state and is bound by
// unpacking them; here up to 16 states share one pass:
//     Y[n][v] = r_n * sum_g scale[v][g] * ( sum_{i in g} x[n][i] * code[v][i]  -  zero[v][g] * sum_{i in g} x[n][i] ).
//
// Mapping onto v_mfma_f32_16x16x32_bf16 (lane = 16*q + c):
//   A operand = codes of row (m0 + c): integers 0..15 are exact in bf16.  A byte that holds a code is the fp8 (E4M3)
//               number code * 2^-9, so one v_cvt_scalef32_pk_bf16_fp8 with scale 2^9 turns two codes into two bf16
//               values: seven instructions per word of eight codes, mask and shift included;
//   B operand = x = h * gamma.  The product of two halves has 22 significant bits and is exact in fp32; it is cut
//               exactly into three bf16 numbers (the top 16 bits of what is left, three times), so that x enters
//               the matrix cores whole, over the full range of fp32: nothing here overflows or loses bits for
//               hidden states that are large or very small, as a split into two halves would;
//   D         = lane holds Y[4q .. 4q+3][c] of a row tile.
// A lane reads LW consecutive words (8 * LW codes) of its row per chunk of 32 * LW elements and uses one word per
// k-step, so k-step j of a chunk covers elements 8 * LW * q + 8 * j .. + 7 for lane group q; inside a word the order
// is (0,2,4,6,1,3,5,7), the one the conversions give.  B is built in that order.  A chunk lies in one quantisation
// group (group % (32 * LW) == 0): after each chunk the lane folds its rows' sums with that group's scale and
// zero-point; the chunk's sum of x was formed in fp32 when B was built.
//
// A workgroup owns 128 rows: wavefront (rw, kh) multiplies two row tiles of 16 with share kh of every stage, and the
// shares are added in ascending order at the end.  128 rows and 32 rows per wavefront because the B operand (its
// construction per workgroup, its LDS reads per wavefront) costs as much as the codes: half as many rows per
// wavefront would make the LDS reads the bound.  B sits in LDS in fragment order, double-buffered: a wavefront's
// read is 64 consecutive 16-byte pieces, without bank conflicts.
//
// Groups of exactly 128 and 64 go to head_states.hip where they gain from the matrix cores; this kernel does the other
// multiples of 32.
//
// Measured against the vector kernel: 32000 x 4096, groups of 256, 2 states 32.1 -> 24.4 us, 16 states 202 -> 26.5;
// 32000 x 3072, groups of 192, 16 states 184 -> 25.8, groups of 96 174 -> 36.5; 50280 x 2048, groups of 32, 172 -> 52.9.
// The time hardly depends on the number of states: the instruction streams (unpacking, building B, folding), the matrix
// cores and the codes (32000 x 4096: 11 us) overlap in part only.
#include "device_utils.h"
#include "kernels.h"

namespace specee {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kQmRows = 128;     // rows per workgroup: four row wavefronts, two tiles each
constexpr int kQmStates = 16;    // hidden states per workgroup
constexpr int kQmKh = 4;         // wavefronts that share a row pair
constexpr int kQmShare = 128;    // elements per stage of each of them
constexpr int kQmStage = kQmKh * kQmShare;
constexpr int kQmThreads = 256 * kQmKh;
constexpr int kQmWaves = kQmThreads / kWave;
constexpr int kQmSteps = kQmStage / 32;                               // k-steps per stage
constexpr int kQmVec = kQmStates * (kQmStage / 8) / kQmThreads;       // vectors of x per thread and stage
constexpr size_t kQmFragBytes = (size_t)2 * kQmSteps * 3 * kWave * 16;
constexpr size_t kQmSumBytes = (size_t)2 * kQmSteps * kQmStates * sizeof(float);
constexpr size_t kQmLdsBudget = 156 * 1024;

static size_t qm_lds_bytes(int d, int group) {
    return kQmFragBytes + kQmSumBytes + (size_t)2 * (d / group) * kQmRows * sizeof(half_t);
}

struct Q4HeadParams {
    int d, V, N, group, blocks_per_wg;  // blocks_per_wg: consecutive blocks of kQmRows rows per workgroup
    float eps;
    const half_t *hidden, *gamma;
    const uint32_t *qweight;
    const half_t *scales, *zeros;
    bool vec_scales;  // eight groups of a row per 16-byte load
    bool vec_out;     // four logits per 16-byte store
    float *out;
    float *best_val;
    int32_t *best_idx;
    const int32_t *gate, *done;
};

// the eight codes of a word as bf16, in the order (0,2,4,6,1,3,5,7)
__device__ __forceinline__ bf16x8 codes_to_bf16(uint32_t w) {
    const uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;
    uintx4 o;
    o[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.f, false));
    o[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.f, true));
    o[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.f, false));
    o[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.f, true));
    return __builtin_bit_cast(bf16x8, o);
}

// upper halves of two words: (a >> 16) | (b & 0xffff0000)
__device__ __forceinline__ uint32_t pack_high(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// LW: words per lane and chunk (group % (32 * LW) == 0, qweight aligned to 4 * LW bytes, d % (32 * LW) == 0)
template <int LW, bool ARGMAX>
__global__ __launch_bounds__(kQmThreads) void lm_head_q4_mfma_kernel(Q4HeadParams p) {
    constexpr int CH = kQmShare / (32 * LW);  // chunks per share
    // stages of loads in flight: with small groups the folds need the registers (two stages spilled 9 to 12 of them at
    // LW = 1, and one stage is faster there: 50280 x 2048 in groups of 32, 16 states, 66 -> 55 us, of 64, 40 -> 37 us)
    constexpr int kQmDepth = LW == 4 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char qm_smem[];
    typedef uintx4 (*frag_t)[kQmSteps][3][kWave];
    frag_t frag = reinterpret_cast<frag_t>(qm_smem);
    typedef float (*sum_t)[kQmSteps][kQmStates];
    sum_t xsum = reinterpret_cast<sum_t>(qm_smem + kQmFragBytes);  // sums of x over 32 elements
    const int d = p.d, ng = d / p.group;
    half_t *sc_lds = reinterpret_cast<half_t *>(qm_smem + kQmFragBytes + kQmSumBytes);  // [ng][kQmRows]
    half_t *zp_lds = sc_lds + (size_t)ng * kQmRows;
    __shared__ float ssq_lds[kQmWaves][kQmStates];
    __shared__ float cand_v[4][kQmStates];
    __shared__ int cand_i[4][kQmStates];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: addresses and branches derive from it
    const int c = lane & 15, q = lane >> 4;
    const int rw = wave & 3, kh = wave >> 2;
    const int n0 = blockIdx.y * kQmStates;
    if (ARGMAX && (p.gate || p.done)) {
        // none of this workgroup's states is to be verified: no pass (the tail kernel fills in the outputs)
        int any = 0;
        if (tid < kQmStates && n0 + tid < p.N)
            any = (!p.gate || p.gate[n0 + tid] != 0) && (!p.done || p.done[n0 + tid] == 0);
        if (__syncthreads_or(any) == 0) return;
    }

    // B side: this thread builds vector bv[i] (eight elements) of every stage for state c of the tile
    const half_t *hrow = p.hidden + (size_t)min(n0 + c, p.N - 1) * d;
    int bpos[kQmVec];
#pragma unroll
    for (int i = 0; i < kQmVec; ++i) {
        const int v = (tid >> 4) + i * (kQmThreads / 16);  // vector within the stage
        const int chunk = v / (4 * LW), off = v % (4 * LW);
        bpos[i] = (chunk * LW + off % LW) * 3 * kWave + (off / LW) * 16 + c;
    }
    const int nstages = (d + kQmStage - 1) / kQmStage;
    const int nblocks = (p.V + kQmRows - 1) / kQmRows;
    const int blk_end = min(nblocks, ((int)blockIdx.x + 1) * p.blocks_per_wg);
    float bv = -INFINITY;
    int bi = 0x7fffffff;

    for (int blk = blockIdx.x * p.blocks_per_wg; blk < blk_end; ++blk) {
        const int m0 = blk * kQmRows;
        // rows past the end repeat the last one and are never stored
        const uint32_t *rowptr[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
            rowptr[t] = p.qweight + (size_t)min(m0 + rw * 32 + t * 16 + c, p.V - 1) * (d >> 3);

        uint32_t a_buf[kQmDepth][2][CH * LW];
        half8 h_buf[kQmDepth][kQmVec], g_buf[kQmDepth][kQmVec];
        auto issue = [&](int s, int slot) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int ch = 0; ch < CH; ++ch) {
                    // clamped into the row: elements past the end meet x = 0
                    const int e = min(s * kQmStage + kh * kQmShare + ch * 32 * LW + 8 * LW * q, d - 8 * LW);
                    const uint32_t *src = rowptr[t] + (e >> 3);
                    if constexpr (LW == 4) {
                        const uintx4 w = *reinterpret_cast<const uintx4 *>(src);
#pragma unroll
                        for (int j = 0; j < 4; ++j) a_buf[slot][t][ch * 4 + j] = w[j];
                    } else if constexpr (LW == 2) {
                        const uint2 w = *reinterpret_cast<const uint2 *>(src);
                        a_buf[slot][t][ch * 2] = w.x;
                        a_buf[slot][t][ch * 2 + 1] = w.y;
                    } else {
                        a_buf[slot][t][ch] = *src;
                    }
                }
#pragma unroll
            for (int i = 0; i < kQmVec; ++i) {
                const int e = min(s * kQmStage + ((tid >> 4) + i * (kQmThreads / 16)) * 8, d - 8);
                h_buf[slot][i] = load_half8(hrow + e);
                g_buf[slot][i] = load_half8(p.gamma + e);
            }
        };
#pragma unroll
        for (int u = 0; u < kQmDepth; ++u) issue(u, u);

        // scales and zero-points of the block's rows, transposed to [group][row]
        if (p.vec_scales) {
            const int gv = ng >> 3;
            for (int i = tid; i < kQmRows * gv; i += kQmThreads) {
                const int m = i & (kQmRows - 1), g0 = (i >> 7) * 8;
                const size_t at = (size_t)min(m0 + m, p.V - 1) * ng + g0;
                const half8 s8 = load_half8(p.scales + at), z8 = load_half8(p.zeros + at);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    sc_lds[(g0 + e) * kQmRows + m] = s8[e];
                    zp_lds[(g0 + e) * kQmRows + m] = z8[e];
                }
            }
        } else {
            for (int i = tid; i < kQmRows * ng; i += kQmThreads) {
                const int m = i & (kQmRows - 1), g = i >> 7;
                const size_t at = (size_t)min(m0 + m, p.V - 1) * ng + g;
                sc_lds[g * kQmRows + m] = p.scales[at];
                zp_lds[g * kQmRows + m] = p.zeros[at];
            }
        }

        floatx4 acc[2];
        acc[0] = acc[1] = floatx4{0.f, 0.f, 0.f, 0.f};
        float ssq = 0.f;
        auto stage = [&](int s, int u) {
            const int b = s & 1;
#pragma unroll
            for (int i = 0; i < kQmVec; ++i) {
                const int v = (tid >> 4) + i * (kQmThreads / 16);
                const half8 h8 = s * kQmStage + v * 8 < d ? h_buf[u][i] : zero_half8(), g8 = g_buf[u][i];
                uint32_t w0[8], w1[8], w2[8];
                float sum = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float h = (float)h8[e], x = h * (float)g8[e];
                    ssq += h * h;
                    sum += x;
                    w0[e] = __builtin_bit_cast(uint32_t, x);
                    const float r1 = x - __builtin_bit_cast(float, w0[e] & 0xffff0000u);
                    w1[e] = __builtin_bit_cast(uint32_t, r1);
                    w2[e] = __builtin_bit_cast(uint32_t, r1 - __builtin_bit_cast(float, w1[e] & 0xffff0000u));
                }
                uintx4 *dst = &frag[b][0][0][0] + bpos[i];
                dst[0] = uintx4{pack_high(w0[0], w0[2]), pack_high(w0[4], w0[6]), pack_high(w0[1], w0[3]),
                                pack_high(w0[5], w0[7])};
                dst[kWave] = uintx4{pack_high(w1[0], w1[2]), pack_high(w1[4], w1[6]), pack_high(w1[1], w1[3]),
                                    pack_high(w1[5], w1[7])};
                dst[2 * kWave] = uintx4{pack_high(w2[0], w2[2]), pack_high(w2[4], w2[6]), pack_high(w2[1], w2[3]),
                                        pack_high(w2[5], w2[7])};
                sum += __shfl_xor(sum, 16, kWave);
                sum += __shfl_xor(sum, 32, kWave);
                if (q == 0) xsum[b][v >> 2][c] = sum;
            }
            uint32_t a_cur[2][CH * LW];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < CH * LW; ++j) a_cur[t][j] = a_buf[u][t][j];
            __syncthreads();
            issue(s + kQmDepth, u);
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) {
                floatx4 tmp[2];
                tmp[0] = tmp[1] = floatx4{0.f, 0.f, 0.f, 0.f};
                float t_x = 0.f;
#pragma unroll
                for (int j = 0; j < LW; ++j) {
                    const int ks = kh * (kQmShare / 32) + ch * LW + j;
                    const bf16x8 a0 = codes_to_bf16(a_cur[0][ch * LW + j]), a1 = codes_to_bf16(a_cur[1][ch * LW + j]);
                    t_x += xsum[b][ks][c];
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) {
                        const bf16x8 x8 = __builtin_bit_cast(bf16x8, frag[b][ks][pl][lane]);
                        tmp[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, x8, tmp[0], 0, 0, 0);
                        tmp[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, x8, tmp[1], 0, 0, 0);
                    }
                }
                const int e0 = s * kQmStage + kh * kQmShare + ch * 32 * LW;
                const int g = min(e0 / p.group, ng - 1);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int at = g * kQmRows + rw * 32 + t * 16 + 4 * q;
                    const half4 s4 = *reinterpret_cast<const half4 *>(sc_lds + at);
                    const half4 z4 = *reinterpret_cast<const half4 *>(zp_lds + at);
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[t][r] += (float)s4[r] * (tmp[t][r] - (float)z4[r] * t_x);
                }
            }
        };
        for (int s0 = 0; s0 < nstages; s0 += kQmDepth) {
#pragma unroll
            for (int u = 0; u < kQmDepth; ++u)
                if (s0 + u < nstages) stage(s0 + u, u);
        }

        // ---- sums of squares, and the shares of a row pair in ascending order
        ssq += __shfl_xor(ssq, 16, kWave);
        ssq += __shfl_xor(ssq, 32, kWave);
        __syncthreads();  // the last stage has been read: its buffers carry the shares
        if (q == 0) ssq_lds[wave][c] = ssq;
        floatx4 *part = reinterpret_cast<floatx4 *>(qm_smem);
        if (kh > 0) {
#pragma unroll
            for (int t = 0; t < 2; ++t) part[(((kh - 1) * 4 + rw) * 2 + t) * kWave + lane] = acc[t];
        }
        __syncthreads();
        if (kh == 0) {
#pragma unroll
            for (int k = 0; k < kQmKh - 1; ++k)
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[t] += part[((k * 4 + rw) * 2 + t) * kWave + lane];
            float total = 0.f;
#pragma unroll
            for (int w = 0; w < kQmWaves; ++w) total += ssq_lds[w][c];
            const float scale = 1.0f / sqrtf(total / (float)d + p.eps);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int m = m0 + rw * 32 + t * 16 + 4 * q;
                const floatx4 y = acc[t] * scale;
                if (ARGMAX) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (m + r < p.V && y[r] > bv) {  // rows ascend: strict '>' keeps the lowest row on ties
                            bv = y[r];
                            bi = m + r;
                        }
                } else if (n0 + c < p.N) {
                    float *dst = p.out + (size_t)(n0 + c) * p.V + m;
                    if (p.vec_out && m + 3 < p.V) {
                        *reinterpret_cast<floatx4 *>(dst) = y;
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (m + r < p.V) dst[r] = y[r];
                    }
                }
            }
        }
        __syncthreads();  // the next block writes the buffers read above
    }

    if (ARGMAX) {
        if (kh == 0) {
#pragma unroll
            for (int off = 16; off <= 32; off <<= 1) {  // the four lane groups of state c
                const float ov = __shfl_xor(bv, off, kWave);
                const int oi = __shfl_xor(bi, off, kWave);
                if (ov > bv || (ov == bv && oi < bi)) {
                    bv = ov;
                    bi = oi;
                }
            }
            if (q == 0) {
                cand_v[rw][c] = bv;
                cand_i[rw][c] = bi;
            }
        }
        __syncthreads();
        if (tid < kQmStates && n0 + tid < p.N) {
            bv = cand_v[0][tid];
            bi = cand_i[0][tid];
            for (int w = 1; w < 4; ++w)
                if (cand_v[w][tid] > bv || (cand_v[w][tid] == bv && cand_i[w][tid] < bi)) {
                    bv = cand_v[w][tid];
                    bi = cand_i[w][tid];
                }
            p.best_val[(size_t)(n0 + tid) * gridDim.x + blockIdx.x] = bv;
            p.best_idx[(size_t)(n0 + tid) * gridDim.x + blockIdx.x] = bi;
        }
    }
}

// Words per lane and chunk that the format allows (0: chunks would cross groups).
static int qm_words(int d, int group, const uint32_t *qweight) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(qweight);
    for (int lw = 4; lw >= 1; lw >>= 1)
        if (group % (32 * lw) == 0 && d % (32 * lw) == 0 && a % (4 * lw) == 0) return lw;
    return 0;
}

// At most 512 workgroups per 16 states: never more arg-max candidates than the vector kernel's launch leaves.
static int qm_blocks_per_wg(int V) {
    return ((V + kQmRows - 1) / kQmRows + 511) / 512;
}

int lm_head_q4_mfma_workgroups(int V) {
    const int rows = kQmRows * qm_blocks_per_wg(V);
    return (V + rows - 1) / rows;
}

// Whether a call goes to the matrix cores.  The format has to keep a chunk inside a group, and the rows' scales have
// to fit in LDS beside the B operand (at most 116 groups in a row: 14848 columns in groups of 128, 7424 in groups of 64,
// 3712 in groups of 32).  One state is cheaper on the vector units (18.4 us at 32000 x 4096), which build no B operand.
// Several states are compared by the time that each kernel takes, in nanoseconds, fitted to 1848 pairs of measurements
// (d = 1024 ... 8192, V = 500 ... 128256, 2 ... 64 states, groups of 128, 64 and 32; where the slower kernel is chosen it
// is so by 15 % at most, in 15 of the pairs by more than 6 %):
//   here, whole rounds of one workgroup per CU and a fixed time per block of 128 rows -- building B, unpacking and
//   folding, the folds of small groups costing more -- however few rows there are;
//   vector kernel, rounds of 512 workgroups (the last one partly filled) of one state's rows each, whose time is a
//   prologue plus the rows; above 64 rows per workgroup the re-reads of the larger head show.
// Groups of 128 and 64 were part of that and hardly come here any more (head_states.hip).  Of those that do, 455 pairs (256,
// 512, 192, 320, 160, 96 and 32; d = 1024 ... 8192, V = 1000 ... 50280, 2 to 16 states): the slower kernel by more than 6 %
// in 23, by 28 % at most (groups of 256, 8000 x 2048, 4 states 16.2 / 12.7 us), by 1.6 % on average.
// Vector kernel against this one, us: groups of 256, 4096 columns, 32000 rows, 2 states 32.1 / 24.3, 8000 rows, 2 states 12.0
// / 20.4, 4 states 21.1 / 20.3, 2000 rows, 16 states 20.2 / 21.6; groups of 192, 3072 columns, 32000 rows, 2 states 29.1 /
// 23.5, 8000 rows, 4 states 18.9 / 21.2, 8 states 33.2 / 21.6; groups of 32, 2048 columns, 50280 rows, 3 states 39.7 / 50.2,
// 4 states 51.6 / 50.4.
bool lm_head_q4_mfma_preferred(int d, int V, int N, int group, const uint32_t *qweight) {
    const int lw = qm_words(d, group, qweight);
    if (N < 2 || lw == 0 || qm_lds_bytes(d, group) > kQmLdsBudget) return false;
    const long long wgs = (long long)lm_head_q4_mfma_workgroups(V) * ((N + kQmStates - 1) / kQmStates);
    const float block_ns = lw == 4 ? 5500.f + 3.85f * d : lw == 2 ? 6600.f + 5.5f * d : 6500.f + 9.6f * d;
    const float here = (float)((wgs + 255) / 256 * qm_blocks_per_wg(V)) * block_ns;

    const long long vwgs = (long long)lm_head_q4_workgroups(V) * N;
    const int rows = (V + lm_head_q4_workgroups(V) - 1) / lm_head_q4_workgroups(V);
    const float rows32 = (float)((rows + 31) / 32) * (rows > 64 ? 1.25f : 1.f);
    const float round_ns = 1600.f + 0.56f * d + (1000.f + 1550.f * ((d + 2047) / 2048)) * rows32;
    const float vector = 2500.f + 0.5f * ((float)vwgs / 512 + (float)((vwgs + 511) / 512)) * round_ns;
    return 1.04f * here < vector;
}

template <int LW, bool ARGMAX>
static hipError_t launch_qm(const Q4HeadParams &p, hipStream_t s) {
    const size_t lds = qm_lds_bytes(p.d, p.group);
    auto kern = lm_head_q4_mfma_kernel<LW, ARGMAX>;
    // per launch: the library keeps no state; a refusal shows as the launch error
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    const dim3 grid(lm_head_q4_mfma_workgroups(p.V), (p.N + kQmStates - 1) / kQmStates);
    hipLaunchKernelGGL(kern, grid, dim3(kQmThreads), lds, s, p);
    return hipGetLastError();
}

template <bool ARGMAX>
static hipError_t launch_qm_words(Q4HeadParams &p, hipStream_t s) {
    const int ng = p.d / p.group;
    p.blocks_per_wg = qm_blocks_per_wg(p.V);
    p.vec_scales = ng % 8 == 0 &&
                   ((reinterpret_cast<uintptr_t>(p.scales) | reinterpret_cast<uintptr_t>(p.zeros)) & 15) == 0;
    p.vec_out = p.V % 4 == 0 && (reinterpret_cast<uintptr_t>(p.out) & 15) == 0;
    switch (qm_words(p.d, p.group, p.qweight)) {
        case 4: return launch_qm<4, ARGMAX>(p, s);
        case 2: return launch_qm<2, ARGMAX>(p, s);
        case 1: return launch_qm<1, ARGMAX>(p, s);
        default: return hipErrorInvalidValue;
    }
}

static Q4HeadParams qm_params(int d, int V, float eps, int N, const half_t *hidden, const half_t *gamma,
                              const uint32_t *qweight, const half_t *scales, const half_t *zeros, int group) {
    Q4HeadParams p{};
    p.d = d; p.V = V; p.N = N; p.group = group; p.eps = eps;
    p.hidden = hidden; p.gamma = gamma; p.qweight = qweight; p.scales = scales; p.zeros = zeros;
    return p;
}

hipError_t launch_lm_head_q4_mfma(int d, int V, float eps, int N, const half_t *hidden, const half_t *gamma,
                                  const uint32_t *qweight, const half_t *scales, const half_t *zeros, int group,
                                  float *out, hipStream_t s) {
    Q4HeadParams p = qm_params(d, V, eps, N, hidden, gamma, qweight, scales, zeros, group);
    p.out = out;
    return launch_qm_words<false>(p, s);
}

hipError_t launch_lm_head_q4_mfma_argmax(int d, int V, float eps, int N, const half_t *hidden, const half_t *gamma,
                                         const uint32_t *qweight, const half_t *scales, const half_t *zeros,
                                         int group, float *best_val, int32_t *best_idx, const int32_t *gate,
                                         const int32_t *done, hipStream_t s) {
    Q4HeadParams p = qm_params(d, V, eps, N, hidden, gamma, qweight, scales, zeros, group);
    p.best_val = best_val;
    p.best_idx = best_idx;
    p.gate = gate;
    p.done = done;
    return launch_qm_words<true>(p, s);
}

}  // namespace specee
