// Full LM head for up to 16 hidden states at once (paper Sec. 4.1: the search space that the predictor replaces; Sec. 4.3.3:
// the logits that a verification needs), on the fp16 head or the 4-bit group-quantised one (Sec. 7.1, 7.3):
//     Y[n][v] = r_n * sum_i x[n][i] * W[v][i],   x = h * gamma,
//     quantised  W[v][i] = scale[v][g] * (code[v][i] - zero[v][g]),  g = i / group.
// One pass over the head is all the memory traffic there is, so the kernel is built around the stream:
//   * the hidden dimension is cut over the wavefronts of a workgroup: wavefront w owns CPW chunks of 128 consecutive
//     elements of it (512, or 256 of some quantised heads: hs_chunks_per_wave) for all rows of the workgroup.  The x of its
//     elements -- the same for every row -- is turned into matrix operands once and stays in registers (32 per chunk);
//     nothing is shared between the wavefronts while they stream, so there is neither LDS traffic nor a barrier per stage;
//   * a tile is 16 rows.  A wavefront's 256 bytes per chunk (fp16) or 64 (codes) of each row come in 16-byte loads, each
//     instruction whole 128-byte lines of eight rows, with the non-temporal hint (hs_hint says when); two such loads become
//     the operands of two matrix steps by exchanging halves of 16 lanes.  Every register of a tile is asked for again, for
//     the next tile, as soon as it has been used: a tile per wavefront is in flight all the time, 128 KB per CU of an fp16
//     row of 4096 (eight wavefronts), 80 KB where a row makes five wavefronts (4608, in two passes), 32 KB of codes;
//   * every 2 * CPW tiles (eight or four) the partial sums meet in LDS and are added in ascending order of elements.
// Shorter rows (d <= 2048) leave room for several workgroups on a CU, or for several groups of wavefronts in one workgroup,
// which take the tiles in turn and meet together.
// Longer rows (d > 4096) are done in passes over the workgroup's rows, 4096 elements or less at a time; the sums of
// the passes wait in LDS.
//
// Matrix operands of v_mfma_f32_16x16x32_f16 (lane = 16 * q + c):
//   A = x of state c, cut into two halves, hi = round(h * gamma) and lo = fma(h, gamma, -hi).  First gamma, as far as it
//       stays below 2^15, and then h are scaled up by powers of two (exactly) so that the norm of the wavefront's x comes
//       to between 2^13 and 2^15: the cut loses what lies below 2^-25, 2^-35 of it.  (Each scaled by its own norm, before
//       the product, lost 1e-5 of the logits where large hidden elements meet weights near zero: |h| 3e4 and 0.1, gamma
//       1e-6 and 1; products in 32 bits cost twice the instructions, on codes 1.6 us.);
//   B = 8 elements of row c of the tile.  fp16 head: as loaded.  Quantised head: a byte that holds a code is the fp8
//       (E4M3) number code * 2^-9, so one conversion with scale 2^9 makes two exact halves of two codes: seven
//       instructions per word of eight, in the order 0,2,4,6,1,3,5,7, in which x is built too.  (Codes as subnormal
//       halves, code * 2^-24, need no conversion at all, but the matrix cores align products by their nominal
//       exponents: relative errors of 2.7e-5 instead of 4e-7.);
//   D = lane holds states 4q .. 4q+3 of row c: on the quantised head a lane folds a group's sums with the one scale and
//       zero-point of its own row.
// Quantised groups: a matrix instruction has to stay inside a group.  A lane holds 32 consecutive elements (16 bytes),
// the four lane groups one chunk; with groups of 128 (LW = 4) that is all.  For groups of 64 (LW = 2) words are
// exchanged between the lane groups first (v_permlane32_swap), so that an instruction sees one half of the chunk.
#pragma once
#include <type_traits>

#include "device_utils.h"

namespace specee {

constexpr int kHsStates = 16;
constexpr int kHsTile = 16;    // rows of a tile
constexpr int kHsChunk = 128;  // elements; CPW of them (4 or 2) per wavefront and pass
constexpr int hs_block(int cpw) {  // tiles between two meetings of the wavefronts
    return 2 * cpw;
}
constexpr int kHsMaxChunks = 32;  // of a pass
constexpr int hs_max_waves(int cpw) {
    return kHsMaxChunks / cpw;
}
constexpr int kHsMaxTiles = 32;  // tiles of a workgroup (their sums wait in LDS when there are several passes)

typedef uint32_t uintx4_a4 __attribute__((ext_vector_type(4), aligned(4)));  // codes: rows start at any word

// How a hidden dimension is cut up; `buffers` of partial sums are alternated when they fit.
struct HsShape {
    int cpw, passes, chunks, waves;  // chunks per pass, cpw for each wavefront
    int subs;                        // quantisation sub-chunks per pass (chunks * 4 / LW), 0 on the fp16 head
    int buffers;
    size_t lds;
};

constexpr size_t kHsLds = 156 * 1024;

inline HsShape hs_shape(int d, int lw, int cpw) {
    HsShape s;
    const int nchunks = (d + kHsChunk - 1) / kHsChunk;
    s.cpw = cpw;
    s.passes = (nchunks + kHsMaxChunks - 1) / kHsMaxChunks;
    s.chunks = cpw * ((nchunks + cpw * s.passes - 1) / (cpw * s.passes));
    s.waves = s.chunks / cpw;
    s.subs = lw ? s.chunks * 4 / lw : 0;
    const size_t part = (size_t)s.waves * hs_block(cpw) * kWave * 16;
    size_t rest = (size_t)2 * s.waves * kHsStates * 4;  // sums of squares, scales
    rest += (size_t)s.subs * kHsStates * 4;             // sums of x
    if (s.passes > 1) rest += (size_t)kHsMaxTiles * kWave * 16;
    s.buffers = 2 * part + rest <= kHsLds ? 2 : 1;
    s.lds = s.buffers * part + rest;
    return s;
}

struct HsParams {
    int d, V, passes, chunks, subs, buffers;
    float eps;
    const half_t *gamma;
    const half_t *lm_head;    // fp16 head, or
    const uint32_t *qweight;  // the quantised one
    const half_t *scales, *zeros;
    int group;  // 128 or 64
};

// the eight codes of a word as eight halves (see above): elements 0, 2, 4, 6, 1, 3, 5, 7
__device__ __forceinline__ half8 hs_codes(uint32_t w) {
    const uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;
    uintx4 o;
    o[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 512.f, false));
    o[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 512.f, true));
    o[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 512.f, false));
    o[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 512.f, true));
    return __builtin_bit_cast(half8, o);
}

// the same order for eight elements of x
__device__ __forceinline__ half8 hs_code_order(half8 v) {
    return half8{v[0], v[2], v[4], v[6], v[1], v[3], v[5], v[7]};
}

// The lane number as something new: what is derived from it is derived here, and not once for the whole kernel and kept
// in registers that the rows need.
__device__ __forceinline__ int hs_opaque(int lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}

// b with |v| < 2^b for every v whose square is part of the sum ssq (what is not finite counts as large)
__device__ __forceinline__ int hs_bound(float ssq) {
    return ((int)(__builtin_bit_cast(uint32_t, ssq) >> 23) - 127 + 2) >> 1;
}

// Sum over the four lane groups: lanes (0, c) ... (3, c), in all of them, on the vector units.
__device__ __forceinline__ float hs_over_q(float v) {
    const uint32_t a = __builtin_bit_cast(uint32_t, v);
    const auto s = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const uint32_t s0 = s[0], s1 = s[1];  // (a bit cast of an element of a vector reads its first one)
    const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, s0) + __builtin_bit_cast(float, s1));
    const auto t = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    const uint32_t t0 = t[0], t1 = t[1];
    return __builtin_bit_cast(float, t0) + __builtin_bit_cast(float, t1);
}

// LW = 2: words between lane groups, so that word j holds elements of sub-chunk j / LW only
template <int LW>
__device__ __forceinline__ void hs_exchange(uint32_t (&w)[4]) {
    if constexpr (LW == 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const auto s = __builtin_amdgcn_permlane32_swap(w[j], w[j + 2], false, false);
            w[j] = s[0];
            w[j + 2] = s[1];
        }
    }
}

// first of the eight elements, within its chunk, that lane group q multiplies in step j
template <int LW>
__device__ __forceinline__ int hs_element(int j, int q) {
    if (LW == 4) return 32 * q + 8 * j;
    if (LW == 2) return 64 * (j >> 1) + 8 * (j & 1) + 32 * (q & 1) + 16 * (q >> 1);
    return 32 * j + 8 * q;  // fp16 head: 64 contiguous bytes of a row
}

// Logits of rows [16 * tile_begin, 16 * tile_end) (tile_begin < tile_end, at most kHsMaxTiles tiles if there are several
// passes) for 16 states, by the whole workgroup of row_groups * chunks / CPW wavefronts (row_groups a power of two, at
// most hs_block(CPW)): state_row(n) is the hidden state of slot n, valid for n < 16.
// emit(row, n, y) is called by the lanes of the first wavefronts, all of a wavefront's lanes together and rows ascending
// for each lane: row may lie past the end (>= V), y[r] is the logit of state n + r, n = 4 * (lane / 16).
// LW: 0 = fp16 head, else the group is 32 * LW.  RAGGED: rows end before the passes do (d != passes * chunks * 128).
// NT: the rows are read with the non-temporal hint.
template <int LW, int CPW, bool RAGGED, bool NT, class StateRow, class Emit>
__device__ __forceinline__ void head_states_rows(const HsParams &p, unsigned char *smem, int row_groups, int tile_begin,
                                                 int tile_end, StateRow state_row, Emit emit) {
    constexpr bool Q4 = LW != 0;
    constexpr int kHsBlock = hs_block(CPW);
    constexpr int kSteps = CPW * 4;            // matrix steps of a tile
    constexpr int kLoads = Q4 ? CPW : kSteps;  // 16-byte loads of a tile
    // Matrix steps added up in a row, fp16 head; what they come to waits in LDS.  (Error against float64 for 16 / 8 / 4 steps,
    // d = 4096: 1.5e-7 / 1.2e-7 / 1.0e-7, the vector kernel's 1.1e-7; 32000 x 4096, verification of 16 states 50.4 / 50.4 /
    // 51.1 us, layer loop of one token 56.6 / 57.6 / 57.8.  LDS additions in place of the reads: 61 and 68.)
    constexpr int kChain = 4;
    constexpr int kDepth = 1;                  // tiles in flight (two or four, with codes: no gain)
    constexpr int kSpw = Q4 ? CPW * 4 / (Q4 ? LW : 1) : 1;  // sub-chunks of a wavefront
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int W = p.chunks / CPW, G = row_groups;
    const int wg_wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = row_groups == 1 ? 0 : wg_wave / W, wave = wg_wave - group * W;
    const int c = lane & 15, q = lane >> 4;
    const int d = p.d, ng = Q4 ? d / (32 * LW) : 1;

    floatx4 *part = reinterpret_cast<floatx4 *>(smem);  // [buffers][W][kHsBlock][64 lanes]
    float *ssq_lds = reinterpret_cast<float *>(part + (size_t)p.buffers * W * kHsBlock * kWave);  // [W][16]
    float *unscale_lds = ssq_lds + W * kHsStates;                                                  // [W][16]
    float *tx = unscale_lds + W * kHsStates;                                                      // [subs][16]
    floatx4 *acc_lds = reinterpret_cast<floatx4 *>(tx + (size_t)p.subs * kHsStates);              // [tiles][64]

    const half_t *hrow = state_row(c);
    float ssq_total = 0.f;
    for (int pass = 0; pass < p.passes; ++pass) {
        const int e0 = (pass * p.chunks + wave * CPW) * kHsChunk;  // this wavefront's first element
        // an element past the end of the row meets x = 0; its load is clamped into the row
        uintx4 a[kDepth][kLoads];
        // (a uniform base and a 32-bit offset, the same for all loads of a row: few registers)
        const uint32_t row_bytes = Q4 ? (uint32_t)d >> 1 : (uint32_t)d * 2;
        const int e0c = e0 < d ? e0 : 0;
        const char *head = reinterpret_cast<const char *>(Q4 ? (const void *)p.qweight : (const void *)p.lm_head) +
                           (Q4 ? e0c >> 1 : e0c * 2);
        const uint32_t limit = Q4 ? (uint32_t)(d - 32 - e0c) >> 1 : (uint32_t)(d - 8 - e0c) * 2;  // of a piece's offset
        auto load_pair = [&](int t, int slot, int i) {  // loads 2i, 2i + 1: 128 bytes of each row
            // Past the last tile all rows are the start of the weight: a branch around the loads would make the compiler wait
            // for too much, and the last tile asked for again came from memory again, with the hint.
            const bool real = t < tile_end;
            const char *base = real ? head + (size_t)t * kHsTile * row_bytes : reinterpret_cast<const char *>(p.gamma);
            const int last = real ? p.V - 1 - t * kHsTile : 0;
            const int ln = RAGGED ? hs_opaque(lane) : lane;
            const uint32_t piece = 16 * ((ln >> 4) + 4 * (ln >> 3 & 1));
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t row = (uint32_t)min((ln & 7) + 8 * u, last) * row_bytes;
                const char *at = RAGGED ? base + (row + min(piece + 128 * i, limit)) : base + (row + piece) + 128 * i;
                typedef std::conditional_t<Q4, uintx4_a4, uintx4> piece_t;
                if constexpr (NT)
                    a[slot][2 * i + u] = __builtin_nontemporal_load(reinterpret_cast<const piece_t *>(at));
                else
                    a[slot][2 * i + u] = *reinterpret_cast<const piece_t *>(at);
            }
        };
        // scales and zero-points of this wavefront's groups of row c of a tile: side by side in memory, one load each (of any
        // alignment), or one by one where the row may end among them
        typedef half_t scales_t __attribute__((ext_vector_type(kSpw), aligned(2)));
        scales_t sc[kDepth], zp[kDepth];
        auto load_scales = [&](int t, int slot) {
            const int ln = hs_opaque(lane);
            const bool real = t < tile_end;
            const size_t tile_at = real ? (size_t)t * kHsTile * ng : 0;
            const half_t *sbase = p.scales + tile_at, *zbase = p.zeros + tile_at;
            const uint32_t row = (uint32_t)min(ln & 15, real ? p.V - 1 - t * kHsTile : 0) * ng;
            if constexpr (RAGGED) {
#pragma unroll
                for (int i = 0; i < kSpw; ++i) {
                    const uint32_t g = (uint32_t)min(e0 / (32 * LW) + i, ng - 1);
                    sc[slot][i] = sbase[row + g];
                    zp[slot][i] = zbase[row + g];
                }
            } else {
                const uint32_t g = (uint32_t)e0 / (32 * LW);
                sc[slot] = *reinterpret_cast<const scales_t *>(sbase + (row + g));
                zp[slot] = *reinterpret_cast<const scales_t *>(zbase + (row + g));
            }
        };

        // ---- x of this wavefront's elements as matrix operands
        half8 xh[kSteps], xl[kSteps];
        auto element = [&](int i) { return e0 + (i >> 2) * kHsChunk + hs_element<LW>(i & 3, q); };
        const half_t *hbase = hrow + (RAGGED ? 0 : e0 + hs_element<LW>(0, q)), *gbase = p.gamma + (RAGGED ? 0 : e0 + hs_element<LW>(0, q));
        auto load_x = [&]() {  // hidden state and weight, side by side in xh and xl
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                // (from one base with constant offsets, where nothing has to be clamped: what does not fit into registers
                // here comes back from memory behind the first tile)
                const int e = RAGGED ? min(element(i), d - 8) : (i >> 2) * kHsChunk + hs_element<LW>(i & 3, 0);
                xh[i] = load_half8(hbase + e);
                xl[i] = load_half8(gbase + e);
            }
        };
        auto store_tx = [&](int i, float sum) {  // a sub-chunk's sum of x is complete; only this wavefront reads it
            sum = hs_over_q(sum);
            if (q == 0) tx[(wave * kSpw + i / (Q4 ? LW : 1)) * kHsStates + c] = sum;
        };
        // the hidden states and the weight are asked for before the rows: loads come back in order, and the operands are made
        // of them while the first rows are on their way
        const half8 gamma8 = load_half8(p.gamma + min(e0 + (lane * 8) % (CPW * kHsChunk), d - 8));  // the share's, once
        load_x();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < kDepth; ++s) {
            const int t = tile_begin + group + s * G;
#pragma unroll
            for (int i = 0; i < kLoads / 2; ++i) load_pair(t, s, i);
            if constexpr (Q4) load_scales(t, s);
        }
        __builtin_amdgcn_sched_barrier(0);
        {
            float ssq = 0.f, ssx = 0.f, ssg = 0.f;
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const half2_t g = {gamma8[e], gamma8[e + 1]};
                ssg = __builtin_amdgcn_fdot2(g, g, ssg, false);
            }
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                if (RAGGED) xh[i] = element(i) < d ? xh[i] : zero_half8();
                float some = 0.f;  // (short chains: all logits of a state share this sum's error)
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const half2_t h = {xh[i][e], xh[i][e + 1]}, x = h * half2_t{xl[i][e], xl[i][e + 1]};
                    some = __builtin_amdgcn_fdot2(h, h, some, false);
                    ssx = __builtin_amdgcn_fdot2(x, x, ssx, false);
                }
                ssq += some;
            }
            ssq = hs_over_q(ssq);
            ssx = hs_over_q(ssx);
            if (__builtin_expect(__any(!(ssx < INFINITY)), 0)) {  // a product that is no half
                ssx = 0.f;
#pragma unroll
                for (int i = 0; i < kSteps; ++i)
#pragma unroll
                    for (int e = 0; e < 8; e += 2) {
                        constexpr half2_t down = {0x1p-9, 0x1p-9};
                        const half2_t x = half2_t{xh[i][e], xh[i][e + 1]} * down * (half2_t{xl[i][e], xl[i][e + 1]} * down);
                        ssx = __builtin_amdgcn_fdot2(x, x, ssx, false);
                    }
                ssx = 0x1p36f * hs_over_q(ssx);
            }
            ssg = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_sum_to_last_row(ssg)), kWave - 1));
            // |x * 2^u| < 2^15 by the norm; of it as much through gamma as leaves that below 2^15 too, the rest through h
            const int u = max(-18, 15 - hs_bound(ssx));
            const int ug = max(0, min(min(u, 15), 15 - hs_bound(ssg))), uh = min(u - ug, max(0, min(15, 15 - hs_bound(ssq))));
            if (q == 0) {
                ssq_lds[wave * kHsStates + c] = ssq;
                unscale_lds[wave * kHsStates + c] = __builtin_bit_cast(float, (uint32_t)(127 - uh - ug) << 23);
            }
            const half_t sh = (half_t)__builtin_bit_cast(float, (uint32_t)(127 + uh) << 23);
            const half_t sg = (half_t)__builtin_bit_cast(float, (uint32_t)(127 + ug) << 23);
            const half2_t s_h = {sh, sh}, s_g = {sg, sg};
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                half8 hi, lo;
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const half2_t h = half2_t{xh[i][e], xh[i][e + 1]} * s_h, g = half2_t{xl[i][e], xl[i][e + 1]} * s_g;
                    const half2_t x = h * g, rest = __builtin_elementwise_fma(h, g, -x);
                    if (Q4) sum = __builtin_amdgcn_fdot2(h, g, sum, false);
                    hi[e] = x[0];
                    hi[e + 1] = x[1];
                    lo[e] = rest[0];
                    lo[e + 1] = rest[1];
                }
                xh[i] = Q4 ? hs_code_order(hi) : hi;
                xl[i] = Q4 ? hs_code_order(lo) : lo;
                if (Q4 && (i + 1) % (Q4 ? LW : 1) == 0) {
                    store_tx(i, sum);
                    sum = 0.f;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // ---- the rows
        float rms = 0.f;  // of state c, once the wavefronts have met
        int buf = 0;
        for (int tb = tile_begin; tb < tile_end; tb += kHsBlock) {
            const int nb = min(kHsBlock, tile_end - tb);
            const int pbuf = p.buffers == 2 ? buf : 0;
            auto tile = [&](int i, int slot) {
                const int tn = tb + i + kDepth * G;
                const int ln = hs_opaque(lane), tq = ln >> 4;
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                if constexpr (Q4) {
#pragma unroll
                    for (int ch = 0; ch < CPW; ++ch) {
                        if (ch % 2 == 0) whole_lines(a[slot][ch], a[slot][ch + 1]);
                        uint32_t w[4] = {a[slot][ch][0], a[slot][ch][1], a[slot][ch][2], a[slot][ch][3]};
                        hs_exchange<LW>(w);
#pragma unroll
                        for (int s = 0; s < 4 / LW; ++s) {
                            floatx4 tmp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int j = s * LW; j < (s + 1) * LW; ++j) {
                                const half8 b = hs_codes(w[j]);
                                tmp = __builtin_amdgcn_mfma_f32_16x16x32_f16(xh[ch * 4 + j], b, tmp, 0, 0, 0);
                                tmp = __builtin_amdgcn_mfma_f32_16x16x32_f16(xl[ch * 4 + j], b, tmp, 0, 0, 0);
                            }
                            const int sub = ch * (4 / LW) + s;
                            const float s_f = (float)sc[slot][sub], z_f = (float)zp[slot][sub];
                            const floatx4 t4 =
                                *reinterpret_cast<const floatx4 *>(tx + (wave * kSpw + sub) * kHsStates + 4 * tq);
#pragma unroll
                            for (int r = 0; r < 4; ++r) acc[r] += s_f * (tmp[r] - z_f * t4[r]);
                        }
                        if (ch % 2 == 1) load_pair(tn, slot, ch / 2);
                        // (without this the scheduler asks for the whole next tile at once, into other registers)
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    load_scales(tn, slot);
                } else {
                    floatx4 acc1 = {0.f, 0.f, 0.f, 0.f};
                    auto cell = [&]() { return part + ((pbuf * W + wave) * kHsBlock + i) * kWave + hs_opaque(lane); };
#pragma unroll
                    for (int k = 0; k < kSteps; k += 2) {
                        if (k > 0 && k % kChain == 0) {
                            floatx4 *at = cell();
                            *at = k == kChain ? acc : *at + acc;
                            acc = floatx4{0.f, 0.f, 0.f, 0.f};
                        }
                        whole_lines(a[slot][k], a[slot][k + 1]);
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            half8 b = __builtin_bit_cast(half8, a[slot][k + u]);
                            // (only the wavefront at the end of a row; what it read there is other elements of the row)
                            if (RAGGED && e0 + CPW * kHsChunk > d)
                                b = e0 + ((k + u) >> 2) * kHsChunk + hs_element<LW>((k + u) & 3, tq) < d ? b : zero_half8();
                            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(xh[k + u], b, acc, 0, 0, 0);
                            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(xl[k + u], b, acc1, 0, 0, 0);
                        }
                        load_pair(tn, slot, k / 2);
                        // (without this the scheduler asks for the whole next tile at once, into other registers)
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    acc += *cell();
                    // (hi * infinity has its sign, lo * infinity may be NaN)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[r] += __builtin_isinf(acc[r]) ? 0.f : acc1[r];
                }
                acc *= *reinterpret_cast<const floatx4 *>(unscale_lds + wave * kHsStates + 4 * tq);
                part[((pbuf * W + wave) * kHsBlock + i) * kWave + ln] = acc;
            };
            static_assert(kDepth == 1, "a block starts with slot 0");
            for (int i = group; i < nb; i += G) tile(i, 0);
            __syncthreads();
            if (tb == tile_begin) {
                for (int w = 0; w < W; ++w) ssq_total += ssq_lds[w * kHsStates + c];
                rms = 1.0f / sqrtf(ssq_total / (float)d + p.eps);  // (used in the last pass)
            }
            for (int i = wg_wave; i < nb; i += G * W) {
                const int ln = hs_opaque(lane), lq = ln >> 4;
                const floatx4 *src = part + (pbuf * W * kHsBlock + i) * kWave + ln;
                double sum[4] = {};  // (a few additions per logit)
#pragma unroll 4
                for (int w = 0; w < W; ++w)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sum[r] += (double)src[w * kHsBlock * kWave][r];
                floatx4 y = {(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
                if (p.passes > 1) {
                    floatx4 *at = acc_lds + (tb - tile_begin + i) * kWave + ln;  // this lane's own cell
                    if (pass > 0) y += *at;
                    if (pass < p.passes - 1) *at = y;
                }
                if (pass == p.passes - 1) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[r] *= __shfl(rms, 4 * lq + r, kWave);
                    emit((tb + i) * kHsTile + (ln & 15), 4 * lq, y);
                }
            }
            // one buffer: read before the next block writes it (two: the next meeting comes before the block after)
            if (p.buffers == 1) __syncthreads();
            buf ^= 1;
        }
        __syncthreads();  // the next pass writes what the last block read
    }
}

// Words of codes per lane: groups of 128 and 64 (0: fp16 head; -1: not done here).
inline int hs_words(int group) {
    return group == 0 ? 0 : group == 128 ? 4 : group == 64 ? 2 : -1;
}

// Chunks of 128 elements per wavefront.  fp16 head: four (two: 32000 x 4096, 16 states 48.7 -> 58 us, 50280 x 2048 42 -> 55).
// Codes: four, if that gives whole multiples of four wavefronts, one for each SIMD, or else two, which gives more and
// leaves less of the last one idle (four / two, 16 states, groups of 128: 32000 x 4096 25.1 / 27.2 us, 50280 x 2048
// 21.5 / 24.2, 32000 x 8192 46.9 / 52.4; 24001 x 4608 36.2 / 27.5, 32000 x 5120 38.0 / 34.5, 32003 x 3072 21.6 / 20.8).
inline int hs_chunks_per_wave(int d, int lw) {
    if (lw == 0) return 4;
    const HsShape sh = hs_shape(d, lw, 4);
    return sh.waves % 4 == 0 && d == sh.passes * sh.chunks * kHsChunk ? 4 : 2;
}

// The hint (us, without / with it).  Only rows of whole 128-byte lines: where a line holds the end of one row and the start
// of the next, the second load that needs it asks memory for it again (fp16, 20011 x 4104, verification of 16 states 62.1
// / 70.3 from memory, 51.0 / 66.6 from the cache, layer loop of one token 56.1 / 61.1, 32001 x 3080 54.3 / 65.0; codes,
// 40000 x 4160, groups of 64, 50.6 / 51.9 and 46.0 / 51.2, 40000 x 4224, groups of 128, 43.7 / 45.2 and 37.8 / 42.0).
// fp16 heads gain wherever they come from memory and lose little where not (16 states, 50280 x 2048 46.9 / 42.0; 16000 x
// 2048, one head after the other 20.2 / 18.4, few heads that stay in the last-level cache 17.2 / 18.0).  Codes: a head is a
// quarter of that, and how much of it that cache still holds at the next verification depends on what the program does in
// between.  The line is where neither side loses much: groups of 128, from the cache and from memory, 32000 x 4096 22.8 /
// 25.5 and 25.5 / 24.7, 24001 x 4608 25.6 / 28.0 and 28.6 / 28.2, 40000 x 4096 24.2 / 27.1 and 29.4 / 28.4, 32000 x 8192
// 49.6 / 47.3 and 50 / 47; groups of 64, 32000 x 5120 39.6 / 39.1 and 40.8 / 39.0.
inline bool hs_hint(int d, int V, int lw) {
    return lw == 0 ? d % 64 == 0 : d % 256 == 0 && (size_t)V * d / 2 > ((size_t)72 << 20);
}

// f(LW, CPW, RAGGED, NT as integral constants, shape) for a head (group 0: fp16)
template <class F>
hipError_t hs_dispatch(int d, int V, int group, F f) {
    const int lw = hs_words(group);
    if (lw < 0) return hipErrorInvalidValue;
    const int cpw = hs_chunks_per_wave(d, lw);
    const HsShape sh = hs_shape(d, lw, cpw);
    const bool ragged = d != sh.passes * sh.chunks * kHsChunk;
    std::integral_constant<int, 0> w0;
    std::integral_constant<int, 2> two;
    std::integral_constant<int, 4> four;
    std::false_type no;
    std::true_type yes;
    const bool hint = hs_hint(d, V, lw);
    if (lw == 0) return !ragged ? f(w0, four, no, yes, sh) : hint ? f(w0, four, yes, yes, sh) : f(w0, four, yes, no, sh);
    auto codes = [&](auto w, auto nt) {
        return cpw == 4 ? f(w, four, no, nt, sh) : ragged ? f(w, two, yes, nt, sh) : f(w, two, no, nt, sh);
    };
    return lw == 4 ? (hint ? codes(four, yes) : codes(four, no)) : hint ? codes(two, yes) : codes(two, no);
}

}  // namespace specee
