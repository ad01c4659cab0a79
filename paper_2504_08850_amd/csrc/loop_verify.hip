// The early-exit decode loop of a batch of tokens down the layer stack (paper Sec. 4.3.3 dataflow -- predict, verify
// after a positive prediction, leave the model at the first accepted verification -- with the active-predictor set of the
// scheduler, Sec. 5.3), in two launches:
//   * the predictors of all active layers of all tokens, side by side (launch_loop_scores).  Nothing in a predictor hangs
//     on a verification -- the probabilities of the layer before are carried on whether or not it fired -- and every
//     layer's hidden state exists before the call, so the layers need not wait for each other: one trip through the
//     predictor (about 4 us) instead of 1.75 us per evaluated layer.  What was scored after a token's exit is taken
//     back below;
//   * here: the verifications.  One persistent grid serves all tokens.  It takes up to 16 of the (layer, token) pairs
//     that fired and are still open -- of every token in turn, its next layers in order -- and makes ONE pass over the
//     head for all of them (head_states.h: the time of a pass hardly depends on the number of states).  Every
//     workgroup takes a share of the rows and leaves its arg-max per state in the workspace (a device-scope maximum over
//     keys that order by logit, then by lowest row).  The last one to arrive reads the winners, looks for them among the
//     ids, and notes for everybody which states hit; all workgroups draw the same conclusions from the note.  A token whose
//     winner is one of its ids leaves at that layer; pairs of its later layers in the same pass count for nothing.
//     The notes lie 128 bytes apart, one per four or eight workgroups: with all of them polling the counter itself, the
//     memory channel that holds it was slow for the others' rows too, and the meeting took 6 us (512 workgroups: 9 us).
// Most tokens are decided in the first pass, where verifying layer by layer took one pass per fired layer and token
// (32000 x 4096, one token, 32 layers, exit at the one that fires: 64.7 -> 58.7 us; eleven that fire 511 -> 59 us).
// Bound by the pass over the head: 46 us of it are the stream (5.7 TB/s), 5 the scores, 2 go by until the first states are
// known and 5 from the last row to the end of the kernel (arrival, winners, note, outputs).
// The meeting needs every workgroup to be resident: the host sizes the grid from the occupancy that the runtime reports,
// and every wait is bounded (spin limit), so a grid that cannot meet (another kernel holds the CUs) ends with status 1
// for the tokens that are still open, instead of hanging.
#include "head_states.h"
#include "kernels.h"

namespace specee {

constexpr int kLoopTokens = 64;

struct LoopVerifyParams {
    HsParams hs;
    int row_groups;
    LoopParams lp;
};

// Keys order by value, then by lowest row; 0 is "nothing yet".  (A zero is made positive; NaN is never a candidate.)
__device__ __forceinline__ unsigned long long arg_max_key(float v, int row) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v + 0.f);
    const uint32_t up = u >> 31 ? ~u : u | 0x80000000u;
    return (unsigned long long)up << 32 | (uint32_t)~row;
}

// The arguments, read where they are used: kept in scalar registers from the start of the kernel on, they crowd out the
// stream's (and what does not fit goes to vector lanes and to memory).
__device__ __forceinline__ const LoopParams &loop_args() {
    auto at = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return ((const LoopVerifyParams *)at)->lp;
}

template <int LW, int CPW, bool RAGGED, bool NT>
__global__ __launch_bounds__(hs_max_waves(CPW) * kWave) void loop_verify_kernel(LoopVerifyParams p) {
    constexpr int kBlock = hs_block(CPW);
    extern __shared__ __attribute__((aligned(16))) unsigned char hs_smem[];
    __shared__ unsigned long long open_lds[kLoopTokens];  // fired, not yet verified layers of the window, per token
    __shared__ int exit_lds[kLoopTokens], token_lds[kLoopTokens], fail_lds[kLoopTokens];
    __shared__ int sel_l[kHsStates], sel_b[kHsStates];
    __shared__ int nsel_lds, met_lds;
    __shared__ float cand_v[kBlock][kHsStates];
    __shared__ int cand_i[kBlock][kHsStates];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = blockDim.x >> 6;
    const int B = p.lp.B, L = p.lp.L, V = p.hs.V;
    const bool writer = blockIdx.x == 0;  // writes all outputs
    const int tiles = (V + kHsTile - 1) / kHsTile;
    const int t_begin = (int)((long long)tiles * blockIdx.x / gridDim.x);
    const int t_end = (int)((long long)tiles * (blockIdx.x + 1) / gridDim.x);
    if (tid < kLoopTokens) exit_lds[tid] = token_lds[tid] = fail_lds[tid] = -1;
    int passes = 0;       // over the head so far: the arrival counter stands at passes * gridDim.x afterwards
    bool failed = false;  // a meeting did not come about

    for (int base = 0; base < L; base += kWave) {
        __syncthreads();
        const LoopParams &lp = loop_args();
        for (int b = wave; b < B; b += W) {
            const int lane = tid & (kWave - 1), l = base + lane;
            const int fired = l < L ? lp.exit_flags[(size_t)l * B + b] : 0;
            const unsigned long long m = __ballot(fired != 0);
            if (lane == 0) open_lds[b] = exit_lds[b] < 0 && fail_lds[b] < 0 ? m : 0;
        }
        __syncthreads();
        while (!failed) {
            if (wave == 0) {  // rounds over the tokens, lane b for token b: its next open layer
                const int lane = hs_opaque(threadIdx.x);
                unsigned long long m = lane < B ? open_lds[lane] : 0;
                int n = 0;
                while (n < kHsStates) {
                    const unsigned long long some = __ballot(m != 0);
                    if (!some) break;
                    const int at = n + (int)__builtin_popcountll(some & ((1ull << lane) - 1));
                    if (m && at < kHsStates) {
                        sel_b[at] = lane;
                        sel_l[at] = base + (int)__builtin_ctzll(m);
                    }
                    m &= m - 1;
                    n += (int)__builtin_popcountll(some);
                }
                if (lane == 0) nsel_lds = min(n, kHsStates);
            }
            __syncthreads();
            const int ns = nsel_lds;
            if (ns == 0) break;

            // ---- one pass over this workgroup's rows
            float bv[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            int bi[4] = {0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff};
            // (several passes over the rows: the sums of as many tiles wait in LDS as there is room for)
            const int most = p.hs.passes > 1 ? kHsMaxTiles : t_end - t_begin;
            for (int t = t_begin; t < t_end; t += most)
                head_states_rows<LW, CPW, RAGGED, NT>(
                    p.hs, hs_smem, p.row_groups, t, min(t + most, t_end),
                    [&](int n) {
                        const int at = n < ns ? n : 0;
                        return p.lp.hidden + ((size_t)sel_l[at] * B + sel_b[at]) * p.hs.d;
                    },
                    [&](int row, int n, floatx4 y) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (row < V && y[r] > bv[r]) {  // rows ascend: strict '>' keeps the lowest row on ties
                                bv[r] = y[r];
                                bi[r] = row;
                            }
                    });
            const int ncand = min(kBlock, W);
            if (wave < ncand) {
                const int lane = hs_opaque(threadIdx.x) & (kWave - 1);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    row16_argmax(bv[r], bi[r]);
                    if ((lane & 15) == 0) {
                        cand_v[wave][4 * (lane >> 4) + r] = bv[r];
                        cand_i[wave][4 * (lane >> 4) + r] = bi[r];
                    }
                }
            }
            __syncthreads();

            // ---- the grid's winners
            if (wave == 0) {
                const LoopParams &lp = loop_args();
                const int lane = hs_opaque(threadIdx.x);
                const int n = lane & 15, part = lane >> 4;  // four lanes per state
                const int b = sel_b[n < ns ? n : 0], l = sel_l[n < ns ? n : 0];
                const int32_t *ids = lp.ids + (size_t)b * lp.K;
                int32_t early[4];  // the deciding workgroup looks for the winner among them
#pragma unroll
                for (int j = 0; j < 4; ++j) early[j] = ids[min(part + 4 * j, lp.K - 1)];
                float v = -INFINITY;
                int i = 0x7fffffff;
                for (int w = part; w < ncand; w += 4)
                    if (cand_v[w][n] > v || (cand_v[w][n] == v && cand_i[w][n] < i)) {
                        v = cand_v[w][n];
                        i = cand_i[w][n];
                    }
#pragma unroll
                for (int off = 16; off <= 32; off <<= 1) {
                    const float ov = __shfl_xor(v, off, kWave);
                    const int oi = __shfl_xor(i, off, kWave);
                    if (ov > v || (ov == v && oi < i)) {
                        v = ov;
                        i = oi;
                    }
                }
                unsigned long long *set = lp.lines + (size_t)(passes % 3) * kHsStates * kLoopLine;
                if (lane < ns && i != 0x7fffffff)
                    (void)__hip_atomic_fetch_max(set + lane * kLoopLine, arg_max_key(v, i), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // they have landed where every XCD reads them
                unsigned at = 0;
                if (lane == 0) at = (unsigned)__hip_atomic_fetch_add(lp.arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const bool last = (unsigned)__builtin_amdgcn_readfirstlane((int)at) + 1 == (unsigned)(passes + 1) * gridDim.x;
                unsigned long long *notes = lp.lines + kLoopKeys * kLoopLine;
                const unsigned long long pass_no = (unsigned long long)(passes + 1) << kHsStates;
                unsigned long long note = 0;  // number of the pass, and below it one bit per state: its winner is an id
                auto winner = [&]() {
                    const unsigned long long key =
                        __hip_atomic_load(set + n * kLoopLine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    return key ? (int)~(uint32_t)key : 0x7fffffff;
                };
                if (last) {
                    const int win = winner();
                    int hit = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) hit |= early[j] == win;
                    for (int k = part + 16; k < lp.K; k += 4) hit |= ids[k] == win;
                    hit |= __shfl_xor(hit, 16, kWave);
                    hit |= __shfl_xor(hit, 32, kWave);
                    note = pass_no | (__ballot(hit != 0) & ((1ull << ns) - 1));
                    // the slots of the pass before, which are used again two passes on, are cleared now: who reads them has
                    // done so before coming here, and who writes them then has heard of the next pass first
                    if (lane < kHsStates)
                        __hip_atomic_store(lp.lines + ((size_t)((passes + 2) % 3) * kHsStates + lane) * kLoopLine, 0ull,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    static_assert(kLoopNotes == kWave, "one lane each");
                    __hip_atomic_store(notes + lane * kLoopLine, note, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else if (lane == 0) {
                    const unsigned long long *mine = notes + (blockIdx.x % kLoopNotes) * kLoopLine;
                    for (long long it = 0; it < lp.spin_limit; ++it) {
                        note = __hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (note >= pass_no) break;
                        note = 0;
                        if (it % 16 == 15 &&
                            __hip_atomic_load(lp.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
                            break;
                        __builtin_amdgcn_s_sleep(4);
                    }
                    if (note == 0) __hip_atomic_store(lp.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                note = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(note >> 32)) << 32 |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)note);
                if (lane == 0) met_lds = note != 0;
                if (note != 0) {
                    const int hits = (int)note & ((1 << kHsStates) - 1);
                    bool counts = lane < ns;  // no earlier layer of the token has been accepted
                    for (int m = 0; m < ns; ++m)
                        if (hits >> m & 1 && sel_b[m] == b && sel_l[m] < l) counts = false;
                    if (counts) {
                        const int hit = hits >> n & 1;
                        if (writer) {
                            const int win = winner();
                            lp.ver_token[(size_t)l * B + b] = win;
                            lp.hit[(size_t)l * B + b] = hit;
                            if (hit) token_lds[b] = win;
                        }
                        if (hit) exit_lds[b] = l;
                    }
                    __builtin_amdgcn_wave_barrier();
                    if (lane < B) {
                        unsigned long long m = open_lds[lane];
                        for (int i = 0; i < ns; ++i)
                            if (sel_b[i] == lane) m &= ~(1ull << (sel_l[i] - base));
                        open_lds[lane] = exit_lds[lane] < 0 ? m : 0;
                    }
                }
            }
            __syncthreads();
            if (!met_lds) failed = true;  // uniform
            ++passes;
        }
        // a token that still has an open layer when the grid fails to meet ends there
        if (failed && tid < B && open_lds[tid]) fail_lds[tid] = base + (int)__builtin_ctzll(open_lds[tid]);
        const bool closed = tid >= B || exit_lds[tid] >= 0 || fail_lds[tid] >= 0;
        if (__syncthreads_and(closed)) break;
    }

    // ---- what was scored but not evaluated: layers after the exit, or from a failed meeting on
    if (!writer) return;
    const LoopParams &lp = loop_args();
    __syncthreads();
    for (size_t i = tid; i < (size_t)L * B; i += blockDim.x) {
        const int l = (int)(i / B), b = (int)(i - (size_t)l * B);
        const int end = fail_lds[b] >= 0 ? fail_lds[b] : exit_lds[b] >= 0 ? exit_lds[b] + 1 : L;
        if (l < end) continue;
        lp.scores[i] = 0.f;
        lp.exit_flags[i] = 0;
        for (int k = 0; k < lp.K; ++k) {
            lp.logits[i * lp.K + k] = 0.f;
            lp.probs[i * lp.K + k] = 0.f;
        }
    }
    if (tid < B) {
        lp.exit_layer[tid] = exit_lds[tid];
        lp.token[tid] = token_lds[tid];
        lp.status[tid] = fail_lds[tid] >= 0 ? 1 : 0;
    }
}

template <int LW, int CPW, bool RAGGED, bool NT>
static hipError_t launch_lv(LoopVerifyParams &p, const HsShape &sh, int max_wgs, hipStream_t s) {
    p.hs.passes = sh.passes; p.hs.chunks = sh.chunks; p.hs.subs = sh.subs; p.hs.buffers = sh.buffers;
    auto kern = loop_verify_kernel<LW, CPW, RAGGED, NT>;
    // per launch: the library keeps no state; a refusal shows as the launch error
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh.lds);
    // every workgroup must be resident while the grid meets: sized from what the runtime says fits on the device
    // (one workgroup per CU: of two, short rows, the older one streamed and the other came after it, and twice as many
    // had to meet: 50280 x 2048, one verification 53.9 us, with two groups of wavefronts in a workgroup instead 46.0)
    const int tiles = (p.hs.V + kHsTile - 1) / kHsTile;
    int dev = 0, cus = 0, per_cu = 0;
    p.row_groups = 1;
    while (2 * p.row_groups * sh.waves <= hs_max_waves(CPW) && p.row_groups < hs_block(CPW) && p.row_groups * 256 < tiles)
        p.row_groups *= 2;
    const int threads = p.row_groups * sh.waves * kWave;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern), threads, sh.lds);
    if (e != hipSuccess) return e;
    int wgs = per_cu > 0 ? cus : 0;
    if (wgs > max_wgs) wgs = max_wgs;
    if (wgs > tiles) wgs = tiles;
    if (wgs < 1) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(threads), sh.lds, s, p);
    return hipGetLastError();
}

hipError_t launch_loop_verify(const LoopParams &lp, int max_wgs, hipStream_t s) {
    LoopVerifyParams p{};
    p.lp = lp;
    p.hs.d = lp.d; p.hs.V = lp.V; p.hs.eps = lp.eps; p.hs.gamma = lp.gamma; p.hs.lm_head = lp.lm_head;
    p.hs.qweight = lp.qweight; p.hs.scales = lp.qscales; p.hs.zeros = lp.qzeros; p.hs.group = lp.group;
    return hs_dispatch(lp.d, lp.V, lp.qweight ? lp.group : 0, [&](auto lw, auto cpw, auto ragged, auto nt, const HsShape &sh) {
        return launch_lv<decltype(lw)::value, decltype(cpw)::value, decltype(ragged)::value, decltype(nt)::value>(
            p, sh, max_wgs, s);
    });
}

}  // namespace specee
