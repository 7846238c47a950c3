// Selective-Rollout gate: mean pairwise prefix edit distance of a group's action sequences
// (paper Section 3.2) compared with the threshold d_L (Eq. 2), in exact integer arithmetic.
//
// Work decomposition.  A lane runs the whole Levenshtein tables of one or two of a group's G(G-1)/2 pairs in registers, a row
// at a time with the row as bit masks (prefix_match.h), so there is no cross-lane traffic in the recurrence.  A workgroup
// of up to 256 lanes serves whole groups (sixteen at G = 8); the equality masks come from LDS tables built once per group
// or from comparing in registers, and the per-group sums are accumulated with LDS integer atomics, which are
// order-independent and therefore deterministic.
//
// Prefix nesting: cell (k,k) of the table of two length-L sequences is the distance of their length-k prefixes, so one
// table serves every requested prefix length.
//
// Bound: memory and vector ALU about equally; the 64 MB of input alone would take 13 us.  65 536 groups of 8, prefixes 5, 10 and
// 15: 18.5 us; 42.2 with a lane per pair, masks of one member per LDS read and 4-byte loads of the symbols.  32 steps: 37
// against 121 us, 16 384 groups of 16 with 16 steps 14 against 29.  Symbols of 64 and more: see prefix_turns.  Compared in registers:
// groups of 5, 12 steps 13.9 us.
#include "prefix_match.h"

namespace sr {

int64_t gate_bound(double d_L, int G, int K) {
    const int64_t den = 1000000;
    const int64_t num = (int64_t)__builtin_llround(d_L * 1e6);
    const int64_t pairs = (int64_t)G * (G - 1) / 2;
    return (num * pairs * (int64_t)K + den - 1) / den;
}

namespace {

__device__ __forceinline__ unsigned min3u(unsigned a, unsigned b, unsigned c) {
    return min(a, min(b, c));
}

__device__ __forceinline__ unsigned wanted_lens(const GateLens &lens) {      // bit k: prefix length k + 1 is asked for
    unsigned wanted = 0;
    for (int l = 0; l < lens.n; ++l) wanted |= 1u << (lens.len[l] - 1);
    return wanted;
}
// Sums of a workgroup's groups, one word of s_sum [distinct prefix length / 2][group] for two lengths: at most 120 * 32 each
__device__ __forceinline__ int len_slot(unsigned wanted, int K) { return __popc(wanted & ((1u << (K - 1)) - 1u)); }
// A lane's distances, shortest prefix first: two of them share an addition
struct LaneSums {
    unsigned word = 0;
    __device__ __forceinline__ void add(unsigned *s_sum, int groups, int g, unsigned wanted, int K, unsigned d) {
        const int u = len_slot(wanted, K);
        word += d << (16 * (u & 1));
        if ((u & 1) || (wanted >> (K - 1)) == 1) {    // uniform
            atomicAdd(&s_sum[(u >> 1) * groups + g], word);
            word = 0;
        }
    }
};
__device__ __forceinline__ void write_sums(const unsigned *s_sum, int groups, int n_here, size_t g0, int n_groups, const GateLens &lens,
                                           unsigned wanted, int32_t *__restrict__ sums, uint8_t *__restrict__ retire) {
    for (int i = threadIdx.x; i < lens.n * n_here; i += blockDim.x) {
        const int l = i / n_here, g = i - l * n_here, u = len_slot(wanted, lens.len[l]);
        const int s = (int)((s_sum[(u >> 1) * groups + g] >> (16 * (u & 1))) & 0xFFFFu);
        if (sums) sums[(size_t)l * n_groups + g0 + g] = s;
        if (retire) retire[(size_t)l * n_groups + g0 + g] = (uint8_t)(s < lens.bound[l]);
    }
}

// Equality masks from tables
template <int KIND>
__global__ __launch_bounds__(kPrefixThreads) void gate_table_kernel(
    const int32_t *__restrict__ actions, int n_groups, int stride, PrefixGeom q, GateLens lens,
    int32_t *__restrict__ sums, uint8_t *__restrict__ retire) {
    extern __shared__ __align__(16) char lds[];      // element ids, tables, sums
    unsigned *s_sum = (unsigned *)(lds + q.total);
    typedef PrefixBits<KIND> Bits;

    const int tid = threadIdx.x, G = q.G;
    const int g0 = blockIdx.x * q.groups;
    const int n_here = min(q.groups, n_groups - g0), rows = n_here * G;
    PrefixRows<KIND> x;
    x.load(q, rows, actions + (size_t)g0 * G * stride, stride, g0 + n_here == n_groups ? rows - 1 : -1);
    prefix_zero(lds, q.body, q.groups * kPrefixSyms * q.row_bytes, tid);
    for (int i = tid; i < 4 * q.groups; i += blockDim.x) s_sum[i] = 0;
    const unsigned beyond = prefix_beyond<KIND>(rows, x);

    const int gl = small_div(tid, 1.0f / (float)q.lanes);      // group within the block
    int i, j;
    prefix_lane<KIND>(tid - gl * q.lanes, G, &i, &j);
    const int ri = gl * G + i;
    const unsigned wanted = wanted_lens(lens);
    const bool second = j + 1 < G;
    auto pairs = [&](int s0, int n, int group_bytes) {           // of the groups s0 .. s0 + n - 1
        if (gl < s0 || gl >= min(s0 + n, n_here)) return;
        const char *column = lds + q.body + (gl - s0) * group_bytes + prefix_column<KIND>(j);
        Bits pv = Bits::all(0xFFFFFFFFu), mv = Bits::all(0);
        LaneSums sum;
#pragma unroll 1
        for (int r0 = 0; r0 < q.L; r0 += 8) {
            unsigned id[8];
            Bits eq[8];
            prefix_ids8<KIND>(lds, ri, r0, id);
#pragma unroll
            for (int t = 0; t < 8; ++t) eq[t] = prefix_masks<KIND>(column, id[t]);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                prefix_row(eq[t], pv, mv);
                if ((wanted >> (r0 + t)) & 1u)        // uniform
                    sum.add(s_sum, q.groups, gl, wanted, r0 + t + 1, prefix_cells(r0 + t + 1, second, pv, mv));
            }
        }
    };
    if (beyond == 0) {
        prefix_mark<KIND, true>(lds, q, rows, x, 0, q.groups, kPrefixSyms * q.row_bytes);
        __syncthreads();
        pairs(0, q.groups, kPrefixSyms * q.row_bytes);
    } else {
        const PrefixTurns t = prefix_turns(q, n_here, beyond);
        for (int s0 = 0; s0 < n_here; s0 += t.groups) {
            prefix_turn<KIND>(lds, q, rows, x, s0, t);
            pairs(s0, t.groups, t.group_bytes);
        }
    }
    __syncthreads();
    write_sums(s_sum, q.groups, n_here, g0, n_groups, lens, wanted, sums, retire);
}

// A lane per pair, symbols compared in registers
template <int KMAX>
__global__ __launch_bounds__(kPrefixThreads) void gate_direct_kernel(
    const int32_t *__restrict__ actions, int n_groups, int stride, PrefixGeom q, GateLens lens,
    int32_t *__restrict__ sums, uint8_t *__restrict__ retire) {
    extern __shared__ __align__(16) char lds[];      // symbols, sums
    unsigned *s_sum = (unsigned *)(lds + q.total);

    const int tid = threadIdx.x, G = q.G;
    const int g0 = blockIdx.x * q.groups;
    const int n_here = min(q.groups, n_groups - g0);
    const unsigned wanted = wanted_lens(lens);
    for (int i = tid; i < 4 * q.groups; i += blockDim.x) s_sum[i] = 0;
    prefix_stage<KMAX>(lds, q, n_here * G, actions + (size_t)g0 * G * stride, stride);

    const int gl = (int)(((float)tid + 0.5f) * (1.0f / (float)q.lanes));   // group within the block
    if (gl < n_here) {
        int i, j;
        pair_members(tid - gl * q.lanes, G, &i, &j);
        unsigned pv = 0xFFFFFFFFu, mv = 0;
        LaneSums sum;
        constexpr int STEP = KMAX % 8 ? 4 : 8;        // rows at a time
        int32_t b[KMAX];
        prefix_symbols<KMAX>(lds, gl * G + j, 0, b);
#pragma unroll
        for (int r0 = 0; r0 < KMAX; r0 += STEP) {
            if (r0 < q.L) {                           // uniform
                unsigned eq[STEP];
                int32_t a[STEP];
                prefix_symbols<KMAX>(lds, gl * G + i, r0, a);
                prefix_equal<KMAX>(a, b, eq);
#pragma unroll
                for (int t = 0; t < STEP; ++t) {
                    prefix_row(eq[t], pv, mv);
                    if ((wanted >> (r0 + t)) & 1u)    // uniform
                        sum.add(s_sum, q.groups, gl, wanted, r0 + t + 1, (unsigned)prefix_cell(r0 + t + 1, r0 + t + 1, pv, mv));
                }
            }
        }
    }
    __syncthreads();
    write_sums(s_sum, q.groups, n_here, g0, n_groups, lens, wanted, sums, retire);
}

// ---------------------------------------------------------------------------------------------
// The other decomposition, kept for comparison: one workgroup per group, every pair's table advanced
// one anti-diagonal at a time by a segment of SEG lanes (lane i owns row i of the table), the last
// three anti-diagonals of every pair in LDS.  256 / SEG pairs advance together; with G = 8 the 28
// pairs take two passes at SEG = 16 and four at SEG = 32.  Cell (k, k), the distance of the two
// length-k prefixes, appears on anti-diagonal 2k in lane k.  A segment never straddles a wavefront,
// and a wavefront's LDS accesses complete in program order, so no workgroup barrier is needed
// between anti-diagonals.  Half of a segment's lanes are idle in the triangular ramp-up and
// ramp-down and every step is an LDS round trip, which is why the library uses the kernels above;
// sr_gate_batch_antidiag exposes this one so that the two can be measured side by side and checked
// against each other.
// ---------------------------------------------------------------------------------------------
template <int SEG>
__global__ __launch_bounds__(kPrefixThreads) void gate_antidiag_kernel(
    const int32_t *__restrict__ actions, int n_groups, int G, int stride, int pairs, int maxlen, GateLens lens,
    int32_t *__restrict__ sums, uint8_t *__restrict__ retire) {
    constexpr int kSlots = kPrefixThreads / SEG;           // pairs that advance together
    __shared__ int32_t s_act[16 * SEG];                      // [member][step], the first SEG steps
    __shared__ unsigned s_d[3][kSlots][SEG + 1];             // anti-diagonals d-2, d-1, d of every slot, by table row
    __shared__ int s_sum[8];

    const int tid = threadIdx.x, g = blockIdx.x;
    if (tid < 8) s_sum[tid] = 0;
    for (int i = tid; i < G * SEG; i += kPrefixThreads) {
        const int r = i / SEG, c = i - r * SEG;
        s_act[i] = (c < stride) ? actions[((size_t)g * G + r) * stride + c] : -1 - c;
    }
    __syncthreads();

    const int slot = tid / SEG, row = tid % SEG + 1;         // this lane owns table row `row` (1-based)
    for (int p0 = 0; p0 < pairs; p0 += kSlots) {
        int p = p0 + slot;
        const bool live = p < pairs;
        int mi = 0;
        if (live) while (p >= G - 1 - mi) { p -= G - 1 - mi; ++mi; }
        const int mj = live ? mi + 1 + p : 1;
        const int32_t a_row = s_act[mi * SEG + row - 1];     // a[row - 1]
        const int32_t *b = s_act + mj * SEG;
        // anti-diagonal 0: D[0][0] = 0; anti-diagonal 1: D[0][1] = D[1][0] = 1
        if (row == 1) { s_d[0][slot][0] = 0; s_d[1][slot][0] = 1; s_d[1][slot][1] = 1; }
        __builtin_amdgcn_wave_barrier();
        for (int d = 2; d <= 2 * maxlen; ++d) {
            const unsigned *prev2 = s_d[(d - 2) % 3][slot], *prev = s_d[(d - 1) % 3][slot];
            unsigned *cur = s_d[d % 3][slot];
            const int col = d - row;                         // this lane's cell is (row, col)
            if (row <= maxlen) {
                if (col == 0) {
                    cur[row] = (unsigned)row;                // first column of the table
                } else if (col >= 1 && col <= maxlen) {
                    const unsigned v = min3u(prev2[row - 1] + (a_row != b[col - 1] ? 1u : 0u), prev[row - 1] + 1u,
                                             prev[row] + 1u);
                    cur[row] = v;
                    if (live && col == row) {                // cell (k, k): the answer for prefix length k
#pragma unroll
                        for (int l = 0; l < 8; ++l)
                            if (l < lens.n && lens.len[l] == row) atomicAdd(&s_sum[l], (int)v);
                    }
                }
            }
            if (row == 1 && d <= maxlen) cur[0] = (unsigned)d;   // first row of the table
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    if (tid < lens.n) {
        const int sum = s_sum[tid];
        if (sums) sums[(size_t)tid * n_groups + g] = sum;
        if (retire) retire[(size_t)tid * n_groups + g] = (uint8_t)(sum < lens.bound[tid]);
    }
}

}  // namespace

int launch_gate_antidiag(const int32_t *actions, int n_groups, int G, int stride, const GateLens &lens,
                         int32_t *sums, uint8_t *retire, hipStream_t stream) {
    if (n_groups <= 0) return SR_OK;
    int maxlen = 0;
    for (int l = 0; l < lens.n; ++l) maxlen = lens.len[l] > maxlen ? lens.len[l] : maxlen;
    const int pairs = G * (G - 1) / 2;
    dim3 grid(n_groups), block(kPrefixThreads);
    if (maxlen <= 16)
        gate_antidiag_kernel<16><<<grid, block, 0, stream>>>(actions, n_groups, G, stride, pairs, maxlen, lens, sums, retire);
    else
        gate_antidiag_kernel<32><<<grid, block, 0, stream>>>(actions, n_groups, G, stride, pairs, maxlen, lens, sums, retire);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_gate(const int32_t *actions, int n_groups, int G, int stride, const GateLens &lens,
                int32_t *sums, uint8_t *retire, hipStream_t stream) {
    if (n_groups <= 0) return SR_OK;
    int maxlen = 0;
    for (int l = 0; l < lens.n; ++l) maxlen = lens.len[l] > maxlen ? lens.len[l] : maxlen;
    GateLayout t;
    if (!gate_layout(n_groups, G, maxlen, &t)) return SR_E_ARG;
    const dim3 grid(ceil_div(n_groups, t.q.groups)), block(t.q.threads);
#define SR_TABLES(KIND) gate_table_kernel<KIND><<<grid, block, t.lds, stream>>>(actions, n_groups, stride, t.q, lens, sums, retire)
#define SR_GATE(K) gate_direct_kernel<K><<<grid, block, t.lds, stream>>>(actions, n_groups, stride, t.q, lens, sums, retire)
    if (t.direct) {
        switch (t.size) {
            case 4: SR_GATE(4); break;
            case 8: SR_GATE(8); break;
            case 12: SR_GATE(12); break;
            case 16: SR_GATE(16); break;
            case 24: SR_GATE(24); break;
            default: SR_GATE(32); break;
        }
    } else if (t.size == PREFIX_TWO16) SR_TABLES(PREFIX_TWO16);
    else if (t.size == PREFIX_TWO32) SR_TABLES(PREFIX_TWO32);
    else SR_TABLES(PREFIX_ONE32);
#undef SR_TABLES
#undef SR_GATE
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace sr

extern "C" int sr_gate_batch(const int32_t *actions, int n_groups, int G, int stride,
                             const int *prefix_lens, int n_lens, double threshold, int32_t *sums,
                             uint8_t *retire, void *stream) {
    if (!actions || !prefix_lens || n_groups < 0 || G < 2 || G > 16 || stride < 1 || n_lens < 1 ||
        n_lens > 8 || !(threshold >= 0.0) || threshold > 1.0)
        return SR_E_ARG;
    sr::GateLens lens{};
    lens.n = n_lens;
    for (int l = 0; l < n_lens; ++l) {
        const int K = prefix_lens[l];
        if (K < 1 || K > 32 || K > stride) return SR_E_ARG;
        lens.len[l] = K;
        lens.bound[l] = (int)sr::gate_bound(threshold, G, K);
    }
    return sr::launch_gate(actions, n_groups, G, stride, lens, sums, retire, (hipStream_t)stream);
}

extern "C" int sr_gate_batch_antidiag(const int32_t *actions, int n_groups, int G, int stride,
                                      const int *prefix_lens, int n_lens, double threshold, int32_t *sums,
                                      uint8_t *retire, void *stream) {
    if (!actions || !prefix_lens || n_groups < 0 || G < 2 || G > 16 || stride < 1 || n_lens < 1 ||
        n_lens > 8 || !(threshold >= 0.0) || threshold > 1.0)
        return SR_E_ARG;
    sr::GateLens lens{};
    lens.n = n_lens;
    for (int l = 0; l < n_lens; ++l) {
        const int K = prefix_lens[l];
        if (K < 1 || K > 32 || K > stride) return SR_E_ARG;
        lens.len[l] = K;
        lens.bound[l] = (int)sr::gate_bound(threshold, G, K);
    }
    return sr::launch_gate_antidiag(actions, n_groups, G, stride, lens, sums, retire, (hipStream_t)stream);
}
