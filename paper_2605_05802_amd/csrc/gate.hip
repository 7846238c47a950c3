// Selective-Rollout gate: mean pairwise prefix edit distance of a group's action sequences
// (paper Section 3.2) compared with the threshold d_L (Eq. 2), in exact integer arithmetic.
//
// Work decomposition.  One lane owns one of the G(G-1)/2 pairs of a group and runs its whole Levenshtein table in
// registers, one row at a time with the row as two bit masks (prefix_match.h), so there is no cross-lane traffic in
// the recurrence.  A workgroup of up to 256 lanes serves whole groups (nine at G = 8); the equality masks come from
// LDS tables built once per group or from comparing in registers, and the per-group sums are accumulated with LDS
// integer atomics, which are order-independent and therefore deterministic.
//
// Prefix nesting: cell (k,k) of the table of two length-L sequences is the distance of their length-k prefixes, so one
// table serves every requested prefix length.
//
// Bound: vector ALU (about 65 % busy, 530 instructions per wavefront: 180 of them the recurrence) with the LDS latency of
// the table build behind it; the 64 MB of input would be 12 us.  65 536 groups of 8, prefixes 5, 10 and 15: 41 us (62 with
// symbols beyond the table's range), 72 us with one table cell at a time in registers; at 32 steps 120 against 284 us.
// Groups of 5, 12 steps: 14 us by comparison, 24 one cell at a time; groups of 16, one step: 44 against 61.
#include "prefix_match.h"

namespace sr {

int64_t gate_bound(double d_L, int G, int K) {
    const int64_t den = 1000000;
    const int64_t num = (int64_t)__builtin_llround(d_L * 1e6);
    const int64_t pairs = (int64_t)G * (G - 1) / 2;
    return (num * pairs * (int64_t)K + den - 1) / den;
}

namespace {

constexpr int kGateThreads = 256;
constexpr int kGateLds = 48 * 1024;      // tables of one workgroup: three workgroups or more per compute unit

__device__ __forceinline__ unsigned min3u(unsigned a, unsigned b, unsigned c) {
    return min(a, min(b, c));
}

template <int KMAX, bool DIRECT>
__global__ __launch_bounds__(kGateThreads) void gate_kernel(
    const int32_t *__restrict__ actions, int n_groups, int stride, int pairs, PrefixGeom q, GateLens lens,
    int32_t *__restrict__ sums, uint8_t *__restrict__ retire) {
    extern __shared__ __align__(16) char lds[];      // prefix tables
    __shared__ unsigned s_sum[4][kGateThreads];      // [len index / 2][group in block]: two sums of at most 120 * 32 each

    const int tid = threadIdx.x, G = q.G;
    const int g0 = blockIdx.x * q.groups;
    const int n_here = min(q.groups, n_groups - g0);
    const PrefixLds off = prefix_lds(q, q.groups, KMAX, DIRECT);
    for (int i = tid; i < q.groups; i += blockDim.x) s_sum[0][i] = s_sum[1][i] = s_sum[2][i] = s_sum[3][i] = 0;
    const int32_t *src = actions + (size_t)g0 * G * stride;
    if constexpr (DIRECT) prefix_stage<KMAX>(lds, q, n_here * G, src, stride);
    else prefix_build<KMAX>(lds, q, off, n_here * G, src, stride);

    const int gl = (int)(((float)tid + 0.5f) * (1.0f / (float)pairs));     // group within the block
    if (gl < n_here) {
        int i, j;
        pair_members(tid - gl * pairs, G, &i, &j);
        unsigned wanted = 0;                          // bit k: prefix length k + 1 is asked for
        for (int l = 0; l < lens.n; ++l) wanted |= 1u << (lens.len[l] - 1);
        unsigned pv = 0xFFFFFFFFu, mv = 0, res[4] = {0, 0, 0, 0};
        constexpr int STEP = KMAX % 8 ? 4 : 8;        // rows at a time
        int32_t b[DIRECT ? KMAX : 4];
        if constexpr (DIRECT) prefix_symbols<KMAX>(lds, gl * G + j, 0, b);
#pragma unroll
        for (int r0 = 0; r0 < KMAX; r0 += STEP) {
            if (r0 < q.L) {                           // uniform
                unsigned eq[STEP];
                if constexpr (DIRECT) {
                    int32_t a[STEP];
                    prefix_symbols<KMAX>(lds, gl * G + i, r0, a);
                    prefix_equal<KMAX>(a, b, eq);
                } else {
                    prefix_masks8<KMAX>(lds, q, off, gl * G + i, gl * G + j, r0, eq);
                }
#pragma unroll
                for (int t = 0; t < STEP; ++t) {
                    prefix_row(eq[t], pv, mv);
                    if ((wanted >> (r0 + t)) & 1u) {  // uniform
                        const unsigned d = (unsigned)prefix_cell(r0 + t + 1, r0 + t + 1, pv, mv);
#pragma unroll
                        for (int l = 0; l < 8; ++l)
                            if (l < lens.n && lens.len[l] == r0 + t + 1) res[l >> 1] += d << (16 * (l & 1));
                    }
                }
            }
        }
#pragma unroll
        for (int l = 0; l < 4; ++l)
            if (2 * l < lens.n) atomicAdd(&s_sum[l][gl], res[l]);
    }
    __syncthreads();

    for (int i = tid; i < lens.n * n_here; i += blockDim.x) {
        const int l = i / n_here, g = i - l * n_here;
        const int s = (int)((s_sum[l >> 1][g] >> (16 * (l & 1))) & 0xFFFFu);
        if (sums) sums[(size_t)l * n_groups + g0 + g] = s;
        if (retire) retire[(size_t)l * n_groups + g0 + g] = (uint8_t)(s < lens.bound[l]);
    }
}

// ---------------------------------------------------------------------------------------------
// The other decomposition, kept for comparison: one workgroup per group, every pair's table advanced
// one anti-diagonal at a time by a segment of SEG lanes (lane i owns row i of the table), the last
// three anti-diagonals of every pair in LDS.  256 / SEG pairs advance together; with G = 8 the 28
// pairs take two passes at SEG = 16 and four at SEG = 32.  Cell (k, k), the distance of the two
// length-k prefixes, appears on anti-diagonal 2k in lane k.  A segment never straddles a wavefront,
// and a wavefront's LDS accesses complete in program order, so no workgroup barrier is needed
// between anti-diagonals.  Half of a segment's lanes are idle in the triangular ramp-up and
// ramp-down and every step is an LDS round trip, which is why the lane-per-pair kernel above is the
// one the library uses; sr_gate_batch_antidiag exposes this one so that the two can be measured
// side by side and checked against each other.
// ---------------------------------------------------------------------------------------------
template <int SEG>
__global__ __launch_bounds__(kGateThreads) void gate_antidiag_kernel(
    const int32_t *__restrict__ actions, int n_groups, int G, int stride, int pairs, int maxlen, GateLens lens,
    int32_t *__restrict__ sums, uint8_t *__restrict__ retire) {
    constexpr int kSlots = kGateThreads / SEG;             // pairs that advance together
    __shared__ int32_t s_act[16 * SEG];                      // [member][step], the first SEG steps
    __shared__ unsigned s_d[3][kSlots][SEG + 1];             // anti-diagonals d-2, d-1, d of every slot, by table row
    __shared__ int s_sum[8];

    const int tid = threadIdx.x, g = blockIdx.x;
    if (tid < 8) s_sum[tid] = 0;
    for (int i = tid; i < G * SEG; i += kGateThreads) {
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
    dim3 grid(n_groups), block(kGateThreads);
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
    const int pairs = G * (G - 1) / 2;
    const bool direct = prefix_direct(n_groups, G, maxlen, 6);
    const int kmax = maxlen <= 4 ? 4 : maxlen <= 8 ? 8 : maxlen <= 12 && direct ? 12 : maxlen <= 16 ? 16 : maxlen <= 24 ? 24 : 32;
    PrefixGeom q{};
    if (!prefix_geometry(n_groups, G, maxlen, kmax, direct, kGateLds, 0, &q)) return SR_E_ARG;
    const size_t lds = prefix_lds(q, q.groups, kmax, direct).total;
    dim3 grid((n_groups + q.groups - 1) / q.groups), block(q.threads);
#define SR_GATE(K, DIRECT) \
    gate_kernel<K, DIRECT><<<grid, block, lds, stream>>>(actions, n_groups, stride, pairs, q, lens, sums, retire)
    switch (kmax) {                       // up to eight steps there are no tables
        case 4: SR_GATE(4, true); break;
        case 8: SR_GATE(8, true); break;
        case 12: SR_GATE(12, true); break;
        case 16: if (direct) SR_GATE(16, true); else SR_GATE(16, false); break;
        case 24: if (direct) SR_GATE(24, true); else SR_GATE(24, false); break;
        default: if (direct) SR_GATE(32, true); else SR_GATE(32, false); break;
    }
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
