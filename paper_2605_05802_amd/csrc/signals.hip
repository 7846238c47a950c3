// In-group divergence signals at step K (paper Appendix B) and the two-clause gate (Appendix E,
// Eq. 3), for groups whose members may have finished before step K.
//
// Member i finished after end_step[i] environment steps, so at step K it contributes the prefix
// a_i[0 : len_i], len_i = min(K, end_step[i]).  Per group and per requested K the kernel produces
//   - d_K: the mean over pairs of the prefix edit distance divided by the longer of the two prefix
//     lengths (Section 3.2), as a double and exactly, in units of 1 / lcm(1..32);
//   - the action-bigram Jaccard distance, the distinct-prefix count, the distinct step-K action and
//     observation counts, the step-K action entropy and the number of finished members;
//   - the decisions  d_K < d_L  (Eq. 2) and  d_K < d_L or tau_K >= tau_H  (Eq. 3) in integers.
//
// Work decomposition, as for the equal-length gate: one lane owns one pair and runs its table bit-parallel
// (prefix_pairs.h).  Cell (r, c) of the table of two sequences is the distance of their prefixes of lengths r and c, so
// one pass serves every requested K: the lane reads cell (K, len_j) when row K is complete, and keeps the masks of row
// end_i for the K beyond it.  The same equality masks give the bigrams: bit u of eq_t & (eq_{t+1} >> 1) says that b holds
// bigram t of a at position u; a bigram position is the first occurrence of its bigram in every prefix that contains it,
// so one mask of first occurrences per member and one mask per position of a serve every K.
// What is per member (first occurrences, step-K counts, entropy terms) is done by one lane per member and K, what is
// per pair (quotients included) by the pair lanes; one thread per (K, group) is left with adding the pair terms in pair
// order (i, j), i < j, and the entropy terms in member order, so that the floating-point results do not depend on
// scheduling.
// Bound: vector ALU (70 % busy).  65 536 groups of 8 with early finishers, K = 5, 10, 15: 126 us; 361 us with one table cell
// at a time, K * K compares per pair for the bigrams and the quotients left to the thread of a (K, group).  At 32 steps
// 272 against 1266 us, at G = 16 and 16 steps 112 against 990 us (16 384 groups).  Groups of 3, 12 steps, symbols compared in
// registers: 18 against 33 us.
#include <type_traits>

#include "prefix_pairs.h"

static_assert(sizeof(sr_signals_t) == 64, "sr_signals_t is part of the C boundary");

namespace sr {
namespace {

constexpr int kSigThreads = 256;
constexpr int kSigLds = 52 * 1024;                   // three workgroups per compute unit where the shape allows it
constexpr int kSigLdsMost = 64 * 1024;               // G = 16 with 32 steps and 8 prefix lengths needs 58.6 KiB
constexpr int kSigMaxLens = 8;
constexpr long long kLcm32 = 144403552893600LL;      // lcm(1..32)

struct SigLens {
    int n;
    int len[kSigMaxLens];
    long long d_bound;                // d_K < d_L  <=>  lev_scaled < d_bound
    long long tau_num;                // tau_K >= tau_H  <=>  n_done * 1e6 >= tau_num * G
    long long lcm_over[33];           // lcm(1..32) / n
};

// What the workgroup keeps behind the prefix tables: byte offsets, 8-byte arrays first.
struct SigLds {
    int d, j, h, out, pair, obs, hold, end, first, total;
};
__host__ __device__ inline SigLds sig_lds(int G, int pairs, int groups, int n_lens) {
    SigLds o;
    const int P = n_lens * groups * pairs, R = n_lens * groups * G;
    o.out = 0;                                    // [K][group] sr_signals_t
    o.d = o.out + n_lens * groups * 64;           // [K][pair] double: distance / longer length
    o.j = o.d + P * 8;                            // [K][pair] double: Jaccard term
    o.h = o.j + P * 8;                            // [K][member] double: log p of an action, at its first holder
    o.obs = o.h + R * 8;                          // [K][member] o_{i,K}
    o.hold = o.obs + R * 4;                       // [K][member] see below
    o.end = o.hold + R * 4;                       // [member]
    o.first = o.end + groups * G * 4;             // [member] positions of first occurrences of bigrams
    o.pair = o.first + groups * G * 4;            // [K][pair] 16 bits: distance | longer length << 6 | equal prefixes << 12
    o.total = o.pair + round_up(P * 2, 16);
    return o;
}

template <int KMAX, bool DIRECT>
__global__ __launch_bounds__(kSigThreads) void signals_kernel(
    const int32_t *__restrict__ actions, const int32_t *__restrict__ obs, const int32_t *__restrict__ end_step,
    int n_groups, int stride, int pairs, PrefixGeom q, SigLens lens, sr_signals_t *__restrict__ out) {
    extern __shared__ __align__(16) char lds[];
    __shared__ long long s_lcm[33];                          // lcm(1..32) / n
    const int tid = threadIdx.x, nt = blockDim.x, G = q.G, NL = lens.n;
    const int g0 = blockIdx.x * q.groups;
    const int n_here = min(q.groups, n_groups - g0);
    const int rows = n_here * G, n_pairs = q.groups * pairs, n_rows = q.groups * G;
    const PrefixLds off = prefix_lds(q, q.groups, KMAX, DIRECT);
    const SigLds so = sig_lds(G, pairs, q.groups, NL);
    char *mine = lds + off.total;
    sr_signals_t *s_out = (sr_signals_t *)(mine + so.out);
    double *s_d = (double *)(mine + so.d), *s_j = (double *)(mine + so.j), *s_h = (double *)(mine + so.h);
    int32_t *s_obs = (int32_t *)(mine + so.obs), *s_end = (int32_t *)(mine + so.end);
    // holders of the member's step-K action if it is the first of them, | 32 the first to hold its observation
    // | 64 its prefix reaches step K | 128 it has finished by step K
    int *s_hold = (int *)(mine + so.hold);
    unsigned *s_first = (unsigned *)(mine + so.first);
    uint16_t *s_pair = (uint16_t *)(mine + so.pair);
    const float inv_G = 1.0f / (float)G, inv_rows = 1.0f / (float)rows;

    if (tid < 33) s_lcm[tid] = lens.lcm_over[tid];
    for (int i = tid; i < rows; i += nt) s_end[i] = end_step ? max(end_step[(size_t)g0 * G + i], 0) : 0x7FFFFFFF;
    for (int w = tid; w < NL * rows; w += nt) {
        const int l = min((int)(((float)w + 0.5f) * inv_rows), NL - 1), r = w - l * rows;
        s_obs[l * n_rows + r] = obs ? obs[((size_t)g0 * G + r) * stride + lens.len[l] - 1] : 0;
    }
    const int32_t *src = actions + (size_t)g0 * G * stride;
    if constexpr (DIRECT) prefix_stage<KMAX>(lds, q, rows, src, stride);
    else prefix_build<KMAX>(lds, q, off, rows, src, stride);
    // what stands for a member's step: its symbol, or the element of the group that represents it
    using Step = std::conditional_t<DIRECT, int32_t, uint16_t>;
    constexpr int SS = DIRECT ? prefix_act_stride(KMAX) : KMAX;
    const Step *steps = (const Step *)(lds + (DIRECT ? off.act : off.id));

    if constexpr (DIRECT) {
        // One lane per member: the positions that are the first occurrence of their bigram
        for (int r = tid; r < rows; r += nt) {
            int32_t b[KMAX];
            prefix_symbols<KMAX>(lds, r, 0, b);
            unsigned eq[KMAX], first = 0;
            prefix_equal<KMAX>(b, b, eq);
#pragma unroll
            for (int t = 0; t + 1 < KMAX; ++t) first |= (eq[t] & (eq[t + 1] >> 1) & low_bits(t)) == 0u ? 1u << t : 0u;
            s_first[r] = first & low_bits(q.L - 1);
        }
    } else {
        // One lane per (member, position): is it the first occurrence of its bigram?  A member's lanes are neighbours, so
        // the wavefront's vote holds the members' masks side by side.
        constexpr int KP = KMAX <= 16 ? 16 : 32;
        for (int e0 = 0; e0 < rows * KP; e0 += nt) {             // whole wavefronts take part
            const int e = e0 + tid, r = e / KP, t = e % KP;
            bool first = false;
            if (r < rows && t + 1 < q.L) {
                const unsigned here = prefix_mask<KMAX>(lds, q, r, steps[r * SS + t]);
                const unsigned next = prefix_mask<KMAX>(lds, q, r, steps[r * SS + t + 1]);
                first = (here & (next >> 1) & low_bits(t)) == 0u;
            }
            const unsigned long long vote = __ballot(first);
            if (t == 0 && r < rows) s_first[r] = (unsigned)(vote >> (tid & 63)) & low_bits(KP);
        }
    }
    // One lane per (member, K): members that reach step K, and whether this one is the first to hold its action or
    // observation
    for (int w = tid; w < NL * rows; w += nt) {
        const int l = min((int)(((float)w + 0.5f) * inv_rows), NL - 1), r = w - l * rows, g = small_div(r, inv_G), K = lens.len[l];
        int hold = s_end[r] <= K ? 128 : 0;
        if (s_end[r] >= K) {
            const unsigned a = steps[r * SS + K - 1];
            const int32_t o = s_obs[l * n_rows + r];
            int n_at = 0, count = 0;
            bool first_act = true, first_obs = true;
#pragma unroll 4
            for (int i = g * G; i < g * G + G; ++i) {
                const bool at = s_end[i] >= K, same = at & ((unsigned)steps[i * SS + K - 1] == a);
                n_at += at ? 1 : 0;
                count += same ? 1 : 0;
                first_act &= !((i < r) & same);
                first_obs &= !((i < r) & at & (s_obs[l * n_rows + i] == o));
            }
            hold |= 64 | (first_act ? count : 0) | (first_obs ? 32 : 0);
            if (first_act) s_h[l * n_rows + r] = log((double)count / (double)n_at);
        }
        s_hold[l * n_rows + r] = hold;
    }
    __syncthreads();

    // per pair
    const int gl = (int)(((float)tid + 0.5f) * (1.0f / (float)pairs));     // group within the block
    if (gl < n_here) {
        int i, j;
        pair_members(tid - gl * pairs, G, &i, &j);
        const int ri = gl * G + i, rj = gl * G + j;
        const int ei = s_end[ri], ej = s_end[rj];
        unsigned wanted = 0;                          // bit k: prefix length k + 1 is asked for
        for (int l = 0; l < NL; ++l) wanted |= 1u << (lens.len[l] - 1);
        int res[kSigMaxLens];
#pragma unroll
        for (int l = 0; l < kSigMaxLens; ++l) res[l] = 0;

        unsigned pv = 0xFFFFFFFFu, mv = 0, pv_end = 0xFFFFFFFFu, mv_end = 0;      // row 0: distance from the empty prefix
        unsigned big[KMAX], eq_last = 0;              // big[t]: positions of b that hold bigram t of a
        int32_t b[DIRECT ? KMAX : 4];
        if constexpr (DIRECT) prefix_symbols<KMAX>(lds, rj, 0, b);
#pragma unroll
        for (int r0 = 0; r0 < KMAX; r0 += 8) {
            unsigned eq[8];
            if (r0 < q.L) {                           // uniform
                if constexpr (DIRECT) {
                    int32_t a[8];
                    prefix_symbols<KMAX>(lds, ri, r0, a);
                    prefix_equal<KMAX>(a, b, eq);
                } else {
                    prefix_masks8<KMAX>(lds, q, off, ri, rj, r0, eq);
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int r = r0 + t + 1;
                    prefix_row(eq[t], pv, mv);
                    if (ei == r) { pv_end = pv; mv_end = mv; }
                    if ((wanted >> (r - 1)) & 1u) {   // uniform
                        const int d = prefix_cell(r, min(r, ej), pv, mv);
#pragma unroll
                        for (int l = 0; l < kSigMaxLens; ++l)
                            if (l < NL && lens.len[l] == r) res[l] = d;
                    }
                }
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t) eq[t] = 0;
            }
            if (r0 > 0) big[r0 - 1] = eq_last & (eq[0] >> 1);
#pragma unroll
            for (int t = 0; t < 7; ++t) big[r0 + t] = eq[t] & (eq[t + 1] >> 1);
            eq_last = eq[7];
        }
        const unsigned first_a = s_first[ri], first_b = s_first[rj];
#pragma unroll
        for (int l = 0; l < kSigMaxLens; ++l) {
            if (l < NL) {
                const int K = lens.len[l], li = min(K, ei), lj = min(K, ej);
                const int lev = ei < K ? prefix_cell(li, lj, pv_end, mv_end) : res[l];
                // a prefix of length n holds bigram positions 0 .. n-2
                const unsigned ma = low_bits(max(li - 1, 0)), mb = low_bits(max(lj - 1, 0));
                unsigned held = 0;
#pragma unroll
                for (int t = 0; t < KMAX - 1; ++t) held |= (big[t] & mb) != 0u ? 1u << t : 0u;
                const int inter = __popc(first_a & ma & held);
                const int uni = __popc(first_a & ma) + __popc(first_b & mb) - inter;
                const int longer = max(li, lj);
                s_d[l * n_pairs + tid] = longer > 0 ? (double)lev / (double)longer : 0.0;
                s_j[l * n_pairs + tid] = uni > 0 ? 1.0 - (double)inter / (double)uni : 0.0;
                s_pair[l * n_pairs + tid] = (uint16_t)(lev | longer << 6 | (lev == 0 && li == lj ? 1 << 12 : 0));
            }
        }
    }
    __syncthreads();

    // Four sums per (K, group), a wavefront for each where the workgroup has four: pair terms in pair order, entropy
    // terms in member order.
    const int n_rec = NL * n_here, waves = nt >> 6;
    const float inv_here = 1.0f / (float)n_here;
    for (int kind = tid >> 6; kind < 4; kind += waves) {
        for (int w = tid & 63; w < n_rec; w += 64) {
            const int l = min((int)(((float)w + 0.5f) * inv_here), NL - 1), g = w - l * n_here;
            sr_signals_t *o = s_out + l * q.groups + g;
            if (kind < 2) {
                const double *t = (kind == 0 ? s_d : s_j) + l * n_pairs + g * pairs;
                double sum = 0.0;
#pragma unroll 4
                for (int k = 0; k < pairs; ++k) sum += t[k];
                sum /= (double)pairs;
                if (kind == 0) o->d_K = sum;
                else o->bigram_jaccard = sum;
            } else if (kind == 2) {
                const uint16_t *t = s_pair + l * n_pairs + g * pairs;
                long long scaled = 0;
                int lev_sum = 0;
                unsigned repeats = 0;                 // members whose prefix an earlier member has
                int i = 0, j = 1;
#pragma unroll 4
                for (int k = 0; k < pairs; ++k) {
                    const int x = t[k], lev = x & 63;
                    lev_sum += lev;
                    scaled += lev * s_lcm[(x >> 6) & 63];
                    repeats |= (unsigned)(x >> 12) << j;
                    if (++j == G) { ++i; j = i + 1; }
                }
                o->lev_scaled = scaled;
                o->lev_sum = lev_sum;
                o->unique_prefix = G - __popc(repeats);
            } else {
                const int *t = s_hold + l * n_rows + g * G;
                const double *lg = s_h + l * n_rows + g * G;
                int n_at = 0, n_done = 0, ua = 0, uo = 0;
                for (int k = 0; k < G; ++k) {
                    n_at += (t[k] >> 6) & 1;
                    n_done += t[k] >> 7;
                    uo += (t[k] >> 5) & 1;
                    ua += (t[k] & 31) ? 1 : 0;
                }
                double H = 0.0;
                for (int k = 0; k < G; ++k)
                    if (t[k] & 31) H = __builtin_fma(-((double)(t[k] & 31) / (double)n_at), lg[k], H);
                o->action_entropy = H;
                o->n_at_step = n_at;
                o->unique_action = ua;
                o->unique_obs = obs ? uo : 0;
                o->n_done = n_done;
            }
        }
    }
    __syncthreads();
    for (int w = tid; w < n_rec; w += nt) {
        const int l = min((int)(((float)w + 0.5f) * inv_here), NL - 1), g = w - l * n_here;
        sr_signals_t *o = s_out + l * q.groups + g;
        o->cut_d = (uint8_t)(o->lev_scaled < lens.d_bound);
        o->cut_or = (uint8_t)(o->cut_d || (long long)o->n_done * 1000000LL >= lens.tau_num * G);
        for (int i = 0; i < 6; ++i) o->reserved[i] = 0;
    }
    __syncthreads();
    for (int w = tid; w < n_rec * 4; w += nt) {              // 16 bytes per lane, whole records of a K in a row
        const int rec = w >> 2, l = min((int)(((float)rec + 0.5f) * inv_here), NL - 1), g = rec - l * n_here;
        ((uint4 *)(out + (size_t)l * n_groups + g0 + g))[w & 3] = ((const uint4 *)(s_out + l * q.groups + g))[w & 3];
    }
}

__global__ void assemble_gate_kernel(const int32_t *__restrict__ src, const int32_t *__restrict__ live_actions,
                                     const int32_t *__restrict__ fin_actions, int n_slots, int max_turns,
                                     int32_t *__restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_slots * max_turns) return;
    const int s = i / max_turns, t = i - s * max_turns;
    const int r = src[s];
    out[i] = r >= 0 ? live_actions[(size_t)r * max_turns + t] : fin_actions[(size_t)(-1 - r) * max_turns + t];
}

__global__ void extract_gate_kernel(const sr_signals_t *__restrict__ sig, int n_groups, int use_or,
                                    int32_t *__restrict__ sums, uint8_t *__restrict__ retire) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_groups) return;
    sums[g] = sig[g].lev_sum;
    retire[g] = use_or ? sig[g].cut_or : sig[g].cut_d;
}

}  // namespace

int launch_assemble_gate(const int32_t *src, const int32_t *live_actions, const int32_t *fin_actions, int n_slots,
                         int max_turns, int32_t *out, hipStream_t stream) {
    const int n = n_slots * max_turns;
    if (n <= 0) return SR_OK;
    assemble_gate_kernel<<<dim3((n + 255) / 256), dim3(256), 0, stream>>>(src, live_actions, fin_actions, n_slots,
                                                                         max_turns, out);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_extract_gate(const sr_signals_t *sig, int n_groups, int use_or, int32_t *sums, uint8_t *retire,
                        hipStream_t stream) {
    if (n_groups <= 0) return SR_OK;
    extract_gate_kernel<<<dim3((n_groups + 255) / 256), dim3(256), 0, stream>>>(sig, n_groups, use_or, sums, retire);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace sr

extern "C" int sr_signals_batch(const int32_t *actions, const int32_t *obs, const int32_t *end_step, int n_groups,
                                int G, int stride, const int *prefix_lens, int n_lens, double d_L, double tau_H,
                                sr_signals_t *out, void *stream) {
    using namespace sr;
    if (!prefix_lens || n_groups < 0 || G < 2 || G > 16 || stride < 1 || n_lens < 1 || n_lens > kSigMaxLens ||
        !(d_L >= 0.0) || d_L > 1.0 || !(tau_H >= 0.0) || tau_H > 4.0)
        return SR_E_ARG;
    if (n_groups > 0 && (!actions || !out)) return SR_E_ARG;
    SigLens lens{};
    lens.n = n_lens;
    int maxlen = 0;
    for (int l = 0; l < n_lens; ++l) {
        const int K = prefix_lens[l];
        if (K < 1 || K > 32 || K > stride) return SR_E_ARG;
        lens.len[l] = K;
        maxlen = K > maxlen ? K : maxlen;
    }
    // d_K < d_L  <=>  lev_scaled * 1e6 < num * P * lcm  <=>  lev_scaled < ceil(num * P * lcm / 1e6)
    const __int128 num = (__int128)__builtin_llround(d_L * 1e6), P = (__int128)G * (G - 1) / 2;
    lens.d_bound = (long long)((num * P * (__int128)kLcm32 + 999999) / 1000000);
    lens.tau_num = (long long)__builtin_llround(tau_H * 1e6);
    if (n_groups == 0) return SR_OK;
    const int pairs = G * (G - 1) / 2;
    const bool direct = prefix_direct(n_groups, G, maxlen, 3);
    const int kmax = maxlen <= 8 ? 8 : maxlen <= 16 ? 16 : maxlen <= 24 ? 24 : 32;
    for (int n = 1; n <= 32; ++n) lens.lcm_over[n] = kLcm32 / n;
    PrefixGeom q{};
    const int extra = sig_lds(G, pairs, 1, n_lens).total;
    if (!prefix_geometry(n_groups, G, maxlen, kmax, direct, kSigLds, extra, &q) &&
        !prefix_geometry(n_groups, G, maxlen, kmax, direct, kSigLdsMost, extra, &q))
        return SR_E_ARG;
    const size_t lds = prefix_lds(q, q.groups, kmax, direct).total + (size_t)sig_lds(G, pairs, q.groups, n_lens).total;
    dim3 grid((n_groups + q.groups - 1) / q.groups), block(q.threads);
    hipStream_t st = (hipStream_t)stream;
#define SR_SIG(K, DIRECT) \
    signals_kernel<K, DIRECT><<<grid, block, lds, st>>>(actions, obs, end_step, n_groups, stride, pairs, q, lens, out)
    switch (kmax) {                       // up to eight steps there are no tables
        case 8: SR_SIG(8, true); break;
        case 16: if (direct) SR_SIG(16, true); else SR_SIG(16, false); break;
        case 24: if (direct) SR_SIG(24, true); else SR_SIG(24, false); break;
        default: if (direct) SR_SIG(32, true); else SR_SIG(32, false); break;
    }
#undef SR_SIG
    SR_HIP(hipGetLastError());
    return SR_OK;
}
