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
// Work decomposition, as for the equal-length gate: a lane runs the tables of one pair, or of two, bit-parallel
// (prefix_match.h).  Cell (r, c) of the table of two sequences is the distance of their prefixes of lengths r and c, so
// one pass serves every requested K: once row K is complete the lane reads cell (K, len_j), or, if a has ended at row
// end_i < K, where the lane's state stays as it was at that row, cell (end_i, len_j).  The same equality masks give the
// bigrams: bit u of eq_t & (eq_{t+1} >> 1) says that b holds bigram t of a at position u, so the positions of b whose bigram
// the first r steps of a hold are a running OR, and the bigrams that the two prefixes share are those positions of it that
// are the first occurrence of their bigram in b.
// What is per member (first occurrences, step-K counts) is done by a lane per member (and K): the members that hold its
// step-K action are one column of the symbol's table row.  Logarithms and quotients of counts come from small tables of a
// workgroup.  Four wavefronts add the terms of every (K, group): pair terms in pair order (i, j), i < j, entropy terms in
// member order, so that the floating-point results do not depend on scheduling.
// Bound: vector ALU (70 % busy, 1570 instructions per wavefront: 300 of them the recurrence, 160 the evaluation at the three K, 150
// the quotients, 200 the sums), with four workgroups per compute unit by LDS.  65 536 groups of 8 with early finishers, K = 5,
// 10, 15: 61.4 us; 120 with a lane per pair, masks of one member per LDS read, bigrams compared position by position for
// every K, a division per pair and K and a logarithm per member and K.  32 steps 80 against 283 us, 16 384 groups of 16 with
// 16 steps 43 against 114, 16 groups of 8 with K = 5, 10, 15 8.3 against 12.7.  Symbols of 64 and more: see prefix_turns.
#include <stddef.h>

#include "prefix_match.h"

static_assert(sizeof(sr_signals_t) == 64, "sr_signals_t is part of the C boundary");

namespace sr {
namespace {

constexpr int kSigMaxLens = 8;
constexpr long long kLcm32 = 144403552893600LL;      // lcm(1..32)

struct SigLens {
    int n;
    unsigned wanted;                  // bit k: prefix length k + 1 is asked for
    unsigned long long packed;        // six bits per length: an argument that lanes index comes through the slowest memory there is
    long long d_bound;                // d_K < d_L  <=>  lev_scaled < d_bound
    long long tau_num;                // tau_K >= tau_H  <=>  n_done * 1e6 >= tau_num * G
    __device__ int len(int l) const { return (int)(packed >> (6 * l)) & 63; }
    __device__ int slot(int K) const { return __popc(wanted & ((1u << (K - 1)) - 1u)); }     // index among the distinct lengths
};

// One pair's integers at one K; distance 0 means equal prefixes
struct SigCode {
    __device__ static unsigned pack(int lev, int longer, int inter, int uni, unsigned j) {
        return (unsigned)(lev | longer << 6 | inter << 12) | ((unsigned)uni << 17 | j << 23);
    }
    __device__ static int lev(unsigned c) { return c & 63; }
    __device__ static int longer(unsigned c) { return (c >> 6) & 63; }       // of the two prefixes
    __device__ static int inter(unsigned c) { return (c >> 12) & 31; }       // shared bigrams
    __device__ static int uni(unsigned c) { return (c >> 17) & 63; }         // bigrams of either
    __device__ static int j(unsigned c) { return c >> 23; }                  // the pair's second member
};

// Members of a group as bits: even ones 0 .. 7, odd ones 16 .. 23, so that a word with the masks of two members adds its two bits
// with one shift
__device__ __forceinline__ int member_bit(int m) { return (m >> 1) + 16 * (m & 1); }
__device__ __forceinline__ unsigned members_before(int m) { return ((1u << ((m + 1) >> 1)) - 1u) | ((1u << (m >> 1)) - 1u) << 16; }
constexpr unsigned kMembers = 0xFF00FFu;

// a / b correctly rounded for whole numbers 0 <= a, b < 64 (0 / 0: 0), r = the rounded 1 / b: the remainder of a * r is exact,
// and one correction with a rounded reciprocal gives the rounded quotient (Markstein 1990; every such a, b compared with the division)
__device__ __forceinline__ double small_quotient(int a, int b, double r) {
    const double q = (double)a * r;
    return __builtin_fma(__builtin_fma(-q, (double)b, (double)a), r, q);
}

// positions of b whose bigram is that of a at rows t, t + 1: eq_t & (eq_{t+1} >> 1), in every mask
template <int KIND>
__device__ __forceinline__ PrefixBits<KIND> bigram_bits(PrefixBits<KIND> eq, PrefixBits<KIND> next) {
    if constexpr (KIND == PREFIX_TWO16) {
        typedef typename PrefixBits<KIND>::u16x2 u16x2;
        return {eq.x & __builtin_bit_cast(unsigned, __builtin_bit_cast(u16x2, next.x) >> (unsigned short)1)};
    } else if constexpr (KIND == PREFIX_TWO32) {
        return {{eq.x[0] & (next.x[0] >> 1), eq.x[1] & (next.x[1] >> 1)}};
    } else {
        return {eq.x & (next.x >> 1)};
    }
}
template <int KIND>
__device__ __forceinline__ PrefixBits<KIND> bits_or(PrefixBits<KIND> a, PrefixBits<KIND> b) {
    if constexpr (KIND == PREFIX_TWO32) return {{a.x[0] | b.x[0], a.x[1] | b.x[1]}};
    else return {a.x | b.x};
}
template <int KIND>
__device__ __forceinline__ PrefixBits<KIND> bits_select(bool c, PrefixBits<KIND> a, PrefixBits<KIND> b) {
    if constexpr (KIND == PREFIX_TWO32) return {{c ? a.x[0] : b.x[0], c ? a.x[1] : b.x[1]}};
    else return {c ? a.x : b.x};
}

// The state of a lane's table(s): vertical differences, positions of b whose bigrams a holds, the last row's equality mask
template <int KIND>
struct SigState {
    typedef PrefixBits<KIND> Bits;
    Bits pv = Bits::all(0xFFFFFFFFu), mv = Bits::all(0), held = Bits::all(0), last = Bits::all(0);
    // row r (1-based) of a sequence that ends at `end`
    __device__ __forceinline__ void row(Bits eq, int r, int end) {
        Bits p = pv, m = mv;
        prefix_row(eq, p, m);
        const Bits h = bits_or<KIND>(held, bigram_bits<KIND>(last, eq));
        const bool live = r <= end;
        pv = bits_select<KIND>(live, p, pv);
        mv = bits_select<KIND>(live, m, mv);
        held = bits_select<KIND>(live, h, held);
        last = eq;
    }
    // the pair (., j) in half h at step K; li, lj: lengths of its prefixes, na: distinct bigrams of the first
    __device__ __forceinline__ unsigned code(int h, unsigned j, int li, int lj, int na, unsigned first_b) const {
        const unsigned cols = KIND == PREFIX_TWO16 ? (1u << lj) - 1u : low_bits(lj);
        const unsigned b = first_b & (cols >> 1);     // a prefix of length n holds bigram positions 0 .. n-2
        const int lev = li + __popc(pv.half(h) & cols) - __popc(mv.half(h) & cols);
        const int inter = __popc(held.half(h) & b);
        return SigCode::pack(lev, max(li, lj), inter, na + __popc(b) - inter, j);
    }
};

// KMAX == 0: equality masks from tables; otherwise a pair a lane, symbols compared in registers, at most KMAX steps
template <int KIND, int KMAX>
__global__ __launch_bounds__(kPrefixThreads) void signals_kernel(
    const int32_t *__restrict__ actions, const int32_t *__restrict__ obs, const int32_t *__restrict__ end_step,
    int n_groups, int stride, PrefixGeom q, SigLens lens, int sums_at, int terms_at_once, sr_signals_t *__restrict__ out) {
    extern __shared__ __align__(16) char lds[];      // symbols and tables, later the quotients; from sums_at on SigLds
    constexpr bool TABLES = KMAX == 0;
    const int tid = threadIdx.x, nt = blockDim.x, G = q.G, NL = lens.n, L = q.L;
    const int g0 = blockIdx.x * q.groups;
    const int n_here = min(q.groups, n_groups - g0);
    const int rows = n_here * G, n_rows = q.groups * G, pairs = G * (G - 1) / 2;
    const SigLds so = sig_lds(G, q.groups, NL);
    char *mine = lds + sums_at;
    sr_signals_t *s_out = (sr_signals_t *)(mine + so.out);
    double *s_lcm = (double *)(mine + so.lcm), *s_recip = (double *)(mine + so.recip), *s_p = (double *)(mine + so.p), *s_log_p = (double *)(mine + so.log_p);
    unsigned *s_code = (unsigned *)(mine + so.code), *s_at = (unsigned *)(mine + so.at), *s_first = (unsigned *)(mine + so.first);
    unsigned *s_repeats = (unsigned *)(mine + so.repeats);
    int32_t *s_obs = (int32_t *)(mine + so.obs), *s_end = (int32_t *)(mine + so.end);
    uint16_t *s_hold = (uint16_t *)(mine + so.hold);
    const float inv_G = 1.0f / (float)G;
    const int32_t *src = actions + (size_t)g0 * G * stride;
    PrefixRows<KIND> x;
    if constexpr (TABLES) x.load(q, rows, src, stride, g0 + n_here == n_groups ? rows - 1 : -1);
    // what else comes from global memory is requested before anything is waited for
    const float inv_rows = 1.0f / (float)rows;
    auto obs_item = [&](int w, int *l, int *r) { *l = min((int)(((float)w + 0.5f) * inv_rows), NL - 1); *r = w - *l * rows; };
    auto load_obs = [&](int w) {
        int l, r;
        obs_item(w, &l, &r);
        return obs ? obs[((size_t)g0 * G + r) * stride + lens.len(l) - 1] : 0;
    };
    auto load_end = [&](int i) { return end_step ? max(end_step[(size_t)g0 * G + i], 0) : 0x7FFFFFFF; };
    int32_t obs_v[2] = {0, 0}, end_v = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (tid + u * nt < NL * rows) obs_v[u] = load_obs(tid + u * nt);
    if (tid < rows) end_v = load_end(tid);
    for (int w = tid; w < NL * q.groups; w += nt) {
        s_repeats[w] = 0;
        s_out[w].lev_scaled = 0;
        s_out[w].lev_sum = 0;
    }
    if constexpr (TABLES) prefix_zero(lds, q.body, q.groups * kPrefixSyms * q.row_bytes, tid);
    // 1 / n, lcm(1..32) / n, c / n and log(c / n), by the last wavefront.  With tables of symbols ahead of its pairs, while the others
    // begin theirs, or ahead of the groups' first turn (within the turns: 127 registers instead of 96).  By comparison at once, where
    // the pairs leave one or two wavefronts' work and the last one's chain would follow it (65 536 groups of 3, 20 steps: 31.7 -> 29.3 us).
    auto small_tables = [&] {
        const int n = nt - 1 - tid;
        const double r = n ? 1.0 / (double)n : 0.0;
        s_recip[n] = r;
        if (n < 33) s_lcm[n] = rint((double)kLcm32 * r);     // exact: below 2^48, the product off by less than 1/16
        if (n == 0) s_p[0] = s_log_p[0] = 0.0;
        for (int e = n; e < G * (G + 1) / 2; e += 64) {       // n * (n - 1) / 2 + c
            const int n = (int)((1.0f + __builtin_amdgcn_sqrtf(8.0f * (float)e + 1.0f)) * 0.5f + 0.0078125f), c = e - n * (n - 1) / 2 + 1;
            const double share = (double)c / (double)n;
            s_p[e + 1] = share;
            s_log_p[e + 1] = log(share);
        }
    };
    if (!TABLES && tid >= nt - 64) small_tables();
    for (int w = tid, u = 0; w < NL * rows; w += nt, ++u) {
        int l, r;
        obs_item(w, &l, &r);
        s_obs[l * n_rows + r] = u == 0 ? obs_v[0] : u == 1 ? obs_v[1] : load_obs(w);
    }
    for (int i = tid; i < rows; i += nt) s_end[i] = i == tid ? end_v : load_end(i);
    unsigned beyond = 0;
    if constexpr (TABLES) {
        beyond = prefix_beyond<KIND>(rows, x);
    } else {
        prefix_stage<KMAX ? KMAX : 8>(lds, q, rows, src, stride);
    }
    // members that reach step K, and how many have finished by then
    for (int w = tid; w < NL * n_here; w += nt) {
        const int l = min((int)(((float)w + 0.5f) * (1.0f / (float)n_here)), NL - 1), g = w - l * n_here, K = lens.len(l);
        unsigned at = 0, done = 0;
#pragma unroll 4
        for (int m = 0; m < G; ++m) {
            const int end = s_end[g * G + m];
            at |= (end >= K ? 1u : 0u) << member_bit(m);
            done += end <= K ? 1u : 0u;
        }
        s_at[l * q.groups + g] = at | done << 24;
    }

    const int gl = small_div(tid, 1.0f / (float)q.lanes);      // group within the block
    int pi, pj;
    prefix_lane<KIND>(tid - gl * q.lanes, G, &pi, &pj);

    // groups s0 .. s0 + n - 1, `group_bytes` of tables each
    auto evaluate = [&](int s0, int n, int group_bytes, int tid, bool with_tables) __attribute__((always_inline)) {
        const int r_lo = s0 * G, here = min(n * G, rows - r_lo);
        auto table = [&](int g) { return lds + q.body + (g - s0) * group_bytes; };
        // Half of the workgroup, a lane per member: the positions that are the first occurrence of their bigram
        auto first_bigrams = [&](int r, int g, int m) __attribute__((always_inline)) {
            unsigned again = 0, last = 0;
            if constexpr (TABLES) {
                const int shift = prefix_shift<KIND>(m);
                const char *column = table(g) + prefix_column<KIND>(m);
#pragma unroll 1
                for (int t0 = 0; t0 < L; t0 += 8) {
                    unsigned id[8], eq[8];
                    prefix_ids8<KIND>(lds, r, t0, id);
#pragma unroll
                    for (int t = 0; t < 8; ++t) eq[t] = *(const unsigned *)(column + id[t]) >> shift;
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        // bigram t0 + t - 1 at an earlier position
                        const unsigned before = last & (eq[t] >> 1) & ((1u << (t0 + t) >> 1) - 1u);
                        again |= (min(before, 1u) << (t0 + t)) >> 1;
                        last = eq[t];
                    }
                }
            } else {
                int32_t b[KMAX ? KMAX : 8];
                unsigned eq[KMAX ? KMAX : 8];
                prefix_symbols<KMAX ? KMAX : 8>(lds, r, 0, b);
                prefix_equal<KMAX ? KMAX : 8>(b, b, eq);
#pragma unroll
                for (int t = 0; t + 1 < KMAX; ++t) again |= min(eq[t] & (eq[t + 1] >> 1) & low_bits(t), 1u) << t;
            }
            s_first[r] = ~again & low_bits(L - 1);
        };
        // The other half, a lane per (member, K): is it the first to hold its action (and how many do), and its observation?
        auto first_holders = [&](int l, int r, int g, int m) __attribute__((always_inline)) {
            const int K = lens.len(l);
            const unsigned at = s_at[l * q.groups + g] & kMembers;
            const int32_t *go = s_obs + l * n_rows + g * G;
            const int32_t o = go[m];
            unsigned same = 0, same_obs = 0;
            if constexpr (TABLES) {
                const unsigned *row = (const unsigned *)(table(g) + ((const uint16_t *)lds)[r * PrefixRows<KIND>::kSteps + K - 1]);
#pragma unroll 4
                for (int c = 0; c < q.Q; ++c) {
                    if constexpr (KIND == PREFIX_TWO16) same |= ((row[c] >> (K - 1)) & 0x10001u) << c;
                    else same |= ((row[2 * c] >> (K - 1)) & 1u) << c | ((row[2 * c + 1] >> (K - 1)) & 1u) << (c + 16);
                }
            } else {
                constexpr int SS = prefix_act_stride(KMAX ? KMAX : 8);
                const int32_t *act = (const int32_t *)lds + g * G * SS + K - 1, a = act[m * SS];
#pragma unroll 4
                for (int i = 0; i < G; ++i) same |= (act[i * SS] == a ? 1u : 0u) << member_bit(i);
            }
#pragma unroll 4
            for (int i = 0; i < G; ++i) same_obs |= (go[i] == o ? 1u : 0u) << member_bit(i);
            const unsigned before = at & members_before(m);
            int hold = ((same & before) == 0u ? __popc(same & at) : 0) | ((same_obs & before) == 0u ? 32 : 0);
            if (!((at >> member_bit(m)) & 1u)) hold = 0;
            s_hold[l * n_rows + r] = (uint16_t)hold;
        };
        int half = nt >> 7 << 6;                                 // whole wavefronts
        // all lanes do both in turn where there are more members than that, and beyond eight steps by comparison, where first_bigrams
        // is as long as a pair and keeps the wavefronts busy that have pairs (65 536 groups of 2, 32 steps: 31.0 -> 28.2 us)
        if (KMAX > 8 || here > nt - half || half == 0) half = 0;
        if (half == 0 || tid < half) {
            const float inv_here = 1.0f / (float)here;
            for (int w = tid; w < NL * here; w += half ? half : nt) {
                const int l = min((int)(((float)w + 0.5f) * inv_here), NL - 1), r = r_lo + w - l * here, g = small_div(r, inv_G);
                first_holders(l, r, g, r - g * G);
            }
        }
        if (tid >= half) {
            for (int r = r_lo + tid - half; r < r_lo + here; r += nt - half) {
                const int g = small_div(r, inv_G);
                first_bigrams(r, g, r - g * G);
            }
        }
        __syncthreads();
        if (TABLES && with_tables && tid >= nt - 64) small_tables();

        if (gl >= s0 && gl < min(s0 + n, n_here)) {
            constexpr int HALVES = KIND == PREFIX_ONE32 ? 1 : 2;
            const int ri = gl * G + pi, ei = s_end[ri];
            const unsigned first_a = s_first[ri];
            unsigned first_b[HALVES];
            int ej[HALVES], at[HALVES];
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                const int j = pj + h, rj = gl * G + min(j, G - 1);
                ej[h] = s_end[rj];
                first_b[h] = s_first[rj];
                at[h] = j > pi && j < G ? gl * so.code_stride + pi * (2 * G - 1 - pi) / 2 + j - pi - 1 : -1;
            }
            SigState<KIND> s;
            auto store = [&](int K) __attribute__((always_inline)) {
                unsigned *c = s_code + lens.slot(K) * (q.groups * so.code_stride);
                const int li = min(K, ei), na = __popc(first_a & (low_bits(li) >> 1));
                unsigned x[HALVES];
#pragma unroll
                for (int h = 0; h < HALVES; ++h) x[h] = s.code(h, pj + h, li, min(K, ej[h]), na, first_b[h]);
#pragma unroll
                for (int h = 0; h < HALVES; ++h)
                    if (HALVES == 1 || at[h] >= 0) c[at[h]] = x[h];
            };
            if constexpr (TABLES) {
                const char *column = table(gl) + prefix_column<KIND>(pj);
#pragma unroll 1
                for (int r0 = 0; r0 < L; r0 += 8) {
                    unsigned id[8];
                    PrefixBits<KIND> eq[8];
                    prefix_ids8<KIND>(lds, ri, r0, id);
#pragma unroll
                    for (int t = 0; t < 8; ++t) eq[t] = prefix_masks<KIND>(column, id[t]);
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        s.row(eq[t], r0 + t + 1, ei);
                        if ((lens.wanted >> (r0 + t)) & 1u) store(r0 + t + 1);        // uniform
                    }
                }
            } else {
                int32_t b[KMAX ? KMAX : 8];
                prefix_symbols<KMAX ? KMAX : 8>(lds, gl * G + pj, 0, b);
#pragma unroll
                for (int r0 = 0; r0 < KMAX; r0 += 8) {
                    if (r0 >= L) break;               // uniform
                    unsigned eq[8];
                    int32_t a[8];
                    prefix_symbols<KMAX ? KMAX : 8>(lds, ri, r0, a);
                    prefix_equal<KMAX ? KMAX : 8>(a, b, eq);
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        s.row({eq[t]}, r0 + t + 1, ei);
                        if ((lens.wanted >> (r0 + t)) & 1u) store(r0 + t + 1);        // uniform
                    }
                }
            }
        }
    };
    if constexpr (TABLES) {
        if (beyond == 0) {
            prefix_mark<KIND, true>(lds, q, rows, x, 0, q.groups, kPrefixSyms * q.row_bytes);
            __syncthreads();
            evaluate(0, q.groups, kPrefixSyms * q.row_bytes, tid, true);
        } else {
            const PrefixTurns t = prefix_turns(q, n_here, beyond);
            if (tid >= nt - 64) small_tables();
            for (int s0 = 0; s0 < n_here; s0 += t.groups) {
                prefix_turn<KIND>(lds, q, rows, x, s0, t);
                evaluate(s0, t.groups, t.group_bytes, turn_tid(), false);
            }
        }
    } else {
        __syncthreads();
        evaluate(0, q.groups, 0, tid, true);
    }
    __syncthreads();

    // The quotients of terms_at_once prefix lengths, in parallel, then the sums: those of quotients in pair order
    const int n_rec = NL * n_here, waves = nt >> 6;
    const float inv_n = 1.0f / (float)n_here;
    const int distinct = __popc(lens.wanted), per_len = q.groups * so.code_stride;
    double *s_d = (double *)lds, *s_j = s_d + terms_at_once * per_len;
    for (int u0 = 0; u0 < distinct; u0 += terms_at_once) {
        const int n_terms = min(terms_at_once, distinct - u0) * per_len;
        if (u0) __syncthreads();
        for (int k = tid; k < n_terms; k += nt) {
            const unsigned c = s_code[u0 * per_len + k];
            const int longer = SigCode::longer(c), uni = SigCode::uni(c);
            s_d[k] = small_quotient(SigCode::lev(c), longer, s_recip[longer]);
            s_j[k] = uni > 0 ? 1.0 - small_quotient(SigCode::inter(c), uni, s_recip[uni]) : 0.0;
        }
        __syncthreads();
        // a lane per (K, group), a wavefront for each kind of sum where the workgroup has four
        for (int kind = tid >> 6; kind < (u0 ? 2 : 4); kind += waves) {
            const int parts = kind == 2 && n_rec < 64 ? 64 / n_rec : 1;      // whole numbers: as many lanes as there are
            const float inv_parts = 1.0f / (float)parts;
            for (int w = tid & 63; w < n_rec * parts; w += 64) {
                const int rec = (int)(((float)w + 0.5f) * inv_parts), l = min((int)(((float)rec + 0.5f) * inv_n), NL - 1), g = rec - l * n_here;
                const int u = lens.slot(lens.len(l)), slot = l * q.groups + g;
                sr_signals_t *o = s_out + slot;
                if (kind < 2) {
                    if (u < u0 || u >= u0 + terms_at_once) continue;
                    const double *t = (kind == 0 ? s_d : s_j) + (u - u0) * per_len + g * so.code_stride;
                    double sum = 0.0;
#pragma unroll 8
                    for (int k = 0; k < pairs; ++k) sum += t[k];
                    sum /= (double)pairs;
                    if (kind == 0) o->d_K = sum;
                    else o->bigram_jaccard = sum;
                } else if (kind == 2) {
                    // at most 60 terms of at most lcm(1..32): whole numbers below 2^53, which 64-bit floats add exactly (and without
                    // 64-bit multiplications)
                    const unsigned *code = s_code + u * per_len + g * so.code_stride;
                    long long scaled = 0;
                    int lev_sum = 0;
                    unsigned repeats = 0;             // members whose prefix an earlier member has
                    for (int k = w - rec * parts; k < pairs;) {
                        double some = 0.0;
                        const int end = min(k + 60 * parts, pairs);
#pragma unroll 4
                        for (; k < end; k += parts) {
                            const unsigned c = code[k];
                            const int lev = SigCode::lev(c);
                            lev_sum += lev;
                            some = __builtin_fma((double)lev, s_lcm[SigCode::longer(c)], some);
                            repeats |= (lev == 0 ? 1u : 0u) << SigCode::j(c);
                        }
                        scaled += (long long)some;
                    }
                    if (parts == 1) {
                        o->lev_scaled = scaled;
                        o->lev_sum = lev_sum;
                        s_repeats[slot] = repeats;
                    } else {
                        atomicAdd((unsigned long long *)&o->lev_scaled, (unsigned long long)scaled);
                        atomicAdd(&o->lev_sum, lev_sum);
                        atomicOr(&s_repeats[slot], repeats);
                    }
                } else {
                    const uint16_t *hold = s_hold + l * n_rows + g * G;
                    const unsigned at = s_at[slot];
                    const int n_at = __popc(at & kMembers), row = n_at * (n_at - 1) / 2;
                    int ua = 0, uo = 0;
                    double H = 0.0;
#pragma unroll 4
                    for (int k = 0; k < G; ++k) {
                        const int h = hold[k], holders = h & 31;
                        uo += h >> 5;
                        ua += holders ? 1 : 0;
                        const int at_row = holders ? row + holders : 0;      // entry 0 is 0
                        H = __builtin_fma(-s_p[at_row], s_log_p[at_row], H);
                    }
                    o->action_entropy = H;
                    o->n_at_step = n_at;
                    o->unique_action = ua;
                    o->unique_obs = obs ? uo : 0;
                    o->n_done = (int)(at >> 24);
                }
            }
        }
    }
    __syncthreads();
    for (int w = tid; w < n_rec * 4; w += nt) {              // 16 bytes per lane, whole records of a K in a row
        const int rec = w >> 2, l = min((int)(((float)rec + 0.5f) * inv_n), NL - 1), g = rec - l * n_here;
        const sr_signals_t *o = s_out + l * q.groups + g;
        uint4 v = ((const uint4 *)o)[w & 3];
        if ((w & 3) == 2) v.x = (unsigned)(G - __popc(s_repeats[l * q.groups + g]));                       // unique_prefix
        if ((w & 3) == 3) {                                                                                // cut_d, cut_or, reserved
            const bool cut = o->lev_scaled < lens.d_bound, either = cut || (long long)o->n_done * 1000000LL >= lens.tau_num * G;
            v.z = (cut ? 1u : 0u) | (either ? 0x100u : 0u);
            v.w = 0;
        }
        ((uint4 *)(out + (size_t)l * n_groups + g0 + g))[w & 3] = v;
    }
}

static_assert(offsetof(sr_signals_t, unique_prefix) == 32 && offsetof(sr_signals_t, cut_d) == 56 && offsetof(sr_signals_t, cut_or) == 57,
              "pieces 2 and 3 of a record");

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
        lens.packed |= (unsigned long long)K << (6 * l);
        lens.wanted |= 1u << (K - 1);
        maxlen = K > maxlen ? K : maxlen;
    }
    // d_K < d_L  <=>  lev_scaled * 1e6 < num * P * lcm  <=>  lev_scaled < ceil(num * P * lcm / 1e6)
    const __int128 num = (__int128)__builtin_llround(d_L * 1e6), P = (__int128)G * (G - 1) / 2;
    lens.d_bound = (long long)((num * P * (__int128)kLcm32 + 999999) / 1000000);
    lens.tau_num = (long long)__builtin_llround(tau_H * 1e6);
    if (n_groups == 0) return SR_OK;
    SignalsLayout t;
    if (!signals_layout(n_groups, G, maxlen, n_lens, __builtin_popcount(lens.wanted), &t)) return SR_E_ARG;
    const dim3 grid(ceil_div(n_groups, t.q.groups)), block(t.q.threads);
    hipStream_t st = (hipStream_t)stream;
#define SR_SIG(KIND, KMAX) \
    signals_kernel<KIND, KMAX><<<grid, block, t.lds, st>>>(actions, obs, end_step, n_groups, stride, t.q, lens, t.sums_at, t.terms_at_once, out)
    if (t.direct) {
        switch (t.size) {
            case 8: SR_SIG(PREFIX_ONE32, 8); break;
            case 16: SR_SIG(PREFIX_ONE32, 16); break;
            case 24: SR_SIG(PREFIX_ONE32, 24); break;
            default: SR_SIG(PREFIX_ONE32, 32); break;
        }
    } else if (t.size == PREFIX_TWO16) SR_SIG(PREFIX_TWO16, 0);
    else if (t.size == PREFIX_TWO32) SR_SIG(PREFIX_TWO32, 0);
    else SR_SIG(PREFIX_ONE32, 0);
#undef SR_SIG
    SR_HIP(hipGetLastError());
    return SR_OK;
}
