// Edit distances of action prefixes, bit-parallel (shared by the gate and the signals kernels).
//
// The table of two sequences a, b of at most 32 symbols is advanced one row (one symbol of a) at a time with its
// vertical differences held as two 32-bit masks -- Myers' bit-vector recurrence (J. ACM 46, 1999) in Hyyro's form
// for the global distance: eleven 32-bit operations per row instead of about five per cell.  Bit u of the masks is
// column u + 1; information only moves from lower to higher bits, so cell (r, c) can be read for every c whatever
// the columns beyond it hold, and one pass serves every prefix length.
//
// What the recurrence needs per row is the mask of positions of b that equal a[r].  Two ways to have it:
// Tables.  A workgroup builds, once per group, the table mask[member][symbol]; a row's mask is then one LDS read.  Symbols
// that all lie in the table's range index it as they are (ids below 64 always do: action ids of a turn are tokens modulo a
// small number).  Where some symbol of the workgroup does not, every symbol is first replaced by the index of one element
// of its group that holds it (hash insertion in LDS, compare-and-swap on the slot; which of several equal elements
// wins does not matter).
// Comparison.  Every pair compares its 2 * K symbols in registers: 2 * K * K more instructions per pair, and nothing to build.
// prefix_direct says which.
#pragma once
#include "sr_internal.h"

namespace sr {

// Sizes of one workgroup's tables; L = longest requested prefix, KMAX = its size class (4, 8, 12, 16, 24 or 32).
struct PrefixGeom {
    int G, L;
    int slots_log2;       // hash slots per group: a power of two, at least twice its elements
    int row_stride;       // mask entries per member: G * L (one per element of the group), at least 64, padded to an odd
                          // number of LDS words so that one symbol's entries of several members lie in several banks
    int groups, threads;  // groups per workgroup and its size
};

__host__ __device__ inline int prefix_mask_bytes(int kmax) { return kmax <= 16 ? 2 : 4; }
// row of the directly compared symbols: an odd multiple of 16 bytes, the rows of sixteen consecutive members in different banks
__host__ __device__ constexpr int prefix_act_stride(int kmax) { return kmax % 8 == 4 ? kmax : kmax + 4; }
// byte offsets of [masks | slots | act | id] for n groups, or of act alone; every part a multiple of 16 bytes
struct PrefixLds {
    int slots, act, id, total;
};
__host__ __device__ inline PrefixLds prefix_lds(const PrefixGeom &q, int n, int kmax, bool direct) {
    PrefixLds o{};
    if (direct) {
        o.total = n * q.G * prefix_act_stride(kmax) * 4;
        return o;
    }
    o.slots = round_up(n * q.G * q.row_stride * prefix_mask_bytes(kmax), 16);
    o.act = o.slots + (n << q.slots_log2) * 4;
    o.id = o.act + round_up(n * q.G * q.L * 4, 16);
    o.total = o.id + n * q.G * kmax * 2;
    return o;
}

// Compare, or build tables?  Up to eight steps the comparisons cost less than zeroing and filling a table, for every group size
// (65 536 groups of 8, 5 steps: gate 17.6 us; with tables 18.7, 26 where symbols lie beyond their range; 3 members: 7.8, 8.3 and
// 19).  Longer prefixes share a table among G - 1 pairs: up to `few` members comparing is cheaper still where the groups
// fill the chip (65 536 groups of 5, 12 steps: gate 14 us, tables 17 and 29; groups of 3: signals 18, tables 28 and 38; 8
// members: gate 41 against 33), and a long chain in too few wavefronts where they do not (64 groups of 3, 32 steps:
// gate 10.0 us, tables 7.7; 16 384 groups of 2: 8.8 and 7.8).
inline bool prefix_direct(int n_groups, int G, int L, int few) {
    return L <= 8 || (G <= few && (long long)n_groups * G >= 1500LL * L);
}

// Groups per workgroup: the count that fills whole wavefronts of pair lanes best (28 pairs: nine groups leave 4 of 256
// lanes idle) within 256 lanes and `lds_limit` bytes of tables plus `extra` bytes per group.  A few groups (an episode's
// gate) are spread over the compute units first: no workgroup takes more than its share of 512.
inline bool prefix_geometry(int n_groups, int G, int L, int kmax, bool direct, int lds_limit, int extra, PrefixGeom *q) {
    const int pairs = G * (G - 1) / 2;
    q->G = G;
    q->L = L;
    q->slots_log2 = 4;
    while ((1 << q->slots_log2) < 2 * G * L) ++q->slots_log2;
    const int per_word = 4 / prefix_mask_bytes(kmax);
    q->row_stride = (ceil_div(G * L > 64 ? G * L : 64, per_word) | 1) * per_word;
    q->groups = 0;
    double best = 0.0;
    for (int n = 1; n * pairs <= 256 && n <= ceil_div(n_groups, 512); ++n) {
        if (prefix_lds(*q, n, kmax, direct).total + n * extra > lds_limit) break;
        const double use = (double)(n * pairs) / round_up(n * pairs, 64);
        if (use >= best) {
            best = use;
            q->groups = n;
        }
    }
    // lanes for the pairs, and no more than eight elements a lane while the tables are built (small groups have more
    // elements than pairs: 16384 groups of 2 with 32 arbitrary symbols take the gate 10.5 us, 25.5 with 64 lanes)
    const int lanes = q->groups * pairs, build = ceil_div(q->groups * G * (kmax <= 16 ? kmax : 32), 8);
    q->threads = round_up(lanes > build ? lanes : build, 64);
    if (q->threads > 256) q->threads = 256;
    return q->groups > 0;
}

#ifdef __HIPCC__
// x / d for 0 <= x < 2^14 and 1 <= d <= 32, inv = 1.0f / d: the distance of (x + 1/2) / d from an integer is at least 1/64,
// far beyond the rounding of two 32-bit operations on values below 2^14
__device__ __forceinline__ int small_div(int x, float inv) { return (int)(((float)x + 0.5f) * inv); }

// Fill the tables for `rows` members starting at `src` ([rows][stride] in global memory).  All threads of the workgroup
// take part; ends with a barrier.
template <int KMAX>
__device__ __forceinline__ void prefix_build(char *lds, const PrefixGeom &q, const PrefixLds &off, int rows,
                                             const int32_t *__restrict__ src, int stride) {
    constexpr int KP = KMAX <= 16 ? 16 : 32;                     // lanes per member
    unsigned *masks = (unsigned *)lds;
    uint16_t *id = (uint16_t *)(lds + off.id);
    int32_t *act = (int32_t *)(lds + off.act);
    const int tid = threadIdx.x, nt = blockDim.x;
    auto mark = [&](int r, int c, unsigned sym) {
        id[r * KMAX + c] = (uint16_t)sym;
        const int m = r * q.row_stride + (int)sym;
        if constexpr (KMAX <= 16) atomicOr(&masks[m >> 1], (1u << c) << (16 * (m & 1)));
        else atomicOr(&masks[m], 1u << c);
    };
    for (int i = tid; i < off.slots / 16; i += nt) ((uint4 *)lds)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    int fits = 1;
    for (int e0 = tid; e0 < rows * KP; e0 += 4 * nt) {           // four loads in flight per lane
        unsigned v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * nt, r = e / KP, c = e % KP;
            v[u] = r < rows && c < q.L ? (unsigned)src[(size_t)r * stride + c] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * nt, r = e / KP, c = e % KP;
            if (r < rows && c < q.L) {
                act[r * q.L + c] = (int32_t)v[u];
                if (v[u] < (unsigned)q.row_stride) mark(r, c, v[u]);
                else fits = 0;
            }
        }
    }
    if (__syncthreads_and(fits)) return;

    unsigned *slots = (unsigned *)(lds + off.slots);
    const int GL = q.G * q.L;
    const float inv_G = 1.0f / (float)q.G;
    for (int i = tid; i < off.act / 16; i += nt) ((uint4 *)lds)[i] = make_uint4(0, 0, 0, 0);   // masks and slots
    __syncthreads();
    const unsigned wrap = (1u << q.slots_log2) - 1u;
    for (int e = tid; e < rows * KP; e += nt) {
        const int r = e / KP, c = e % KP;
        if (c >= q.L) continue;
        const int g = small_div(r, inv_G);
        const int32_t v = act[r * q.L + c];
        unsigned *table = slots + ((size_t)g << q.slots_log2);
        const int32_t *ga = act + g * GL;
        const unsigned mine = (unsigned)((r - g * q.G) * q.L + c) + 1u;      // element within the group; 0 = free slot
        unsigned rep = mine;
        unsigned h = ((unsigned)v * 0x9E3779B1u) >> (32 - q.slots_log2);
        for (unsigned probe = 0; probe <= wrap; ++probe) {                   // at most half of the slots are ever taken
            const unsigned old = atomicCAS(&table[h], 0u, mine);
            if (old == 0u) break;
            if (ga[old - 1u] == v) { rep = old; break; }
            h = (h + 1u) & wrap;
        }
        mark(r, c, rep - 1u);
    }
    __syncthreads();
}

// Without tables: the symbols of `rows` members as they are, [row][prefix_act_stride].  Entries from L on hold anything: they
// only reach bits and rows that nobody reads.  Ends with a barrier.
template <int KMAX>
__device__ __forceinline__ void prefix_stage(char *lds, const PrefixGeom &q, int rows, const int32_t *__restrict__ src, int stride) {
    constexpr int KP = KMAX <= 8 ? KMAX : KMAX <= 16 ? 16 : 32;  // lanes per member
    int32_t *act = (int32_t *)lds;
    const int nt = blockDim.x;
    for (int e0 = threadIdx.x; e0 < rows * KP; e0 += 4 * nt) {   // four loads in flight per lane
        int32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * nt, r = e / KP, c = e % KP;
            v[u] = r < rows && c < q.L ? src[(size_t)r * stride + c] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * nt, r = e / KP, c = e % KP;
            if (r < rows && c < q.L) act[r * prefix_act_stride(KMAX) + c] = v[u];
        }
    }
    __syncthreads();
}

// a member's staged symbols c0 .. c0 + N - 1 (multiples of four)
template <int KMAX, int N>
__device__ __forceinline__ void prefix_symbols(const char *lds, int row, int c0, int32_t (&x)[N]) {
    const int4 *p = (const int4 *)((const int32_t *)lds + row * prefix_act_stride(KMAX) + c0);
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        const int4 v = p[i];
        x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
    }
}

// m[i] = positions of b that hold a[i], for N symbols (a multiple of four): a compare and an add with carry (m = 2 m + equal)
// per symbol and position.  Four symbols take turns in one asm block, because a vector instruction may read a compare's
// scalar result only two instructions later; left to the compiler the same sum took two more instructions and a wait each.
template <int KMAX, int N>
__device__ __forceinline__ void prefix_equal(const int32_t (&a)[N], const int32_t (&b)[KMAX], unsigned (&m)[N]) {
#pragma unroll
    for (int i = 0; i < N; i += 4) {
        unsigned m0 = 0, m1 = 0, m2 = 0, m3 = 0;
#pragma unroll
        for (int c = KMAX - 1; c >= 0; --c) {
            unsigned long long t0, t1, t2, t3;
            asm("v_cmp_eq_u32_e64 %4, %8, %12\n\t"
                "v_cmp_eq_u32_e64 %5, %9, %12\n\t"
                "v_cmp_eq_u32_e64 %6, %10, %12\n\t"
                "v_cmp_eq_u32_e64 %7, %11, %12\n\t"
                "v_addc_co_u32_e64 %0, %4, %0, %0, %4\n\t"
                "v_addc_co_u32_e64 %1, %5, %1, %1, %5\n\t"
                "v_addc_co_u32_e64 %2, %6, %2, %2, %6\n\t"
                "v_addc_co_u32_e64 %3, %7, %3, %3, %7"
                : "+v"(m0), "+v"(m1), "+v"(m2), "+v"(m3), "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3)
                : "v"(a[i]), "v"(a[i + 1]), "v"(a[i + 2]), "v"(a[i + 3]), "v"(b[c]));
        }
        m[i] = m0; m[i + 1] = m1; m[i + 2] = m2; m[i + 3] = m3;
    }
}

// positions of member `row` that hold the symbol `id`
template <int KMAX>
__device__ __forceinline__ unsigned prefix_mask(const char *lds, const PrefixGeom &q, int row, int id) {
    const int m = row * q.row_stride + id;
    if constexpr (KMAX <= 16) return ((const uint16_t *)lds)[m];
    else return ((const unsigned *)lds)[m];
}

// The masks of rows r0 .. r0 + 7 of the table of members ri (a) and rj (b), requested together so that the LDS latency is
// paid once; rows from L on, which nobody asks for, get 0.
template <int KMAX>
__device__ __forceinline__ void prefix_masks8(const char *lds, const PrefixGeom &q, const PrefixLds &off, int ri, int rj,
                                              int r0, unsigned (&eq)[8]) {
    const uint4 raw = *(const uint4 *)(lds + off.id + (ri * KMAX + r0) * 2);      // eight 16-bit ids
    const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int t = 0; t < 8; ++t)
        eq[t] = r0 + t < q.L ? prefix_mask<KMAX>(lds, q, rj, (int)((w[t >> 1] >> (16 * (t & 1))) & 0xFFFFu)) : 0u;
}

// Pair p of a group of G -> (i, j), i < j, pairs in the order (0,1), (0,2), ..., (G-2,G-1): the largest i with
// i * (2G - 1 - i) / 2 <= p.  (b - sqrt(b^2 - 8p)) / 2, b = 2G - 1, is an integer exactly at the first pair of an i;
// the added 1/128 keeps rounding from missing it and is too little to reach the next one (G <= 16).
__device__ __forceinline__ void pair_members(int p, int G, int *i, int *j) {
    const float b = (float)(2 * G - 1);
    const int a = (int)((b - __builtin_amdgcn_sqrtf(b * b - 8.0f * (float)p)) * 0.5f + 0.0078125f);
    *i = a;
    *j = p - a * (2 * G - 1 - a) / 2 + a + 1;
}

// One row of the table: eq = positions of b that equal the row's symbol of a.
__device__ __forceinline__ void prefix_row(unsigned eq, unsigned &pv, unsigned &mv) {
    const unsigned xv = eq | mv;
    const unsigned xh = (((eq & pv) + pv) ^ pv) | eq;
    const unsigned ph = ((mv | ~(xh | pv)) << 1) | 1u;
    const unsigned mh = (pv & xh) << 1;
    pv = mh | ~(xv | ph);
    mv = ph & xv;
}
// bits 0 .. n-1, 0 <= n <= 32
__device__ __forceinline__ unsigned low_bits(int n) { return n >= 32 ? 0xFFFFFFFFu : (1u << n) - 1u; }
// cell (r, c) once row r is complete
__device__ __forceinline__ int prefix_cell(int r, int c, unsigned pv, unsigned mv) {
    return r + __popc(pv & low_bits(c)) - __popc(mv & low_bits(c));
}
#endif

}  // namespace sr
