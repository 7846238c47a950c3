// Edit distances of action prefixes, bit-parallel (shared by the gate and the signals kernels).
//
// The table of two sequences a, b of at most 32 symbols is advanced one row (one symbol of a) at a time with its
// vertical differences held as bit masks -- Myers' bit-vector recurrence (J. ACM 46, 1999) in Hyyro's form
// for the global distance: eleven operations per row instead of about five per cell.  Bit u of the masks is
// column u + 1; information only moves from lower to higher bits, so cell (r, c) can be read for every c whatever
// the columns beyond it hold, and one pass serves every prefix length.
//
// What the recurrence needs per row is the mask of positions of b that equal a[r].  Two ways to have it:
//
// Tables.  A workgroup builds mask[symbol][member] for its groups.  A symbol's masks of all members lie side by side, so one
// LDS read gives a lane those of two neighbouring members, and the lane runs one a against both: the pairs (i, 2q) and
// (i, 2q + 1).  Up to 16 steps the two masks are the halves of one register, and a step of the recurrence is one bitwise or
// packed 16-bit instruction for both pairs; beyond, two registers.  A group of eight takes 16 lanes instead of 28.
// Small symbols (action ids of a turn are tokens modulo a small number) index the tables as they are: the groups of a workgroup
// all at once where every symbol is below 64, otherwise with as many rows as the largest symbol of the workgroup asks for, the
// groups taking turns in the LDS, as many at a time as fit.  Where fewer would fit than by hashing, every symbol is first
// replaced by the index of one element of its group that holds it (hash insertion in LDS, compare-and-swap on the slot; which
// of several equal elements wins does not matter), with turns too.
//
// Comparison.  Every pair compares its 2 * K symbols in registers: 2 * K * K more instructions per pair, and nothing to build.
// prefix_direct says which (prefix_plan.h, as how a workgroup lays out its groups).
#pragma once
#include "prefix_plan.h"
#include "sr_internal.h"

namespace sr {

#ifdef __HIPCC__
// x / d for 0 <= x < 2^14 and d >= 1 (members, steps, the up to 120 lanes of a group), inv = 1.0f / d: (x + 1/2) / d is 1 / 2d or more
// from an integer, and the roundings of inv and of the product move it by less than 2^-22 (x + 1) / d
__device__ __forceinline__ int small_div(int x, float inv) { return (int)(((float)x + 0.5f) * inv); }

// ---------------------------------------------------------------------------------------------
// tables
// ---------------------------------------------------------------------------------------------
// The masks of a lane's two pairs: halves of one register (16 steps), or a register each (32 steps)
template <int KIND>
struct PrefixBits;
template <>
struct PrefixBits<PREFIX_TWO16> {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    unsigned x;
    __device__ static PrefixBits all(unsigned v) { return {v}; }
    __device__ unsigned half(int h) const { return h ? x >> 16 : x & 0xFFFFu; }
};
template <>
struct PrefixBits<PREFIX_TWO32> {
    unsigned x[2];
    __device__ static PrefixBits all(unsigned v) { return {{v, v}}; }
    __device__ unsigned half(int h) const { return x[h]; }
};
template <>
struct PrefixBits<PREFIX_ONE32> {
    unsigned x;
    __device__ static PrefixBits all(unsigned v) { return {v}; }
    __device__ unsigned half(int) const { return x; }
};

// One row of the table: eq = positions of b that equal the row's symbol of a.
__device__ __forceinline__ void prefix_row(unsigned eq, unsigned &pv, unsigned &mv) {
    const unsigned xv = eq | mv;
    const unsigned xh = (((eq & pv) + pv) ^ pv) | eq;
    const unsigned ph = ((mv | ~(xh | pv)) << 1) | 1u;
    const unsigned mh = (pv & xh) << 1;
    pv = mh | ~(xv | ph);
    mv = ph & xv;
}
__device__ __forceinline__ void prefix_row(PrefixBits<PREFIX_ONE32> eq, PrefixBits<PREFIX_ONE32> &pv, PrefixBits<PREFIX_ONE32> &mv) {
    prefix_row(eq.x, pv.x, mv.x);
}
__device__ __forceinline__ void prefix_row(PrefixBits<PREFIX_TWO32> eq, PrefixBits<PREFIX_TWO32> &pv, PrefixBits<PREFIX_TWO32> &mv) {
    prefix_row(eq.x[0], pv.x[0], mv.x[0]);
    prefix_row(eq.x[1], pv.x[1], mv.x[1]);
}
__device__ __forceinline__ void prefix_row(PrefixBits<PREFIX_TWO16> eq, PrefixBits<PREFIX_TWO16> &pv, PrefixBits<PREFIX_TWO16> &mv) {
    typedef PrefixBits<PREFIX_TWO16>::u16x2 u16x2;
    auto v = [](unsigned x) { return __builtin_bit_cast(u16x2, x); };
    auto u = [](u16x2 x) { return __builtin_bit_cast(unsigned, x); };
    const unsigned xv = eq.x | mv.x;
    const unsigned xh = (u(v(eq.x & pv.x) + v(pv.x)) ^ pv.x) | eq.x;
    const unsigned ph = u(v(mv.x | ~(xh | pv.x)) * (unsigned short)2 + (unsigned short)1);
    const unsigned mh = u(v(pv.x & xh) << (unsigned short)1);
    pv.x = mh | ~(xv | ph);
    mv.x = ph & xv;
}
// bits 0 .. n-1, 0 <= n <= 32
__device__ __forceinline__ unsigned low_bits(int n) { return n >= 32 ? 0xFFFFFFFFu : (1u << n) - 1u; }
// cell (r, c) once row r is complete
__device__ __forceinline__ int prefix_cell(int r, int c, unsigned pv, unsigned mv) {
    return r + __popc(pv & low_bits(c)) - __popc(mv & low_bits(c));
}
// cells (K, K) of a lane's two pairs, added; the second only if there is one
__device__ __forceinline__ unsigned prefix_cells(int K, bool second, PrefixBits<PREFIX_TWO16> pv, PrefixBits<PREFIX_TWO16> mv) {
    const unsigned m = low_bits(K) * (second ? 0x10001u : 1u);
    return (unsigned)((second ? 2 * K : K) + __popc(pv.x & m) - __popc(mv.x & m));
}
__device__ __forceinline__ unsigned prefix_cells(int K, bool, PrefixBits<PREFIX_ONE32> pv, PrefixBits<PREFIX_ONE32> mv) {
    return (unsigned)prefix_cell(K, K, pv.x, mv.x);
}
__device__ __forceinline__ unsigned prefix_cells(int K, bool second, PrefixBits<PREFIX_TWO32> pv, PrefixBits<PREFIX_TWO32> mv) {
    return (unsigned)(prefix_cell(K, K, pv.x[0], mv.x[0]) + (second ? prefix_cell(K, K, pv.x[1], mv.x[1]) : 0));
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
// Lane p of a group -> its member i and the (first) member j it is compared with.  With two pairs a lane, the members 2q and
// 2q + 1 have the lanes q^2 .. q^2 + 2q, i = 0 .. 2q: the first is no pair when i == 2q (its distance is 0), the second when the
// group ends at 2q.
template <int KIND>
__device__ __forceinline__ void prefix_lane(int p, int G, int *i, int *j) {
    if constexpr (KIND == PREFIX_ONE32) {
        pair_members(p, G, i, j);
    } else {
        const int q = (int)__builtin_amdgcn_sqrtf((float)p + 0.5f);
        *i = p - q * q;
        *j = 2 * q;
    }
}

// The members' rows as every lane holds them while the tables are built: 16-byte pieces tid, tid + threads, ... of [row][16 or
// 32 steps].  Steps from L on are 0.  `tail`: the last row of the whole input, behind which nothing may be read.
template <int KIND>
struct PrefixRows {
    static constexpr int kSteps = prefix_steps(KIND), kRowVecs = kSteps / 4;
    int32_t v[kPrefixVecs][4];

    __device__ static bool used(int u, int rows) { return u * (int)blockDim.x < rows * kRowVecs; }       // uniform
    // lanes beyond the last row take it once more
    __device__ static int row(int u, int rows, int tid) { return min((tid + u * (int)blockDim.x) / kRowVecs, rows - 1); }
    __device__ static int step(int u, int tid) { return ((tid + u * (int)blockDim.x) % kRowVecs) * 4; }

    __device__ __forceinline__ void load(const PrefixGeom &q, int rows, const int32_t *__restrict__ src, int stride, int tail) {
        typedef int32_t piece __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int u = 0; u < kPrefixVecs; ++u) {
            if (!used(u, rows)) break;
            const int r = row(u, rows, threadIdx.x), c = step(u, threadIdx.x);
            const int32_t *p = src + (size_t)r * stride + c;
            piece x = {0, 0, 0, 0};
            if (c < q.L) {
                if (c + 4 <= stride && r != tail) x = *(const piece *)p;
                else x = piece{p[0], p[min(1, q.L - 1 - c)], p[min(2, q.L - 1 - c)], p[min(3, q.L - 1 - c)]};
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[u][e] = c + e < q.L ? x[e] : 0;
        }
    }
    // every symbol of this lane's indexes the tables as it is
    __device__ __forceinline__ bool fits(int rows) const {
        unsigned any = 0;
#pragma unroll
        for (int u = 0; u < kPrefixVecs; ++u) {
            if (!used(u, rows)) break;
            any |= (unsigned)(v[u][0] | v[u][1]) | (unsigned)(v[u][2] | v[u][3]);
        }
        return any < (unsigned)kPrefixSyms;
    }
    // of this lane's symbols, as unsigned numbers
    __device__ __forceinline__ unsigned largest(int rows) const {
        unsigned most = 0;
#pragma unroll
        for (int u = 0; u < kPrefixVecs; ++u) {
            if (!used(u, rows)) break;
            most = max(most, max(max((unsigned)v[u][0], (unsigned)v[u][1]), max((unsigned)v[u][2], (unsigned)v[u][3])));
        }
        return most;
    }
};

// byte offset of the word that holds member m's mask within a table row, and the mask's shift in it
template <int KIND>
__device__ __forceinline__ int prefix_column(int m) { return KIND == PREFIX_TWO16 ? (m >> 1) * 4 : m * 4; }
template <int KIND>
__device__ __forceinline__ int prefix_shift(int m) { return KIND == PREFIX_TWO16 ? (m & 1) * 16 : 0; }

// threadIdx.x anew in every turn: what the compiler works out from it ahead of the turns costs 20 to 30 registers, and with them a
// fourth of the wavefronts (signals of 65 536 groups of 8: 72 us instead of 62, whatever the symbols)
__device__ __forceinline__ int turn_tid() {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

__device__ __forceinline__ void prefix_zero(char *lds, int from, int bytes, int tid) {
    for (int i = tid * 16; i < bytes; i += blockDim.x * 16) *(uint4 *)(lds + from + i) = make_uint4(0, 0, 0, 0);
}

// 0 if all of the workgroup's symbols index tables of kPrefixSyms rows, otherwise the largest of them, as an unsigned number.
// A barrier, behind which the tables are zero too.
template <int KIND>
__device__ __forceinline__ unsigned prefix_beyond(int rows, const PrefixRows<KIND> &x) {
    __shared__ unsigned s_most[4];
    unsigned most = 0;
    if (!__all(x.fits(rows))) {                                  // the wavefront's: within rows of 16 lanes by rotation, then across them
        most = x.largest(rows);
        most = max(most, (unsigned)__builtin_amdgcn_update_dpp(0, (int)most, 0x128, 0xF, 0xF, false));
        most = max(most, (unsigned)__builtin_amdgcn_update_dpp(0, (int)most, 0x124, 0xF, 0xF, false));
        most = max(most, (unsigned)__builtin_amdgcn_update_dpp(0, (int)most, 0x122, 0xF, 0xF, false));
        most = max(most, (unsigned)__builtin_amdgcn_update_dpp(0, (int)most, 0x121, 0xF, 0xF, false));
        const auto h = __builtin_amdgcn_permlane32_swap(most, most, false, false);
        most = max(h[0], h[1]);
        const auto q = __builtin_amdgcn_permlane16_swap(most, most, false, false);
        most = max(q[0], q[1]);
    }
    s_most[threadIdx.x >> 6] = most;                             // every lane of a wavefront writes the same
    __syncthreads();
    most = 0;
#pragma unroll 1
    for (int w = 0; w < (int)blockDim.x >> 6; ++w) most = max(most, s_most[w]);
    return __builtin_amdgcn_readfirstlane(most);
}

// Tables of the groups g0 .. g0 + n - 1 (ALL: of every group), `group_bytes` each, from symbols that index them as they are; the
// tables are zero.  The caller's barrier follows.
template <int KIND, bool ALL>
__device__ __forceinline__ void prefix_mark(char *lds, const PrefixGeom &q, int rows, const PrefixRows<KIND> &x, int g0, int n,
                                            int group_bytes) {
    typedef PrefixRows<KIND> R;
    const float inv_G = 1.0f / (float)q.G;
    const int tid = ALL ? (int)threadIdx.x : turn_tid();
#pragma unroll
    for (int u = 0; u < kPrefixVecs; ++u) {
        if (!R::used(u, rows)) break;
        const int r = R::row(u, rows, tid), c = R::step(u, tid), g = small_div(r, inv_G), m = r - __mul24(g, q.G);
        if (!ALL && (unsigned)(g - g0) >= (unsigned)n) continue;
        unsigned id[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) id[e] = (unsigned)__mul24(x.v[u][e], q.row_bytes);
        *(uint2 *)(lds + (r * R::kSteps + c) * 2) = make_uint2(id[0] | id[1] << 16, id[2] | id[3] << 16);
        if (c < q.L) {                               // steps from L on set bits of symbol 0 that nobody looks at
            char *t = lds + q.body + __mul24(ALL ? g : g - g0, group_bytes) + prefix_column<KIND>(m);
            const unsigned bit = 1u << (c + prefix_shift<KIND>(m));
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicOr((unsigned *)(t + id[e]), bit << e);
        }
    }
}

// Tables of the groups g0 .. g0 + n - 1 from any symbols, in the place of the last round's.  Ends with a barrier.
template <int KIND>
__device__ __forceinline__ void prefix_hash(char *lds, const PrefixGeom &q, int rows, const PrefixRows<KIND> &x, int g0, int n) {
    typedef PrefixRows<KIND> R;
    const int tid = turn_tid(), nt = blockDim.x, GL = q.G * q.L, r0 = g0 * q.G, here = min(n * q.G, rows - r0);
    const int slots_at = q.body + q.hash_groups * round_up(prefix_hash_rows(q), 16);
    unsigned *slots = (unsigned *)(lds + slots_at);
    int32_t *act = (int32_t *)(lds + slots_at + (q.hash_groups * 4 << q.slots_log2));
    prefix_zero(lds, q.body, slots_at - q.body + (q.hash_groups * 4 << q.slots_log2), tid);        // masks and slots
#pragma unroll
    for (int u = 0; u < kPrefixVecs; ++u) {
        if (!R::used(u, rows)) break;
        const int r = R::row(u, rows, tid) - r0, c = R::step(u, tid);
        if (r >= 0 && r < here) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (c + e < q.L) act[r * q.L + c + e] = x.v[u][e];
                else ((uint16_t *)lds)[(r0 + r) * R::kSteps + c + e] = 0;
            }
        }
    }
    __syncthreads();
    const float inv_G = 1.0f / (float)q.G;
    const unsigned wrap = (1u << q.slots_log2) - 1u;
    const float inv_L = 1.0f / (float)q.L;
    for (int e = tid; e < here * q.L; e += nt) {
        const int r = small_div(e, inv_L), c = e - r * q.L, g = small_div(r, inv_G), m = r - g * q.G;
        const int32_t v = act[r * q.L + c];
        unsigned *table = slots + ((size_t)g << q.slots_log2);
        const int32_t *ga = act + g * GL;
        const unsigned mine = (unsigned)(m * q.L + c) + 1u;                  // element within the group; 0 = free slot
        unsigned rep = mine;
        unsigned h = ((unsigned)v * 0x9E3779B1u) >> (32 - q.slots_log2);
        for (unsigned probe = 0; probe <= wrap; ++probe) {                   // at most half of the slots are ever taken
            const unsigned old = atomicCAS(&table[h], 0u, mine);
            if (old == 0u) break;
            if (ga[old - 1u] == v) { rep = old; break; }
            h = (h + 1u) & wrap;
        }
        const unsigned id = (rep - 1u) * (unsigned)q.row_bytes;              // below 512 * 64
        ((uint16_t *)lds)[(r0 + r) * R::kSteps + c] = (uint16_t)id;
        atomicOr((unsigned *)(lds + q.body + g * round_up(prefix_hash_rows(q), 16) + prefix_column<KIND>(m) + id),
                 1u << (c + prefix_shift<KIND>(m)));
    }
    __syncthreads();
}

// Tables of a turn's groups, from g0 on, in the place of the turn before.  Begins and ends with a barrier.
template <int KIND>
__device__ __forceinline__ void prefix_turn(char *lds, const PrefixGeom &q, int rows, const PrefixRows<KIND> &x, int g0,
                                            const PrefixTurns &t) {
    __syncthreads();                                 // nobody reads the tables of the turn before
    if (t.hashed) {
        prefix_hash<KIND>(lds, q, rows, x, g0, t.groups);
    } else {
        prefix_zero(lds, q.body, t.groups * t.group_bytes, turn_tid());
        __syncthreads();
        prefix_mark<KIND, false>(lds, q, rows, x, g0, t.groups, t.group_bytes);
        __syncthreads();
    }
}

// Eight steps of member row `r`, from step c on (a multiple of eight): table rows as byte offsets
template <int KIND>
__device__ __forceinline__ void prefix_ids8(const char *lds, int r, int c, unsigned (&id)[8]) {
    const uint4 raw = *(const uint4 *)(lds + (r * prefix_steps(KIND) + c) * 2);
    const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int t = 0; t < 8; ++t) id[t] = t & 1 ? w[t >> 1] >> 16 : w[t >> 1] & 0xFFFFu;
}
// the lane's masks of table row `id` (byte offset); `column`: the group's tables and the word of member j
template <int KIND>
__device__ __forceinline__ PrefixBits<KIND> prefix_masks(const char *column, unsigned id) {
    if constexpr (KIND != PREFIX_TWO32) {
        return {*(const unsigned *)(column + id)};
    } else {
        const uint2 m = *(const uint2 *)(column + id);
        return {{m.x, m.y}};
    }
}

// ---------------------------------------------------------------------------------------------
// comparison
// ---------------------------------------------------------------------------------------------
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
#endif

}  // namespace sr
