// How the gate and the signals kernels lay out their groups over workgroups and LDS (prefix_match.h), in plain C++ so that it can
// be evaluated and tested without a GPU.
#pragma once
#include "plan.h"

namespace sr {

constexpr int kPrefixThreads = 256;     // most threads of a workgroup

// row of the directly compared symbols: an odd multiple of 16 bytes, the rows of sixteen consecutive members in different banks
SR_HD constexpr int prefix_act_stride(int kmax) { return kmax % 8 == 4 ? kmax : kmax + 4; }

// Compare, or build tables?  The symbols are not known here, and comparing takes the same time whatever they are, where tables win with
// symbols below 64, are about even below 100 and lose up to three times with all different ones: comparing is taken where the most that it
// can lose is less than the most that tables can.  Up to eight steps (65 536 groups of 8, 5 steps: gate 17.0 us; with tables 13.2, 24.8 and
// 31.4; 8 steps 17.8, and 12.8, 19.0 and 49.0; 3 members, 5 steps 8.7, and 9.1, 11.2 and 13.9).  Longer prefixes share a table among
// G - 1 pairs: up to `few` members where the groups fill the chip (65 536 groups of 5, 12 steps: gate 14.0 us, and 11.0, 16.2 and 42.8; groups
// of 3: signals 17.8, and 18.0, 24.7 and 41.8), but not in too few wavefronts (64 groups of 3, 32 steps: gate 9.7 us, with tables 7.9).
inline bool prefix_direct(int n_groups, int G, int L, int few) {
    return L <= 8 || (G <= few && (long long)n_groups * G >= 1500LL * L);
}

// How a workgroup lays out its groups; L = longest requested prefix.
struct PrefixGeom {
    int G, L, Q;          // Q = member pairs: columns of the tables
    int groups, threads;  // groups per workgroup and its size
    int lanes;            // lanes per group: its pairs when comparing, (member, member pair) combinations with tables
    // tables only: bytes of LDS
    int row_bytes;        // one symbol's masks
    int body;             // offset of the tables, behind the element ids [member][16 or 32] (16 bits: symbol * row_bytes)
    int slots_log2;       // hash slots per group: a power of two, at least twice its elements
    int hash_groups;      // groups that take part in a turn where symbols are hashed
    int total;
};
constexpr int kPrefixSyms = 64;         // table rows of a group whose symbols need no hashing

// How a lane runs its pairs: two in the halves of a register (up to 16 steps), two in a register each, or one.  The last takes
// more lanes and a shorter chain of instructions each: for launches that do not fill the chip.
enum PrefixKind { PREFIX_TWO16, PREFIX_TWO32, PREFIX_ONE32 };
SR_HD constexpr int prefix_steps(int kind) { return kind == PREFIX_TWO16 ? 16 : 32; }
// a group's tables when its symbols are hashed: a row per element, the slots, the symbols themselves
SR_HD inline int prefix_hash_rows(const PrefixGeom &q) { return q.G * q.L * q.row_bytes; }
SR_HD inline int prefix_hash_bytes(const PrefixGeom &q) {
    return round_up(prefix_hash_rows(q), 16) + (4 << q.slots_log2) + round_up(q.G * q.L * 4, 16);
}

// x / d for 0 <= x < 2^14 and 1 <= d < 2^14.  On the device by a reciprocal, a few instructions instead of 35: (x + 1/2) / d is 1 / 2d
// or more from an integer, and the three roundings move it by less than 2^-21 x / d
SR_HD inline int short_quotient(int x, int d) {
#ifdef __HIP_DEVICE_COMPILE__
    return (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)d));
#else
    return x / d;
#endif
}

// How the groups of a workgroup take turns when some symbol is not below kPrefixSyms; `most`: the largest symbol.  Tables with a row
// for every number up to it where at least as many groups fit as by hashing, which is so for every symbol below the number of a
// group's elements.  65 536 groups of 8, prefixes 5, 10 and 15, gate / signals in us: symbols below 64 18.5 / 61.5, all groups at once;
// below 100 25.8 / 78.1 in turns, hashed 50.0 / 108 (and with 16-bit masks of one member a read, whose tables held 120 symbols, 42.1 /
// 120); below 200 34.2 / 96.7, hashed 50.9 / 110; below 1000 53.5 / 116, hashed; all different 82 / 148.  32 steps, below 128: 66 / 124,
// hashed 147 / 352.
struct PrefixTurns {
    bool hashed;
    int groups, group_bytes;            // groups of a turn; one group's tables
};
SR_HD inline PrefixTurns prefix_turns(const PrefixGeom &q, int n_here, unsigned most) {
    if (most < 2048) {                               // no group has more rows, hashed or not
        const int pieces = (((int)most + 1) * q.row_bytes + 15) >> 4, fit = short_quotient((q.total - q.body) >> 4, pieces);
        if (fit >= q.hash_groups) {
            const int turns = short_quotient(n_here + fit - 1, fit);
            return PrefixTurns{false, short_quotient(n_here + turns - 1, turns), pieces * 16};       // turns of equal size
        }
    }
    return PrefixTurns{true, q.hash_groups, round_up(prefix_hash_rows(q), 16)};
}

// Groups per workgroup: the count that fills whole wavefronts of lanes best within 256 lanes.  A few groups (an episode's
// gate) are spread over the compute units first: no workgroup takes more than its share of 512.
inline bool prefix_geometry_direct(int n_groups, int G, int L, int kmax, int lds_limit, int extra, PrefixGeom *q) {
    *q = PrefixGeom{};
    q->G = G;
    q->L = L;
    q->lanes = G * (G - 1) / 2;
    double best = 0.0;
    for (int n = 1; n * q->lanes <= 256 && n <= ceil_div(n_groups, 512); ++n) {
        if (n * (G * prefix_act_stride(kmax) * 4 + extra) > lds_limit) break;
        const double use = (double)(n * q->lanes) / round_up(n * q->lanes, 64);
        if (use >= best) {
            best = use;
            q->groups = n;
        }
    }
    q->total = q->groups * G * prefix_act_stride(kmax) * 4;
    // lanes for the pairs, and no more than eight elements a lane while the symbols are staged (small groups have more
    // elements than pairs: 16384 groups of 2 with 32 arbitrary symbols take the gate 10.5 us, 25.5 with 64 lanes)
    const int lanes = q->groups * q->lanes, build = ceil_div(q->groups * G * (kmax <= 16 ? kmax : 32), 8);
    q->threads = round_up(lanes > build ? lanes : build, 64);
    if (q->threads > 256) q->threads = 256;
    return q->groups > 0;
}

constexpr int kPrefixVecs = 4;          // 16-byte pieces of the members' rows that a lane loads at most
// Of the counts that fill the wavefronts equally well the largest within `lds_limit` bytes is taken; with two pairs in a register, and more
// workgroups than two per compute unit, the largest within `four` bytes, of which four workgroups fit: groups of four had taken 51 KB
// (65 536 groups of 4, 16 steps, signals: 88.6 -> 76.3 us with all different symbols, 76.1 before the tables held pairs; 21.9 -> 21.1 with
// symbols below 64; with three prefix lengths 92.9 -> 73.6 and 33.3 -> 29.5; groups of 6 139 -> 114 and 52.9 -> 45.8).  With two registers
// groups of 5 lose what they gain (20 steps: 143 -> 112, and 46.3 -> 50.0).
inline bool prefix_geometry_tables(int n_groups, int G, int L, int kind, int lds_limit, int four, int hash_lds, int extra, PrefixGeom *q) {
    *q = PrefixGeom{};
    q->G = G;
    q->L = L;
    q->Q = ceil_div(G, 2);
    q->lanes = kind == PREFIX_ONE32 ? G * (G - 1) / 2 : q->Q * q->Q - (G & 1);
    q->row_bytes = q->Q * (kind == PREFIX_TWO16 ? 4 : 8);
    q->slots_log2 = 4;
    while ((1 << q->slots_log2) < 2 * G * L) ++q->slots_log2;
    const int steps = prefix_steps(kind), hash = prefix_hash_bytes(*q);
    auto body = [&](int n) { const int b = n * kPrefixSyms * q->row_bytes; return round_up(b > hash ? b : hash, 16); };
    double best = 0.0;
    for (int n = 1; n * q->lanes <= 256 && n * G * (steps / 4) <= 256 * kPrefixVecs && n <= ceil_div(n_groups, 512); ++n) {
        const int bytes = n * (G * steps * 2 + extra) + body(n);
        if (bytes > lds_limit) break;
        const double use = (double)(n * q->lanes) / round_up(n * q->lanes, 64);
        const bool roomy = kind != PREFIX_TWO16 || bytes <= four || ceil_div(n_groups, n) <= 512;
        if (use > best || (use == best && roomy)) {
            best = use;
            q->groups = n;
        }
    }
    if (q->groups == 0) return false;
    q->body = round_up(q->groups * G * steps * 2, 16);
    // hashed symbols: all groups at once where that costs no workgroup its place; otherwise two at least
    const int all = q->groups * hash, most = lds_limit - q->groups * extra - q->body;
    int room = hash_lds - q->groups * extra - q->body;
    if (room < 2 * hash) room = 2 * hash;
    if (room > most || ceil_div(n_groups, q->groups) <= 512) room = most;
    int bytes = round_up(room < all ? room / hash * hash : all, 16);
    if (bytes < body(q->groups)) bytes = body(q->groups);
    q->hash_groups = bytes / hash;
    if (q->hash_groups > q->groups) q->hash_groups = q->groups;
    q->total = q->body + bytes;
    const int lanes = q->groups * q->lanes, build = ceil_div(q->groups * G * steps, ceil_div(n_groups, q->groups) <= 1024 ? 2 : 8);
    q->threads = round_up(lanes > build ? lanes : build, 64);
    if (q->threads > 256) q->threads = 256;
    return true;
}

// ---------------------------------------------------------------------------------------------
// gate
// ---------------------------------------------------------------------------------------------
constexpr int kGateLds = 40 * 1024;      // LDS of one workgroup: four workgroups or more per compute unit
// ... where symbols are hashed, whose tables are larger: 65 536 groups of 12, 12 steps 95 us, 109 with 16 KiB, 113 with 32, 147 with 40
// (groups of 8, 15 steps: 86, 80, 89 and 113); 40 and more take occupancy from calls that hash nothing (20 -> 26 us)
constexpr int kGateHashLds = 24 * 1024;

struct GateLayout {
    bool direct;          // symbols compared in registers
    int size;             // steps the kernel is compiled for when comparing, PrefixKind otherwise
    PrefixGeom q;
    int lds;
};
inline bool gate_layout(int n_groups, int G, int maxlen, GateLayout *t) {
    t->direct = prefix_direct(n_groups, G, maxlen, 6);
    if (t->direct) {
        t->size = maxlen <= 4 ? 4 : maxlen <= 8 ? 8 : maxlen <= 12 ? 12 : maxlen <= 16 ? 16 : maxlen <= 24 ? 24 : 32;
        if (!prefix_geometry_direct(n_groups, G, maxlen, t->size, kGateLds, 16, &t->q)) return false;
    } else {
        // Beyond 16 steps a lane with two pairs has twice the instructions: one pair where that still leaves no more than eight
        // wavefronts per compute unit (300 groups of 8, 32 steps: 6.6 us, 7.6 with two; 2000 groups 6.2)
        t->size = maxlen <= 16 ? PREFIX_TWO16 : (long long)n_groups * G * (G - 1) / 2 <= 256 * 512 ? PREFIX_ONE32 : PREFIX_TWO32;
        if (!prefix_geometry_tables(n_groups, G, maxlen, t->size, kGateLds, kGateLds, kGateHashLds, 16, &t->q)) return false;
    }
    t->lds = t->q.total + 16 * t->q.groups;           // and the sums
    return true;
}

// ---------------------------------------------------------------------------------------------
// signals
// ---------------------------------------------------------------------------------------------
constexpr int kSigLds = 52 * 1024;                   // LDS of symbols, tables and sums: three workgroups per compute unit or more
constexpr int kSigHashLds = 40 * 1024;               // ... where symbols are hashed: four
constexpr int kSigThird = 53744;                      // a third of a compute unit's LDS, in its granules of 1280 bytes, less the kernels' own 16
constexpr int kSigTerms = 24 * 1024;                 // LDS that the quotients may take: three K of sixteen groups of 8 at once

// What the workgroup keeps behind symbols and tables: byte offsets, 8-byte arrays first.
struct SigLds {
    int out, lcm, recip, p, log_p, repeats, code, obs, at, end, first, hold, total;
    int code_stride;                  // pairs of a group, made odd: the groups' terms in different banks
};
SR_HD inline SigLds sig_lds(int G, int groups, int n_lens) {
    SigLds o;
    const int pairs = G * (G - 1) / 2, members = groups * G;
    o.code_stride = pairs | 1;
    o.out = 0;                                    // [K][group] sr_signals_t
    o.lcm = o.out + n_lens * groups * 64;         // lcm(1..32) / n
    o.recip = o.lcm + 33 * 8;                     // 1 / n, n = 1 .. 63 (0: 0)
    o.p = o.recip + 64 * 8;                       // 0, then c / n, 1 <= c <= n <= G
    o.log_p = o.p + (G * (G + 1) / 2 + 1) * 8;    // log(c / n)
    o.repeats = o.log_p + (G * (G + 1) / 2 + 1) * 8;    // [K][group] members whose prefix an earlier member has
    o.code = o.repeats + n_lens * groups * 4;     // [distinct K][group][pair] see SigCode
    o.obs = o.code + n_lens * groups * o.code_stride * 4;        // [K][member] o_{i,K}
    o.at = o.obs + n_lens * members * 4;          // [K][group] bits of the members that reach step K | finished by K << 24
    o.end = o.at + n_lens * groups * 4;           // [member]
    o.first = o.end + members * 4;                // [member] positions of first occurrences of bigrams
    o.hold = o.first + members * 4;               // [K][member] holders of its step-K action if it is the first of them, | 32 the
    o.total = round_up(o.hold + n_lens * members * 2, 16);       // first to hold its observation (16 bits)
    return o;
}

struct SignalsLayout {
    bool direct;
    int size;             // both as in GateLayout
    PrefixGeom q;
    int terms_at_once;    // prefix lengths whose quotients are there at a time, in the place of symbols and tables
    int sums_at;          // offset of SigLds
    int lds;
};
inline bool signals_layout(int n_groups, int G, int maxlen, int n_lens, int distinct, SignalsLayout *t) {
    // LDS behind symbols and tables: at most `extra` for every group, and `fixed`
    const int extra = sig_lds(G, 2, n_lens).total - sig_lds(G, 1, n_lens).total + 16, fixed = sig_lds(G, 1, n_lens).total - extra + 16;
    PrefixGeom &q = t->q;
    // Up to eight steps the tables are nevertheless cheaper for large groups that fill the chip (65 536 groups of 8, 5 steps: 47.4 us by
    // comparison, 34.8 with tables of symbols below 64, 42.5 below 100, 49.2 all different; 8 steps: 48.1, and 39.1, 42.8 and 78.6; groups
    // of 16, 8 steps: 232, and 142, 147 and 217)
    const bool many = (long long)n_groups * G >= 32000 && (G >= 12 || (G >= 8 && maxlen <= 6));
    t->direct = prefix_direct(n_groups, G, maxlen, 3) && !many;
    if (t->direct) {
        t->size = maxlen <= 8 ? 8 : maxlen <= 16 ? 16 : maxlen <= 24 ? 24 : 32;
        if (!prefix_geometry_direct(n_groups, G, maxlen, t->size, kSigLds - fixed, extra, &q)) return false;
    } else {
        // beyond 16 steps a pair a lane where the pairs leave eight wavefronts per compute unit or fewer, as in the gate
        t->size = maxlen <= 16 ? PREFIX_TWO16 : (long long)n_groups * G * (G - 1) / 2 <= 256 * 512 ? PREFIX_ONE32 : PREFIX_TWO32;
        if (!prefix_geometry_tables(n_groups, G, maxlen, t->size, kSigLds - fixed, kSigHashLds - fixed, kSigHashLds - fixed, extra, &q)) return false;
    }
    // A launch that does not fill the chip takes whole workgroups: four wavefronts share the phases of a group.  By comparison up to
    // four workgroups per compute unit, which are resident together (16 384 groups of 2 or 3, 5 steps: 9.4 and 10.0 -> 7.8 us, 2, 4 and 8
    // steps: 13.5 and 12.6 -> 8.7 and 9.1; at 2048 workgroups no gain)
    if (ceil_div(n_groups, q.groups) <= (t->direct ? 1024 : q.groups <= 4 ? 512 : 0)) q.threads = kPrefixThreads;
    // quotients take the place of symbols and tables: of every length at once up to kSigTerms bytes, while three workgroups fit
    const SigLds sums = sig_lds(G, q.groups, n_lens);
    const int per_len = q.groups * sums.code_stride * 16, left = kSigThird - sums.total;
    int room = left < kSigTerms ? left : kSigTerms;
    if (room < q.total) room = q.total;
    t->terms_at_once = room / per_len < 1 ? 1 : room / per_len < distinct ? room / per_len : distinct;
    t->sums_at = round_up(q.total > t->terms_at_once * per_len ? q.total : t->terms_at_once * per_len, 16);
    t->lds = t->sums_at + sums.total;
    return true;
}

}  // namespace sr
