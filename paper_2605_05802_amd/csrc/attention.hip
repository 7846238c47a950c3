// Grouped-query attention over the paged KV cache, for decode and for chunked prefill.
//
// A work item is one wavefront.  It owns up to 16*RT query rows -- consecutive query tokens of
// one unit times the n_rep query heads that share one kv head -- and one split of a token
// range.  The page layout is the MFMA operand layout: where a KV byte is used by one wavefront
// (a sequence's private context in decode) K and V tiles go from HBM straight into operand
// registers, each 16-byte lane load part of a contiguous 1 KiB run; where several items walk the
// same blocks (prefill, the shared prompt in decode) four of them share each block through LDS.
//
// Per 32-token block:   S^T = K Q^T   (tokens x rows; the accumulator leaves each lane holding
// four consecutive tokens of one query row), online softmax with the row maximum reduced across
// four lanes, then  O^T += V^T P^T  where the probabilities of the two 16-token
// tiles are packed, in-lane, into the P^T operand (the V block's slot order matches).
// Splits leave (un-normalised O, running max, running sum); a merge kernel combines the splits
// of the shared-prompt phase and of the private phase in fixed order.  Short contexts of a few sequences take one kernel for all of
// it (attn_whole_kernel).
//
// Group batching: during decode the prompt pages shared by the G members of a group are read
// once per group (the members' G*n_rep query rows form the row tiles of the work item)
// instead of once per member.
#include <type_traits>

#include "sr_internal.h"

namespace sr {
namespace {

constexpr float kNegBig = -1.0e30f;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A 16-byte K/V fragment.  STREAM: with the non-temporal hint, for tokens that exactly one work item reads in
// this launch (a sequence's private context): the caches do not retain the line and a long stream gains 8 %.
// Blocks that sibling work items re-read (the shared prompt, prefill) keep the default policy.
template <bool STREAM>
__device__ __forceinline__ bf16x8 load_frag(const uint16_t *p) {
    if constexpr (STREAM) return __builtin_bit_cast(bf16x8, __builtin_nontemporal_load((const u32x4 *)p));
    else return __builtin_bit_cast(bf16x8, *(const u32x4 *)p);
}

// An entry of the page table or of a unit map: the index is uniform and nothing writes the tables while the kernel runs.
// Read from the constant address space, because the compiler then loads it into a scalar register whatever code it stands
// in; as an ordinary load it came through a vector register where a launch has one phase, and the wait for it drained the
// K/V fragments in flight (chunks of one token over a context of 300 for 4 groups of 8 at head size 128: 20.1 us, 16.8 with
// scalar loads; of two tokens for 16 groups of 8 at head size 64: 13.2 against 9.6).
__device__ __forceinline__ int table_entry(const int32_t *table, int i) {
    return ((const __attribute__((address_space(4))) int32_t *)(uintptr_t)table)[i];
}

// The pages of a work item's token range: lane i holds the entry of the (first + i)th page, so that a page number inside the block
// loop costs a register read instead of a load whose wait would drain the K/V fragments (vector) or LDS reads (scalar) in
// flight.  64 pages at a time; the lanes past the last page hold it once more.
struct PageWindow {
    const int32_t *pt;
    int shift, last, first, entry;
    __device__ __forceinline__ void load(int page) {
        first = page;
        entry = pt[min(page + (int)(threadIdx.x & 63), last)];
    }
    // of tokens t_lo .. t_end - 1; nothing behind the page of t_end - 1 is read, whatever t_lo is
    __device__ __forceinline__ PageWindow(const int32_t *table, int page_shift, int t_lo, int t_end)
        : pt(table), shift(page_shift), last((t_end - 1) >> page_shift) { load(min(t_lo >> page_shift, last)); }
    // token t, uniform and within the range; the first page asked for never decreases
    __device__ __forceinline__ int page(int t) {
        const int i = t >> shift;
        if (i - first >= 64) {                       // uniform
            load(i);
            asm volatile("" : "+v"(entry));          // waits in here, not behind the branch in every iteration
        }
        return __builtin_amdgcn_readlane(entry, i - first);
    }
};

// Online softmax of one 32-token block for one row tile.  s holds the raw scores of tokens t0 + tt*16 + 4g + e of query row
// c; tokens above `lim` are invisible (MASKED; otherwise every token is visible to every used row).  The running maximum is
// kept in units of score * scale * log2(e), the scale is folded into the exponent's multiply-add, and the exponentials are
// the hardware's base-2 exponential as it is (arguments <= 0; results below 2^-126 of the row maximum may flush to zero).
// Leaves the probabilities packed for the P^T operand and the factor by which earlier sums shrink.
template <bool MASKED>
__device__ __forceinline__ void softmax_block(f32x4 (&s)[2], int t, int lim, float scale_log2, float &mrun, float &lrun,
                                              bf16x8 &pf, float &alpha) {
    bool ok[2][4];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            ok[tt][e] = !MASKED || t + tt * 16 + e <= lim;
            if (MASKED) s[tt][e] = ok[tt][e] ? s[tt][e] : kNegBig;
        }
    const float bmax = row_max(fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                                     fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3]))));
    const float mnew = fmaxf(mrun, bmax * scale_log2);
    alpha = __builtin_amdgcn_exp2f(mrun - mnew);
    mrun = mnew;
    float pv[8], psum = 0.f;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float pe = __builtin_amdgcn_exp2f(fmaf(s[tt][e], scale_log2, -mnew));
            pv[tt * 4 + e] = ok[tt][e] ? pe : 0.f;
            psum += pv[tt * 4 + e];
        }
    lrun = lrun * alpha + psum;
    pf = __builtin_bit_cast(bf16x8, make_uint4(pack_bf16x2(pv[0], pv[1]), pack_bf16x2(pv[2], pv[3]),
                                               pack_bf16x2(pv[4], pv[5]), pack_bf16x2(pv[6], pv[7])));
}

// query token of row `row` of a tile (row < 32, at most 16 rows to a token: the product is at least 1 / 32 from an integer)
__device__ __forceinline__ int row_token(const AttnArgs &a, int row) { return (int)(((float)row + 0.5f) * a.inv_rep); }

// Write the results of one work item: O^T tile lane (c, g) holds head dims dt*16 + 4g .. 4g+3 of row (rt, c).
template <int D, int RT>
__device__ __forceinline__ void store_item(const AttnArgs &a, const AttnPhase &p, const f32x4 (&o)[D / 16][RT],
                                           const float (&mrun)[RT], const float (&lrun)[RT], const int (&limit)[RT],
                                           int item, size_t first_tok, int kvh, int c, int g) {
    constexpr int DT = D / 16;
    const int n_rep = a.n_rep;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const float l = row_sum(lrun[rt]);
        if (limit[rt] < 0) continue;            // padding row of the tile: nobody reads it
        const int row = rt * 16 + c;
        if (a.direct_out) {
            // the only partial result of its rows: what the merge of one item computes, o / l (0 for an empty row)
            const int qi = row_token(a, row), col = (kvh * n_rep + row - qi * n_rep) * D + 4 * g;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                float r[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) r[e] = l > 0.f ? o[dt][rt][e] / l : 0.f;
                *(uint2 *)(a.direct_out + frag_offset((int)(first_tok + qi), col + dt * 16, a.out_mt_total)) =
                    make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
            }
            continue;
        }
        const size_t prow = (size_t)item * (16 * RT) + row;
        float *po = p.part_o + prow * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *(f32x4 *)(po + dt * 16 + 4 * g) = o[dt][rt];
        if (g == 0) *(float2 *)(p.part_ml + prow * 2) = make_float2(mrun[rt], l);
    }
}

// Queries of one work item: operand fragments, and the last visible token of each row (-1 = row unused)
template <int D, int RT>
__device__ __forceinline__ void load_queries(const AttnArgs &a, const AttnPhase &p, bf16x8 (&qf)[RT][D / 32], int (&limit)[RT],
                                             int qtile, int u_row0, int u_count, int kvh, int c, int g) {
    const int n_rep = a.n_rep;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int row = rt * 16 + c, tok = row_token(a, row);
        const int qi = qtile * p.q_per_item + tok;               // query token within the unit
        const int hr = row - tok * n_rep;
        const bool used = qtile < p.items_per_unit && row < p.q_per_item * n_rep && qi < u_count;
        limit[rt] = used ? p.causal_pos0 + qi * p.causal_stride : -1;
        const uint16_t *qp = a.q + (((size_t)u_row0 + qi) * a.n_q + kvh * n_rep + hr) * D + 8 * g;
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
            uint4 raw = make_uint4(0, 0, 0, 0);
            if (used) raw = *(const uint4 *)(qp + ks * 32);
            qf[rt][ks] = __builtin_bit_cast(bf16x8, raw);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// One work item alone (a sequence's private context during decode; units with few query tiles).
// ---------------------------------------------------------------------------------------------
// finish(o, mrun, lrun, limit, first query token) takes the results.
template <int D, int RT, typename F>
__device__ __forceinline__ void walk_item(const AttnArgs &a, const AttnPhase &p, int unit, int kvh, int split, int qtile, int lane, F &&finish) {
    constexpr int KS = D / 32;     // k-steps of the QK^T contraction
    constexpr int DT = D / 16;     // 16-wide tiles of the head dimension

    const int c = lane & 15, g = lane >> 4;
    const int u_row0 = p.unit_row0 ? table_entry(p.unit_row0, unit) : unit * p.q_per_unit;   // first query token of the unit
    const int u_count = p.unit_count ? table_entry(p.unit_count, unit) : p.q_per_unit;       // its query tokens
    const int32_t *pt = a.page_table + (size_t)(p.unit_row0 ? u_row0 : unit * p.pt_row_stride) * a.pt_stride;
    const size_t block_elems = (size_t)32 * D;
    const int t_lo = p.t_begin + split * p.split_tokens;
    PageWindow pages(pt, a.page_shift, t_lo, min(p.t_end, t_lo + p.split_tokens));
    auto block_base = [&](int t0) __attribute__((always_inline)) -> size_t {
        const int page = pages.page(t0);
        const int blk = (t0 & (a.page_tokens - 1)) >> 5;
        return ((((size_t)page * a.n_kv + kvh) << (a.page_shift - 5)) + blk) * block_elems;
    };
    bf16x8 qf[RT][KS];
    int limit[RT];
    load_queries<D, RT>(a, p, qf, limit, qtile, u_row0, u_count, kvh, c, g);

    // token range of this split, clipped to what any row of the item can see
    int max_limit = -1;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) max_limit = max(max_limit, limit[rt]);
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) max_limit = max(max_limit, __shfl_xor(max_limit, off, 64));
    // the same in every lane after the reduction; kept in scalar registers so that the block loop, the
    // page-table lookups and the block addresses stay on the scalar unit
    const int t_hi = __builtin_amdgcn_readfirstlane(min(min(p.t_end, t_lo + p.split_tokens), max_limit + 1));

    f32x4 o[DT][RT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) o[dt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun[RT], lrun[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) { mrun[rt] = kNegBig; lrun[rt] = 0.f; }
    const float scale_log2 = a.scale * 1.4426950408889634f;

    bf16x8 kf[2][KS], vf[DT];
    auto load_k = [&](auto stream, const uint16_t *kb) {
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                kf[tt][ks] = load_frag<decltype(stream)::value>(kb + ((ks * 32 + tt * 16 + c) * 32 + 8 * g));
    };
    auto load_v = [&](auto stream, const uint16_t *vb) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            vf[dt] = load_frag<decltype(stream)::value>(vb + ((dt * 16 + c) * 32 + 8 * g));
    };
    // S^T = K Q^T for all row tiles
    auto scores = [&](f32x4 (&s)[RT][2]) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                s[rt][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    s[rt][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tt][ks], qf[rt][ks], s[rt][tt], 0, 0, 0);
            }
    };
    // O^T = alpha O^T + V^T P^T
    auto accumulate = [&](const bf16x8 (&pf)[RT], const float (&alpha)[RT]) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                o[dt][rt] *= alpha[rt];
                o[dt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pf[rt], o[dt][rt], 0, 0, 0);
            }
    };

    // Software pipeline without spare registers: the K fragments of the next block are requested
    // into the registers of the current ones as soon as the score MFMAs have consumed them, and
    // the V fragments likewise after the P.V MFMAs, so 8 KiB per wavefront (d = 128) are in
    // flight behind the softmax and behind the next block's scores.  With one row tile (decode) the register
    // budget stays low enough for three wavefronts per SIMD, so every item of a decode step is resident at once.
    auto block_loop = [&](auto stream) {
        if (t_lo < t_hi) {
            const size_t base = block_base(t_lo);
            load_k(stream, a.kpool + base);
            load_v(stream, a.vpool + base);
        }
        for (int t0 = t_lo; t0 < t_hi; t0 += 32) {          // t_lo is a multiple of 32
            const int tn = t0 + 32 < t_hi ? t0 + 32 : t0;   // after the last block: harmless re-read
            const size_t base_n = block_base(tn);
            f32x4 s[RT][2];
            scores(s);
            // the scheduling fences keep each refill where it is written: right behind the last use
            // of the registers it overwrites, a whole softmax (or score pass) ahead of its first use
            __builtin_amdgcn_sched_barrier(0);
            load_k(stream, a.kpool + base_n);
            __builtin_amdgcn_sched_barrier(0);
            bf16x8 pf[RT];
            float alpha[RT];
            // with the visibility tests in every block: a second copy of the softmax without them, as in shared_tiles, splits
            // the loop body and costs the chain of a block more than the tests (36 against 43 us with all loads hits)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                softmax_block<true>(s[rt], t0 + 4 * g, min(limit[rt], t_hi - 1), scale_log2, mrun[rt], lrun[rt], pf[rt], alpha[rt]);
            accumulate(pf, alpha);
            __builtin_amdgcn_sched_barrier(0);
            load_v(stream, a.vpool + base_n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (p.stream_loads) block_loop(std::true_type{});       // uniform: one of two copies of the loop runs
    else block_loop(std::false_type{});
    finish(o, mrun, lrun, limit, (size_t)u_row0 + qtile * p.q_per_item);
}

template <int D, int RT>
__device__ __forceinline__ void single_item(const AttnArgs &a, const AttnPhase &p, int item, int lane) {
    // item -> (unit, kv head, split, q tile): the q tiles of one split are neighbours
    const int set = quotient(item, p.by_items), qtile = item - set * p.items_per_unit;
    const int rest = quotient(set, p.by_splits), split = set - rest * p.n_splits;
    const int unit = quotient(rest, a.by_kv), kvh = rest - unit * a.n_kv;
    walk_item<D, RT>(a, p, unit, kvh, split, qtile, lane, [&](const auto &o, const auto &mrun, const auto &lrun, const auto &limit, size_t first_tok) {
        store_item<D, RT>(a, p, o, mrun, lrun, limit, item, first_tok, kvh, lane & 15, lane >> 4);
    });
}

// One launch may cover two phases (decode: the shared-prompt phase followed by the private phase), so
// that the short, narrow shared phase overlaps the private one instead of running alone.
template <int D, int RT>
__global__ __launch_bounds__(256, RT == 1 ? 3 : 2) void attn_kernel(AttnArgs a, AttnPhase p0, AttnPhase p1, int n0, int n_items) {
    // the wavefront index is uniform: tell the compiler, so that everything derived from the work item
    // (phase, token range, page-table reads) lives in scalar registers
    const int gitem = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (gitem >= n_items) return;
    const bool second = gitem >= n0;
    single_item<D, RT>(a, second ? p1 : p0, second ? gitem - n0 : gitem, threadIdx.x & 63);
}

// ---------------------------------------------------------------------------------------------
// Four query tiles of one (unit, kv head, split) per workgroup: they need the same K/V blocks (prefill: consecutive query
// tiles of a chunk; decode: the members of a group over their shared prompt), so a block goes from global memory to LDS
// once per workgroup and every wavefront takes its MFMA operands from there.  The copies are direct-to-LDS loads, a
// quarter of a block per wavefront, two blocks ahead through three buffers (96 to 144 KiB of a compute unit's LDS in
// flight or in use at two or three workgroups), with one barrier per block; they are issued from inline assembly, so
// that the compiler does not wait for them before LDS reads, and the wait is placed by hand: a wavefront's
// vector-memory operations retire in order, so "all but the newest block's copies" is a count.  Page numbers come from a
// register (PageWindow): as a vector load behind the copies, whose wait drained them, they kept one block in flight
// instead of two; scalar loads kept two, but their wait covers the LDS reads.  Prompts of 4096 (32 groups of 16) 120.8 -> 112.6 us
// with the private contexts and the merge, of 1024 (16 groups of 8) 43.5 -> 42.2; no change in prefill.
//
// In LDS a 1 KiB tile of 16 rows lies as the MFMA's lanes take it, lane (c, g)'s 16 bytes at 16 (c + 16 g): the copy's source address
// is what is permuted.  As the tile lies in the page, reads counted conflict cycles worth a quarter of the kernel's.  Four
// fragments are on their way before the first MFMA of a product; the compiler had kept two and waited for both.  Prefill of 128 x 64
// tokens 278 -> 270 us a launch (order of the page: 275), of 128 x 32 91 -> 87.  The vector unit is 82 % busy there: softmax
// and the issue of MFMAs.
// ---------------------------------------------------------------------------------------------
constexpr int kShBufs = 3;

template <int D, int RT>
__device__ __forceinline__ void shared_tiles(const AttnArgs &a, const AttnPhase &p, int wg, u32x4 *lds) {
    constexpr int KS = D / 32, DT = D / 16;
    constexpr int SLOTS = 32 * D / 8;              // 16-byte slots of one K (or V) block
    constexpr int SEGS = SLOTS / 256;              // 1 KiB copies per wavefront of one K (or V) block
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // workgroup -> (set = unit, kv head, split; four of its query tiles)
    int set, qg;
    shared_tiles_of(wg, p.n_units * a.n_kv * p.n_splits, (p.items_per_unit + 3) >> 2, p.by_set, &set, &qg);
    const int rest = quotient(set, p.by_splits), split = set - rest * p.n_splits;
    const int unit = quotient(rest, a.by_kv), kvh = rest - unit * a.n_kv;
    const int qtile = qg * 4 + wave;               // beyond items_per_unit: this wavefront only helps with the copies

    const int c = lane & 15, g = lane >> 4;
    const int u_row0 = p.unit_row0 ? table_entry(p.unit_row0, unit) : unit * p.q_per_unit;
    const int u_count = p.unit_count ? table_entry(p.unit_count, unit) : p.q_per_unit;
    const int32_t *pt = a.page_table + (size_t)(p.unit_row0 ? u_row0 : unit * p.pt_row_stride) * a.pt_stride;
    const int page_shift = a.page_shift;           // 32, 64 or 128 tokens
    const int t_lo = p.t_begin + split * p.split_tokens, t_end = min(p.t_end, t_lo + p.split_tokens);
    PageWindow pages(pt, page_shift, t_lo, t_end);

    bf16x8 qf[RT][KS];
    int limit[RT];
    load_queries<D, RT>(a, p, qf, limit, qtile, u_row0, u_count, kvh, c, g);
    int max_limit = -1, min_limit = 0x7FFFFFFF;      // over the used rows of this wavefront
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        max_limit = max(max_limit, limit[rt]);
        min_limit = min(min_limit, limit[rt] < 0 ? 0x7FFFFFFF : limit[rt]);
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        max_limit = max(max_limit, __shfl_xor(max_limit, off, 64));
        min_limit = min(min_limit, __shfl_xor(min_limit, off, 64));
    }
    // this wavefront's range, and the workgroup's: its last query token sees the most
    const int t_hi = __builtin_amdgcn_readfirstlane(min(t_end, max_limit + 1));
    // tokens below t_vis are visible to every used row (unused rows hold zero queries and are never written out)
    const int t_vis = __builtin_amdgcn_readfirstlane(min(t_hi, min_limit == 0x7FFFFFFF ? 0 : min_limit + 1));
    const int last_q = min((qg * 4 + 4) * p.q_per_item, u_count) - 1;
    const int t_hi_wg = min(t_end, p.causal_pos0 + last_q * p.causal_stride + 1);
    const int n_blocks = __builtin_amdgcn_readfirstlane((t_hi_wg - t_lo + 31) >> 5);       // t_lo is a multiple of 32

    f32x4 o[DT][RT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) o[dt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun[RT], lrun[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) { mrun[rt] = kNegBig; lrun[rt] = 0.f; }
    const float scale_log2 = a.scale * 1.4426950408889634f;

    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void *)lds;
    auto copy = [&](int blk, int buf) __attribute__((always_inline)) {      // past the end: a harmless re-read of the last block
        const int t0 = t_lo + 32 * min(blk, n_blocks - 1), page = pages.page(t0);
        const int in_page = (t0 & (a.page_tokens - 1)) >> 5;
        const size_t base = ((((size_t)page * a.n_kv + kvh) << (page_shift - 5)) + in_page) * SLOTS + wave * (SEGS * 64) + c * 4 + g;
        const unsigned dst = lds0 + (unsigned)(buf * 2 * SLOTS + wave * (SEGS * 64)) * 16;
#pragma unroll
        for (int i = 0; i < SEGS; ++i) lds_dma16((const u32x4 *)a.kpool + base + i * 64, dst + i * 1024);
#pragma unroll
        for (int i = 0; i < SEGS; ++i) lds_dma16((const u32x4 *)a.vpool + base + i * 64, dst + (SLOTS + i * 64) * 16);
    };

    // N fragments from LDS, each for RT MFMAs: four are requested before the first MFMA, the others as their registers become free
    auto reads_ahead = [](auto n) __attribute__((always_inline)) {
        constexpr int N = decltype(n)::value, AHEAD = 4;
        __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);         // LDS reads
#pragma unroll
        for (int i = 0; i < N; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, RT, 0);        // MFMAs
            if (i + AHEAD < N) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };

    if (n_blocks > 0) {
        copy(0, 0);
        copy(1, 1);
        int buf = 0;
        for (int blk = 0; blk < n_blocks; ++blk) {
            // this wavefront's part of block blk has landed, and its LDS reads of block blk - 1, whose buffer the copies below
            // overwrite, are back (lgkmcnt; by now they always are: MFMAs took them)
            __builtin_amdgcn_s_waitcnt(0x0070 | (2 * SEGS));
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();                         // ... and everybody's; nobody reads block blk - 1 any more
            asm volatile("" ::: "memory");
            copy(blk + 2, buf == 0 ? 2 : buf - 1);
            const int t0 = t_lo + 32 * blk;
            const u32x4 *kb = lds + buf * 2 * SLOTS, *vb = kb + SLOTS;
            buf = buf == kShBufs - 1 ? 0 : buf + 1;
            if (t0 >= t_hi) continue;               // uniform per wavefront: invisible to all its rows
            f32x4 s[RT][2];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) s[rt][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
            // k-steps outermost: 2 x RT independent accumulators take turns, so an MFMA never waits for the one before it
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    const bf16x8 kf = __builtin_bit_cast(bf16x8, kb[(ks * 2 + tt) * 64 + lane]);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        s[rt][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[rt][ks], s[rt][tt], 0, 0, 0);
                }
            reads_ahead(std::integral_constant<int, 2 * KS>{});
            __builtin_amdgcn_sched_barrier(0);
            bf16x8 pf[RT];
            float alpha[RT];
            if (t0 + 32 <= t_vis) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    softmax_block<false>(s[rt], 0, 0, scale_log2, mrun[rt], lrun[rt], pf[rt], alpha[rt]);
            } else {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    softmax_block<true>(s[rt], t0 + 4 * g, min(limit[rt], t_hi - 1), scale_log2, mrun[rt], lrun[rt], pf[rt], alpha[rt]);
            }
            // the accumulators are rescaled only when some row's maximum moved (after the first blocks it rarely does)
            bool moved = false;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) moved |= alpha[rt] != 1.0f;
            if (__any(moved)) {
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) o[dt][rt] *= alpha[rt];
            }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const bf16x8 vf = __builtin_bit_cast(bf16x8, vb[dt * 64 + lane]);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    o[dt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[rt], o[dt][rt], 0, 0, 0);
            }
            reads_ahead(std::integral_constant<int, DT>{});
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);        // the copies past the end have landed before LDS goes away
    }
    const int item = ((unit * a.n_kv + kvh) * p.n_splits + split) * p.items_per_unit + qtile;
    store_item<D, RT>(a, p, o, mrun, lrun, limit, item, (size_t)u_row0 + qtile * p.q_per_item, kvh, c, g);
}

// Prefill: one phase
template <int D, int RT>
__global__ __launch_bounds__(256, 2) void attn_prefill_shared_kernel(AttnArgs a, AttnPhase p) {
    __shared__ u32x4 lds[kShBufs * 2 * 32 * D / 8];
    shared_tiles<D, RT>(a, p, blockIdx.x, lds);
}

// Decode: the groups' query tiles over their shared prompt first, a workgroup for four of them, then the sequences'
// private contexts, a wavefront each.
template <int D>
__global__ __launch_bounds__(256, 3) void attn_decode_kernel(AttnArgs a, AttnPhase p0, AttnPhase p1, int wgs0, int n1) {
    __shared__ u32x4 lds[kShBufs * 2 * 32 * D / 8];
    if ((int)blockIdx.x < wgs0) {
        shared_tiles<D, 1>(a, p0, blockIdx.x, lds);
    } else {
        const int item = ((int)blockIdx.x - wgs0) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (item < n1) single_item<D, 1>(a, p1, item, threadIdx.x & 63);
    }
}

// Decode over a short context: a workgroup per (sequence, kv head), whose wavefronts share the whole context out, prompt included, and
// merge through LDS with the arithmetic of attn_merge_kernel.  The members of a group then read the prompt once each instead of once
// together, but nothing goes through memory and the merge launch is gone (whole_context says where that pays).  Bound: a chain of
// a quarter of the context's blocks.
template <int D>
__global__ __launch_bounds__(64 * kWholeWaves) void attn_whole_kernel(AttnArgs a, AttnPhase p) {
    constexpr int DT = D / 16, WAVES = kWholeWaves;
    __shared__ f32x4 s_o[WAVES][DT][64];             // [dims dt * 16 + 4 g of row c]
    __shared__ float s_m[WAVES][16], s_l[WAVES][16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int unit = quotient(blockIdx.x, a.by_kv), kvh = (int)blockIdx.x - unit * a.n_kv;
    const int c = lane & 15, g = lane >> 4;
    size_t tok = 0;
    walk_item<D, 1>(a, p, unit, kvh, wave, 0, lane, [&](const auto &o, const auto &mrun, const auto &lrun, const auto &, size_t first_tok) {
        tok = first_tok;
        const float l = row_sum(lrun[0]);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) s_o[wave][dt][lane] = o[dt][0];
        if (g == 0) { s_m[wave][c] = mrun[0]; s_l[wave][c] = l; }
    });
    __syncthreads();
    if (c >= a.n_rep) return;
    float m[WAVES], l[WAVES], best = kNegBig, den = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        m[w] = s_m[w][c];
        l[w] = s_l[w][c];
        best = fmaxf(best, l[w] > 0.f ? m[w] : kNegBig);
    }
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        m[w] = l[w] > 0.f ? exp2f(m[w] - best) : 0.f;
        den += l[w] * m[w];
    }
    const int col = (kvh * a.n_rep + c) * D + 4 * g;
#pragma unroll
    for (int dt = wave; dt < DT; dt += WAVES) {
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) num += s_o[w][dt][lane] * m[w];
        float r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = den > 0.f ? num[e] / den : 0.f;
        *(uint2 *)(a.direct_out + frag_offset((int)tok, col + dt * 16, a.out_mt_total)) = make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
    }
}

// One phase of the merge: partial result i of (query token, query head) lies in row base + i * step of the phase's items
struct MergePhase {
    const int32_t *unit_row0, *row_unit;
    FastDiv by_unit, by_item;        // divisions by query tokens per unit and per item
    int q_per_unit, q_per_item, n_splits, step;      // step: rows of the items of one split
    unsigned row0;                   // first row of the phase in the buffer that the phases share
    const float *part_ml;
};
struct MergeArgs {
    MergePhase ph[2];
    int n_phases;
    FastDiv by_rep;
    int n_rep, n_q, n_kv, tile_rows, mt_total;       // tile_rows: 16 * rt
    const float *part_o;
    uint16_t *out;
    float *out32;       // non-null: row-major fp32 output instead of `out`
};

// One wavefront per (query token, query head), D / 64 head dimensions per lane.  Lane i works out where partial result i
// lies and fetches its (max, sum) pair; the partial outputs, whose rows the other lanes read from it, are requested four
// at a time in the same round trip.  The weighted sum runs over the items in a fixed order.  No LDS and no barrier: a
// workgroup of its own for every (token, head) with three barriers took 17.4 us at 296 rows and 4 items.  Bound: the latency of
// a chain of a few steps; with both phases' arguments read in a loop and divisions by them it was 11.9 us at
// 296 rows and 4 items and 5.1 at 8, 9.3 and 4.5 now.
constexpr int kMaxMergeItems = 64;

template <int D>
__global__ __launch_bounds__(256) void attn_merge_kernel(MergeArgs a) {
    constexpr int E = D / 64;
    typedef float vec __attribute__((ext_vector_type(E)));
    const int lane = threadIdx.x & 63;
    const int qt = blockIdx.x, h = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (h >= a.n_q) return;
    const int kvh = quotient(h, a.by_rep), hr = h - kvh * a.n_rep;

    // row of the first partial result in a phase
    auto base = [&](const MergePhase &p) __attribute__((always_inline)) {
        int unit, qi;
        if (p.row_unit) {
            unit = table_entry(p.row_unit, qt);
            qi = qt - table_entry(p.unit_row0, unit);
        } else {
            unit = quotient(qt, p.by_unit);
            qi = qt - unit * p.q_per_unit;
        }
        const int qtile = quotient(qi, p.by_item);
        return ((unit * a.n_kv + kvh) * p.n_splits) * p.step + qtile * a.tile_rows + (qi - qtile * p.q_per_item) * a.n_rep + hr;
    };
    const int n0 = a.ph[0].n_splits, n_items = n0 + (a.n_phases > 1 ? a.ph[1].n_splits : 0);
    const int base0 = base(a.ph[0]), base1 = a.n_phases > 1 ? base(a.ph[1]) : 0;
    unsigned row = 0;                                // lane i: row of partial result i
    float m = kNegBig, l = 0.f;
    if (lane < n_items) {
        const bool first = lane < n0;
        const int prow = first ? base0 + lane * a.ph[0].step : base1 + (lane - n0) * a.ph[1].step;
        row = (first ? a.ph[0].row0 : a.ph[1].row0) + (unsigned)prow;
        const float2 ml = *(const float2 *)((first ? a.ph[0].part_ml : a.ph[1].part_ml) + (size_t)prow * 2);
        m = ml.x;
        l = ml.y;
    }
    const float *po = a.part_o + lane * E;
    vec v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u < n_items) v[u] = *(const vec *)(po + (size_t)__builtin_amdgcn_readlane(row, u) * D);
    float mbest = l > 0.f ? m : kNegBig;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mbest = fmaxf(mbest, __shfl_xor(mbest, off, 64));
    const float w = l > 0.f ? exp2f(m - mbest) : 0.f;
    const float lw = l * w;
    auto of_lane = [](float x, int i) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), i)); };
    float den = 0.f;
    for (int i = 0; i < n_items; ++i) den += of_lane(lw, i);
    vec num = {};
    for (int i = 0; i < n_items; i += 4) {
        vec nx[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + 4 + u < n_items) nx[u] = *(const vec *)(po + (size_t)__builtin_amdgcn_readlane(row, i + 4 + u) * D);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u < n_items) {
                const float wu = of_lane(w, i + u);
#pragma unroll
                for (int e = 0; e < E; ++e) num[e] += v[u][e] * wu;
            }
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = nx[u];
    }
    float r[E];
#pragma unroll
    for (int e = 0; e < E; ++e) r[e] = den > 0.f ? num[e] / den : 0.f;
    const int col = h * D + lane * E;
    if (a.out32) {
#pragma unroll
        for (int e = 0; e < E; ++e) a.out32[(size_t)qt * a.n_q * D + col + e] = r[e];
    } else if constexpr (E == 2) {
        *(uint32_t *)(a.out + frag_offset(qt, col, a.mt_total)) = pack_bf16x2(r[0], r[1]);
    } else {
        a.out[frag_offset(qt, col, a.mt_total)] = f32_to_bf16(r[0]);
    }
}

}  // namespace

int launch_attention_whole(const AttnArgs &args, int n_seq, int ctx, hipStream_t stream) {
    AttnArgs a = args;
    if (n_seq <= 0) return SR_OK;
    a.n_rep = a.n_q / a.n_kv;
    const long long wgs = (long long)n_seq * a.n_kv;
    if (a.n_rep > 16 || ctx < 1 || !a.direct_out || wgs > 0x7FFFFFFF) return SR_E_ARG;
    a.by_kv = fast_div(a.n_kv);
    a.inv_rep = 1.0f / (float)a.n_rep;
    a.page_shift = 31 - __builtin_clz(a.page_tokens);
    const AttnPhase p = whole_phase(n_seq, ctx);
    const dim3 grid((unsigned)wgs), block(64 * kWholeWaves);
    if (a.d == 128) attn_whole_kernel<128><<<grid, block, 0, stream>>>(a, p);
    else if (a.d == 64) attn_whole_kernel<64><<<grid, block, 0, stream>>>(a, p);
    else return SR_E_ARG;
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_attention(const AttnArgs &args, const AttnPhase *phase_args, int n_phases, hipStream_t stream) {
    if (n_phases < 1 || n_phases > 2) return SR_E_ARG;
    long long n[2] = {0, 0};
    AttnArgs a = args;
    AttnPhase phases[2] = {phase_args[0], phase_args[n_phases - 1]};
    const int n_rep = a.n_q / a.n_kv;
    a.by_kv = fast_div(a.n_kv);
    a.n_rep = n_rep;
    a.inv_rep = 1.0f / (float)n_rep;
    a.page_shift = 31 - __builtin_clz(a.page_tokens);
    for (int i = 0; i < n_phases; ++i) {
        AttnPhase &p = phases[i];
        p.by_items = fast_div(p.items_per_unit);
        p.by_splits = fast_div(p.n_splits);
        p.by_set = fast_div((p.items_per_unit + 3) / 4);
        n[i] = (long long)p.n_units * a.n_kv * p.items_per_unit * p.n_splits;
        if (p.t_end <= p.t_begin) n[i] = 0;
        if ((p.t_begin & 31) || (p.split_tokens & 31) || p.split_tokens <= 0 || p.q_per_item * n_rep > 16 * p.rt ||
            p.rt != phases[0].rt)
            return SR_E_ARG;
        // no split without a token of its own
        if (n[i] && p.t_begin + (long long)(p.n_splits - 1) * p.split_tokens >= p.t_end) return SR_E_ARG;
    }
    if (a.direct_out && (n_phases != 1 || phases[0].n_splits != 1)) return SR_E_ARG;
    const long long n_items = n[0] + n[1];
    if (n_items <= 0) return SR_OK;
    if (n_items > 0x7FFFFFFF) return SR_E_ARG;
    const AttnPhase &p0 = phases[0], &p1 = phases[n_phases - 1];
    const int rt = p0.rt, n0 = (int)n[0], nt = (int)n_items;
    // workgroups of a phase whose query tiles share their blocks through LDS: four tiles of a set each
    auto shared_wgs = [&](const AttnPhase &p) -> long long {
        return (long long)p.n_units * a.n_kv * p.n_splits * ((p.items_per_unit + 3) / 4);
    };
    if (n_phases == 1 && p0.share) {
        const long long wgs = shared_wgs(p0);
        if (wgs > 0x7FFFFFFF) return SR_E_ARG;
        dim3 sgrid((unsigned)wgs);
        if (a.d == 128 && rt == 1) attn_prefill_shared_kernel<128, 1><<<sgrid, dim3(256), 0, stream>>>(a, p0);
        else if (a.d == 128 && rt == 2) attn_prefill_shared_kernel<128, 2><<<sgrid, dim3(256), 0, stream>>>(a, p0);
        else if (a.d == 64 && rt == 1) attn_prefill_shared_kernel<64, 1><<<sgrid, dim3(256), 0, stream>>>(a, p0);
        else if (a.d == 64 && rt == 2) attn_prefill_shared_kernel<64, 2><<<sgrid, dim3(256), 0, stream>>>(a, p0);
        else return SR_E_ARG;
        SR_HIP(hipGetLastError());
        return SR_OK;
    }
    if (n_phases == 2 && p0.share && rt == 1 && n0 > 0) {
        const long long wgs0 = shared_wgs(p0), wgs = wgs0 + (n[1] + 3) / 4;
        if (wgs > 0x7FFFFFFF) return SR_E_ARG;
        dim3 sgrid((unsigned)wgs);
        if (a.d == 128) attn_decode_kernel<128><<<sgrid, dim3(256), 0, stream>>>(a, p0, p1, (int)wgs0, (int)n[1]);
        else if (a.d == 64) attn_decode_kernel<64><<<sgrid, dim3(256), 0, stream>>>(a, p0, p1, (int)wgs0, (int)n[1]);
        else return SR_E_ARG;
        SR_HIP(hipGetLastError());
        return SR_OK;
    }
    dim3 grid((unsigned)((n_items + 3) / 4)), block(256);
    if (a.d == 128 && rt == 1) attn_kernel<128, 1><<<grid, block, 0, stream>>>(a, p0, p1, n0, nt);
    else if (a.d == 128 && rt == 2) attn_kernel<128, 2><<<grid, block, 0, stream>>>(a, p0, p1, n0, nt);
    else if (a.d == 64 && rt == 1) attn_kernel<64, 1><<<grid, block, 0, stream>>>(a, p0, p1, n0, nt);
    else if (a.d == 64 && rt == 2) attn_kernel<64, 2><<<grid, block, 0, stream>>>(a, p0, p1, n0, nt);
    else return SR_E_ARG;
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_attn_merge(const AttnArgs &a, const AttnPhase *phases, int n_phases, int n_qtok, uint4 *out,
                      int mt_total, float *out32, hipStream_t stream) {
    if (n_qtok <= 0) return SR_OK;
    if (n_phases < 1 || n_phases > 2) return SR_E_ARG;
    int total = 0;
    for (int i = 0; i < n_phases; ++i) total += phases[i].n_splits;
    if (total > kMaxMergeItems) return SR_E_ARG;
    MergeArgs m{};
    m.n_phases = n_phases;
    m.n_q = a.n_q; m.n_kv = a.n_kv; m.mt_total = mt_total;
    m.n_rep = a.n_q / a.n_kv;
    m.by_rep = fast_div(m.n_rep);
    m.tile_rows = 16 * phases[0].rt;
    m.part_o = phases[0].part_o;
    for (int i = 0; i < n_phases; ++i) {
        const AttnPhase &p = phases[i];
        MergePhase &q = m.ph[i];
        q.unit_row0 = p.unit_row0;
        q.row_unit = p.row_unit;
        q.by_unit = fast_div(p.q_per_unit);
        q.by_item = fast_div(p.q_per_item);
        q.q_per_unit = p.q_per_unit;
        q.q_per_item = p.q_per_item;
        q.n_splits = p.n_splits;
        q.step = p.items_per_unit * 16 * p.rt;
        q.row0 = (unsigned)((p.part_o - phases[0].part_o) / a.d);        // phases share one buffer
        q.part_ml = p.part_ml;
        if (p.rt != phases[0].rt) return SR_E_ARG;
    }
    m.out = (uint16_t *)out;
    m.out32 = out32;
    const dim3 grid(n_qtok, ceil_div(a.n_q, 4)), block(256);
    if (a.d == 128) attn_merge_kernel<128><<<grid, block, 0, stream>>>(m);
    else if (a.d == 64) attn_merge_kernel<64><<<grid, block, 0, stream>>>(m);
    else return SR_E_ARG;
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace sr
