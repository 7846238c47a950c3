// What happens to a projection's sums before they go back to memory, for the kernels that hold them in registers.
#pragma once
#include "sr_internal.h"

namespace sr {

// RowScale: the sums of squares of a row, dealt out over THREADS threads, each of which adds those of one row; then the row's factor.
// request() where the round trip is hidden, leave() ahead of a barrier, scale() behind it.  The order of the sum is the same for all rows of a
// launch, but follows the power of two that holds M and THREADS: a sequence's factor may change in its last bits with the
// batch, and between QKV, gate|up and LM head, as the sums of a projection do with its K splits.
template <int THREADS>
struct RowSquares {
    static constexpr int N = 4;      // values of 16 bytes that a thread requests at once; the first ones of more are added on the way
    f32x4 v[N], sum;
    int rows, groups;                // rows: 8 or the power of two from 16 on that holds M
    __device__ __forceinline__ void request(const RowScale &s, int M, int tid) {
        if (!s.squares) return;
        rows = M <= 8 ? 8 : M <= 16 ? 16 : M <= 32 ? 32 : M <= 64 ? 64 : 128;
        groups = THREADS / rows;
        const f32x4 *p = (const f32x4 *)(s.squares + (size_t)(tid & (rows - 1)) * s.ld);
        const int n = s.ld >> 2;
        int i = tid / rows;
        sum = f32x4{0.f, 0.f, 0.f, 0.f};
        for (; i + N * groups < n; i += groups) sum += p[i];
#pragma unroll
        for (int u = 0; u < N; ++u, i += groups) v[u] = i < n ? p[i] : f32x4{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void leave(const RowScale &s, float *lds, int tid) {
        if (!s.squares) return;
#pragma unroll
        for (int u = 0; u < N; ++u) sum += v[u];
        lds[tid] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    }
    __device__ __forceinline__ float scale(const RowScale &s, const float *lds, int row) const {
        float t = 0.f;
        for (int g = 0; g < groups; ++g) t += lds[g * rows + (row & (rows - 1))];
        return 1.0f / sqrtf(t * s.inv_h + s.eps);
    }
};

// What finish_qkv needs besides the sums; requested early where a round trip can be hidden.
struct QkvExtras { uint2 bias_lo, bias_hi; f32x4 cos, sin; int page, pos; };

// Queries, keys and values of row m and `head` (queries first, then keys, then values): four consecutive dims i .. i+3 of the low
// half of the head and their rotation partners i + d/2 ..
__device__ __forceinline__ void fetch_bias_and_rotation(const QkvPostArgs &a, int head, int i, QkvExtras &x) {
    const int kind = head < a.n_q ? 0 : head < a.n_q + a.n_kv ? 1 : 2;
    const int h = kind == 0 ? head : kind == 1 ? head - a.n_q : head - a.n_q - a.n_kv, half = a.d >> 1;
    const uint16_t *bias = kind == 0 ? a.bq : kind == 1 ? a.bk : a.bv;
    x.bias_lo = x.bias_hi = make_uint2(0, 0);
    x.cos = f32x4{1.f, 1.f, 1.f, 1.f};
    x.sin = f32x4{0.f, 0.f, 0.f, 0.f};
    if (bias) {
        x.bias_lo = *(const uint2 *)(bias + h * a.d + i);
        x.bias_hi = *(const uint2 *)(bias + h * a.d + i + half);
    }
    if (kind != 2) {
        x.cos = *(const f32x4 *)(a.rope_cos + (size_t)x.pos * half + i);
        x.sin = *(const f32x4 *)(a.rope_sin + (size_t)x.pos * half + i);
    }
}

// Add the bias, rotate, and write the query row or the K/V page.
__device__ __forceinline__ void finish_qkv(const QkvPostArgs &a, int m, int head, int i, f32x4 lo, f32x4 hi, const QkvExtras &x) {
    const int kind = head < a.n_q ? 0 : head < a.n_q + a.n_kv ? 1 : 2;       // 0 q, 1 k, 2 v
    const int h = kind == 0 ? head : kind == 1 ? head - a.n_q : head - a.n_q - a.n_kv, half = a.d >> 1;
    const uint16_t *bias = kind == 0 ? a.bq : kind == 1 ? a.bk : a.bv;
    if (bias) {
        lo += f32x4{__uint_as_float(x.bias_lo.x << 16), __uint_as_float(x.bias_lo.x & 0xFFFF0000u), __uint_as_float(x.bias_lo.y << 16),
                    __uint_as_float(x.bias_lo.y & 0xFFFF0000u)};
        hi += f32x4{__uint_as_float(x.bias_hi.x << 16), __uint_as_float(x.bias_hi.x & 0xFFFF0000u), __uint_as_float(x.bias_hi.y << 16),
                    __uint_as_float(x.bias_hi.y & 0xFFFF0000u)};
    }
    if (kind != 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float rlo = lo[e] * x.cos[e] - hi[e] * x.sin[e], rhi = hi[e] * x.cos[e] + lo[e] * x.sin[e];
            lo[e] = rlo; hi[e] = rhi;
        }
    }
    const uint2 plo = make_uint2(pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]));
    const uint2 phi = make_uint2(pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3]));
    if (kind == 0) {
        uint16_t *q = a.q_out + ((size_t)m * a.n_q + h) * a.d;
        *(uint2 *)(q + i) = plo;
        *(uint2 *)(q + i + half) = phi;
        return;
    }
    const int tok = x.pos & (a.page_tokens - 1), blk = tok >> 5, t = tok & 31;
    const size_t base = ((((size_t)x.page * a.n_kv + h) << (a.page_shift - 5)) + blk) * (size_t)(32 * a.d);
    if (kind == 1) {
        // K block [d/32][32 tok][32]: four consecutive dims stay inside one 32-dim group
        uint16_t *k = a.kpool + base;
        *(uint2 *)(k + (((i >> 5) * 32 + t) << 5) + (i & 31)) = plo;
        const int i2 = i + half;
        *(uint2 *)(k + (((i2 >> 5) * 32 + t) << 5) + (i2 & 31)) = phi;
    } else {
        uint16_t *v = a.vpool + base;
        const int slot = 8 * ((t & 15) >> 2) + 4 * (t >> 4) + (t & 3);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[(i + e) * 32 + slot] = f32_to_bf16(lo[e]);
            v[(i + half + e) * 32 + slot] = f32_to_bf16(hi[e]);
        }
    }
}

}  // namespace sr
