// Row-wise kernels between the GEMMs: residual update + RMSNorm, QKV epilogue (bias, RoPE,
// KV page write), greedy argmax, and small utilities.  All reductions of these kernels run in a fixed order that does not depend on
// the row index or on the batch size.  (K splits and attention splits do depend on the batch size, and so does the order in which a
// norm that is finished behind the next projection adds up its squares: see RowSquares.  Rows of one batch are treated alike everywhere.)
#include "epilogue.h"

namespace sr {
namespace {

// deterministic block-wide sums of ROWS values over 512 threads (the same order of additions for every row)
template <int ROWS>
__device__ __forceinline__ void block_sums_512(float (&v)[ROWS], float (*s_red)[8]) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v[r] += __shfl_xor(v[r], off, 64);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) s_red[r][wave] = v[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        v[r] = ((s_red[r][0] + s_red[r][1]) + (s_red[r][2] + s_red[r][3])) + ((s_red[r][4] + s_red[r][5]) + (s_red[r][6] + s_red[r][7]));
}

// lo += p[s * stride .. + 3], hi += p[s * stride + apart .. + 3] for s = 0 .. n-1, in that order, N of them requested before
// the first is added.  More than four at a time gains nothing (nine, for the norm behind a projection in nine splits: 6.5 us at
// 128 rows either way, 4.9 instead of 4.5 at 8) and costs registers.
template <int N>
__device__ __forceinline__ void add_partials_exactly(const float *p, size_t stride, int apart, f32x4 &lo, f32x4 &hi) {
    f32x4 pl[N], ph[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const float *q = p + (size_t)u * stride;
        pl[u] = *(const f32x4 *)q;
        ph[u] = *(const f32x4 *)(q + apart);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) { lo += pl[u]; hi += ph[u]; }
}
__device__ __forceinline__ void add_partials(const float *p, size_t stride, int n, int apart, f32x4 &lo, f32x4 &hi) {
    for (; n >= 4; n -= 4, p += 4 * stride) add_partials_exactly<4>(p, stride, apart, lo, hi);
    switch (n) {                                     // uniform
        case 1: return add_partials_exactly<1>(p, stride, apart, lo, hi);
        case 2: return add_partials_exactly<2>(p, stride, apart, lo, hi);
        case 3: return add_partials_exactly<3>(p, stride, apart, lo, hi);
    }
}

// x = resid (+ partials) or embedding row; resid <- x (if write_resid); out <- bf16(x * rsqrt(mean(x^2)+eps) * gain)
// H <= 8192: each thread keeps its (at most 2 x 8) values per row in registers between the two passes.
// A workgroup takes ROWS consecutive output rows and requests all of their data before the first reduction:
// one row at decode time (few rows, every compute unit should get one), four for prefill-sized batches, where
// a row's three dependent memory round trips would otherwise leave the memory system mostly idle.  The
// arithmetic of a row does not depend on ROWS.
template <bool F32OUT, int ROWS>
__global__ __launch_bounds__(512) void resid_norm_kernel(NormArgs a) {
    __shared__ float s_red[ROWS][8];
    const int nvec = a.H >> 3;                       // groups of 8 consecutive features
    float xv[ROWS][2][8];
    float ss[ROWS];
    // the gains do not depend on the reduction: fetch them first, so that the second pass starts from registers
    uint4 graw[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int v = threadIdx.x + it * 512;
        graw[it] = v < nvec ? *(const uint4 *)(a.gain + v * 8) : make_uint4(0, 0, 0, 0);
    }

#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int m = blockIdx.x * ROWS + r;
        ss[r] = 0.f;
        if (m >= a.rows_out) continue;               // uniform across the workgroup
        const size_t row = (size_t)quotient(m, a.by_dup) * a.src_stride + a.src_off;
        float *x = a.resid + row * a.H;
        const uint16_t *e = nullptr;
        if (a.embed) {
            const int unit = quotient(m, a.by_chunk);
            const int tok = a.tokens[(size_t)unit * a.tok_stride + a.tok_off + m - unit * a.tok_chunk];
            e = a.embed + (size_t)tok * a.H;
        }
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int v = threadIdx.x + it * 512;
            if (v < nvec) {
                float *f = xv[r][it];
                if (e) {
                    const uint4 raw = *(const uint4 *)(e + v * 8);
                    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        f[2 * i] = __uint_as_float(w[i] << 16);
                        f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
                    }
                } else {
                    f32x4 lo = *(const f32x4 *)(x + v * 8), hi = *(const f32x4 *)(x + v * 8 + 4);
                    const float *p0 = a.partials + row * a.H + v * 8;
                    if (F32OUT && a.sums_first) {
                        f32x4 slo = {0.f, 0.f, 0.f, 0.f}, shi = {0.f, 0.f, 0.f, 0.f};
                        add_partials(p0, a.partial_stride, a.n_partials, 4, slo, shi);
                        lo += slo;
                        hi += shi;
                    } else add_partials(p0, a.partial_stride, a.n_partials, 4, lo, hi);
#pragma unroll
                    for (int i = 0; i < 4; ++i) { f[i] = lo[i]; f[4 + i] = hi[i]; }
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) ss[r] += f[i] * f[i];
                if (a.write_resid) {
                    *(f32x4 *)(x + v * 8) = f32x4{f[0], f[1], f[2], f[3]};
                    *(f32x4 *)(x + v * 8 + 4) = f32x4{f[4], f[5], f[6], f[7]};
                }
            }
        }
    }
    block_sums_512<ROWS>(ss, s_red);

#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int m = blockIdx.x * ROWS + r;
        if (m >= a.rows_out) continue;
        const float inv = 1.0f / sqrtf(ss[r] / (float)a.H + a.eps);
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int v = threadIdx.x + it * 512;
            if (v < nvec) {
                const float *f = xv[r][it];
                const uint32_t gw[4] = {graw[it].x, graw[it].y, graw[it].z, graw[it].w};
                float y[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    y[2 * i] = f[2 * i] * inv * __uint_as_float(gw[i] << 16);
                    y[2 * i + 1] = f[2 * i + 1] * inv * __uint_as_float(gw[i] & 0xFFFF0000u);
                }
                if constexpr (F32OUT) {
                    float *dst = a.out32 + (size_t)m * a.H + v * 8;
                    *(f32x4 *)dst = f32x4{y[0], y[1], y[2], y[3]};
                    *(f32x4 *)(dst + 4) = f32x4{y[4], y[5], y[6], y[7]};
                } else {
                    uint4 o = make_uint4(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]),
                                         pack_bf16x2(y[6], y[7]));
                    *(uint4 *)((uint16_t *)a.out + frag_offset(m, v * 8, a.mt_total)) = o;
                }
            }
        }
    }
}

// One block per (row, group of heads): 64 threads at decode time, up to 640 (all heads of a row) for prefill-sized
// batches, where tens of thousands of one-wavefront blocks would cost more than they move.  A thread owns four
// consecutive dims i .. i+3 of the low half of a head and their rotation partners i + d/2 .. (16-byte loads of the
// fp32 partials); d/8 threads make a head.
// EARLY (decode): what does not depend on the partial sums (bias, rotation) is requested before them; a full chip hides that
// round trip, and needs the registers.
template <bool EARLY>
__global__ __launch_bounds__(640) void qkv_post_kernel(QkvPostArgs a) {
    const int half = a.d >> 1, tph = half >> 2;               // threads per head
    const int at = (int)(((float)threadIdx.x + 0.5f) * __builtin_amdgcn_rcpf((float)tph));       // 640 at most: far from an integer
    const int m = blockIdx.x, head = blockIdx.y * a.heads_per_block + at, i = ((int)threadIdx.x - at * tph) * 4;
    if (head >= a.n_q + 2 * a.n_kv) return;
    const int unit = quotient(m, a.by_chunk);
    QkvExtras x;
    x.pos = a.pos0 + m - unit * a.chunk;
    // the page table does not change while the kernel runs: a uniform entry comes through a scalar load
    x.page = ((const __attribute__((address_space(4))) int32_t *)(uintptr_t)a.page_table)[(size_t)unit * a.pt_row_stride *
                                                                                         a.pt_stride + (x.pos >> a.page_shift)];
    if (EARLY) fetch_bias_and_rotation(a, head, i, x);
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
    add_partials(a.partials + (size_t)m * a.ld + head * a.d + qkv_column(i), a.partial_stride, a.n_partials, 16, lo, hi);
    if (!EARLY) fetch_bias_and_rotation(a, head, i, x);
    finish_qkv(a, m, head, i, lo, hi, x);
}

struct MaxIdx {
    float v;
    int i;
};
__device__ __forceinline__ MaxIdx better(MaxIdx a, MaxIdx b) {
    return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}

__device__ __forceinline__ uint64_t smx_finalize(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

// One 1024-thread block per row: strided scan, wavefront shuffle reduction, then 16 wave results.
// With inv_temperature > 0 every logit is scaled and perturbed by a standard Gumbel variate drawn from a
// counter-based SplitMix64 stream keyed (seed, original sequence id, position), counter = vocabulary
// index: the argmax of the perturbed scores is a draw from softmax(logits / T).
__global__ __launch_bounds__(1024) void argmax_kernel(const float *__restrict__ logits, int vocab,
                                                      const int32_t *forced, int32_t *greedy_out,
                                                      int32_t *chosen, int32_t *actions, int max_turns,
                                                      int turn_idx, int action_mod, float inv_temperature,
                                                      uint64_t seed, const int32_t *__restrict__ orig_seq, int pos) {
    __shared__ MaxIdx s_best[16];
    const int r = blockIdx.x;
    const float *row = logits + (size_t)r * vocab;
    MaxIdx best{-INFINITY, 0x7FFFFFFF};
    const int nvec = vocab >> 2;
    if (inv_temperature > 0.f) {
        const uint64_t golden = 0x9E3779B97F4A7C15ULL;
        const uint64_t stream = ((uint64_t)(uint32_t)orig_seq[r] << 32) | (uint32_t)pos;
        const uint64_t key = smx_finalize(smx_finalize(seed + golden) ^ (stream * 0xD1342543DE82EF95ULL + 1ULL));
        for (int v = threadIdx.x; v < vocab; v += 1024) {
            const uint64_t rnd = smx_finalize(key + ((uint64_t)v + 1ULL) * golden);
            const float u = ((float)(uint32_t)(rnd >> 41) + 0.5f) * (1.0f / 8388608.0f);
            best = better(best, MaxIdx{row[v] * inv_temperature - logf(-logf(u)), v});
        }
    } else {
        for (int v0 = threadIdx.x; v0 < nvec; v0 += 4096) {      // four loads in flight; past the end the last one again
            f32x4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = *(const f32x4 *)(row + min(v0 + u * 1024, nvec - 1) * 4);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) best = better(best, MaxIdx{x[u][e], min(v0 + u * 1024, nvec - 1) * 4 + e});
        }
        for (int v = nvec * 4 + threadIdx.x; v < vocab; v += 1024) best = better(best, MaxIdx{row[v], v});
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        MaxIdx o{__shfl_xor(best.v, off, 64), __shfl_xor(best.i, off, 64)};
        best = better(best, o);
    }
    if ((threadIdx.x & 63) == 0) s_best[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) best = better(best, s_best[w]);
        const int greedy = best.i;
        const int tok = forced ? forced[r] : greedy;       // before the write: greedy_out may be the same buffer
        if (greedy_out) greedy_out[r] = greedy;
        chosen[r] = tok;
        if (actions) actions[(size_t)r * max_turns + turn_idx] = tok % action_mod;
    }
}

__global__ void fill_i32_kernel(int32_t *dst, size_t n, int32_t value) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = value;
}

template <typename T>
__global__ void gather_rows_kernel(T *dst, const T *src, const int32_t *src_rows, size_t row_vec) {
    const int r = blockIdx.y;
    const size_t s = (size_t)src_rows[r];
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < row_vec; i += (size_t)gridDim.x * blockDim.x)
        dst[(size_t)r * row_vec + i] = src[s * row_vec + i];
}

// One page of every layer, K and V, per (pair, layer); the pairs of a call go in one launch (a prompt that ends inside a
// page gives every member but one a copy: 112 launches of 4.8 us at 16 x 8 sequences before).
__global__ void copy_pages_kernel(uint4 *kpool, uint4 *vpool, size_t layer_vec, size_t page_vec, const int2 *__restrict__ pairs) {
    const int layer = blockIdx.y;
    const int2 pr = pairs[blockIdx.x];               // source, destination
    uint4 *k = kpool + layer * layer_vec, *v = vpool + layer * layer_vec;
    for (size_t i = (size_t)blockIdx.z * blockDim.x + threadIdx.x; i < page_vec; i += (size_t)gridDim.z * blockDim.x) {
        const uint4 kx = k[(size_t)pr.x * page_vec + i], vx = v[(size_t)pr.x * page_vec + i];
        k[(size_t)pr.y * page_vec + i] = kx;
        v[(size_t)pr.y * page_vec + i] = vx;
    }
}

}  // namespace

int launch_resid_norm(const NormArgs &args, hipStream_t stream) {
    NormArgs a = args;
    if (a.rows_out <= 0) return SR_OK;
    if (a.H % 8 || a.H > 8192 || a.src_dup < 1 || (a.embed && a.tok_chunk < 1)) return SR_E_ARG;
    a.by_dup = fast_div(a.src_dup);
    a.by_chunk = fast_div(a.embed ? a.tok_chunk : 1);
    if (a.out32) resid_norm_kernel<true, 1><<<dim3(a.rows_out), dim3(512), 0, stream>>>(a);
    else if (a.rows_out >= 2048) resid_norm_kernel<false, 4><<<dim3(ceil_div(a.rows_out, 4)), dim3(512), 0, stream>>>(a);
    else resid_norm_kernel<false, 1><<<dim3(a.rows_out), dim3(512), 0, stream>>>(a);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_qkv_post(const QkvPostArgs &args, hipStream_t stream) {
    QkvPostArgs a = args;
    if (a.rows <= 0) return SR_OK;
    if (a.d > 128 || a.d % 32 || a.rows > 0x7FFFFFF || a.chunk < 1) return SR_E_ARG;
    set_divisions(&a);
    const int heads_per_wave = 64 / (a.d / 8);                 // d/8 threads per head
    const int heads = a.n_q + 2 * a.n_kv;
    int waves = 1;                                             // wavefronts per block
    if (a.rows >= 2048) {
        waves = ceil_div(heads, heads_per_wave);
        if (waves > 10) waves = 10;
    }
    a.heads_per_block = heads_per_wave * waves;
    const dim3 grid(a.rows, ceil_div(heads, heads_per_wave * waves)), block(64 * waves);
    if (waves == 1) qkv_post_kernel<true><<<grid, block, 0, stream>>>(a);
    else qkv_post_kernel<false><<<grid, block, 0, stream>>>(a);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_argmax(const float *logits, int rows, int vocab, const int32_t *forced, int32_t *greedy_out,
                  int32_t *chosen, int32_t *actions, int max_turns, int turn_idx, int action_mod,
                  float inv_temperature, uint64_t seed, const int32_t *orig_seq, int pos, hipStream_t stream) {
    if (rows <= 0) return SR_OK;
    argmax_kernel<<<dim3(rows), dim3(1024), 0, stream>>>(logits, vocab, forced, greedy_out, chosen, actions,
                                                         max_turns, turn_idx, action_mod, inv_temperature, seed,
                                                         orig_seq, pos);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_fill_i32(int32_t *dst, size_t n, int32_t value, hipStream_t stream) {
    if (n == 0) return SR_OK;
    fill_i32_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(dst, n, value);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_gather_rows(void *dst, const void *src, const int32_t *src_rows, int n_out, size_t row_bytes,
                       hipStream_t stream) {
    if (n_out <= 0 || row_bytes == 0) return SR_OK;
    if (row_bytes % 4) return SR_E_ARG;
    const bool wide = row_bytes % 16 == 0;
    const size_t row_vec = row_bytes / (wide ? 16 : 4);
    unsigned bx = (unsigned)((row_vec + 255) / 256);
    if (bx > 256) bx = 256;
    if (wide)
        gather_rows_kernel<uint4><<<dim3(bx, n_out), dim3(256), 0, stream>>>((uint4 *)dst, (const uint4 *)src, src_rows, row_vec);
    else
        gather_rows_kernel<uint32_t><<<dim3(bx, n_out), dim3(256), 0, stream>>>((uint32_t *)dst, (const uint32_t *)src, src_rows, row_vec);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_copy_pages(uint16_t *kpool, uint16_t *vpool, size_t layer_stride, int n_layers, size_t page_elems,
                      const int2 *pairs, int n_pairs, hipStream_t stream) {
    if (n_pairs <= 0) return SR_OK;
    const size_t page_vec = page_elems / 8;
    unsigned bz = (unsigned)((page_vec + 1023) / 1024);      // four 16-byte pieces of K and of V per thread
    if (bz > 64) bz = 64;
    copy_pages_kernel<<<dim3(n_pairs, n_layers, bz), dim3(256), 0, stream>>>((uint4 *)kpool, (uint4 *)vpool, layer_stride / 8,
                                                                             page_vec, pairs);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace sr
