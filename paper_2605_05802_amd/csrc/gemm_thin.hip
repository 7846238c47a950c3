// Thin projections (QKV, O, down) of a few rows, with what follows them.
#include "epilogue.h"

namespace sr {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A workgroup owns 16 output features (O, down) or 16 rotation pairs of a head (QKV) and all rows.  Its four wavefronts share K out
// between them, each with W and X straight from global memory into a ring of registers -- wavefronts with different k-steps
// have nothing to share, so there is no LDS and no barrier in the loop -- and their sums meet in LDS once, in a fixed order.
// So no partial sums go through memory, and what had to wait for them in a kernel of its own happens here:
//   O, down: the residual stream takes the result, and x * gain (bf16) and x^2 summed over the workgroup's features are left for the
//            projection behind the norm, which finishes the norm by scaling its results (RowScale);
//   QKV:     bias, rotation, queries and K/V pages.
// A layer of a decode step is then five or six launches instead of nine.  Bound: launch latency for small matrices; else a compute
// unit's vector-memory path, about 50 GB/s, through which W and, as many times as there are workgroups, X come.  Eight rows read only
// their half of X's 16-row tiles.  Alone, in us, this kernel against gemm_stream_kernel without what follows it (norm 4.4 us at 8 rows,
// QKV epilogue 4.6): K = 3584, 8 rows: O 6.4 / 7.0, QKV 9.6 / 8.6, down 22.6 / 24.4; 16 rows: 7.7 / 7.4, 11.1 / 8.7, 28.8 / 24.8; K = 256, 32
// rows: 2.7 / 2.8 and 3.0 / 3.2.  More wavefronts and deeper rings are no faster.
constexpr int kWaves = kThinSplits;
constexpr int ring_steps(int mt) { return mt == 1 ? 8 : mt == 2 ? 4 : 2; }

// X as it is needed by both kernels: acc[NT][MT] of this wavefront's k-steps
template <int NT, int MT, bool HALF>
__device__ __forceinline__ void multiply(const ThinArgs &a, int wave, int lane, f32x4 (&acc)[NT][MT]) {
    constexpr int D = ring_steps(MT);
    int k0, k1;
    split_range(a.ks_total, 1, kWaves, wave, &k0, &k1);
    const int last = k1 - 1;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (k0 >= k1) return;
    const u32x4 *wp = (const u32x4 *)a.W + (size_t)blockIdx.x * NT * a.ks_total * 64 + lane;
    const u32x4 *xp = (const u32x4 *)a.X + (HALF ? lane & ~8 : lane);        // rows 8 .. 15 repeat 0 .. 7: the same lines
    const size_t xs = (size_t)a.mt_total * 64, ws = (size_t)a.ks_total * 64;
    u32x4 w[D][NT], x[D][MT];
    auto load = [&](int d, int k) __attribute__((always_inline)) {           // past the end: the last k-step again, never used
        const int kk = min(k, last);
#pragma unroll
        for (int i = 0; i < NT; ++i) w[d][i] = __builtin_nontemporal_load(wp + i * ws + (size_t)kk * 64);
#pragma unroll
        for (int j = 0; j < MT; ++j) x[d][j] = xp[kk * xs + j * 64];
    };
    auto step = [&](int d) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[d][i]), __builtin_bit_cast(bf16x8, x[d][j]),
                                                                     acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, k0 + d);
    int k = k0;
    for (; k + D <= k1; k += D)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            __builtin_amdgcn_sched_barrier(0);
            step(d);
            load(d, k + d + D);
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (k + d < k1) step(d);
}

template <int NT, int MT>
struct ThinLds {
    f32x4 acc[kWaves][NT][MT][64];
    float squares[64 * kWaves];
};
template <int NT, int MT>
__device__ __forceinline__ f32x4 sum_of_waves(const ThinLds<NT, MT> &s, int i, int j, int lane) {
    f32x4 v = s.acc[0][i][j][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += s.acc[w][i][j][lane];
    return v;
}
template <int MT, bool HALF>
__global__ __launch_bounds__(64 * kWaves) void thin_resid_kernel(ThinArgs a) {
    __shared__ ThinLds<1, MT> lds;
    constexpr int TILES = (MT + kWaves - 1) / kWaves;          // row tiles that a wavefront finishes
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4, n = blockIdx.x * 16 + 4 * g;
    // what the end needs besides the sums, requested first
    const uint2 gain = *(const uint2 *)(a.gain + n);
    f32x4 x[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) x[t] = *(const f32x4 *)(a.resid + (size_t)min((wave + t * kWaves) * 16 + c, a.M - 1) * a.N + n);
    f32x4 acc[1][MT];
    multiply<1, MT, HALF>(a, wave, lane, acc);
#pragma unroll
    for (int j = 0; j < MT; ++j) lds.acc[wave][0][j][lane] = acc[0][j];
    __syncthreads();
    const float gn[4] = {__uint_as_float(gain.x << 16), __uint_as_float(gain.x & 0xFFFF0000u), __uint_as_float(gain.y << 16),
                         __uint_as_float(gain.y & 0xFFFF0000u)};
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int j = wave + t * kWaves, m = j * 16 + c;
        if (j >= MT) break;
        const f32x4 v = x[t] + sum_of_waves(lds, 0, j, lane);
        const float squares = row_sum((v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]));
        if (m >= a.M) continue;
        *(f32x4 *)(a.resid + (size_t)m * a.N + n) = v;
        *(uint2 *)(a.xg + frag_offset(m, n, a.mt_total)) = make_uint2(pack_bf16x2(v[0] * gn[0], v[1] * gn[1]), pack_bf16x2(v[2] * gn[2], v[3] * gn[3]));
        if (g == 0) a.squares[(size_t)m * a.squares_ld + blockIdx.x] = squares;
    }
}

template <int MT, bool HALF>
__global__ __launch_bounds__(64 * kWaves) void thin_qkv_kernel(ThinArgs a) {
    __shared__ ThinLds<2, MT> lds;
    constexpr int TILES = (MT + kWaves - 1) / kWaves;
    const QkvPostArgs &q = a.qkv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    // the workgroup's two tiles: dims 16 t .. and d/2 + 16 t .. of a head
    const int per_head = q.d >> 5, head = (int)blockIdx.x / per_head, i = ((int)blockIdx.x - head * per_head) * 16 + 4 * g;
    QkvExtras x[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int m = min((wave + t * kWaves) * 16 + c, a.M - 1), unit = quotient(m, q.by_chunk);
        x[t].pos = q.pos0 + m - unit * q.chunk;
        x[t].page = q.page_table[(size_t)unit * q.pt_row_stride * q.pt_stride + (x[t].pos >> q.page_shift)];
        fetch_bias_and_rotation(q, head, i, x[t]);
    }
    RowSquares<64 * kWaves> squares;
    squares.request(a.scale, a.M, threadIdx.x);
    f32x4 acc[2][MT];
    multiply<2, MT, HALF>(a, wave, lane, acc);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < MT; ++j) lds.acc[wave][h][j][lane] = acc[h][j];
    squares.leave(a.scale, lds.squares, threadIdx.x);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int j = wave + t * kWaves, m = j * 16 + c;
        if (j >= MT || m >= a.M) break;
        const float s = a.scale.squares ? squares.scale(a.scale, lds.squares, m) : 1.f;
        finish_qkv(q, m, head, i, sum_of_waves(lds, 0, j, lane) * s, sum_of_waves(lds, 1, j, lane) * s, x[t]);
    }
}

}  // namespace

#define SR_THIN(KERNEL, GRID)                                                                   \
    do {                                                                                        \
        const dim3 grid(GRID), block(64 * kWaves);                                              \
        if (a.M <= 8) KERNEL<1, true><<<grid, block, 0, stream>>>(a);                           \
        else if (a.M <= 16) KERNEL<1, false><<<grid, block, 0, stream>>>(a);                    \
        else if (a.M <= 32) KERNEL<2, false><<<grid, block, 0, stream>>>(a);                    \
        else if (a.M <= 64) KERNEL<4, false><<<grid, block, 0, stream>>>(a);                    \
        else KERNEL<8, false><<<grid, block, 0, stream>>>(a);                                   \
        SR_HIP(hipGetLastError());                                                              \
    } while (0)

int launch_thin_resid(const ThinArgs &a, hipStream_t stream) {
    if (a.M <= 0) return SR_OK;
    if (a.M > kThinRows || a.mt_total < kThinRows / 16 || a.N % 16 || a.ks_total < 1 || a.scale.squares || a.squares_ld < a.N / 16) return SR_E_ARG;
    SR_THIN(thin_resid_kernel, a.N / 16);
    return SR_OK;
}

int launch_thin_qkv(const ThinArgs &args, hipStream_t stream) {
    ThinArgs a = args;
    if (a.M <= 0) return SR_OK;
    if (a.M > kThinRows || a.mt_total < kThinRows / 16 || a.ks_total < 1 || (a.qkv.d != 64 && a.qkv.d != 128) || a.qkv.chunk < 1 ||
        a.N != (a.qkv.n_q + 2 * a.qkv.n_kv) * a.qkv.d || (a.scale.squares && a.scale.ld % 4))
        return SR_E_ARG;
    set_divisions(&a.qkv);
    SR_THIN(thin_qkv_kernel, a.N / 32);
    return SR_OK;
}

}  // namespace sr
