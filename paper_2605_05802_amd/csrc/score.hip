// Teacher-forced log-likelihood (paper Appendix C.2) and the policy-gradient loss (Section 2.1).
//
// More than 256 rows at a time: the LM head's epilogue leaves a (maximum, sum of exponentials) pair per row and 128
// columns and the target's logit (EPI_LSE in gemm.hip), and score_reduce_kernel turns them into log-probabilities; the
// logits themselves are stored for the last row of a unit only.  Writing the logits of a block of rows, reading them back
// and computing the last rows' a second time took 0.7 ms more (of 7.8) at 4096 rows of 152 064 columns.
// Fewer rows (the weight stream bounds the LM head) and the chunk's first token go through the logits:
// logprob_rows_kernel: one workgroup per logits row.  log softmax(row)[target] needs the row's
// maximum and the sum of exponentials; every thread keeps a running (max, sum) pair over its
// strided part of the row, so the row (vocab x 4 bytes, 608 KiB at the 7B shape) is read once, and
// the pairs are combined through LDS.  Rows whose next token is not an action token are skipped.
//
// accumulate_logprob_kernel: one thread per sequence adds the per-token values of a chunk to the
// sequence's running log-likelihood in token order (double), so the sum does not depend on scheduling.
//
// grpo_share_kernel: one thread per group computes the advantages of Eq. 1 (population standard
// deviation; exactly zero when all rewards of the group are equal) and the group's share of
// sum_i A_i log p(tau_i).  The shares are added in group order, by one lane, so that the loss is the
// same to the last bit whatever the launch shape: a chain of dependent 64-bit additions, which is
// what bounds the call from a few hundred groups on.  The lane reads from LDS only, and finds no zeros there: a share of
// exactly zero, which every group with equal rewards has, changes no sum, so the wavefronts that bring the shares in leave
// them out.  4096 groups of 8, two fifths of them with equal rewards: 16.7 us; 30 with every share added and a group's
// rewards read one after another, 336 with the shares read from global memory by the adding lane.  65 536 groups: 189 us
// (292 without a zero among them), 348 before.
#include <mutex>

#include "sr_internal.h"

namespace sr {
namespace {

constexpr int kLpThreads = 1024;

__device__ __forceinline__ void lse_merge(float &m, float &s, float m2, float s2) {
    const float mn = fmaxf(m, m2);
    s = s * expf(m - mn) + s2 * expf(m2 - mn);
    m = mn;
}

__global__ __launch_bounds__(kLpThreads) void logprob_rows_kernel(LogprobArgs a) {
    __shared__ float s_m[kLpThreads / 64], s_s[kLpThreads / 64];
    const int row = blockIdx.x, tid = threadIdx.x;
    // row -> (unit, token index in the chunk whose probability this row's logits give)
    const int u = (a.row0 + row) / a.rows_per_unit;
    const int t = a.tok0 + (a.row0 + row) % a.rows_per_unit;
    if (t >= a.chunk_len) return;                             // the chunk's last row predicts nothing here
    float *dst = a.out + (size_t)u * a.chunk_len + t;
    if (a.mask && !a.mask[(size_t)u * a.chunk_len + t]) {
        if (tid == 0) *dst = 0.f;
        return;
    }
    const float *lg = a.logits + (size_t)row * a.vocab;
    float m = -3.0e38f, s = 0.f;
    const int v4 = a.vocab & ~3;
    // four 16-byte loads in flight per thread and one rescaling for the sixteen values: a row has one workgroup, so a
    // call of 128 rows is bound by what a workgroup keeps in flight (152 064 columns: 55 us with 512 threads and one
    // load each, 31 now)
    for (int v0 = tid * 4; v0 < v4; v0 += kLpThreads * 16) {
        float4 x[4];
        float mx = -3.0e38f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = v0 + u * kLpThreads * 4;
            x[u] = v < v4 ? *(const float4 *)(lg + v) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) mx = fmaxf(mx, fmaxf(fmaxf(x[u].x, x[u].y), fmaxf(x[u].z, x[u].w)));
        const float mn = fmaxf(m, mx);
        s *= expf(m - mn);
#pragma unroll
        for (int u = 0; u < 4; ++u) s += (expf(x[u].x - mn) + expf(x[u].y - mn)) + (expf(x[u].z - mn) + expf(x[u].w - mn));
        m = mn;
    }
    for (int v = v4 + tid; v < a.vocab; v += kLpThreads) lse_merge(m, s, lg[v], 1.f);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) lse_merge(m, s, __shfl_xor(m, off, 64), __shfl_xor(s, off, 64));
    if ((tid & 63) == 0) { s_m[tid >> 6] = m; s_s[tid >> 6] = s; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kLpThreads / 64; ++w) lse_merge(m, s, s_m[w], s_s[w]);
        const int target = a.tokens[(size_t)u * a.chunk_len + t];
        *dst = (lg[target] - m) - logf(s);
    }
}

// Row r of a pass -> its (unit, token index in the chunk whose probability it gives); false: predicts nothing here
__device__ __forceinline__ bool scored_token(const LogprobArgs &a, int row, size_t *at) {
    const int u = (a.row0 + row) / a.rows_per_unit, t = a.tok0 + (a.row0 + row) % a.rows_per_unit;
    *at = (size_t)u * a.chunk_len + t;
    return t < a.chunk_len;
}

__global__ void score_targets_kernel(LogprobArgs a, int rows, int32_t *__restrict__ target) {
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= rows) return;
    size_t at;
    const bool scored = scored_token(a, row, &at) && (!a.mask || a.mask[at]);
    target[row] = scored ? a.tokens[at] : -1;
}

// Sixteen rows per workgroup, sixteen threads for the column blocks of each; the pairs lie row by row, so a wavefront
// reads runs of 128 bytes.  Column blocks are merged in a fixed order.
__global__ __launch_bounds__(256) void score_reduce_kernel(LogprobArgs a, int rows, ScoreOut s, int n_parts) {
    __shared__ float s_m[16][17], s_s[16][17];
    const int r = threadIdx.x & 15, q = threadIdx.x >> 4, row = blockIdx.x * 16 + r;
    float m = -3.0e38f, sum = 0.f;
    if (row < rows)
        for (int p0 = q; p0 < n_parts; p0 += 128) {          // eight loads in flight
            float2 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                x[u] = p0 + 16 * u < n_parts ? s.lse[(size_t)(p0 + 16 * u) * s.lse_ld + row] : make_float2(-3.0e38f, 0.f);
#pragma unroll
            for (int u = 0; u < 8; ++u) lse_merge(m, sum, x[u].x, x[u].y);
        }
    s_m[q][r] = m;
    s_s[q][r] = sum;
    __syncthreads();
    if (q != 0 || row >= rows) return;
    for (int k = 1; k < 16; ++k) lse_merge(m, sum, s_m[k][r], s_s[k][r]);
    size_t at;
    if (!scored_token(a, row, &at)) return;
    a.out[at] = s.target[row] < 0 ? 0.f : (s.target_logit[row] - m) - logf(sum);
}

__global__ void last_rows_kernel(float4 *__restrict__ dst, const float4 *__restrict__ src, int period, int vec) {
    const float4 *from = src + ((size_t)blockIdx.y * period + period - 1) * vec;
    float4 *to = dst + (size_t)blockIdx.y * vec;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < vec; i += gridDim.x * blockDim.x) to[i] = from[i];
}

__global__ void accumulate_logprob_kernel(const float *__restrict__ tok_lp, int n_seq, int chunk_len,
                                          double *__restrict__ logprob) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n_seq) return;
    double acc = logprob[u];
    for (int t = 0; t < chunk_len; ++t) acc += (double)tok_lp[(size_t)u * chunk_len + t];
    logprob[u] = acc;
}

constexpr int kAddBlock = 32;          // shares added between two looks at LDS (16: 17.8 instead of 16.7 us; reading a block ahead: 19.8)

// Up to 64 shares, one per lane of a wavefront (0 where there is none), appended to v[0 .. n) without the zeros, in lane order;
// returns the new n.
__device__ __forceinline__ int append_shares(double *v, int n, double x) {
    const unsigned long long some = __ballot(x != 0.0);          // NaN is not 0
    const int lane = threadIdx.x & 63;
    if (x != 0.0) v[n + __popcll(some & ((1ull << lane) - 1ull))] = x;
    return n + __popcll(some);
}
// v[n .. next multiple of kAddBlock) = 0, by one wavefront; returns the number of blocks.  Zeros change no sum: it starts as +0 and
// no sum of it and others rounds to -0.
__device__ __forceinline__ int pad_shares(double *v, int n) {
    const int end = (n + kAddBlock - 1) / kAddBlock * kAddBlock, lane = threadIdx.x & 63;
    if (n + lane < end) v[n + lane] = 0.0;
    return end / kAddBlock;
}
// acc + v[0] + ... + v[kAddBlock * blocks - 1], in that order; v in LDS
__device__ __forceinline__ double add_in_order(double acc, const double *v, int blocks) {
    for (int b = 0; b < blocks; ++b) {
        double x[kAddBlock];
#pragma unroll
        for (int k = 0; k < kAddBlock; ++k) x[k] = v[b * kAddBlock + k];
#pragma unroll
        for (int k = 0; k < kAddBlock; ++k) acc += x[k];
    }
    return acc;
}

constexpr int kShareThreads = 64;      // many small workgroups: the groups spread over the compute units
// Up to so many groups and members one workgroup does shares and sum in one launch: groups of 8 400 of them (7.6 us either way; 37: 4.3
// and 5.6), of 16 200 (7.4 either way; 512: 14.0 and 8.8), of 2 all 512 (6.4 and 7.6)
constexpr int kOneBlock = 512, kOneMembers = 3200;
constexpr int kSegment = 512;          // shares that one wavefront brings in, without zeros, ...
constexpr int kSegments = 4;           // ... and how many of these an LDS buffer of the ordered sum holds

// Advantages and share of one group of at most MOST members, everything requested before anything is used; MOST = 0: of any size.
template <int MOST>
__device__ __forceinline__ double group_share(const double *__restrict__ lp, const float *__restrict__ r, int G, double eps,
                                              float *__restrict__ adv) {
    float rr[MOST ? MOST : 1];
    double ll[MOST ? MOST : 1];
#pragma unroll
    for (int i = 0; i < MOST; ++i) rr[i] = r[min(i, G - 1)];
#pragma unroll
    for (int i = 0; i < MOST; ++i) ll[i] = lp[min(i, G - 1)];
    auto each = [&](auto &&f) __attribute__((always_inline)) {   // f(i, reward, log-likelihood) in member order
        if constexpr (MOST > 0) {
#pragma unroll
            for (int i = 0; i < MOST; ++i)
                if (i < G) f(i, rr[i], ll[i]);       // uniform
        } else {
            for (int i = 0; i < G; ++i) f(i, r[i], lp[i]);
        }
    };
    const float r0 = MOST ? rr[0] : r[0];
    bool all_equal = true;
    double mean = 0.0;
    each([&](int, float x, double) {
        all_equal &= x == r0;
        mean += (double)x;
    });
    mean /= G;
    double var = 0.0;
    each([&](int, float x, double) { var += ((double)x - mean) * ((double)x - mean); });
    const double sigma = sqrt(var / G);
    double acc = 0.0;
    each([&](int i, float x, double l) {
        const double A = all_equal ? 0.0 : ((double)x - mean) / (sigma + eps);
        if (adv) adv[i] = (float)A;
        acc += A * l;
    });
    return acc;
}

// ONE: a single workgroup of kOneBlock threads holds every group and adds the shares itself
template <bool ONE>
__global__ void grpo_share_kernel(const double *__restrict__ logprob, const float *__restrict__ rewards, int n_groups,
                                  int G, double eps, float *__restrict__ adv, double *__restrict__ share,
                                  double *__restrict__ loss) {
    __shared__ __align__(16) double s_share[ONE ? kOneBlock : 1];
    __shared__ int s_blocks[ONE ? kOneBlock / 64 : 1];
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    double mine = 0.0;
    if (g < n_groups) {
        const size_t at = (size_t)g * G;
        float *a = adv ? adv + at : nullptr;
        mine = G <= 4    ? group_share<4>(logprob + at, rewards + at, G, eps, a)
               : G <= 8  ? group_share<8>(logprob + at, rewards + at, G, eps, a)
               : G <= 16 ? group_share<16>(logprob + at, rewards + at, G, eps, a)
                         : group_share<0>(logprob + at, rewards + at, G, eps, a);
        share[g] = mine;
    }
    if (!ONE) return;
    const int wave = threadIdx.x >> 6;
    const int blocks = pad_shares(s_share + wave * 64, append_shares(s_share + wave * 64, 0, mine));
    if ((threadIdx.x & 63) == 0) s_blocks[wave] = blocks;
    __syncthreads();
    if (threadIdx.x == 0) {
        double acc = 0.0;
        for (int w = 0; w < kOneBlock / 64; ++w) acc = add_in_order(acc, s_share + w * 64, s_blocks[w]);
        *loss = -acc / ((double)n_groups * G);
    }
}

__global__ __launch_bounds__(256) void grpo_sum_kernel(const double *__restrict__ share, int n_groups, int G,
                                                       double *__restrict__ loss) {
    constexpr int kChunk = kSegments * kSegment;
    __shared__ __align__(16) double buf[2][kChunk];
    __shared__ int s_blocks[2][kSegments];
    const int n_chunks = (n_groups + kChunk - 1) / kChunk;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    auto fetch = [&](int c, int seg) {                // by one wavefront
        double x[kSegment / 64];
        const int at = c * kChunk + seg * kSegment + lane;
#pragma unroll
        for (int j = 0; j < kSegment / 64; ++j) x[j] = at + 64 * j < n_groups ? share[at + 64 * j] : 0.0;
        double *v = buf[c & 1] + seg * kSegment;
        int n = 0;
#pragma unroll
        for (int j = 0; j < kSegment / 64; ++j) n = append_shares(v, n, x[j]);
        const int blocks = pad_shares(v, n);
        if (lane == 0) s_blocks[c & 1][seg] = blocks;
    };
    fetch(0, wave);
    double acc = 0.0;
    for (int c = 0; c < n_chunks; ++c) {
        __syncthreads();                 // chunk c is in LDS, and nobody reads the other buffer any more
        if (wave > 0) {
            if (c + 1 < n_chunks)
                for (int seg = wave - 1; seg < kSegments; seg += 3) fetch(c + 1, seg);
        } else if (lane == 0) {
            for (int seg = 0; seg < kSegments; ++seg) acc = add_in_order(acc, buf[c & 1] + seg * kSegment, s_blocks[c & 1][seg]);
        }
    }
    if (threadIdx.x == 0) *loss = -acc / ((double)n_groups * G);
}

int launch_grpo_loss(const double *logprob, const float *rewards, int n_groups, int G, double eps, float *advantages,
                     double *share, double *loss, hipStream_t stream) {
    if (n_groups <= kOneBlock && (long long)n_groups * G <= kOneMembers) {
        grpo_share_kernel<true><<<dim3(1), dim3(kOneBlock), 0, stream>>>(logprob, rewards, n_groups, G, eps, advantages,
                                                                         share, loss);
        SR_HIP(hipGetLastError());
        return SR_OK;
    }
    grpo_share_kernel<false><<<dim3((n_groups + kShareThreads - 1) / kShareThreads), dim3(kShareThreads), 0, stream>>>(
        logprob, rewards, n_groups, G, eps, advantages, share, loss);
    SR_HIP(hipGetLastError());
    grpo_sum_kernel<<<dim3(1), dim3(256), 0, stream>>>(share, n_groups, G, loss);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace

int launch_logprob_rows(const LogprobArgs &a, int rows, hipStream_t stream) {
    if (rows <= 0) return SR_OK;
    if (a.rows_per_unit < 1 || a.vocab < 1 || a.chunk_len < 1) return SR_E_ARG;
    logprob_rows_kernel<<<dim3(rows), dim3(kLpThreads), 0, stream>>>(a);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_score_targets(const LogprobArgs &a, int rows, int32_t *target, hipStream_t stream) {
    if (rows <= 0) return SR_OK;
    if (a.rows_per_unit < 1 || a.chunk_len < 1) return SR_E_ARG;
    score_targets_kernel<<<dim3((rows + 255) / 256), dim3(256), 0, stream>>>(a, rows, target);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_score_reduce(const LogprobArgs &a, int rows, const ScoreOut &s, hipStream_t stream) {
    if (rows <= 0) return SR_OK;
    if (a.rows_per_unit < 1 || a.chunk_len < 1 || a.vocab < 1) return SR_E_ARG;
    score_reduce_kernel<<<dim3((rows + 15) / 16), dim3(256), 0, stream>>>(a, rows, s, 2 * ceil_div(a.vocab, 256));
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_last_rows(float *dst, const float *src, int n, int period, int vocab, hipStream_t stream) {
    if (n <= 0) return SR_OK;
    if (vocab % 4) return SR_E_ARG;
    const int vec = vocab / 4;
    last_rows_kernel<<<dim3(vec < 64 * 256 ? (vec + 255) / 256 : 64, n), dim3(256), 0, stream>>>((float4 *)dst, (const float4 *)src,
                                                                                             period, vec);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

int launch_accumulate_logprob(const float *tok_lp, int n_seq, int chunk_len, double *logprob, hipStream_t stream) {
    if (n_seq <= 0) return SR_OK;
    accumulate_logprob_kernel<<<dim3((n_seq + 63) / 64), dim3(64), 0, stream>>>(tok_lp, n_seq, chunk_len, logprob);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace sr

extern "C" int sr_grpo_loss(const double *logprob, const float *rewards, int n_groups, int G, double eps,
                            float *advantages, double *group_scratch, double *loss, void *stream) {
    if (!logprob || !rewards || !group_scratch || !loss || n_groups < 1 || G < 1 || !(eps >= 0.0)) return SR_E_ARG;
    return sr::launch_grpo_loss(logprob, rewards, n_groups, G, eps, advantages, group_scratch, loss, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------------
// The same loss for callers that cannot allocate: the per-group shares live in a file-scope device
// array instead of a buffer the caller brings.
// ---------------------------------------------------------------------------------------------
namespace {

constexpr int kStaticMaxGroups = SR_GRPO_STATIC_MAX_GROUPS;
static __device__ __align__(256) double scratch[kStaticMaxGroups];   // every GPU holds its own copy

constexpr int kMaxDevices = 64;
double *g_scratch_ptr[kMaxDevices];        // device address of `scratch` on each GPU, looked up once
bool g_scratch_known[kMaxDevices];
std::mutex g_scratch_mutex;

// Device address of this GPU's copy of `scratch` (the array's name is only a host-side stand-in).
int static_scratch(double **out) {
    int dev = -1;
    SR_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return SR_E_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_known[dev]) {
        void *p = nullptr;
        SR_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_scratch_ptr[dev] = (double *)p;
        g_scratch_known[dev] = true;
    }
    *out = g_scratch_ptr[dev];
    return SR_OK;
}

}  // namespace

extern "C" int sr_grpo_loss_static(const double *logprob, const float *rewards, int n_groups, int G, double eps,
                                   float *advantages, double *loss, void *stream) {
    if (!logprob || !rewards || !loss || n_groups < 1 || G < 1 || !(eps >= 0.0)) return SR_E_ARG;
    if (n_groups > kStaticMaxGroups) return SR_E_LIMIT;
    double *share = nullptr;
    SR_TRY(static_scratch(&share));
    // every share[g], g < n_groups, is written before it is read: nothing of an earlier call is used
    return sr::launch_grpo_loss(logprob, rewards, n_groups, G, eps, advantages, share, loss, (hipStream_t)stream);
}
