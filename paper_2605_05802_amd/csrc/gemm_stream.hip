// Decode-time projection GEMM  Y[M][N] = X[M][K] * W[N][K]^T  for M <= 256 on the bf16 matrix cores:
// the weight-streaming kernel that carries most of a decode step's HBM traffic.
#include "epilogue.h"

namespace sr {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// k-steps (of 32) per LDS chunk of X: three chunks of four fit in 160 KiB up to 192 rows
constexpr int chunk_steps(int mt32) { return mt32 <= 6 ? 4 : 2; }
// uint4 per k-step of X in LDS: the 16-row tiles a launch computes, at least eight
constexpr int kstep_vec(int mt32) { return (mt32 <= 4 ? 8 : 2 * mt32) * 64; }

// Every weight byte is used once per launch, so the load carries the non-temporal hint: the caches do
// not retain the line, and a pure streaming read measures 13 % faster with it (6.97 against 6.15 TB/s).
__device__ __forceinline__ u32x4 load_w_stream(const u32x4 *p) { return __builtin_nontemporal_load(p); }

// ---------------------------------------------------------------------------------------------
// Weight-streaming kernel (M <= 256) with a loader wavefront.
//
// A workgroup owns 32 * WAVES output features and all rows; each of its WAVES computing wavefronts
// owns 32 features and streams their weights through a register ring of RING k-steps (2 KiB each),
// refilling a slot as soon as its MFMAs are issued, so RING * 2 KiB per wavefront stay in flight
// across the workgroup barriers.  The loop body has no branch: the compiler counts outstanding
// loads exactly, and prefetches past the end re-read the last valid k-step.
//
// The activations are brought in by one extra wavefront that does nothing else: it copies X chunks
// (four k-steps, 32 KiB at 128 rows) from global memory straight into LDS with lane-linear 16-byte direct-to-LDS
// loads, two chunks ahead of the MFMAs, through three buffers.  Vector-memory loads return in order
// within a wavefront, so an activation load inside a computing wavefront would make its wait drain
// the older weight loads too; with the loader the computing wavefronts carry only weight loads,
// never wait for an activation and keep no staging registers, and the loader's wait for its own
// copies stalls nobody.
//
// Two forms of the MFMA.  LEAN is 16x16x32, whose operands are 16-row tiles as they lie in memory; it draws less power for the same
// product (2.12 against 1.88 PFLOP/s in a loop without memory), and from 65 rows on the chip's clock follows: gate|up at the 7B
// shape 46.99 -> 46.52 us at 72 rows, 56.5 -> 55.8 at 144, 68.8 -> 66.1 at 224, 76.8 -> 72.7 at 256; prefill of 8 x 17 tokens 838 -> 811; up to 64
// rows no difference.  32x32x16 has half the instructions, and short launches and those that leave the chip partly idle keep it
// (stream_lean).  Its operands (32 rows x 16 k) are assembled from the
// 16-row fragment layout by addressing: lane (r = lane % 32, g = lane / 32) of k-half h takes the 16 bytes of row tile r / 16, lane slot
// (r % 16) + 16 * (2h + g).
//
// MT32 = number of 32-row tiles computed (M <= 32 * MT32): smaller batches skip the idle rows'
// copies, LDS reads and MFMAs.  Up to four tiles the fragments of a whole k-step are read ahead; five to eight
// (129 to 256 rows) read half a k-step ahead, which keeps 128 accumulators, the ring and the fragments within 256 registers.
// At the 7B shape gate|up, QKV, O and down take 53, 17, 14 and 40 us at 136 rows and 79, 22, 20 and 54 at 256; the tiled kernels took
// 76, 25, 18 and 58, and 87, 26, 19 and 59.  Workgroup width matters because with one workgroup per CU a matrix
// should break into about 256 equal workgroups: 37 888 packed gate|up rows give 148 workgroups of
// 256 features (108 CUs idle) but 237 of 160.
// ---------------------------------------------------------------------------------------------
constexpr int kRing = 8;                   // k-steps of W in flight per computing wavefront (16 measured slower at every width)
constexpr int kStBufs = 3;                 // LDS chunk buffers: the loader runs two chunks ahead
constexpr int st_x_bytes(int mt32) { return kStBufs * chunk_steps(mt32) * kstep_vec(mt32) * 16; }
// ... and, where a norm is finished, a float for every computing thread behind them (RowScale)
constexpr int st_lds_bytes(int mt32, int waves, bool scaled) { return st_x_bytes(mt32) + (scaled ? 256 * waves : 0); }

// RING = k-steps of W each computing wavefront keeps in flight (2 KiB per k-step); LEAN: the 16x16x32 MFMA
template <int EPI, int WAVES, int MT32, int RING, bool SCALED, bool LEAN>
__global__ __launch_bounds__(64 * (WAVES + 1)) void gemm_stream_kernel(GemmArgs a) {
    extern __shared__ u32x4 lds_dyn[];     // [kStBufs][k-step in chunk][16-row tile][lane]
    constexpr int kKC = chunk_steps(MT32), kStepVec = kstep_vec(MT32), kChunkVec = kKC * kStepVec;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = blockIdx.x, sp = blockIdx.z;
    int ks0, ks1;
    split_range(a.ks_total, RING, a.splits, sp, &ks0, &ks1);
    const int last = ks1 - 1;

    if (wave == WAVES) {
        // ---- loader.  Chunk c lives in buffer c % 3.  Barrier c (c = 0, 1, ...) is passed by the
        // computing wavefronts once they are done with chunk c - 1, and by the loader once chunk c has
        // landed; after it the loader may overwrite the buffer of chunk c - 1 with chunk c + 2.
        if (ks0 >= ks1) return;
        const u32x4 *xp = (const u32x4 *)a.X + lane;
        const size_t x_ks_stride = (size_t)a.mt_total * 64;
        constexpr int kCopies = kKC * 2 * MT32;         // direct-to-LDS loads per chunk (<= 48)
        auto copy_chunk = [&](int kc, int buf) {
#pragma unroll
            for (int kk = 0; kk < kKC; ++kk) {
                const u32x4 *src = xp + (size_t)min(kc + kk, last) * x_ks_stride;
#pragma unroll
                for (int b = 0; b < 2 * MT32; ++b)
                    __builtin_amdgcn_global_load_lds(
                        (const __attribute__((address_space(1))) void *)(src + b * 64),
                        (__attribute__((address_space(3))) void *)&lds_dyn[buf * kChunkVec + kk * kStepVec + b * 64], 16,
                        0, 0);
            }
        };
        // wait until at most one chunk of copies is outstanding: vmcnt(kCopies), other counters untouched
        constexpr int kWaitOlder = 0x0F70 | (kCopies & 15) | ((kCopies >> 4) << 14);
        copy_chunk(ks0, 0);
        copy_chunk(ks0 + kKC, 1);
        int buf = 2;
        for (int kc = ks0; kc < ks1; kc += kKC) {
            __builtin_amdgcn_s_waitcnt(kWaitOlder);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            copy_chunk(kc + 2 * kKC, buf);               // past the end: re-copies the last k-step, never read
            buf = buf == kStBufs - 1 ? 0 : buf + 1;
        }
        __builtin_amdgcn_s_waitcnt(kWaitOlder);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_s_waitcnt(0x0F70);              // nothing may still be writing LDS at exit
        return;
    }

    const int nt32 = nb * WAVES + wave;             // this wavefront's 32 output features
    // The norm in front of this projection: its sums of squares are dealt out over the computing threads, requested before the first
    // weights and added up behind them.  (By the loader, in a few round trips before the first barrier, it cost 3.5 us at 8 rows.)
    RowSquares<64 * WAVES> squares;
    if constexpr (SCALED) squares.request(a.scale, a.M, tid);

    // LEAN: acc16[row tile][feature tile], lane (c, g) holds features 4g .. 4g+3 of row c.  Else acc32[32 rows], lane (r32 = row, g2)
    // holds, in register v, feature 8 * (v / 4) + 4 * g2 + v % 4 of the wavefront's 32.
    const int c = lane & 15, g = lane >> 4, r32 = lane & 31, g2 = lane >> 5;
    f32x4 acc16[LEAN ? 2 * MT32 : 1][2];
    f32x16 acc32[LEAN ? 1 : MT32];
#pragma unroll
    for (auto &t : acc16)
#pragma unroll
        for (f32x4 &x : t) x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (f32x16 &t : acc32)
#pragma unroll
        for (int v = 0; v < 16; ++v) t[v] = 0.f;

    if (ks0 < ks1) {
        constexpr int NF = 2 * MT32;                // X fragments per k-step
        // The two W fragments of a k-step: LEAN the feature tiles, else the k-halves of both
        const int sub = LEAN ? 0 : r32 >> 4, slot0 = LEAN ? lane : (r32 & 15) + 16 * g2;
        const u32x4 *wp0 = (const u32x4 *)a.W + ((size_t)(nt32 * 2 + sub) * a.ks_total) * 64 + slot0;
        const u32x4 *wp1 = wp0 + (LEAN ? (size_t)a.ks_total * 64 : 32);
        // X fragment f: LEAN row tile f, else k-half f % 2 of rows 32 (f / 2) ..
        const int xoff = sub * 64 + slot0;
        auto x_at = [](int f) { return LEAN ? f * 64 : (f >> 1) * 128 + (f & 1) * 32; };
        auto multiply = [&](int f, const bf16x8 &wa, const bf16x8 &wb, const bf16x8 &x) __attribute__((always_inline)) {
            if constexpr (LEAN) {
                acc16[f][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, x, acc16[f][0], 0, 0, 0);
                acc16[f][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb, x, acc16[f][1], 0, 0, 0);
            } else acc32[f >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f & 1 ? wb : wa, x, acc32[f >> 1], 0, 0, 0);
        };
        constexpr int PER = LEAN ? 2 : 1;           // MFMAs per X fragment

        u32x4 w0[RING], w1[RING];
#pragma unroll
        for (int i = 0; i < RING; ++i) {
            w0[i] = load_w_stream(wp0 + (size_t)(ks0 + i) * 64);
            w1[i] = load_w_stream(wp1 + (size_t)(ks0 + i) * 64);
        }
        if constexpr (SCALED) squares.leave(a.scale, (float *)lds_dyn + st_x_bytes(MT32) / 4, tid);
        __syncthreads();                                         // barrier 0: chunk 0 is in LDS

        int buf = 0;
        for (int ks = ks0; ks < ks1; ks += RING) {
#pragma unroll
            for (int q = 0; q < RING / kKC; ++q) {
                const int kc0 = ks + q * kKC;
                const u32x4 *xb = &lds_dyn[buf * kChunkVec + xoff];
                buf = buf == kStBufs - 1 ? 0 : buf + 1;
                // STEPS parts of the chunk, each with NX fragments that are read while the part before it is multiplied: whole k-steps, or
                // their halves (LEAN of the rows, else of k)
                constexpr int HALVES = MT32 <= 4 ? 1 : 2, PARTS = HALVES * kKC, NX = NF / HALVES;
                auto part = [](int p, int j) { return HALVES == 1 ? j : LEAN ? (p & 1) * MT32 + j : 2 * j + (p & 1); };      // its fragments
                bf16x8 xf[2][NX];
#pragma unroll
                for (int j = 0; j < NX; ++j) xf[0][j] = __builtin_bit_cast(bf16x8, xb[x_at(part(0, j))]);
#pragma unroll
                for (int p = 0; p < PARTS; ++p) {
                    const int kk = p / HALVES, i = q * kKC + kk;
                    __builtin_amdgcn_sched_barrier(0);
                    const bf16x8 wa = __builtin_bit_cast(bf16x8, w0[i]), wb = __builtin_bit_cast(bf16x8, w1[i]);
                    if (p + 1 < PARTS) {
#pragma unroll
                        for (int j = 0; j < NX; ++j)
                            xf[(p + 1) & 1][j] = __builtin_bit_cast(bf16x8, xb[(p + 1) / HALVES * kStepVec + x_at(part(p + 1, j))]);
                    }
#pragma unroll
                    for (int j = 0; j < NX; ++j) multiply(part(p, j), wa, wb, xf[p & 1][j]);
                    // refill the slots just consumed
                    const int kn = min(kc0 + kk + RING, last);
                    const bool done0 = HALVES == 1 || !LEAN ? p % HALVES == 0 : p % 2 == 1, done1 = p % HALVES == HALVES - 1;
                    if (done0) w0[i] = load_w_stream(wp0 + (size_t)kn * 64);
                    if (done1) w1[i] = load_w_stream(wp1 + (size_t)kn * 64);
                    if (p + 1 < PARTS) {
#pragma unroll
                        for (int j = 0; j < NX; ++j) {
                            __builtin_amdgcn_sched_group_barrier(0x008, PER, 0); // MFMAs
                            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // 1 LDS read
                        }
                    } else {
                        __builtin_amdgcn_sched_group_barrier(0x008, PER * NX, 0);
                    }
                    if (done0 && done1) __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);           // W refills
                    else if (done0 || done1) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                __syncthreads();
            }
        }
    }

    if constexpr (SCALED) {
        // four (two) lanes have the same rows: each forms a quarter (half) of their factors
        const float *left = (const float *)lds_dyn + st_x_bytes(MT32) / 4;
        constexpr int ROWS = LEAN ? 16 : 32, LANES = 64 / ROWS, TILES = 32 * MT32 / ROWS;
        float mine[(TILES + LANES - 1) / LANES];
        const int which = LEAN ? g : g2, row = LEAN ? c : r32;
#pragma unroll
        for (int u = 0; u * LANES < TILES; ++u) mine[u] = squares.scale(a.scale, left, (LANES * u + which) * ROWS + row);
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const float f = __shfl(mine[t / LANES], t % LANES * ROWS + row);
            if constexpr (LEAN) {
                acc16[t][0] *= f;
                acc16[t][1] *= f;
            } else acc32[t] *= f;
        }
    }
    // Four consecutive features from n on of row m; of SwiGLU's 32, 0 .. 15 are gate and 16 .. 31 the matching up features.
    auto store = [&](int m, int n, const f32x4 &v) __attribute__((always_inline)) {
        if (n < a.N) *(f32x4 *)((float *)a.out + (size_t)sp * a.split_stride + (size_t)m * a.ld_out + n) = v;
    };
    auto store_swiglu = [&](int m, int f, const f32x4 &gate, const f32x4 &up) __attribute__((always_inline)) {
        if (f >= a.ld_out) return;
        float r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = gate[e] / (1.0f + __expf(-gate[e])) * up[e];
        *(uint2 *)((uint16_t *)a.out + frag_offset(m, f, a.mt_total)) = make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
    };
    if constexpr (LEAN) {
#pragma unroll
        for (int t = 0; t < 2 * MT32; ++t) {
            const int m = t * 16 + c;
            if (m >= a.M) continue;
            if constexpr (EPI == EPI_F32) {
                store(m, nt32 * 32 + 4 * g, acc16[t][0]);
                store(m, nt32 * 32 + 16 + 4 * g, acc16[t][1]);
            } else store_swiglu(m, nt32 * 16 + 4 * g, acc16[t][0], acc16[t][1]);
        }
    } else {
#pragma unroll
        for (int mt = 0; mt < MT32; ++mt) {
            const int m = mt * 32 + r32;
            if (m >= a.M) continue;
            auto four = [&](int vq) { return f32x4{acc32[mt][4 * vq], acc32[mt][4 * vq + 1], acc32[mt][4 * vq + 2], acc32[mt][4 * vq + 3]}; };
#pragma unroll
            for (int vq = 0; vq < (EPI == EPI_F32 ? 4 : 2); ++vq) {
                if constexpr (EPI == EPI_F32) store(m, nt32 * 32 + 8 * vq + 4 * g2, four(vq));
                else store_swiglu(m, nt32 * 16 + 8 * vq + 4 * g2, four(vq), four(vq + 2));
            }
        }
    }
}

}  // namespace

int launch_gemm_stream(const GemmArgs &a, GemmEpilogue epi, hipStream_t stream) {
    if (a.M <= 0) return SR_OK;
    if (a.M > 256 || a.mt_total < (a.M > 128 ? 16 : 8) || a.splits < 1 || a.splits > 65535) return SR_E_ARG;
    if (a.ks_total % kRing || (a.wide != 2 && a.wide != 4 && a.wide != 5 && a.wide != 8 && a.wide != 10)) return SR_E_ARG;
    dim3 sgrid(ceil_div(a.N, 32 * a.wide), 1, epi == EPI_F32 ? a.splits : 1), lblock(64 * (a.wide + 1));
    const int mt32 = ceil_div(a.M, 32);
    hipError_t attr = hipSuccess;
    const bool scaled = a.scale.squares != nullptr;
    const bool lean = stream_lean(a.M, a.wide, a.ks_total, epi == EPI_F32 ? a.splits : 1, scaled);
#define SR_STREAM_CASE(E, W, T, S, L)                                                                      \
    (attr = hipFuncSetAttribute((const void *)gemm_stream_kernel<E, W, T, kRing, S, L>,                    \
                        hipFuncAttributeMaxDynamicSharedMemorySize, st_lds_bytes(T, W, S)),                \
     gemm_stream_kernel<E, W, T, kRing, S, L><<<sgrid, lblock, st_lds_bytes(T, W, S), stream>>>(a))
#define SR_STREAM_SCALED(E, W, T, L) (scaled ? SR_STREAM_CASE(E, W, T, true, L) : SR_STREAM_CASE(E, W, T, false, L))
#define SR_STREAM_PLAIN(E, W, T) SR_STREAM_CASE(E, W, T, false, false)
#define SR_STREAM_TALL(E, W, T) (lean ? SR_STREAM_CASE(E, W, T, false, true) : SR_STREAM_PLAIN(E, W, T))
#define SR_STREAM_LEAN(E, W, T) (scaled ? SR_STREAM_CASE(E, W, T, true, false) : SR_STREAM_TALL(E, W, T))
    // nine and eleven wavefronts put three on one SIMD: 168 registers, too few for more than four row tiles, and for four without LEAN
#define SR_STREAM_MT4(E, W, LEAN)                                                                          \
    (mt32 == 1 ? SR_STREAM_SCALED(E, W, 1, false) : mt32 == 2 ? SR_STREAM_SCALED(E, W, 2, false)           \
     : mt32 == 3 ? LEAN(E, W, 3) : LEAN(E, W, 4))
#define SR_STREAM_ALWAYS(E, W, T) SR_STREAM_SCALED(E, W, T, true)
#define SR_STREAM_MT(E, W, TALLEST)                                                                        \
    (mt32 <= 4 ? SR_STREAM_MT4(E, W, SR_STREAM_LEAN)                                                       \
     : mt32 == 5 ? SR_STREAM_TALL(E, W, 5) : mt32 == 6 ? SR_STREAM_TALL(E, W, 6)                           \
     : mt32 == 7 ? TALLEST(E, W, 7) : TALLEST(E, W, 8))
#define SR_STREAM_W(E)                                                                                     \
    (a.wide == 2 ? SR_STREAM_MT(E, 2, SR_STREAM_PLAIN) : a.wide == 4 ? SR_STREAM_MT(E, 4, SR_STREAM_TALL)  \
     : a.wide == 5 ? SR_STREAM_MT(E, 5, SR_STREAM_TALL)                                                    \
     : a.wide == 8 ? SR_STREAM_MT4(E, 8, SR_STREAM_ALWAYS) : SR_STREAM_MT4(E, 10, SR_STREAM_ALWAYS))
    if (mt32 > 4 && (a.wide >= 8 || scaled)) return SR_E_ARG;
    if (scaled && (a.scale.ld % 4 || a.splits != 1)) return SR_E_ARG;
    if (epi == EPI_F32) SR_STREAM_W(EPI_F32); else SR_STREAM_W(EPI_SWIGLU);
    SR_HIP(attr);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace sr
