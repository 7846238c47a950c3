// Projection GEMMs  Y[M][N] = X[M][K] * W[N][K]^T  on the bf16 matrix cores, for more than 256 rows (up to there the
// weight stream bounds all but small matrices: gemm_stream.hip).  W and X are stored pre-tiled in MFMA operand order.  Three
// kernels, chosen per launch by measured cost (plan_projection in plan.h): 128 x 128 tiles, tiles of 128 to 384 rows x 64 to 256
// features, and all rows of a batch of a few hundred in one workgroup of 160 features.
#include <type_traits>

#include "sr_internal.h"

namespace sr {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kKC = 4;                    // k-steps (of 32) per LDS chunk of X
constexpr int kChunkVec = kKC * 512;      // uint4 per chunk: 8 row tiles x 64 lanes per k-step

// 128 x 128 tiles, two workgroups per CU.  Each wavefront reads its 32 output features as two contiguous runs with
// 16-byte loads per lane straight into registers; X is staged through LDS and shared by the four wavefronts.  grid.y walks
// 128-row blocks; thin matrices are split along K across workgroups (grid.z) and the fp32 partial results are summed, in
// fixed order, by the kernel that consumes them.
//
// Software pipeline per wavefront: a ring of kPF k-steps of W lives in registers; every k-step is
// consumed by 16 MFMAs and its slot is refilled at once with the k-step kPF further on, so 16 KiB of
// weights per wavefront are always in flight.  X chunks (kKC k-steps, 32 KiB) are double buffered
// in LDS: the next chunk is fetched into registers while the current one is being consumed.
// The loop body spans kPF k-steps (two X chunks) and contains no branch: the k extent of X and W is
// padded to a multiple of kPF k-steps with zeros, every split covers whole groups of kPF k-steps,
// prefetches past the end re-read the last valid k-step (never used), and rows of X beyond M are
// computed and never stored.  Without branches the compiler can count outstanding loads exactly,
// so the weight prefetch survives across the workgroup barriers.
template <int EPI>
__global__ __launch_bounds__(kThreads, 2) void gemm_kernel(GemmArgs a) {
    __shared__ u32x4 lds[2][kChunkVec];   // 2 x 32 KiB

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nb = blockIdx.x, mb = blockIdx.y, sp = blockIdx.z;
    int ks0, ks1;                                              // whole groups of kPF k-steps
    split_range(a.ks_total, kPF, a.splits, sp, &ks0, &ks1);
    const int nt0 = nb * 8 + wave * 2;    // first of this wavefront's two 16-feature tiles

    f32x4 acc[8][2];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (ks0 < ks1) {
        const u32x4 *wp0 = (const u32x4 *)a.W + ((size_t)nt0 * a.ks_total) * 64 + lane;
        const u32x4 *wp1 = wp0 + (size_t)a.ks_total * 64;
        // X: thread's r-th vector of a chunk is k-step (tid + 256 r) / 512, position (tid + 256 r) % 512
        const u32x4 *xp = (const u32x4 *)a.X + (size_t)mb * 8 * 64 + tid;
        const size_t x_ks_stride = (size_t)a.mt_total * 64;
        const int last = ks1 - 1;

        u32x4 w0[kPF], w1[kPF], xr[8];
#pragma unroll
        for (int i = 0; i < kPF; ++i) {
            w0[i] = *(wp0 + (size_t)(ks0 + i) * 64);
            w1[i] = *(wp1 + (size_t)(ks0 + i) * 64);
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) xr[r] = xp[(size_t)(ks0 + (r >> 1)) * x_ks_stride + ((r & 1) << 8)];
#pragma unroll
        for (int r = 0; r < 8; ++r) lds[0][tid + kThreads * r] = xr[r];
        __syncthreads();

        for (int ks = ks0; ks < ks1; ks += kPF) {
#pragma unroll
            for (int half = 0; half < kPF / kKC; ++half) {
                const int kc0 = ks + half * kKC;                 // first k-step of the chunk in LDS buffer `half`
#pragma unroll
                for (int r = 0; r < 8; ++r) {                    // next chunk of X (clamped at the end)
                    const int k = min(kc0 + kKC + (r >> 1), last);
                    xr[r] = xp[(size_t)k * x_ks_stride + ((r & 1) << 8)];
                }
                __builtin_amdgcn_sched_barrier(0);
                // X fragments come from LDS one k-step ahead of their MFMAs, the two streams interleaved
                bf16x8 xf[2][8];
#pragma unroll
                for (int mt = 0; mt < 8; ++mt)
                    xf[0][mt] = __builtin_bit_cast(bf16x8, lds[half][mt * 64 + lane]);
#pragma unroll
                for (int kk = 0; kk < kKC; ++kk) {
                    const int i = half * kKC + kk;
                    __builtin_amdgcn_sched_barrier(0);
                    const bf16x8 wa = __builtin_bit_cast(bf16x8, w0[i]);
                    const bf16x8 wb = __builtin_bit_cast(bf16x8, w1[i]);
                    if (kk + 1 < kKC) {
#pragma unroll
                        for (int mt = 0; mt < 8; ++mt)
                            xf[(kk + 1) & 1][mt] = __builtin_bit_cast(bf16x8, lds[half][(kk + 1) * 512 + mt * 64 + lane]);
                    }
#pragma unroll
                    for (int mt = 0; mt < 8; ++mt) {
                        acc[mt][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, xf[kk & 1][mt], acc[mt][0], 0, 0, 0);
                        acc[mt][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb, xf[kk & 1][mt], acc[mt][1], 0, 0, 0);
                    }
                    const int kn = min(kc0 + kk + kPF, last);    // refill the slot just consumed
                    w0[i] = *(wp0 + (size_t)kn * 64);
                    w1[i] = *(wp1 + (size_t)kn * 64);
                    if (kk + 1 < kKC) {
#pragma unroll
                        for (int mt = 0; mt < 8; ++mt) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // 2 MFMA
                            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // 1 LDS read
                        }
                    } else {
                        __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);           // W refills
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < 8; ++r) lds[half ^ 1][tid + kThreads * r] = xr[r];
                __syncthreads();
            }
        }
    }

    // accumulator tile: lane (j = lane%16, g = lane/16) holds output features 4g..4g+3 of batch row j
    const int j = lane & 15, g = lane >> 4;
    if constexpr (EPI == EPI_F32) {
        float *out = (float *)a.out + (size_t)sp * a.split_stride;
#pragma unroll
        for (int mt = 0; mt < 8; ++mt) {
            const int m = mb * 128 + mt * 16 + j;
            if (m < a.M) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int n = (nt0 + t) * 16 + 4 * g;
                    if (n < a.N) *(f32x4 *)(out + (size_t)m * a.ld_out + n) = acc[mt][t];
                }
            }
        }
    } else {
        // tile 0 = gate, tile 1 = up, for features f0..f0+15
        uint16_t *out = (uint16_t *)a.out;
        const int f = (nt0 >> 1) * 16 + 4 * g;
        if (f < a.ld_out) {
#pragma unroll
            for (int mt = 0; mt < 8; ++mt) {
                const int m = mb * 128 + mt * 16 + j;
                if (m < a.M) {
                    float r[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float gt = acc[mt][0][e];
                        r[e] = gt / (1.0f + __expf(-gt)) * acc[mt][1][e];
                    }
                    uint2 v = make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
                    *(uint2 *)(out + frag_offset(m, f, a.mt_total)) = v;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Kernel for more than 256 rows: compute bound, so the tile is sized for the matrix cores.
//
// A workgroup owns 64 * RT rows x 32 * NT features and one split of K (see plan_projection for which).  Eight wavefronts in a
// 2 x 4 arrangement each take 16 * NT features x 16 * RT rows with 16x16x32 MFMAs; both operands reach them
// through LDS, so every byte crosses the vector-memory path once per workgroup.  Each wavefront copies its share of a
// k-step from global memory straight into LDS (direct-to-LDS loads issued from inline assembly and waited for by hand),
// three k-steps ahead through four buffers, with one workgroup barrier per k-step.
//
// The fragments of k-step s + 1 are read from LDS while the MFMAs of k-step s run, into a second register set: the
// barrier that starts k-step s therefore waits for the copies of s + 1, and the reads are spread over the whole k-step
// instead of standing in front of its first MFMA.  With eight wavefronts (two per SIMD) there are 256 registers for
// 4 * RT * NT accumulators and two sets of NT + RT fragments.
//
// MFMAs, LDS reads and copies are issued in the order in which they are written, a copy behind every second of the first MFMAs: a
// copy takes half a dozen scalar instructions, and those of a whole k-step in front of its first MFMA, where both wavefronts of a SIMD
// stand at the same time, kept the matrix pipes idle for 200 to 330 cycles a k-step.  For the same reason addresses are added up, not
// multiplied out, and wavefronts with one copy less have a loop without branches of their own.  Cycles a k-step (of which MFMAs), before ->
// now: {NT, RT} = {7, 4} 1218 -> 970 (896), {6, 4} 1096 -> 847 (768), {5, 4} 936 -> 750 (640), {4, 5} 952 -> 730 (640), {8, 4} 1245 -> 1140
// (1024) in one round of workgroups, 1265 -> 1250 in eight.  The chip answers with a lower clock (1.9 -> 1.65 GHz), so that 8192 rows
// of down take 830 -> 749 us, QKV 222 -> 196, O 165 -> 151; 296 rows of down 45.4 -> 40.7, 512 of gate|up 134 -> 117.  The MFMA is the
// 16x16x32 form: 32x32x16 draws more power for the same product (the loop without copies 1.95 against 1.75 PFLOP/s).
//
// The tiles are numbered split by split, in panels of eight row blocks, column by column, and every XCD takes a contiguous eighth of
// that order: the 32 workgroups that run together on one XCD form an 8 x 4 block of tiles (2048 rows x 128 * NT
// features) whose operands they share through that XCD's L2, and no XCD has more than one tile above its share.
// ---------------------------------------------------------------------------------------------
constexpr int kPfThreads = 512;
constexpr int pf_tiles(int nt, int rt) { return 2 * nt + 4 * rt; }      // 1 KiB tiles per k-step: W, then X
constexpr int pf_lds_bytes(int nt, int rt) { return kPfBufs * pf_tiles(nt, rt) * 1024; }

template <int EPI, int NT, int RT>
__global__ __launch_bounds__(kPfThreads) void gemm_prefill_kernel(GemmArgs a, int m_blocks, int n_blocks, int per_xcd) {
    extern __shared__ u32x4 pf_lds[];      // [kPfBufs][tile][lane]
    constexpr int TILES = pf_tiles(NT, RT), SV = TILES * 64;
    constexpr int COPIES = (TILES + 7) / 8;          // per wavefront and k-step; some wavefronts have one less

    // linear id -> XCD -> place in its share -> split, tile
    int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const int sp = t / (m_blocks * n_blocks);
    if (sp >= a.splits) return;
    t -= sp * m_blocks * n_blocks;
    const int panel = t / (8 * n_blocks), in_panel = t - panel * 8 * n_blocks;
    const int panel_rows = min(8, m_blocks - panel * 8);
    const int nb = in_panel / panel_rows, mb = panel * 8 + in_panel - nb * panel_rows;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, wm = wave >> 1;
    int ks0, ks1;
    split_range(a.ks_total, a.split_steps, a.splits, sp, &ks0, &ks1);
    const int n_stages = ks1 - ks0;

    // copies of one k-step: tiles wave, wave + 8, ...
    const char *src[COPIES];               // of the next k-step to copy
    unsigned step[COPIES];
#pragma unroll
    for (int k = 0; k < COPIES; ++k) {
        const int tile = min(wave + 8 * k, TILES - 1);
        const bool is_w = tile < 2 * NT;
        step[k] = is_w ? 1024u : (unsigned)a.mt_total * 1024u;
        src[k] = (is_w ? (const char *)a.W + (size_t)(nb * 2 * NT + tile) * a.ks_total * 1024
                       : (const char *)a.X + (size_t)(mb * 4 * RT + tile - 2 * NT) * 1024) + (size_t)ks0 * step[k];
    }
    const unsigned voff = lane * 16;
    const unsigned lds0 =
        __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) void *)pf_lds) + wave * 1024;
    // more: there is a k-step behind this one; else the next copy reads the last one again, and nothing consumes it
    auto copy = [&](int k, int buf, bool more) __attribute__((always_inline)) {
        lds_dma16_uniform(src[k], voff, lds0 + (unsigned)(buf * SV * 16 + k * 8 * 1024));
        src[k] += more ? step[k] : 0u;
    };

    f32x4 up[RT];                           // see the SwiGLU epilogue
    f32x4 acc[NT][RT];                      // [feature tile][row tile]: lane (c, g) holds features 4g .. 4g+3 of row c
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int woff = wn * NT * 64 + lane, xoff = (2 * NT + wm * RT) * 64 + lane;
    bf16x8 wf[2][NT], xf[2][RT];           // [k-step parity]
    auto read_frag = [&](int f, int set, int buf) __attribute__((always_inline)) {
        const u32x4 *base = pf_lds + buf * SV;
        if (f < RT) xf[set][f] = __builtin_bit_cast(bf16x8, base[xoff + f * 64]);
        else wf[set][f - RT] = __builtin_bit_cast(bf16x8, base[woff + (f - RT) * 64]);
    };

    // C: this wavefront's copies per k-step
    auto run = [&](auto copies) __attribute__((always_inline)) {
        constexpr int C = decltype(copies)::value;
        // all LDS reads of this wavefront are done and at most `stages` k-steps of its copies are still on their way; then the
        // barrier
        auto wait_and_meet = [&](auto stages) __attribute__((always_inline)) {
            constexpr int S = decltype(stages)::value;
            static_assert(C * S < 16, "the count's low four bits");
            __builtin_amdgcn_s_waitcnt(0x0070 | (C * S));
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
#pragma unroll
        for (int i = 0; i < kPfBufs; ++i)
#pragma unroll
            for (int k = 0; k < C; ++k) copy(k, i, i + 1 < n_stages);
        wait_and_meet(std::integral_constant<int, 3>{});
#pragma unroll
        for (int f = 0; f < NT + RT; ++f) read_frag(f, 0, 0);
        for (int s0 = 0; s0 < n_stages; s0 += kPfBufs) {          // a split is a multiple of four k-steps
#pragma unroll
            for (int q = 0; q < kPfBufs; ++q) {
                const int s = s0 + q, set = q & 1;
                wait_and_meet(std::integral_constant<int, 2>{});      // k-step s + 1 has landed; k-step s is in everybody's registers
                const bool more = s + kPfBufs + 1 < n_stages;
                constexpr int MFMAS = RT * NT, READS = NT + RT, PER = MFMAS >= 2 * READS ? 2 : 1;    // MFMAs per LDS read
                static_assert(MFMAS >= PER * READS && MFMAS >= 2 * C, "everything fits between the MFMAs");
#pragma unroll
                for (int m = 0; m < MFMAS; ++m) {
                    const int i = m / RT, j = m % RT;
                    __builtin_amdgcn_sched_barrier(0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[set][i], xf[set][j], acc[i][j], 0, 0, 0);
                    if (m % PER == PER - 1 && m / PER < READS) read_frag(m / PER, set ^ 1, (q + 1) % kPfBufs);
                    __builtin_amdgcn_sched_barrier(0);
                    if (m % 2 && m / 2 < C) copy(m / 2, q, more);         // into the buffer of k-step s
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if (TILES % 8 == 0 || wave + 8 * (COPIES - 1) < TILES) run(std::integral_constant<int, COPIES>{});
    else run(std::integral_constant<int, COPIES - 1>{});
    __builtin_amdgcn_s_waitcnt(0x0070);              // the copies past the end have landed before LDS goes away

    const int c = lane & 15, g = lane >> 4;
    if constexpr (EPI == EPI_F32) {
        float *out = (float *)a.out + (size_t)sp * a.split_stride;
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            const int m = (mb * 4 * RT + wm * RT + j) * 16 + c;
            if (m < a.M) {
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    const int n = (nb * 2 * NT + wn * NT + i) * 16 + 4 * g;
                    if (n < a.N) *(f32x4 *)(out + (size_t)m * a.ld_out + n) = acc[i][j];
                }
            }
        }
    } else if constexpr (EPI == EPI_LSE) {
        // a wavefront's 128 columns of a row lie in four lanes.  The exponentials are the hardware's base-2 exponential in fp32 as it
        // is: arguments <= 0, results below 2^-126 of the row's maximum may flush to zero, which no sum near 1 or above sees (the
        // error against 64 bits is the stored logits': 0.00101 both at 152 064 columns).
        const ScoreOut &so = a.score;
        const int n0 = (nb * 2 * NT + wn * NT) * 16 + 4 * g;         // + 16 i + e
        auto value = [&](int i, int e, int j) { return n0 + 16 * i < a.N ? acc[i][j][e] : -3.0e38f; };      // N is a multiple of 16
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            const int m = (mb * 4 * RT + wm * RT + j) * 16 + c;
            float mx = -3.0e38f, sum = 0.f;
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) mx = fmaxf(mx, value(i, e, j));
            mx = row_max(mx);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    sum += n0 + 16 * i < a.N ? __builtin_amdgcn_exp2f((acc[i][j][e] - mx) * 1.4426950408889634f) : 0.f;
            sum = row_sum(sum);
            if (m >= a.M) continue;
            if (g == 0) so.lse[(size_t)(nb * 2 + wn) * so.lse_ld + m] = make_float2(mx, sum);
            const int at = so.target[m] - n0;
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (at == 16 * i + e) so.target_logit[m] = acc[i][j][e];
            if (so.last && m % so.rows_per_unit == so.rows_per_unit - 1) {
                float *dst = so.last + (size_t)(m / so.rows_per_unit) * a.N + n0;
#pragma unroll
                for (int i = 0; i < NT; ++i)
                    if (n0 + 16 * i < a.N) *(f32x4 *)(dst + 16 * i) = acc[i][j];
            }
        }
    } else {
        // Packed tiles alternate gate and up.  With an odd NT the middle pair's gate is the last tile of the first wavefront column
        // and its up the first of the second, which hands it over through LDS.
        constexpr bool ODD = NT % 2 != 0;
        if constexpr (ODD) {
            __syncthreads();                         // nobody reads fragments any more
            f32x4 *mid = (f32x4 *)pf_lds;            // [row tile][lane]
            if (wn == 1) {
#pragma unroll
                for (int j = 0; j < RT; ++j) mid[(wm * RT + j) * 64 + lane] = acc[0][j];
            }
            __syncthreads();
            if (wn == 0) {
#pragma unroll
                for (int j = 0; j < RT; ++j) up[j] = mid[(wm * RT + j) * 64 + lane];
            }
        }
        uint16_t *out = (uint16_t *)a.out;
        auto store = [&](int m, int f, const f32x4 &gate, const f32x4 &up4) __attribute__((always_inline)) {   // features f .. f + 3
            if (f < a.ld_out) {
                float r[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) r[e] = gate[e] / (1.0f + __expf(-gate[e])) * up4[e];
                *(uint2 *)(out + frag_offset(m, f, a.mt_total)) = make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
            }
        };
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            const int m = (mb * 4 * RT + wm * RT + j) * 16 + c;
            if (m >= a.M) continue;
            if constexpr (ODD) {
                const int f0 = nb * NT * 16 + 4 * g;             // features of the workgroup's first pair
                if (wn == 0) {
#pragma unroll
                    for (int i = 0; i < NT / 2; ++i) store(m, f0 + i * 16, acc[2 * i][j], acc[2 * i + 1][j]);
                    store(m, f0 + NT / 2 * 16, acc[NT - 1][j], up[j]);
                } else {
#pragma unroll
                    for (int i = 0; i < NT / 2; ++i)
                        store(m, f0 + (NT / 2 + 1 + i) * 16, acc[2 * i + 1][j], acc[2 * i + 2][j]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < NT / 2; ++i) store(m, (nb * NT + wn * (NT / 2) + i) * 16 + 4 * g, acc[2 * i][j], acc[2 * i + 1][j]);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Batches of 321 to 512 rows against a wide matrix (more than 32 784 rows) of less than 3072 inputs; with more inputs tiles of
// 160 to 256 features and 192 to 320 rows are faster (plan_projection: gate|up of the 7B shape at 512 rows 117 us, a round of this
// kernel 139).  Neither a weight stream (the matrix pipe, not HBM, bounds 512 rows) nor a large tiled GEMM (two row blocks of 256 leave
// 1.16 rounds of tiles and fetch every weight from HBM with only two workgroups sharing it).  One workgroup takes ALL rows (up
// to 512) of 160 packed features, so every weight byte is fetched from HBM exactly once and 37 888 packed
// gate|up rows break into 237 workgroups, one round.  Eight wavefronts, each 64 rows x 160 features
// (2 x 5 accumulator tiles of 32 x 32 = 160 registers; seven LDS fragment reads per ten MFMAs).  Both operands go
// global -> LDS with direct-to-LDS loads, one barrier per k-step: X (32 KiB per k-step, L2 resident) two k-steps
// ahead through three buffers, W (10 KiB per k-step, from HBM) five k-steps ahead through six;
// each wavefront copies the X rows it consumes itself and its share of the ten W tiles.  The copies are issued
// from inline assembly: the compiler's wait-count pass then neither sees them nor waits for them before the LDS
// reads, and the wait for the stage that is needed is placed by hand (vector-memory operations of a wavefront
// retire in order, so "all but the newer stage's copies" is a count).
// ---------------------------------------------------------------------------------------------
constexpr int kMidThreads = 512;
constexpr int kMidWTiles = 10;                                     // 160 packed features
constexpr int kMidXTiles = 32;                                     // 512 rows
constexpr int kMidXBufs = 3, kMidWBufs = 6;                        // k-steps of X (from L2) and of W (from HBM) in LDS
constexpr int kMidXVec = kMidXTiles * 64, kMidWVec = kMidWTiles * 64;       // u32x4 per k-step: 32 KiB and 10 KiB
constexpr int kMidLdsBytes = (kMidXBufs * kMidXVec + kMidWBufs * kMidWVec) * 16;   // 156 KiB

// wait until at most n of this wavefront's vector-memory operations are outstanding (n uniform, 0..8) and its LDS reads are
// back: the buffers they came from are overwritten behind the barrier that follows
__device__ __forceinline__ void wait_vm_at_most(int n) {
    switch (n) {
        case 0: __builtin_amdgcn_s_waitcnt(0x0070); break;
        case 1: __builtin_amdgcn_s_waitcnt(0x0071); break;
        case 2: __builtin_amdgcn_s_waitcnt(0x0072); break;
        case 3: __builtin_amdgcn_s_waitcnt(0x0073); break;
        case 4: __builtin_amdgcn_s_waitcnt(0x0074); break;
        case 5: __builtin_amdgcn_s_waitcnt(0x0075); break;
        case 6: __builtin_amdgcn_s_waitcnt(0x0076); break;
        case 7: __builtin_amdgcn_s_waitcnt(0x0077); break;
        default: __builtin_amdgcn_s_waitcnt(0x0078); break;
    }
}

__global__ __launch_bounds__(kMidThreads) void gemm_mid_kernel(GemmArgs a) {
    extern __shared__ u32x4 mid_lds[];      // X ring [kMidXBufs][32 tiles x 64], then W ring [kMidWBufs][10 tiles x 64]

    const int nb = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool active = wave * 64 < a.M;               // this wavefront's 64 rows hold valid rows
    const int n_stages = a.ks_total;

    // copies of one k-step: this wavefront's four X tiles (if it has rows) and W tiles wave, wave + 8
    const int n_w = wave + 8 < kMidWTiles ? 2 : 1;
    const u32x4 *xsrc = (const u32x4 *)a.X + (size_t)(wave * 4) * 64 + lane;                       // + ks * mt_total * 64
    const u32x4 *wsrc = (const u32x4 *)a.W + ((size_t)(nb * kMidWTiles + wave) * a.ks_total) * 64 + lane;   // + ks * 64
    const unsigned lds_x = (unsigned)(size_t)(__attribute__((address_space(3))) void *)mid_lds;
    const unsigned lds_w = lds_x + (unsigned)(kMidXBufs * kMidXVec) * 16;
    auto copy_x = [&](int st) {             // past the end: a harmless re-read of the last k-step, never consumed
        if (!active) return;
        const int ks = min(st, n_stages - 1);
        const unsigned base = lds_x + (unsigned)((st % kMidXBufs) * kMidXVec + wave * 4 * 64) * 16;
#pragma unroll
        for (int t = 0; t < 4; ++t) lds_dma16(xsrc + ((size_t)ks * a.mt_total + t) * 64, base + (unsigned)(t * 64) * 16);
    };
    auto copy_w = [&](int st) {
        const int ks = min(st, n_stages - 1);
        const unsigned base = lds_w + (unsigned)((st % kMidWBufs) * kMidWVec + wave * 64) * 16;
        lds_dma16(wsrc + (size_t)ks * 64, base);
        if (n_w == 2) lds_dma16(wsrc + ((size_t)8 * a.ks_total + ks) * 64, base + (unsigned)(8 * 64) * 16);
    };

    f32x16 acc[5][2];                        // [feature group of 32][row group of 32]
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int r32 = lane & 31, g2 = lane >> 5;
    const int sub = r32 >> 4, slot0 = (r32 & 15) + 16 * g2;
    const int woff = kMidXBufs * kMidXVec + sub * 64 + slot0;              // + W buffer + i * 128 + h * 32
    const int xoff = (wave * 4 + sub) * 64 + slot0;                        // + X buffer + j * 128 + h * 32

    // Vector-memory operations of a wavefront retire in order.  Every iteration issues X of k-step s + 2, then W of
    // k-step s + 5; the prologue issues the same pattern for the two iterations before the first, behind W 0..2.
    // So when iteration s begins, what was issued after X(s) is W(s+3), X(s+1), W(s+4), and W(s) is older than X(s).
    copy_w(0); copy_w(1); copy_w(2);
    copy_x(0); copy_w(3);
    copy_x(1); copy_w(4);
    const int n_newer = (active ? 4 : 0) + 2 * n_w;
    int bx = 0, bw = 0;
    for (int s = 0; s < n_stages; ++s) {
        wait_vm_at_most(n_newer);            // X(s) and W(s) have landed
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();        // ... for every wavefront, and nobody reads k-step s - 1 any more
        asm volatile("" ::: "memory");
        copy_x(s + 2);                       // into the buffers k-step s - 1 used
        copy_w(s + 5);
        const u32x4 *xb = mid_lds + bx * kMidXVec, *wb = mid_lds + bw * kMidWVec;
        bx = bx == kMidXBufs - 1 ? 0 : bx + 1;
        bw = bw == kMidWBufs - 1 ? 0 : bw + 1;
        if (active) {
            bf16x8 wf[2][5], xf[2][2];       // [k-half parity][group]
#pragma unroll
            for (int i = 0; i < 5; ++i) wf[0][i] = __builtin_bit_cast(bf16x8, wb[woff + i * 128]);
#pragma unroll
            for (int j = 0; j < 2; ++j) xf[0][j] = __builtin_bit_cast(bf16x8, xb[xoff + j * 128]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 5; ++i) wf[1][i] = __builtin_bit_cast(bf16x8, wb[woff + i * 128 + 32]);
#pragma unroll
            for (int j = 0; j < 2; ++j) xf[1][j] = __builtin_bit_cast(bf16x8, xb[xoff + j * 128 + 32]);
#pragma unroll
            for (int i = 0; i < 5; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[0][i], xf[0][j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int f = 0; f < 7; ++f) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // 1 LDS read
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
#pragma unroll
            for (int i = 0; i < 5; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[1][i], xf[1][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);      // the copies past the end have landed before LDS goes away
    if (!active) return;

    // accumulator (i, j): lane (r32 = row within the 32-row group, g2) holds, in register v,
    // feature 8 * (v / 4) + 4 * g2 + v % 4 of the 32-feature group: 16 gate, then 16 up features
    uint16_t *out = (uint16_t *)a.out;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int m = wave * 64 + j * 32 + r32;
        if (m < a.M) {
#pragma unroll
            for (int i = 0; i < 5; ++i)
#pragma unroll
                for (int vq = 0; vq < 2; ++vq) {
                    const int f = nb * 80 + i * 16 + 8 * vq + 4 * g2;
                    if (f < a.ld_out) {
                        float r[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float gt = acc[i][j][4 * vq + e];
                            r[e] = gt / (1.0f + __expf(-gt)) * acc[i][j][4 * (vq + 2) + e];
                        }
                        uint2 v = make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
                        *(uint2 *)(out + frag_offset(m, f, a.mt_total)) = v;
                    }
                }
        }
    }
}

// The same kernel for 257 .. 384 rows on 16x16x32 MFMAs: with 64-row slabs five (or six) of the eight wavefronts
// would have rows, two of them on one SIMD, and that SIMD would carry 128 rows.  Here the 16-row tiles are dealt
// out round robin, wavefront w owning tiles w, w + 8, w + 16 (at most three), so 19 tiles (304 rows) put 5, 5, 5
// and 4 on the four SIMDs.  A 16-row fragment-major tile is one MFMA operand as it lies in LDS (one 16-byte read per
// lane): 10 W + up to 3 X reads for up to 30 MFMAs per k-step.  Copies, rings, barrier and wait counts as above.
template <int EPI>
__global__ __launch_bounds__(kMidThreads) void gemm_mid16_kernel(GemmArgs a) {
    constexpr int RT = 3;
    extern __shared__ u32x4 mid_lds[];

    const int nb = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_tiles = (a.M + 15) >> 4;
    const int my_tiles = wave < n_tiles ? min(RT, (n_tiles - wave + 7) >> 3) : 0;     // tiles wave, wave + 8, ...
    const int n_stages = a.ks_total;

    const int n_w = wave + 8 < kMidWTiles ? 2 : 1;
    const u32x4 *xsrc = (const u32x4 *)a.X + (size_t)wave * 64 + lane;                             // + (ks * mt_total + 8 t) * 64
    const u32x4 *wsrc = (const u32x4 *)a.W + ((size_t)(nb * kMidWTiles + wave) * a.ks_total) * 64 + lane;
    const unsigned lds_x = (unsigned)(size_t)(__attribute__((address_space(3))) void *)mid_lds;
    const unsigned lds_w = lds_x + (unsigned)(kMidXBufs * kMidXVec) * 16;
    auto copy_x = [&](int st) {
        const int ks = min(st, n_stages - 1);
        const unsigned base = lds_x + (unsigned)((st % kMidXBufs) * kMidXVec + wave * 64) * 16;
#pragma unroll
        for (int t = 0; t < RT; ++t)
            if (t < my_tiles) lds_dma16(xsrc + ((size_t)ks * a.mt_total + 8 * t) * 64, base + (unsigned)(8 * t * 64) * 16);
    };
    auto copy_w = [&](int st) {
        const int ks = min(st, n_stages - 1);
        const unsigned base = lds_w + (unsigned)((st % kMidWBufs) * kMidWVec + wave * 64) * 16;
        lds_dma16(wsrc + (size_t)ks * 64, base);
        if (n_w == 2) lds_dma16(wsrc + ((size_t)8 * a.ks_total + ks) * 64, base + (unsigned)(8 * 64) * 16);
    };

    f32x4 acc[kMidWTiles][RT];               // [feature tile of 16][row tile]: lane (c, g) holds features 4g..4g+3 of row c
#pragma unroll
    for (int i = 0; i < kMidWTiles; ++i)
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int woff = kMidXBufs * kMidXVec + lane;                          // + W buffer + i * 64
    const int xoff = wave * 64 + lane;                                     // + X buffer + t * 512

    copy_w(0); copy_w(1); copy_w(2);
    copy_x(0); copy_w(3);
    copy_x(1); copy_w(4);
    const int n_newer = my_tiles + 2 * n_w;  // issued after X(s): W(s+3), X(s+1), W(s+4)
    int bx = 0, bw = 0;
    for (int s = 0; s < n_stages; ++s) {
        wait_vm_at_most(n_newer);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        copy_x(s + 2);
        copy_w(s + 5);
        const u32x4 *xb = mid_lds + bx * kMidXVec, *wb = mid_lds + bw * kMidWVec;
        bx = bx == kMidXBufs - 1 ? 0 : bx + 1;
        bw = bw == kMidWBufs - 1 ? 0 : bw + 1;
        if (my_tiles > 0) {
            // tiles 0 and 1 unconditionally (a wavefront with one tile computes it twice and stores it once), tile 2
            // where it exists: one uniform branch per k-step
            bf16x8 xf[RT], wf[kMidWTiles];
            xf[0] = __builtin_bit_cast(bf16x8, xb[xoff]);
            xf[1] = __builtin_bit_cast(bf16x8, xb[xoff + (my_tiles > 1 ? 512 : 0)]);
#pragma unroll
            for (int i = 0; i < kMidWTiles; ++i) wf[i] = __builtin_bit_cast(bf16x8, wb[woff + i * 64]);
            if (my_tiles == 3) xf[2] = __builtin_bit_cast(bf16x8, xb[xoff + 1024]);
#pragma unroll
            for (int i = 0; i < kMidWTiles; ++i)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i], xf[t], acc[i][t], 0, 0, 0);
            if (my_tiles == 3) {
#pragma unroll
                for (int i = 0; i < kMidWTiles; ++i)
                    acc[i][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i], xf[2], acc[i][2], 0, 0, 0);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    if (my_tiles == 0) return;

    const int c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int m = (wave + 8 * t) * 16 + c;
        if (t >= my_tiles || m >= a.M) continue;
        if constexpr (EPI == EPI_F32) {
            float *out = (float *)a.out + (size_t)m * a.ld_out;
#pragma unroll
            for (int i = 0; i < kMidWTiles; ++i) {
                const int n = nb * 160 + i * 16 + 4 * g;
                if (n < a.N) *(f32x4 *)(out + n) = acc[i][t];
            }
        } else {
            uint16_t *out = (uint16_t *)a.out;
#pragma unroll
            for (int i = 0; i < kMidWTiles / 2; ++i) {      // tile 2i = gate, tile 2i + 1 = up of features f..f+15
                const int f = nb * 80 + i * 16 + 4 * g;
                if (f < a.ld_out) {
                    float r[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float gt = acc[2 * i][t][e];
                        r[e] = gt / (1.0f + __expf(-gt)) * acc[2 * i + 1][t][e];
                    }
                    *(uint2 *)(out + frag_offset(m, f, a.mt_total)) =
                        make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
                }
            }
        }
    }
}

// One wavefront per 16-row tile and kPackSteps k-steps: a lane holds one 16-byte slot of the packed tile, so the writes are
// whole 1 KiB runs, and the reads use each row's lines up within the wavefront.  Bound: HBM (read once, written once).
// 1.05 GB of weights took 1.28 ms with a thread per slot in source order (16-byte writes 256 bytes apart), 0.47 now.
constexpr int kPackSteps = 8;
template <bool ALIGNED>                    // the source pointer is a multiple of 16 bytes
__global__ __launch_bounds__(256) void pack_rows_kernel(const uint16_t *__restrict__ src, int n_rows, int K,
                                                        uint16_t *__restrict__ dst, int ks_total, int dst_row0,
                                                        int interleave16, int which, int half_tiles) {
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = tile * 16 + (lane & 15), kg = lane >> 4;
    if (i >= n_rows) return;
    size_t ptile = interleave16 ? 2 * tile + which : (dst_row0 >> 4) + tile;
    if (half_tiles) {                                    // tiles of a head's low half, then of its high half -> in turn
        const int u = tile % (2 * half_tiles);
        ptile += (u < half_tiles ? 2 * u : 2 * (u - half_tiles) + 1) - u;
    }
    const int ks0 = blockIdx.y * kPackSteps;
    const uint16_t *row = src + (size_t)i * K;
    uint4 v[kPackSteps];
#pragma unroll
    for (int u = 0; u < kPackSteps; ++u) {
        const int k0 = (ks0 + u) * 32 + kg * 8;          // K is a multiple of 8: a slot is inside the row or all padding
        v[u] = make_uint4(0, 0, 0, 0);
        if (k0 < K) {
            if constexpr (ALIGNED) {
                v[u] = *(const uint4 *)(row + k0);
            } else {
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = (uint32_t)row[k0 + 2 * e] | ((uint32_t)row[k0 + 2 * e + 1] << 16);
                v[u] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
    uint4 *d = (uint4 *)dst + (ptile * ks_total + ks0) * 64 + lane;
#pragma unroll
    for (int u = 0; u < kPackSteps; ++u)
        if (ks0 + u < ks_total) d[u * 64] = v[u];
}

}  // namespace

int launch_pack_rows(const uint16_t *src, int n_rows, int K, uint16_t *dst, int ks_total, int dst_row0,
                     int interleave16, int which, int head_dim, hipStream_t stream) {
    if (n_rows <= 0 || ks_total <= 0) return SR_OK;
    if (K % 8 || dst_row0 % 16 || (head_dim && (head_dim % 32 || n_rows % head_dim))) return SR_E_ARG;
    const dim3 grid(ceil_div(ceil_div(n_rows, 16), 4), ceil_div(ks_total, kPackSteps)), block(256);
    if (((uintptr_t)src & 15) == 0)
        pack_rows_kernel<true><<<grid, block, 0, stream>>>(src, n_rows, K, dst, ks_total, dst_row0, interleave16, which, head_dim / 32);
    else
        pack_rows_kernel<false><<<grid, block, 0, stream>>>(src, n_rows, K, dst, ks_total, dst_row0, interleave16, which, head_dim / 32);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

namespace {

// Tiles of 64 * RT rows x 32 * NT features over all of `a`
template <int EPI, int NT, int RT>
int launch_tiles(const GemmArgs &a, hipStream_t stream) {
    SR_HIP(hipFuncSetAttribute((const void *)gemm_prefill_kernel<EPI, NT, RT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               pf_lds_bytes(NT, RT)));
    const int mb = ceil_div(a.M, 64 * RT), nb = ceil_div(a.N, 32 * NT), per_xcd = ceil_div(mb * nb * a.splits, 8);
    if (mb * 4 * RT > a.mt_total || (a.split_steps != kPfBufs && a.split_steps != kPF) || a.splits > a.ks_total / a.split_steps ||
        (EPI != EPI_F32 && a.splits != 1))
        return SR_E_ARG;
    gemm_prefill_kernel<EPI, NT, RT><<<dim3((unsigned)(per_xcd * 8)), dim3(kPfThreads), pf_lds_bytes(NT, RT), stream>>>(a, mb, nb, per_xcd);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

// 128 x 128 tiles over all of `a`
int launch_tiles128(const GemmArgs &a, GemmEpilogue epi, hipStream_t stream) {
    dim3 grid(ceil_div(a.N, 128), ceil_div(a.M, 128), epi == EPI_F32 ? a.splits : 1), block(kThreads);
    if (epi == EPI_F32) gemm_kernel<EPI_F32><<<grid, block, 0, stream>>>(a);
    else gemm_kernel<EPI_SWIGLU><<<grid, block, 0, stream>>>(a);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

// All rows (at most 512) of 160 packed features per workgroup; no K split.  The last workgroup reads whole tiles
// past N: the packed matrix is allocated (and zero) up to a multiple of 160 rows.
int launch_mid(const GemmArgs &a, GemmEpilogue epi, hipStream_t stream) {
    static bool attr_set = false;
    if (!attr_set) {
        SR_HIP(hipFuncSetAttribute((const void *)gemm_mid_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMidLdsBytes));
        SR_HIP(hipFuncSetAttribute((const void *)gemm_mid16_kernel<EPI_F32>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   kMidLdsBytes));
        SR_HIP(hipFuncSetAttribute((const void *)gemm_mid16_kernel<EPI_SWIGLU>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   kMidLdsBytes));
        attr_set = true;
    }
    if (a.M > (epi == EPI_SWIGLU ? 512 : 384) || a.splits != 1 || a.ks_total < 1 || round_up(a.M, 64) > a.mt_total * 16)
        return SR_E_ARG;
    dim3 grid((unsigned)ceil_div(a.N, 160)), block(kMidThreads);
    if (a.M > 256 && a.M <= 384) {           // 17 .. 24 row tiles: three per wavefront, dealt out round robin
        if (epi == EPI_F32) gemm_mid16_kernel<EPI_F32><<<grid, block, kMidLdsBytes, stream>>>(a);
        else gemm_mid16_kernel<EPI_SWIGLU><<<grid, block, kMidLdsBytes, stream>>>(a);
    } else gemm_mid_kernel<<<grid, block, kMidLdsBytes, stream>>>(a);
    SR_HIP(hipGetLastError());
    return SR_OK;
}

}  // namespace

int launch_gemm(const GemmArgs &a, GemmEpilogue epi, hipStream_t stream) {
    if (a.M <= 0) return SR_OK;
    const int m_blocks = ceil_div(a.M, 128);
    if (m_blocks * 8 > a.mt_total || a.splits < 1 || m_blocks > 65535 || a.splits > 65535 || a.ks_total % kPF)
        return SR_E_ARG;
    if (a.wide) return launch_gemm_stream(a, epi, stream);
    if (a.scale.squares) return SR_E_ARG;
    if (epi == EPI_LSE) return launch_tiles<EPI_LSE, 8, 4>(a, stream);
    if (epi == EPI_SWIGLU && a.splits != 1) return SR_E_ARG;
    int nt = a.nt, rt = a.rt;
    if (!nt) {
        const GemmPlan plan = plan_gemm(a.M, a.N, a.ks_total, a.mt_total, epi == EPI_SWIGLU, a.splits, a.splits);
        if (plan.kernel == KERNEL_128) return launch_tiles128(a, epi, stream);
        if (plan.kernel == KERNEL_MID) return launch_mid(a, epi, stream);
        nt = kTileShapes[plan.kernel].nt;
        rt = kTileShapes[plan.kernel].rt;
    }
#define SR_TILE_F32(NT, RT) if (epi == EPI_F32 && nt == NT && rt == RT) return launch_tiles<EPI_F32, NT, RT>(a, stream);
#define SR_TILE_SWIGLU(NT, RT) if (epi == EPI_SWIGLU && nt == NT && rt == RT) return launch_tiles<EPI_SWIGLU, NT, RT>(a, stream);
    SR_TILE_SWIGLU(8, 4) SR_TILE_SWIGLU(7, 4) SR_TILE_SWIGLU(6, 4) SR_TILE_SWIGLU(5, 4) SR_TILE_SWIGLU(6, 5) SR_TILE_SWIGLU(5, 5)
    SR_TILE_SWIGLU(8, 3) SR_TILE_SWIGLU(7, 3) SR_TILE_SWIGLU(5, 3)
    SR_TILE_F32(8, 4) SR_TILE_F32(7, 4) SR_TILE_F32(6, 4) SR_TILE_F32(5, 4) SR_TILE_F32(4, 4) SR_TILE_F32(3, 4) SR_TILE_F32(2, 4)
    SR_TILE_F32(6, 5) SR_TILE_F32(5, 5) SR_TILE_F32(4, 5) SR_TILE_F32(3, 5) SR_TILE_F32(2, 5) SR_TILE_F32(4, 6)
    SR_TILE_F32(7, 3) SR_TILE_F32(5, 3) SR_TILE_F32(4, 3) SR_TILE_F32(3, 3)
    SR_TILE_F32(8, 2) SR_TILE_F32(7, 2) SR_TILE_F32(6, 2) SR_TILE_F32(5, 2) SR_TILE_F32(4, 2)
    return SR_E_ARG;
}

}  // namespace sr
