// Host-side rules that decide how work is laid out over the chip, in plain C++ so that they can be evaluated (and tested)
// without a GPU or the HIP headers; kernels use the parts marked SR_HD.
#pragma once
#include <cmath>
#include <initializer_list>
#include <vector>

#ifdef __HIPCC__
#define SR_HD __host__ __device__
#else
#define SR_HD
#endif

namespace sr {

SR_HD inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
SR_HD inline int round_up(int a, int b) { return ceil_div(a, b) * b; }

// n / d for 0 <= n < 2^31 by a multiplication: mul = ceil(2^shift / d) with shift = 31 + ceil(log2 d), so that mul exceeds
// 2^shift / d by less than 2^(shift - 31) / d.  A division by a number that only the launch knows takes the scalar unit about
// 35 dependent instructions, and the kernels of a decode step began with up to twelve of them.
struct FastDiv { unsigned mul, shift; };
inline FastDiv fast_div(int d) {
    unsigned s = 31;
    while ((1ull << (s - 31)) < (unsigned long long)d) ++s;
    return FastDiv{(unsigned)(((1ull << s) + d - 1) / d), s};
}
SR_HD inline int quotient(int n, FastDiv f) { return (int)(((unsigned long long)(unsigned)n * f.mul) >> f.shift); }

// Attention whose query tiles share K/V blocks: workgroup `wg` -> set (unit, kv head, split) and which of the set's `per_set`
// workgroups.  Consecutive workgroups go to consecutive XCDs.  Of every eight sets each goes to one XCD, whose L2 then
// serves the set's workgroups; the last n_sets % 8 sets are dealt out over all XCDs, because whole sets would leave
// XCDs idle (one group's prompt of 5000 tokens and two kv heads of 128: 549 us on two XCDs, 202 on eight).
SR_HD inline void shared_tiles_of(int wg, int n_sets, int per_set, FastDiv by_set, int *set, int *part) {
    const int rest0 = (n_sets & ~7) * per_set, t = wg - rest0, n = t < 0 ? wg >> 3 : t, q = quotient(n, by_set);
    *set = t < 0 ? q * 8 + (wg & 7) : (n_sets & ~7) + q;
    *part = n - q * per_set;
}
inline void shared_tiles_of(int wg, int n_sets, int per_set, int *set, int *part) {
    shared_tiles_of(wg, n_sets, per_set, fast_div(per_set), set, part);
}

// ---------------------------------------------------------------------------------------------
// projections
// ---------------------------------------------------------------------------------------------
// k-steps [*k0, *k1) of split sp when `units` groups of `unit` k-steps are dealt out evenly
SR_HD inline void split_range(int ks_total, int unit, int splits, int sp, int *k0, int *k1) {
    const int units = ks_total / unit, q = units / splits, r = units % splits;
    const int u0 = sp * q + (sp < r ? sp : r);
    *k0 = u0 * unit;
    *k1 = (u0 + q + (sp < r ? 1 : 0)) * unit;
}

constexpr int kMaxSplitK = 16;
// k-steps that a kernel's splits cover a multiple of: kPfBufs (its LDS buffers) where tiles of 32 nt features x 64 rt rows run, kPF
// (the k-steps of W it holds in registers) in the other kernels
constexpr int kPfBufs = 4, kPF = 8;
// k-steps of 32 that hold K, the projections' inner dimension, padded with zeros to whole groups of kPF, which is what every kernel
// consumes at a time.  (Padded to twice that, the model with hidden size 256 multiplied as many zeros as weights.)
inline int padded_k_steps(int K) { return round_up(ceil_div(K, 32), kPF); }

// Projections of up to kStreamRows rows go to the weight-streaming kernel, except that above kStreamThinRows rows small
// matrices (up to 8192 rows and 16 MB) stay on the tiled kernels: with seven or eight row tiles a k-step of the streaming
// kernel costs more than one of 128 x 128 tiles, and there is little weight to stream (256 rows, K = 1024: QKV 16.5 against
// 15.1 us, O 15.5 against 14.1, gate|up 17.1 against 14.2; at 192 rows they are even, at 160 streaming is 10 % faster).
// Larger matrices stream: at K = 3584 the whole decode step of 224 rows takes 255 us, 267 with tiles for its thin ones.
constexpr int kStreamRows = 256, kStreamThinRows = 192;
inline bool small_matrix(int N, int ks_total) { return N <= 8192 && (long long)N * ks_total * 64 <= 16 << 20; }
// The number of computing wavefronts per workgroup (32 features each) is picked so that the matrix breaks into about 256
// workgroups; 0 = a tiled kernel.
inline int stream_waves(int M, int N, int ks_total, bool swiglu) {
    if (M > kStreamRows || (M > kStreamThinRows && small_matrix(N, ks_total))) return 0;
    // Thin (QKV, O, down): split along K so that about one workgroup per CU is in flight -- more than that only adds
    // partial-sum traffic.  Shallow ones take two computing wavefronts, which gives enough workgroups with three or four K
    // splits instead of seven: the projection itself takes the same time (13.9 against 13.0 us, 11.4 against 11.8 us at
    // the 7B shape) and the kernel that adds the partial sums reads half as many.
    if (!swiglu && N < 8192) return ks_total < 256 ? 2 : 4;
    // Otherwise: the width w with the cheapest rounds of workgroups on 256 CUs, the widest of equals.  A round costs w and a
    // part that does not depend on it, which grows with the rows (the activations' way through LDS): 0.5 up to 32 rows, 1 up
    // to 64, 4 beyond, in halves below; at K = 3584 a round of w = 2, 4, 5, 8, 10 takes 22, 40, 49, 77, 96 us at 8 rows and 34,
    // 49, 60, 89, 109 at 128.  gate|up at the 7B shape (37 888 packed rows): 237 workgroups of 160 features; LM head (152 064):
    // 476 of 320 in two rounds (594 of 256 in three: 246 against 226 us); 49 152 rows at 128: 192 of 256 features, 77 us, 99
    // with 768 of 64 in three rounds; 106 496: 416 of 256, 164 us, 212 with 64; 16 384 rows: 256 of 64 features, 20 against
    // 41 us with 64 of 256 at 8 rows, 33 against 56 at 128.
    int best = 2, least = 0;
    const int fixed = M <= 32 ? 1 : M <= 64 ? 2 : 8;
    for (int w : {10, 8, 5, 4, 2}) {
        if (w >= 8 && M > 128) continue;             // not enough registers for more than four row tiles
        const int cost = ceil_div(ceil_div(N, 32 * w), 256) * (2 * w + fixed);
        if (least == 0 || cost < least) { least = cost; best = w; }
    }
    return best;
}

// Whether the streaming kernel of `wide` computing wavefronts takes the 16x16x32 MFMA, which draws less power, instead of the 32x32x16,
// which has half the instructions (gemm_stream.hip).  From 65 rows on, where the chip's clock follows the power.
//   4 and 5 wavefronts: from 24 k-steps of a split on (76.8 -> 72.7 us for gate|up of the 7B shape at 256 rows, 51.5 and 51.8 at 128; a
//     launch of fewer k-steps spends 0.2 to 0.3 us more on fetching its instructions).
//   2 wavefronts: up to 192 rows and from K = 3072 on only (gate|up of 16 384 rows, K = 3072, 160 rows: 30.4 -> 29.7 us; QKV, O and LM head at
//     K = 5120 28.8 -> 28.1).  Shorter ones leave the chip partly idle and lose (K = 896 at 160 rows: 12.6 -> 13.2 us, K = 2048 14.05
//     -> 14.4), and so do 224 and 256 rows at any K (K = 3584: 22.1 -> 22.9 and 23.8 -> 25.0; K = 4096 at 224 rows 38.5 -> 39.8).
//   8 and 10 wavefronts have registers for nothing else beyond 64 rows.
// Where a norm is finished the 2 to 5 wavefronts keep 32x32x16: above 64 rows that is in front of short inner dimensions (thin_resid).
inline bool stream_lean(int M, int wide, int ks_total, int splits, bool scaled) {
    if (M <= 64) return false;
    if (wide >= 8) return true;
    if (scaled) return false;
    return wide >= 4 ? ks_total / splits >= 24 : M <= 192 && ks_total >= 96;
}

// K splits up to kStreamRows rows, whichever kernel it is
inline int pick_splits(int M, int N, int ks_total) {
    const int n_blocks = ceil_div(N, 32 * stream_waves(M < kStreamThinRows ? M : kStreamThinRows, N, ks_total, false));
    const int target = 256 / n_blocks;
    if (target <= 1) return 1;
    const int units = ks_total / 8;                 // a split covers whole groups of 8 k-steps
    const int ups = ceil_div(units, target);        // units per split at the target count ...
    int s = ceil_div(units, ups);                   // ... and the fewest splits that keep it
    if (s > kMaxSplitK) s = kMaxSplitK;
    // Beyond 128 rows at least four groups each.  Not for speed: without it short inner dimensions are split further and gain (136
    // rows: O at K = 1024 12.2 -> 8.2 us, at 2048 12.9 -> 10.0, at 3584 16.0 -> 15.1; from 4096 on nothing changes; a whole
    // step at hidden 1024 166 -> 148).  But a scoring pass split into several agrees with one pass to 1e-3 only while
    // batches on both sides of 128 rows group the sums of a short inner dimension alike; split further it was 1.4e-3.
    if (M > 128 && s > (units + 1) / 4) s = (units + 1) / 4;     // seven groups (K = 1792) as eight
    return s < 1 ? 1 : s;
}

// Thin projections of up to kThinRows rows that finish in the kernel (gemm_thin.hip).  A workgroup reads its own part of W and all of X,
// at about 50 KB / us, and saves the kernel that adds partial sums (norm or QKV epilogue, 3.3 to 5 us) and their way through
// memory; gemm_stream_kernel shares X between several times as many features.  The limits are where the two come out even.  Whole
// calls of two layers, us, without these -> with them: K = 3584, decode of 8 rows 246 -> 227, 16 rows (all but down) 249 -> 244, 24
// rows (none; QKV or O alone would be +- 1 %) 252; hidden 256, decode of 32 rows 80 -> 65, 128 rows 104 -> 89, prefill of 40 rows 98 -> 82;
// hidden 512 with down projections of 8192 inputs (which stay), 8 rows 95 -> 90, 32 rows 107 -> 99; QKV at 64 rows there 108 -> 110.
// K is dealt out evenly over kThinSplits wavefronts, k-step by k-step (split_range with a unit of one).
constexpr int kThinRows = 128, kThinSplits = 4;
inline long long thin_bytes(int M, int features, int N, int ks_total) {
    const int rows = M <= 8 ? 8 : round_up(M, 16), rounds = ceil_div(ceil_div(N, features), 256);
    return (long long)rounds * (features + rows) * ks_total * 64;
}
// Sums of squares that every workgroup of the projection behind adds up (a float for each row and 16 of the N features, rows as RowSquares
// deals them out).  Up to 24 KB that is hidden behind its weights; beyond, it costs more than the norm kernel saves.  Whole decode steps of two
// layers with O in its own kernel, against without: 80 rows at hidden 768 (24 KB) 1 % faster, 896 (28 KB) 1 % slower, 1024 (32 KB) 4 %,
// 1280 (40 KB) 4 %; hidden 4096 with 256 inputs, 16 rows (16 KB) 3 % faster, 48 (64 KB) 1.4 % slower, 80 to 128 (128 KB) 4 to 5 %.
inline int squares_bytes(int M, int N) { return (M <= 8 ? 8 : M <= 16 ? 16 : M <= 32 ? 32 : M <= 64 ? 64 : 128) * (N / 4); }
// O and down.  Eight rows at any depth where the matrix has a workgroup for most compute units: down of the 7B shape streams no
// faster otherwise (23 and 24 us; whole steps with all three at hidden 3200 and 4096 10 % faster than without any, down alone 4 %).
inline bool thin_resid(int M, int N, int ks_total) {
    return M <= kThinRows && squares_bytes(M, N) <= 24 << 10 &&
           (thin_bytes(M, 16, N, ks_total) <= 256 << 10 || (M <= 8 && N >= 3200 && N <= 4096));
}
inline bool thin_qkv(int M, int N, int ks_total) {
    return M <= kThinRows && thin_bytes(M, 32, N, ks_total) <= (M <= 32 ? 360 << 10 : 88 << 10);
}

// The tiled kernels: which one, and how many K splits, except where plan_projection below decides by itself: 257 to 2048 rows of 2048 features
// and more from K = 3072 on.  Times in us, fitted to launches of the 7B shape's projections at 8192, 5120, 4096, 2048, 1280, 768, 512 and
// 296 rows, of which those up to 2048 rows are launches that plan_projection has taken over since (marked *): they are why
// the prices are what they are, and the prices go on deciding shorter inner dimensions.  k = K / 3584.  A launch has about 3
// us of its own, the same for all.
//   64 RT x 32 NT tiles, one to a CU: a round takes 2.33 RT (NT + 1.5) k.  O at 4096 rows 86 (NT = 7) and 88 (8), QKV at
//     8192 rows 186 (6, three rounds), 202 (7, three), 207 (5, four) and 212 (8, three), O at 5120 rows 126 (5), 142 (6),
//     155 (7) and 165 (8), two rounds each.  Every shape is looked at: what decides is how full the last round is.  The
//     narrow ones (NT = 2, 3) give a few hundred rows a whole round where 128 x 128 tiles need two or more K splits (* 16 384
//     columns at 296 rows: 45 us with {2, 5} and 55 with 128 x 128).  Every one of their many column blocks reads all of X again, so
//     they count as 0.4 to 1 features more (`edge`).  With the 1.5 of the others they won where they lose (* without edge -> with it: QKV at 600
//     rows {2, 4} 47.3 -> {4, 5} in three splits 42.2; O at 800 rows {2, 4} 53.7 -> {4, 5} in three 47.6).  They still win where they should:
//     512 columns, K = 8192 at 2560 rows {3, 4} in four 40.4 ({4, 5} in eight 42.0).  The model with hidden 512, where projections are
//     short and a change of kernel costs about a us, takes them from 1281 rows on (whole prefill of 360 rows 208 -> 202 us).
//     SwiGLU takes NT = 8 and 6, and {5, 4} from K = 3072 on, which counts as 0.65 more (* at 900 rows 238, {6, 5} 225; * at 1000 in a warm
//     loop 268, {8, 4} 254; at K = 2048 they are even, at 1024 and below it is 2 to 8 % slower); {7, 4} is within 2 % either way of
//     {8, 4} up to 3000 rows and 4 % slower at 4096, {5, 5} within 3 % of {6, 5}.
//   128 x 128 tiles, two to a CU: 39 k up to 256 of them (36 k up to 512 rows: * O at 450 rows in two splits 29.3 us with the norm behind it,
//     {3, 4} in three 30.6) and 60 k up to 512 (16 384 matrix rows at 512 rows: 24.1 us at K = 1024,
//     {6, 4} 27.1; 38.8 and 42.6 at 2048); then 0.166 k a tile up to 1024 rows, and above 0.095 k a tile and 15 k (W read
//     through L2 by many row blocks), from 16 384 matrix rows on, which no L2 holds, 0.137 k (22 016 rows, K = 4096: 658 us at
//     3072 rows, where tiles of {6, 4} take 458).
//   All rows in one workgroup of 160 features, up to 512 rows: 108 k a round up to 384 rows, 139 k up to 512 (SwiGLU only: no
//     fp32 matrix is cheapest there).  Only for matrices of 16 384 rows and more, where it makes a round of workgroups; cheapest
//     for some of more than 32 784 rows at 321 to 512 rows.
//   S splits divide k, cost a fixed 6 and S times the output, written here and read by the next kernel, at 4.5 TB/s.
struct TileShape { int nt, rt; double edge; };
constexpr TileShape kTileShapes[] = {{8, 4, 1.5}, {7, 4, 1.5}, {6, 4, 1.5}, {5, 4, 1.5}, {6, 5, 1.5}, {5, 5, 1.5}, {4, 5, 1.5}, {4, 6, 1.5},
                                     {2, 4, 2.5}, {3, 4, 1.9}, {2, 5, 1.9}, {3, 5, 2.0}};      // {5, 6} and up spill
inline double edge(TileShape t, bool swiglu) { return swiglu && t.nt == 5 ? 2.15 : t.edge; }
inline bool swiglu_shape(TileShape t, int ks_total) { return t.nt == 8 || t.nt == 6 || (t.nt == 5 && t.rt == 4 && ks_total >= 96); }
enum { KERNEL_128 = -2, KERNEL_MID = -1 };             // otherwise an index into kTileShapes

// us that n tiles of 128 x 128 take per 112 k-steps (see above)
inline double tiles128_us(int M, int N, long long n) {
    if (n <= 256) return M <= 512 ? 36.0 : 39.0;
    if (n <= (M > 1024 ? 473 : 512)) return 60.0;
    return M <= 1024 ? 0.166 * n : (N < 16384 ? 0.095 : 0.137) * n + 15.0;
}
struct GemmPlan { int kernel, splits; };
// splits: 0 = choose up to max_splits, otherwise given
inline GemmPlan plan_gemm(int M, int N, int ks_total, int mt_total, bool swiglu, int splits, int max_splits) {
    const double k = ks_total / 112.0;
    const long long t128 = (long long)ceil_div(M, 128) * ceil_div(N, 128);
    const int s_lo = splits ? splits : 1;
    int s_hi = splits ? splits : max_splits;
    if (!splits && s_hi > (ks_total + 8) / 32) s_hi = (ks_total + 8) / 32;     // at least 32 k-steps each (28 of 56): filling the pipeline is not free
    // what does not depend on S: workgroups of a split, of each shape that may run
    constexpr int n_shapes = sizeof kTileShapes / sizeof kTileShapes[0];
    long long tiles[n_shapes];
    double round[n_shapes];
    for (int i = 0; i < n_shapes; ++i) {
        const int nt = kTileShapes[i].nt, rt = kTileShapes[i].rt, mb = ceil_div(M, 64 * rt);
        const bool may = (!swiglu || swiglu_shape(kTileShapes[i], ks_total)) && mb * 4 * rt <= mt_total;
        tiles[i] = may ? (long long)mb * ceil_div(N, 32 * nt) : 0;
        round[i] = rt * (nt + edge(kTileShapes[i], swiglu));
    }
    GemmPlan best{KERNEL_128, s_lo};
    double least = 0.0;
    for (int S = s_lo; S == s_lo || S <= s_hi; ++S) {
        const double more = (swiglu ? 0.0 : 8.0e-6 / 4.5 * S * M * N) + (S > 1 ? 6.0 : 0.0);
        if (least != 0.0 && more >= least) break;         // grows with S: nothing from here on is cheaper
        auto offer = [&](int kernel, double us) {
            if (least == 0.0 || us + more < least) { least = us + more; best = GemmPlan{kernel, S}; }
        };
        offer(KERNEL_128, k / S * tiles128_us(M, N, t128 * S));
        if (S <= ks_total / kPfBufs)
            for (int i = 0; i < n_shapes; ++i)
                if (tiles[i]) offer(i, ((tiles[i] * S + 255) >> 8) * round[i] * 2.33 * k / S);      // equal shapes stay equal
        if (S == 1 && M <= (swiglu ? 512 : 384) && N >= 16384)
            offer(KERNEL_MID, k * ceil_div(ceil_div(N, 160), 256) * (M <= 384 ? 108.0 : 139.0));
    }
    return best;
}

// What split_range deals out at a time in the kernel that plan_gemm (or the streaming rule) names for a projection with these splits
inline int split_steps(int M, int N, int ks_total, int mt_total, int splits) {
    if (splits == 1 || stream_waves(M, N, ks_total, false)) return kPF;
    return plan_gemm(M, N, ks_total, mt_total, false, splits, splits).kernel >= 0 ? kPfBufs : kPF;
}
// K splits of a projection whose partial sums another kernel adds (fp32 output)
inline int projection_splits(int M, int N, int ks_total, int mt_total) {
    return M <= kStreamRows ? pick_splits(M, N, ks_total) : plan_gemm(M, N, ks_total, mt_total, false, 0, kMaxSplitK).splits;
}

// ---- which kernel a projection runs on and its K splits ----
// wide: computing wavefronts of the streaming kernel; nt, rt: tiles of 32 nt features x 64 rt rows; neither: what plan_gemm says.
// steps: what split_range deals out at a time, in that kernel and in the debugging path that mirrors it.
struct ProjectionPlan { int wide, nt, rt, splits, steps; };

// From 96 k-steps (K = 3072) on tiles may also have 128 or 192 rows, and a batch of a few hundred rows then takes whole rounds of them;
// up to 2048 rows, beyond which large tiles fill any number of rounds.  With K = 512 a launch is mostly its beginning and end, and a
// matrix of a few hundred rows is all splits (512 rows, K = 8192: whole steps of 384 rows 213 us as plan_gemm has it, 217 this way).
constexpr int kDeepSteps = 96, kDeepCols = 2048, kDeepRows = 2048;
struct DeepShape { int nt, rt; bool f32, swiglu; };
constexpr DeepShape kDeepShapes[] = {
    {4, 2, true, false}, {5, 2, true, false}, {6, 2, true, false}, {7, 2, true, false}, {8, 2, true, false}, {3, 3, true, false},
    {4, 3, true, false}, {5, 3, true, true}, {7, 3, true, true}, {8, 3, false, true}, {3, 4, true, false}, {4, 4, true, false},
    {5, 4, true, true}, {6, 4, true, true}, {7, 4, true, true}, {8, 4, true, true}, {3, 5, true, false}, {4, 5, true, false},
    {5, 5, true, true}, {6, 5, true, true}, {4, 6, true, false}};
// us that 112 k-steps of such a tile take: matrix instructions, and the operands' way through L2 and LDS, where a row tile costs more
// than a feature tile (its 64 rows are four 16-row tiles, the features' 32 two).  Fitted, with the constants below, to launches of
// every shape and number of splits at 31 batches of 72 to 2048 rows of the 7B shape's projections and a 16 384-row LM head (8000
// launches); {4, 3} 34.7 measured, {5, 4} 51.1, {8, 4} 72.1.  At the 19 of these above 256 rows its choice is within 0.3 % of the
// fastest on average and 2.9 % at most, plan_gemm's within 4.6 % on average: at 576 rows gate|up 152 -> 125 us, QKV 36.0 -> 29.6, down 84.7 -> 76.6; at 384 the LM
// head 63.5 -> 52.0 and down 65.4 -> 58.7; at 896 gate|up 221 -> 198, O 37.6 -> 33.6.  Whole decode steps of two layers: 336 rows 649 ->
// 621 us, 384 671 -> 639, 416 763 -> 725, 576 917 -> 805, 640 935 -> 899, 768 1046 -> 970, 960 1328 -> 1225.  At other widths, fitted to none
// (264 to 2000 rows; plan_gemm's choice -> this one): hidden 5120, gate|up of 27 648 rows at 440, 576 and 1280 rows 112 -> 108, 183 -> 159 and 295 ->
// 260, its down 66 -> 63, 76.5 -> 74 and 144 -> 131; hidden 4096, 28 672 rows 95 -> 89, 150 -> 130 and 234 -> 216; hidden 6144, 32 768 rows 146 ->
// 143, 245 -> 193 and 382 -> 356.  Of 300 projections there 11 are 4 to 7 % slower, all short (down of hidden 4096 at 512 rows 55.5 -> 59;
// O of 5120 at 440 32.7 -> 34.3).  Shapes of {2, 4} and {2, 5} are not among them: no size of this range chose them.
// Up to 256 rows the streaming kernel keeps them: tiles take less time there in a loop of their own (down at 192 rows 41 -> 36 us), but
// with activations that another kernel has just written, and a chip that then runs at a lower clock, whole steps of 72 to 192
// rows were 3 to 8 % slower with down on tiles, of 176 to 224 rows 4 % with gate|up on them, and of 240 and 256 rows as fast.
inline double deep_us(int nt, int rt) { return 1.22 * nt * rt + 1.97 * nt + 3.8 * rt + (rt == 2 ? 4.0 : 2.0); }

// max_splits 1: nothing adds partial sums behind it.
inline ProjectionPlan plan_projection(int M, int N, int ks_total, int mt_total, bool swiglu, int max_splits) {
    ProjectionPlan p{stream_waves(M, N, ks_total, swiglu), 0, 0, 1, kPF};
    if (max_splits > 1) p.splits = projection_splits(M, N, ks_total, mt_total);
    if (p.splits > max_splits) p.splits = max_splits;
    p.steps = split_steps(M, N, ks_total, mt_total, p.splits);
    if (ks_total < kDeepSteps || N < kDeepCols || M <= kStreamRows || M > kDeepRows) return p;
    const int units = ks_total / kPfBufs;
    int most = (ks_total + 8) / 32;
    if (most > max_splits) most = max_splits;
    if (most > kMaxSplitK) most = kMaxSplitK;
    double least = 0.0;
    // The SwiGLU shapes are all wide and tall.  Matrices of a few thousand rows fill the compute units better with 128 x 128 tiles, where
    // plan_gemm takes them: gate|up at K = 4096, 4096 and 8192 packed rows, 37 to 39 us at 280 and 512 rows, 52 to 54 on {5, 3}.
    if (swiglu && plan_gemm(M, N, ks_total, mt_total, true, 1, 1).kernel == KERNEL_128)
        least = ks_total / 112.0 * tiles128_us(M, N, (long long)ceil_div(M, 128) * ceil_div(N, 128));
    for (int S = 1; S <= most; ++S) {
        const double partials = swiglu ? 0.0 : 1.5e-6 * S * M * N;        // written, and read by the kernel behind
        if (least != 0.0 && partials >= least) break;
        const double steps = ceil_div(units, S) * (kPfBufs / 112.0);
        for (const DeepShape &t : kDeepShapes) {
            const int mb = ceil_div(M, 64 * t.rt);
            if (!(swiglu ? t.swiglu : t.f32) || mb * 4 * t.rt > mt_total) continue;
            const int rounds = (mb * ceil_div(N, 32 * t.nt) * S + 255) >> 8;
            const double us = partials + rounds * (1.2 + steps * deep_us(t.nt, t.rt));
            if (least == 0.0 || us < least) { least = us; p = ProjectionPlan{0, t.nt, t.rt, S, kPfBufs}; }
        }
    }
    return p;
}

// Scoring through stored logits: rows of the LM head at a time.  All of them where it has at most 16 tiles of 256 x 256, too few for
// the epilogue that reduces its rows (512 rows of 1024 columns: 23.5 us for the projection and 4.8 for the reduction behind
// it; 8.9 and 4.4 with stored logits; the whole call with two layers at hidden 256 167 -> 147 us).
constexpr int kSmallScore = 16 * 256 * 256;            // logits that such a pass stores at most
inline int score_rows(int M, int vocab, int rows) {
    return (long long)ceil_div(M, 256) * ceil_div(vocab, 256) <= 16 && M > rows ? M : rows;
}

// ---------------------------------------------------------------------------------------------
// rotary embedding
// ---------------------------------------------------------------------------------------------
// Tables [pos][i] of cos and sin(pos * theta^(-2i/d)), formed in double.  The library's cosine and sine are taken for every 32nd position
// and the first 32, the rest by the sum of two angles: two products and a sum each, off by a few 2^-53 before they are
// rounded to single precision, less than the rounding of the angle itself.  1208 positions of 64 angles: 1.04 ms with a
// cosine and a sine each, a fortieth part of a whole gated rollout of 16 x 8 sequences at the 7B width, 0.1 ms this way.
inline void rope_tables(int len, int d, double theta, float *cos_out, float *sin_out) {
    const int half = d / 2;
    std::vector<double> freq(half), c0(32 * half), s0(32 * half), c(half), s(half);
    for (int i = 0; i < half; ++i) freq[i] = std::pow(theta, -2.0 * i / d);
    for (int b = 0; b < 32 && b < len; ++b)
        for (int i = 0; i < half; ++i) {
            c0[b * half + i] = std::cos(b * freq[i]);
            s0[b * half + i] = std::sin(b * freq[i]);
        }
    for (int p0 = 0; p0 < len; p0 += 32) {
        for (int i = 0; i < half; ++i) {
            c[i] = std::cos(p0 * freq[i]);
            s[i] = std::sin(p0 * freq[i]);
        }
        for (int b = 0; b < 32 && p0 + b < len; ++b) {
            const double *cb = &c0[b * half], *sb = &s0[b * half];
            float *co = cos_out + (size_t)(p0 + b) * half, *so = sin_out + (size_t)(p0 + b) * half;
            for (int i = 0; i < half; ++i) {
                co[i] = (float)(c[i] * cb[i] - s[i] * sb[i]);
                so[i] = (float)(s[i] * cb[i] + c[i] * sb[i]);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// decode attention
// ---------------------------------------------------------------------------------------------
// `want` splits of a token range, or fewer: each holds a multiple of 32 tokens, and rounding up may leave the last ones nothing
// (2080 tokens in 16 splits of 160: the last three).  Work items of an empty split would look for pages behind the context, take
// a wavefront and add a row to the merge.
struct TokenSplits { int n, tokens; };
inline TokenSplits token_splits(int tokens, int want) {
    const int each = round_up(ceil_div(tokens, want), 32);
    return TokenSplits{ceil_div(tokens, each), each};
}

// K/V splits of the sequences' private contexts in a decode step.  waves1: wavefronts of the private phase with one split
// (sequences x kv heads); shared_waves: those of the shared-prompt phase in the same launch; tokens: private tokens of a
// sequence.  At first about 1024 wavefronts, at least 128 tokens each, at most 16.  But a launch takes as long as its
// fullest compute unit, and 256 of them take the workgroups (four wavefronts) in rounds: fewer splits are taken where the
// rounds they save outweigh the longer chain of 32-token blocks.  The three terms of the cost were fitted to attention and
// merge at 28 query and 4 kv heads of 128, 1 to 200 groups of 2, 4, 8 and 16, private contexts of 150 to 1000 tokens (147 shapes,
// each with up to eight splits): 2.4 % on average, nothing more than 3 % slower; whole steps of two layers there and at 14 query and 2 kv
// heads of 128 and 4 and 2 of 64 (150 of them, 2 to 100 groups, private contexts of 150 to 1000): 2 % on average, up to 10 % faster, and
// 3 % slower at most (14 heads: 28 groups of 8 with 150 tokens, 32 of 16 with 1000).  In us, before and after: 8 groups of 8 with 500
// tokens 27.8 with four splits (384 workgroups), 25.2 with two (256); 20 groups 55.0 with two (640), 47.4 with one (480);
// 24 groups of 4 with 150 tokens 26.7 and 21.5.  A second split where one leaves the last of its rounds emptier by 8 %: 37
// groups of 8, 300 tokens, 66.7 -> 62.8, 1000 tokens 153 -> 141; 28 groups, whose 784 workgroups begin a fourth
// round, 48.6 -> 54.3, keep one.  Whole steps of four layers at 37 groups 1293 -> 1268 us, of two at 16 groups of 4 344 -> 333, at
// 6 groups of 8 319 -> 313.
inline int private_splits(long long waves1, long long shared_waves, int tokens, int max_splits) {
    int most = (int)((1024 + waves1 / 2) / waves1);
    if (most > ceil_div(tokens, 128)) most = ceil_div(tokens, 128);
    if (most > max_splits) most = max_splits;
    if (most < 1) most = 1;
    auto wgs = [&](int s) { return (double)((shared_waves + waves1 * s + 3) / 4); };
    auto rounds = [&](int s) { return (double)(((shared_waves + waves1 * s + 3) / 4 + 255) / 256); };
    auto filled = [&](int s) { return wgs(s) > 256 ? wgs(s) / (256 * rounds(s)) : 1.0; };
    auto cost = [&](int s) {
        return (1 + 0.15 * (rounds(s) - 1)) / filled(s) + 0.06 * ceil_div(ceil_div(tokens, s), 32) / rounds(s);
    };
    int best = most;
    for (int s = most - 1; s >= 1; --s)
        if (cost(s) < cost(best) - 1e-9) best = s;
    if (most == 1 && max_splits > 1 && tokens >= 256 && filled(2) >= 0.85 && filled(2) >= filled(1) + 0.08) best = 2;
    return best;
}

// Decode attention over the whole context in one launch (attn_whole_kernel) instead of shared prompt and private context side by side
// and a merge.  It saves 4 to 8 us a layer where its workgroups, one to a (sequence, kv head), are one round of the compute units,
// and pays with every member reading the prompt for itself: even at 1000 to 1300 tokens of head size 128 and about twice that
// of 64.  More workgroups keep the other kernel busy too (512: 1 to 3 % faster below 300 tokens, 4 % slower at 1000) and stay there.
// Whole steps of two layers, us, two launches -> one: 4 and 2 kv heads of 64, 32 sequences, 272 tokens 54.4 -> 47.8, 688 61.7 -> 51.7, 1356
// 60.9 -> 57.3, 2432 63.3 -> 65.2; 28 and 4 of 128, 8 sequences, 272 tokens 225 -> 215, 832 229.5 -> 226.6, 1356 230.4 -> 230.8; 64
// sequences, 832 tokens 273 -> 268.  Eight wavefronts to a workgroup are never faster than four.
// What the members of a group read again of their `shared` prompt tokens comes from L2 where the workgroups of a kv head lie on one XCD
// (consecutive workgroups go to consecutive XCDs, so that is where n_kv is a multiple of 8), and from HBM once for every other XCD that they lie
// on.  4 us of launches pay for about 40 MB of that.  us a layer gained by one launch, around 256 workgroups, by MB read again: n_kv = 8, 0 MB
// 3.8 (G = 2) and 4.8 (G = 8); n_kv = 4, 14 MB 1.4, 39 MB -0.9 and 52 MB -2.2 (G = 2); n_kv = 2, 29 MB 0.3; n_kv = 5 with G = 8, 43 MB
// -0.7, 64 MB -3.4 and 86 MB -5.8 (whole decode steps of hidden 3200, 48 sequences, 900 tokens 206 -> 220); n_kv = 1, 74 MB -4.0.
constexpr int kWholeWaves = 4;
constexpr long long kWholeRereads = 36 << 20;
inline bool whole_context(long long seqs, int n_kv, int head_dim, int ctx, int groups, int G, int shared) {
    if (seqs * n_kv > 256 || (long long)ctx * head_dim > 1024 * 128) return false;
    const int xcds = n_kv % 8 == 0 ? 1 : n_kv % 4 == 0 ? 2 : n_kv % 2 == 0 ? 4 : 8, reads = G < xcds ? G : xcds;
    return (long long)groups * n_kv * shared * head_dim * 4 * (reads - 1) <= kWholeRereads;
}

}  // namespace sr
