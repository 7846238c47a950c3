"""The rules that lay work out over the chip (csrc/plan.h), evaluated on the CPU."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("per_set", [1, 2, 3, 7, 313])
@pytest.mark.parametrize("n_sets", [1, 2, 4, 7, 8, 9, 12, 16, 37])
def test_shared_query_tiles_use_every_xcd(plan, n_sets, per_set):
    """Every (set, part) has one workgroup, whole rounds of eight sets stay on one XCD each, and no XCD (workgroup index
    modulo 8) has more than a workgroup above its share: one group's two kv heads used to leave six XCDs idle."""
    n = n_sets * per_set
    s, p = (ctypes.c_int * n)(), (ctypes.c_int * n)()
    plan.shared_tiles(n_sets, per_set, s, p)
    assert sorted(zip(s, p)) == [(a, b) for a in range(n_sets) for b in range(per_set)]
    load = [0] * 8
    home = {}
    for wg in range(n):
        load[wg % 8] += 1
        if s[wg] < n_sets // 8 * 8:
            assert home.setdefault(s[wg], wg % 8) == wg % 8
    assert max(load) <= -(-n // 8)


def test_division_by_multiplication(plan):
    """Every divisor up to 4096 and some large ones, at both sides of multiples up to 2^31 - 1."""
    top = 2 ** 31 - 1
    for d in list(range(1, 4097)) + [65535, 65536, 1000003, 2 ** 30, 2 ** 30 + 1, top]:
        k = top // d
        for m in {0, 1, k // 2, k - 1, k}:
            for n in {m * d - 1, m * d, m * d + d - 1, m * d + 1}:
                if 0 <= n <= top:
                    assert plan.divide(n, d) == n // d, (n, d)


@pytest.mark.parametrize("M", [1, 128, 129, 192, 193, 256, 257])
def test_small_matrices_leave_the_streaming_kernel_at_193_rows(plan, M):
    """Matrices of up to 16 MB lost 10 % on the streaming kernel at 193 to 256 rows; larger ones gain up to half."""
    for N, ks, swiglu in ((3072, 32, 0), (1024, 32, 0), (5632, 32, 1), (8192, 16, 1), (8192, 32, 0), (512, 256, 0)):
        assert (plan.stream_waves(M, N, ks, swiglu) == 0) == (M > 192)
    for N, ks, swiglu in ((16384, 112, 0), (37888, 112, 1), (8208, 16, 0), (3584, 592, 0), (4608, 112, 0)):
        assert (plan.stream_waves(M, N, ks, swiglu) == 0) == (M > 256)
    for N, ks in ((3584, 592), (3072, 32), (512, 256)):
        assert 1 <= plan.projection_splits(M, N, ks, 512) <= 16


@pytest.mark.parametrize("N,M,waves", [(49152, 128, 8), (45056, 64, 8), (106496, 128, 8), (114688, 64, 8), (65536, 8, 8), (98304, 8, 4),
                                       (152064, 128, 10), (152064, 8, 10), (81920, 128, 10), (37888, 128, 5), (37888, 160, 5),
                                       (16384, 8, 2), (16384, 128, 2), (32768, 128, 4), (106496, 160, 5), (49152, 160, 4)])
def test_workgroup_widths_of_wide_matrices(plan, N, M, waves):
    """The widths measured best or within a few per cent of it: a round of narrow workgroups is not proportionally cheaper."""
    assert plan.stream_waves(M, N, 112, 0) == waves


def test_mfma_form_of_the_weight_streams(plan):
    """16x16x32 where it measured faster: four and five wavefronts from 65 rows and 24 k-steps on, two at K >= 3072 up to 192 rows only, eight and
    ten always (registers), never the first three in front of a norm's factors, and never up to 64 rows."""
    for M in (1, 64, 65, 128, 129, 192, 193, 256):
        for ks, splits in ((8, 1), (24, 1), (32, 1), (32, 2), (64, 2), (96, 4), (112, 1), (160, 5), (592, 16)):
            for wide in (4, 5):
                assert plan.stream_lean(M, wide, ks, splits, 0) == (M > 64 and ks // splits >= 24)
                assert not plan.stream_lean(M, wide, ks, splits, 1)
            assert plan.stream_lean(M, 2, ks, splits, 0) == (64 < M <= 192 and ks >= 96)
            assert not plan.stream_lean(M, 2, ks, splits, 1)
            assert plan.stream_lean(M, 8, ks, splits, 1) == plan.stream_lean(M, 10, ks, splits, 0) == (M > 64)


def test_tiled_kernel_choice_of_wide_matrices(plan):
    """More than 1024 rows against 16 384 matrix rows or more: never the 128 x 128 tiles (658 us where others took 458).  512 such
    tiles are one round of two to a CU: 8192 and 16 384 matrix rows at 1024 and 512 rows take them."""
    for ks in (16, 64, 112, 128, 352):
        for N in (16384, 22016, 37888):
            for M in range(1025, 8193, 41):
                assert plan.plan_kernel(M, N, ks, 512, 1, 1) != -2
    for ks in (16, 32, 64):
        assert plan.plan_kernel(1024, 8192, ks, 512, 1, 1) == -2 and plan.plan_kernel(512, 16384, ks, 512, 1, 1) == -2


def test_debug_path_deals_k_out_like_the_kernel_it_mirrors(plan):
    """The single-precision debugging path covers the same k-step ranges per split as the kernel that the normal path runs, because both
    take them from the plan of the projection: tiles deal out four k-steps at a time, the streaming kernel and the 128 x 128
    tiles eight."""
    tiled = 0
    for M in (64, 136, 224, 257, 296, 384, 512, 600, 768, 1536, 2048, 2304):
        for N, ks in ((3584, 592), (1504, 400), (1024, 592), (2048, 352), (3584, 112)):
            name, s = plan.projection(M, N, 32 * ks, max_splits=16)
            cuts, unit = split_cuts(plan, M, N, ks, s), 4 if name.startswith("tiles") else 8
            assert cuts[0] == 0 and cuts[-1] == ks and all((b - a) % unit == 0 and b > a for a, b in zip(cuts, cuts[1:]))
            assert max(np.diff(cuts)) - min(np.diff(cuts)) <= unit
            tiled += unit == 4 and s > 1 and (ks // 8) % s != 0       # the two units give different ranges
    assert tiled >= 3


def split_cuts(plan, M, N, ks, splits):
    out = (ctypes.c_int * 17)()
    plan.split_ranges(M, N, ks, 512, 0, 16, out)
    return list(out)[:splits + 1]


def test_no_split_is_longer_than_the_tile_rule_reckons_with(plan):
    """A launch lasts as long as its longest split, which the rule takes to be the groups of four k-steps divided evenly.  Where plan_gemm
    would have taken the 128 x 128 tiles, groups of eight were dealt out instead: 516 to 614 rows of 2048 features at K = 4096 had
    splits of 48 k-steps and were reckoned with 44."""
    for M in range(257, 2049, 23):
        for N in (2048, 3072, 3584, 4608, 5120, 10240):
            for ks in (96, 112, 128, 160, 344, 432, 592):
                name, s = plan.projection(M, N, 32 * ks, max_splits=16)
                if name.startswith("tiles") and s > 1:
                    assert max(np.diff(split_cuts(plan, M, N, ks, s))) == 4 * -(-(ks // 4) // s), (M, N, ks, name, s)


def test_small_lm_heads_are_scored_through_stored_logits(plan):
    """Up to 16 tiles of 256 x 256 in one block, within the buffer sized for it; beyond, blocks of 256 rows (or the epilogue)."""
    for vocab in (16, 272, 1024, 2048, 2064, 4096, 152064):
        for M in (1, 256, 257, 512, 513, 1024, 4096, 4097, 8192):
            rows = plan.score_rows(M, vocab, 256)
            tiles = -(-M // 256) * -(-vocab // 256)
            assert rows == (M if M > 256 and tiles <= 16 else 256)
            assert rows == 256 or rows * vocab <= 16 * 65536


@pytest.mark.parametrize("M,N,K,kernel,splits", [
    (360, 2304, 512, "128", 1), (600, 512, 1792, "128", 2),
    # ... and where they do gain
    (2560, 512, 8192, "tiles 2x5", 4), (2560, 2304, 512, "tiles 3x4", 1)])
def test_narrow_tiles_only_where_they_gain(plan, M, N, K, kernel, splits):
    """Kernel and K splits that measured fastest, or within 2 % of it, among all shapes, the kernel that adds the splits included: where
    plan_gemm decides.  (Of more than 2047 features and 3071 inputs at 257 to 2048 rows: test_deep_projections_of_a_few_hundred_rows.)"""
    assert plan.projection(M, N, K, max_splits=16) == (kernel, splits)


@pytest.mark.parametrize("M,kernel", [(450, "tiles 5x4"), (512, "tiles 5x4"), (800, "tiles 8x3"), (960, "tiles 8x3"), (1000, "tiles 7x4"),
                                      (2049, "tiles 6x4"), (4096, "tiles 8x4")])
def test_gate_up_tiles_of_160_only_up_to_512_rows(plan, M, kernel):
    """37 888 packed rows, K = 3584: beyond 512 rows wider tiles, plan_projection's up to 2048 and plan_gemm's from there on."""
    assert plan.projection(M, 37888, 3584, swiglu=True)[0] == kernel


@pytest.mark.parametrize("waves1,shared,tokens,splits", [
    (256, 512, 500, 2), (640, 1280, 500, 1), (768, 1152, 300, 1), (512, 1024, 500, 2), (32, 64, 500, 4),
    (1184, 1184, 300, 2), (1184, 1184, 255, 1), (896, 1344, 300, 1), (2048, 2048, 300, 1), (1, 0, 100000, 16)])
def test_private_splits_where_measured(plan, waves1, shared, tokens, splits):
    assert plan.private_splits(waves1, shared, tokens, 16) == splits


def test_private_splits_stay_within_their_limits(plan):
    """At most what about 1024 wavefronts of 128 tokens each would take, or two; never none, never beyond the buffers' limit."""
    for waves1 in [*range(1, 70), 129, 255, 256, 257, 500, 1023, 1024, 1025, 1184, 2048, 4096, 200000]:
        for shared in (0, 1, 4, 63, 256, 1024, 1184, 100000):
            for tokens in (1, 31, 32, 127, 128, 129, 255, 256, 480, 1000, 16384, 1 << 20):
                for limit in (1, 3, 16):
                    most = max(1, min((1024 + waves1 // 2) // waves1, -(-tokens // 128), limit))
                    s = plan.private_splits(waves1, shared, tokens, limit)
                    assert 1 <= s <= max(most, min(2, limit))
                    assert s == 1 or -(-tokens // s) >= 32


def test_no_attention_split_is_empty(plan):
    """Every split of a token range begins within it, and the splits cover it: for any number of splits asked for (the prompt, a
    prefill chunk's context, a probe), and for the number that decode asks for."""
    each = ctypes.c_int()

    def check(tokens, want):
        n = plan.token_splits(tokens, want, ctypes.byref(each))
        assert 1 <= n <= want and each.value % 32 == 0, (tokens, want)
        assert (n - 1) * each.value < tokens <= n * each.value, (tokens, want, n, each.value)

    for tokens in [*range(1, 4200), 5000, 8191, 16384, 100001, 1 << 20]:
        for want in range(1, 17):
            check(tokens, want)
        for waves1 in (4, 32, 64, 100, 150, 256):
            check(tokens, plan.private_splits(waves1, 64, tokens, 16))


@pytest.mark.parametrize("n_lens", [0, 1, 3, 8])
@pytest.mark.parametrize("G", range(2, 17))
def test_symbols_below_the_elements_of_a_group_are_not_hashed(plan, n_lens, G):
    """Gate (no n_lens) and signals: symbols below 64 or the number of a group's elements index the tables as they are, whatever the
    shape; the groups of a turn lie within the workgroup's tables and their ids within 16 bits; turns of equal size."""
    v, t = (ctypes.c_int * 10)(), (ctypes.c_int * 3)()
    for n_groups in (1, 3, 300, 2000, 5000, 16384, 65536):
        for K in range(max(1, n_lens), 33):
            ok = plan.signals_layout(n_groups, G, K, n_lens, n_lens, v) if n_lens else plan.gate_layout(n_groups, G, K, v)
            assert ok
            direct, _, groups, _, _, row_bytes, body, hash_groups, total, _ = v
            if direct:
                continue
            for most in {64, 99, 127, max(64, G * K) - 1, G * K, 255, 511, 1000, 4095, 4096, 2 ** 31, 2 ** 32 - 1}:
                plan.prefix_turns(n_groups, G, K, n_lens, ctypes.c_uint(most), t)
                hashed, per_turn, group_bytes = t
                if most < max(64, G * K):
                    assert not hashed, (n_groups, G, K, most)
                if hashed:
                    assert per_turn == hash_groups
                else:
                    assert group_bytes >= (most + 1) * row_bytes and group_bytes % 16 == 0 and most * row_bytes < 65536
                    assert per_turn * group_bytes <= total - body
                    turns = -(-groups // per_turn)
                    assert per_turn == -(-groups // turns) and turns <= -(-groups // hash_groups)


@pytest.mark.parametrize("G", range(2, 17))
def test_gate_and_signals_fit_the_lds_that_their_occupancy_counts_on(plan, G):
    """Nothing is refused, and a workgroup stays within 40 KiB (gate: four per compute unit) or a third of 160 KiB (signals) whatever the
    number of groups, steps and prefix lengths; whole wavefronts, and lanes for every pair of the workgroup's groups."""
    v = (ctypes.c_int * 10)()
    for n_groups in (1, 2, 100, 511, 513, 1000, 2000, 5000, 8000, 16384, 30000, 65536, 200000):
        for K in range(1, 33):
            for n_lens in range(9):
                for distinct in ({0} if n_lens == 0 else {1, (n_lens + 1) // 2, min(n_lens, K)}):
                    ok = plan.signals_layout(n_groups, G, K, n_lens, distinct, v) if n_lens else plan.gate_layout(n_groups, G, K, v)
                    assert ok
                    direct, size, groups, threads, lanes, row_bytes, body, hash_groups, total, lds = v
                    assert total <= lds and 3 * (-(-(lds + 16) // 1280)) * 1280 <= 160 * 1024, (n_groups, K, n_lens, distinct, lds)
                    assert n_lens or lds <= 40 * 1024
                    assert groups >= 1 and threads % 64 == 0 and groups * lanes <= threads <= 256


@pytest.mark.parametrize("G", [4, 5, 6, 8, 12, 16])
def test_signals_of_up_to_16_steps_fit_four_workgroups_per_compute_unit(plan, G):
    """... where there are more than 1024 of them: groups of four had taken 51 KB of LDS, and with all different symbols a sixth more time than
    a lane per pair."""
    v = (ctypes.c_int * 10)()
    for K in range(9, 17):
        for n_lens in (1, 2, 3):
            assert plan.signals_layout(65536, G, K, n_lens, n_lens, v) and not v[0]
            assert 65536 / v[2] > 1024 and 4 * (-(-(v[9] + 16) // 1280)) * 1280 <= 160 * 1024, (K, n_lens, v[9])


def test_quotients_of_small_numbers_are_correctly_rounded():
    """The signals kernel divides whole numbers below 64 by multiplying with the rounded reciprocal and correcting once with the
    remainder: the same double as the division, for every pair."""
    libm = ctypes.CDLL("libm.so.6")
    libm.fma.argtypes, libm.fma.restype = [ctypes.c_double] * 3, ctypes.c_double
    for b in range(1, 64):
        r = 1.0 / b
        for a in range(64):
            q = a * r
            assert libm.fma(libm.fma(-q, float(b), float(a)), r, q) == a / b
        if b <= 32:                                   # lcm(1..32) / b from the same reciprocal
            assert round(144403552893600.0 * r) * b == 144403552893600


def test_small_divisions_by_a_rounded_reciprocal():
    """Indexes of lanes, members and steps: (x + 1/2) times the rounded 1 / d in single precision, cut off, is x / d for every x below 2^14 and
    every d of the kernels (up to 16 members, 32 steps, 120 lanes, and beyond)."""
    x = np.arange(1 << 14)
    for d in range(1, 1025):
        for inv in (np.float32(1) / np.float32(d), np.nextafter(np.float32(1) / np.float32(d), np.float32(0)), np.nextafter(np.float32(1) / np.float32(d), np.float32(2))):
            q = ((x.astype(np.float32) + np.float32(0.5)) * np.float32(inv)).astype(np.int64)
            assert np.array_equal(q, x // d), d


@pytest.mark.parametrize("K", [32, 256, 257, 272, 512, 688, 1792, 3584, 18944])
@pytest.mark.parametrize("M", [8, 128, 129, 200, 256, 257, 512, 3000])
def test_inner_dimensions_of_an_odd_number_of_groups(plan, K, M):
    """K is padded to whole groups of eight k-steps and no further, and no projection has more K splits than groups of what its
    kernel deals out; seven groups (1792) are split above 128 rows as eight are."""
    ks = plan.padded_k_steps(K)
    assert ks % 8 == 0 and 0 <= ks * 32 - K < 256
    for N in (256, 512, 2304, 4608, 16384):
        splits = plan.projection_splits(M, N, ks, 512)
        assert 1 <= splits <= max(1, ks // plan.split_steps(M, N, ks, 512, splits))
    if K == 1792 and 128 < M <= 256:
        assert plan.projection_splits(M, 512, ks, 512) == plan.projection_splits(M, 512, 64, 512) == 2


def test_thin_projections_where_they_come_out_ahead(plan):
    """Up to 128 rows of small matrices, up to 8 (all) and 16 (not down) of the 7B shape's; never above 128 rows, the size of their buffer."""
    for M in (1, 8):
        assert plan.thin_qkv(M, 4608, 112) and plan.thin_resid(M, 3584, 112) and plan.thin_resid(M, 3584, 592)
    for M in (9, 16):
        assert plan.thin_qkv(M, 4608, 112) and plan.thin_resid(M, 3584, 112) and not plan.thin_resid(M, 3584, 592)
    assert not plan.thin_qkv(17, 4608, 112) and not plan.thin_resid(17, 3584, 112)
    for M in (1, 32, 128):
        assert plan.thin_qkv(M, 512, 8) and plan.thin_resid(M, 256, 8) and plan.thin_resid(M, 256, 24)
    assert plan.thin_qkv(32, 2304, 16) and not plan.thin_qkv(64, 2304, 16) and not plan.thin_resid(8, 512, 256)
    for M in (129, 200, 4000):
        for N in (16, 256, 3584):
            assert not plan.thin_qkv(M, N, 8) and not plan.thin_resid(M, N, 8)


@pytest.mark.parametrize("M,N,ks,thin", [(64, 1024, 32, True), (65, 1024, 32, False), (80, 768, 24, True), (80, 896, 32, False), (128, 768, 24, True),
                                         (16, 4096, 8, True), (17, 4096, 8, False), (48, 4096, 8, False), (128, 4096, 8, False), (8, 8192, 8, True)])
def test_sums_of_squares_that_fit_behind_the_weights(plan, M, N, ks, thin):
    """Up to 24 KB of them for each workgroup behind; more made whole steps 1 to 5 % slower than the norm kernel does."""
    assert plan.thin_resid(M, N, ks) == thin


def test_whole_contexts_where_they_come_out_ahead(plan):
    """Up to 1024 tokens of 128 dims and 2048 of 64, for one round of workgroups."""
    assert plan.whole_context(8, 128, 1024, 4, 8, 0) and plan.whole_context(8, 64, 2048, 1, 8, 0) and plan.whole_context(1, 64, 1, 1, 2, 0)
    assert not plan.whole_context(8, 128, 1025, 4, 8, 0) and not plan.whole_context(8, 64, 2049, 1, 8, 0)
    assert not plan.whole_context(8, 128, 32, 3, 11, 0)


@pytest.mark.parametrize("n_kv,d,groups,G,shared,whole", [
    (8, 128, 16, 2, 900, True), (8, 128, 4, 8, 900, True),            # a group's kv head on one XCD
    (4, 128, 8, 8, 900, True), (4, 128, 32, 2, 400, True), (4, 128, 32, 2, 832, False),
    (2, 128, 16, 8, 576, True), (5, 128, 6, 8, 384, False), (5, 128, 6, 8, 896, False), (5, 128, 3, 8, 384, True), (5, 128, 3, 16, 576, True),
    (1, 64, 32, 8, 640, True), (1, 64, 32, 8, 1280, False), (7, 128, 1, 8, 960, True)])
def test_whole_contexts_where_members_read_the_prompt_from_one_l2(plan, n_kv, d, groups, G, shared, whole):
    """One launch as long as what the members read again from HBM stays below 36 MB: with five kv heads they lie on eight XCDs, and 48
    sequences with a prompt of 900 tokens took 206 us a step in two launches and 220 in one."""
    assert plan.whole_context(n_kv, d, shared + 40, groups, G, shared) == whole


@pytest.mark.parametrize("M,N,K,swiglu,kernel,splits", [
    (296, 37888, 3584, True, "tiles 5x5", 1), (384, 37888, 3584, True, "tiles 5x3", 1), (512, 37888, 3584, True, "tiles 5x4", 1),
    (576, 37888, 3584, True, "tiles 7x3", 1), (768, 37888, 3584, True, "tiles 7x4", 1), (896, 37888, 3584, True, "tiles 8x3", 1),
    (2048, 37888, 3584, True, "tiles 8x4", 1), (296, 3584, 18944, False, "tiles 4x5", 9), (384, 3584, 18944, False, "tiles 7x3", 8),
    (768, 3584, 18944, False, "tiles 7x3", 4), (384, 3584, 3584, False, "tiles 4x2", 3), (704, 3584, 3584, False, "tiles 4x3", 2),
    (512, 4608, 3584, False, "tiles 5x2", 2), (640, 4608, 3584, False, "tiles 6x2", 2)])
def test_deep_projections_of_a_few_hundred_rows(plan, M, N, K, swiglu, kernel, splits):
    """Kernel and K splits within 2.9 % of the fastest of all shapes measured there, the partial sums' way included."""
    assert plan.projection(M, N, K, swiglu, 1 if swiglu else 16) == (kernel, splits)


@pytest.mark.parametrize("M,N,K,kernel", [(264, 4096, 4096, "128"), (280, 8192, 4096, "128"), (512, 8192, 4096, "128"), (768, 4096, 3072, "128"),
                                          (264, 10912, 3072, "tiles 5x3"), (768, 8192, 4096, "tiles 5x3"), (512, 22016, 4096, "tiles 6x4")])
def test_deep_gate_up_of_a_few_thousand_rows(plan, M, N, K, kernel):
    """Too few features for tiles of 160 and more to fill the compute units: 128 x 128 as before (37 to 39 us at K = 4096; 52 to 54 on {5, 3})."""
    assert plan.projection(M, N, K, True) == (kernel, 1)


def test_projections_without_tile_shapes_of_their_own(plan):
    """Up to 256 and beyond 2048 rows, and below 3072 inputs, the choice is plan_gemm's and the streaming kernel's, splits included; never more
    splits than asked for, nor a split of less than two groups of eight k-steps."""
    for M in (1, 128, 256, 257, 600, 2048, 2049, 8192):
        for N, K in ((3584, 3584), (3584, 18944), (4608, 3072), (2304, 512), (16384, 2048), (37888, 3584)):
            ks = plan.padded_k_steps(K)
            for most in (1, 2, 16):
                name, splits = plan.projection(M, N, K, max_splits=most)
                assert 1 <= splits <= most and (splits == 1 or ks // splits >= 8)
                if not 256 < M <= 2048 or K < 3072:
                    want = min(most, plan.projection_splits(M, N, ks, 512)) if most > 1 else 1
                    assert (name, splits) == (plan.kernel(M, N, K, splits=want), want)
                else:
                    assert name.startswith("tiles")


@pytest.mark.parametrize("length,d,theta", [(1, 64, 1e6), (31, 128, 1e6), (32, 64, 1e4), (33, 128, 1e4), (1208, 128, 1e6), (16389, 64, 5e5)])
def test_rope_tables_by_sums_of_angles(plan, length, d, theta):
    """Against a cosine and a sine for every entry: angles of up to `length` are rounded to 2^-53 of themselves on both sides and the sum adds
    a few 2^-53, so entries agree but for those next to a rounding boundary of single precision, which may go either way."""
    half = d // 2
    got = np.empty((2, length, half), dtype=np.float32)
    at = lambda x: x.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
    plan.rope_tables(length, d, ctypes.c_double(theta), at(got[0]), at(got[1]))
    angle = np.arange(length)[:, None] * theta ** (-2.0 * np.arange(half) / d)
    bound = 4 * (length + 4) * 2.0 ** -53
    for table, exact in zip(got, (np.cos(angle), np.sin(angle))):
        assert np.all(np.abs(table - exact) <= np.spacing(np.abs(exact).astype(np.float32)) / 2 + bound)
        assert np.mean(table != exact.astype(np.float32)) < 1e-4
