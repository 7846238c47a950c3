"""GPU gate vs the CPU checker: every pairwise-distance sum and every retire bit must be equal."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_05802_amd as sr
import synth

pytestmark = pytest.mark.gpu


def run_gpu(acts, lens, thr, fn=None):
    a = torch.from_numpy(acts).cuda()
    n_groups = acts.shape[0]
    sums = torch.full((len(lens), n_groups), -7, dtype=torch.int32, device="cuda")
    retire = torch.full((len(lens), n_groups), 9, dtype=torch.uint8, device="cuda")
    (fn or sr.sr_gate_batch)(a, lens, thr, sums, retire)
    torch.cuda.synchronize()
    return sums.cpu().numpy(), retire.cpu().numpy()


def check(acts, lens, thr):
    """Both decompositions of the gate (one lane per pair; one workgroup per group with anti-diagonals in LDS)
    against the checker: every sum and every decision equal."""
    s_ref, r_ref = oracle.gate_batch(acts, lens, thr)
    for fn in (sr.sr_gate_batch, sr.sr_gate_batch_antidiag):
        s_gpu, r_gpu = run_gpu(acts, lens, thr, fn)
        assert np.array_equal(s_gpu, s_ref), fn.__name__
        assert np.array_equal(r_gpu, r_ref), fn.__name__
    return s_ref, r_ref


def test_gate_workload_full_size():
    """65536 groups x G=8 x length 30 over 64 symbols; prefixes 5, 10, 15; threshold 0.3."""
    acts, pidx = synth.gate_actions(65536, 8, 30, 64, seed=0)
    sums, retire = check(acts, [5, 10, 15], 0.3)
    assert np.all(sums[:, pidx == 3] == 0) and np.all(retire[:, pidx == 3] == 1)
    assert 0.3 < retire[1].mean() < 0.8          # the workload straddles the threshold


@pytest.mark.parametrize("G", [2, 3, 5, 8, 11, 16])
@pytest.mark.parametrize("lens", [[1], [8], [3, 9, 16], [17, 24], [30], [32], [1, 2, 3, 4, 5, 6, 7, 8]])
def test_gate_shapes(G, lens):
    stride = max(lens) + (3 if max(lens) < 30 else 0)
    n_groups = 517                                  # several workgroups and a ragged tail
    acts, _ = synth.gate_actions(n_groups, G, stride, 5, seed=G * 100 + len(lens))
    check(acts, lens, 0.25)


def test_gate_adversarial_sequences():
    rng = np.random.default_rng(0)
    G, K = 8, 16
    cases = []
    base = rng.integers(0, 3, size=K)
    cases.append(np.tile(base, (G, 1)))                                           # identical
    cases.append(np.arange(G)[:, None] * 100 + np.arange(K)[None, :])             # nothing shared
    cases.append(np.stack([np.roll(base, s) for s in range(G)]))                  # shifts: insert+delete paths
    cases.append(np.stack([np.repeat(np.arange(K // 2), 2) if i % 2 else np.tile(np.arange(K // 2), 2)
                           for i in range(G)]))
    cases.append(np.stack([np.full(K, i % 2) for i in range(G)]))                 # two constant camps
    cases.append(rng.integers(-2**31, 2**31 - 1, size=(G, K)))                    # full int32 range
    acts = np.stack(cases).astype(np.int32)
    for thr in (0.0, 0.12, 0.3, 1.0):
        check(acts, [4, 10, 16], thr)


def test_gate_threshold_edge_is_strict():
    """One member differs in one step: S = G-1 = 7; choose d_L so that 7 sits exactly on the bound."""
    G, K = 8, 10
    acts = np.tile(np.arange(K, dtype=np.int32), (1, G, 1))
    acts[0, 3, 4] = 99
    s, r = check(acts, [K], 7 / 280)          # d_K == d_L: not cut
    assert s[0, 0] == 7 and r[0, 0] == 0
    s, r = check(acts, [K], 0.025001)
    assert r[0, 0] == 1


def test_gate_empty_batch_is_a_noop():
    a = torch.zeros((1, 8, 30), dtype=torch.int32, device="cuda")
    import ctypes
    lens = (ctypes.c_int * 1)(5)
    assert sr.lib().sr_gate_batch(a.data_ptr(), 0, 8, 30, lens, 1, 0.3, None, None, None) == 0


def test_device_weight_fill_matches_host_generator():
    """The device fill used for multi-gigabyte models is bit-identical to the host generator."""
    shape = synth.ModelShape(2, 128, 4, 2, 64, 256, 512)
    host = synth.make_weights(shape, seed=7)
    embed, lm, fn, layers = synth.make_weights_device(shape, seed=7)
    same = lambda t, a: np.array_equal(t.cpu().numpy().view(np.uint16), a)
    assert same(embed, host.embed) and same(lm, host.lm_head) and same(fn, host.final_norm)
    for l in range(2):
        for k, v in host.layers[l].items():
            assert same(layers[l][k], v), (l, k)


@pytest.mark.parametrize("n_groups,G,lens", [(14337, 2, [32]), (9001, 3, [8, 1]), (6001, 12, [24, 7]), (1537, 16, [32, 31, 17]),
                                             (4099, 8, [32]), (4099, 8, [16, 9]), (1, 16, [16]), (1025, 7, [24])])
def test_gate_groups_per_workgroup(n_groups, G, lens):
    """Enough groups that a workgroup takes as many as its lanes and LDS tables hold, a ragged last workgroup, symbols at
    both ends of the 32-bit range (the empty-slot marker of the symbol table is not a symbol)."""
    acts, _ = synth.gate_actions(n_groups, G, max(lens), 6, seed=n_groups)
    values = np.array([0, -1, 1, -2 ** 31, 2 ** 31 - 1, 0x01000000], dtype=np.int32)
    acts = values[acts]
    s_ref, r_ref = oracle.gate_batch(acts, lens, 0.25)
    s_gpu, r_gpu = run_gpu(acts, lens, 0.25)
    assert np.array_equal(s_gpu, s_ref) and np.array_equal(r_gpu, r_ref)


def test_rows_further_apart_than_a_32_bit_index_reaches():
    """The members' rows may lie any distance apart (views into long histories): 16 rows of 143 165 580 entries, 9.2 GB, of
    which the first eight are looked at; gate and signals."""
    stride = 143165580                          # 15 * stride > 2^31
    acts, _ = synth.gate_actions(1, 16, 8, 5, seed=3)
    s_ref, r_ref = oracle.gate_batch(acts, [8, 3], 0.25)
    a = torch.empty((1, 16, stride), dtype=torch.int32, device="cuda")
    a[:, :, :8] = torch.from_numpy(acts).cuda()
    sums = torch.full((2, 1), -7, dtype=torch.int32, device="cuda")
    retire = torch.full((2, 1), 9, dtype=torch.uint8, device="cuda")
    sr.sr_gate_batch(a, [8, 3], 0.25, sums, retire)
    out = torch.zeros((2, 1, sr.SIGNALS_BYTES), dtype=torch.uint8, device="cuda")
    sr.sr_signals_batch(a, [8, 3], 0.25, 0.5, out)
    torch.cuda.synchronize()
    assert np.array_equal(sums.cpu().numpy(), s_ref) and np.array_equal(retire.cpu().numpy(), r_ref)
    dtype = np.dtype([(f[0], f[1]) + tuple(f[2:]) for f in sr.SIGNALS_FIELDS], align=True)
    assert np.array_equal(out.cpu().numpy().view(dtype)[..., 0]["lev_sum"], s_ref)


@pytest.mark.parametrize("n_groups,G,lens", [(24001, 2, [32, 31]), (16001, 3, [30, 1]), (9001, 4, [24, 9]), (4801, 5, [16, 3]),
                                             (3001, 6, [12, 11]), (2251, 6, [9]), (777, 16, [8, 5]), (1025, 16, [4, 1]),
                                             (513, 7, [3]), (1, 2, [1])])
def test_gate_by_comparison(n_groups, G, lens):
    """The symbols compared in registers: the smallest group counts of each size class that take it, prefixes at both ends of a
    class, a ragged last workgroup, symbols at both ends of the 32-bit range."""
    acts, _ = synth.gate_actions(n_groups, G, max(lens) + 1, 6, seed=n_groups)
    acts = np.array([0, -1, 1, -2 ** 31, 2 ** 31 - 1, 0x01000000], dtype=np.int32)[acts]
    s_ref, r_ref = oracle.gate_batch(acts, lens, 0.25)
    s_gpu, r_gpu = run_gpu(acts, lens, 0.25)
    assert np.array_equal(s_gpu, s_ref) and np.array_equal(r_gpu, r_ref)


@pytest.mark.parametrize("n_groups,G,lens,stride", [(9001, 8, [15, 10, 5], 15), (9001, 8, [16], 16), (8193, 7, [9, 13], 13), (2049, 16, [16, 9], 30),
                                                    (4097, 12, [9], 9), (4099, 8, [32, 17], 32), (601, 11, [29], 29), (1025, 16, [32], 33),
                                                    (70000, 2, [24], 25), (3, 5, [9], 9), (1, 2, [18], 18)])
@pytest.mark.parametrize("beyond", [False, True])
def test_gate_tables(n_groups, G, lens, stride, beyond):
    """Tables of symbols in their range (0 .. 63) and, with one symbol just beyond it in every hundredth group, workgroups that hash and
    workgroups that do not in one launch: up to 16 steps, beyond 16 with one and with two pairs a lane; rows that end inside a
    16-byte piece, no element behind the last one; odd groups, a ragged last workgroup, a prefix length asked for twice."""
    rng = np.random.default_rng(n_groups + G)
    lead = rng.integers(0, 64, size=(n_groups, 1, stride))
    acts = np.where(rng.random((n_groups, G, stride)) < 0.8, lead, rng.integers(0, 64, size=(n_groups, G, stride))).astype(np.int32)
    acts[0] = acts[0, :1]                           # a group that agrees
    acts[-1, :, 0], acts[-1, 0, -1] = 63, 0
    if beyond:
        acts[::100, 0, lens[0] - 1] = 64
        acts[50::100, G - 1, 0] = -1
    lens = lens + lens[:1]
    s_ref, r_ref = oracle.gate_batch(acts, lens, 0.25)
    s_gpu, r_gpu = run_gpu(acts, lens, 0.25)
    assert np.array_equal(s_gpu, s_ref) and np.array_equal(r_gpu, r_ref)


# alphabets: just beyond 64; an action modulus of 100; elements of a group; the first that does not fit a turn at its shape, and more
@pytest.mark.parametrize("n_groups,G,lens,stride", [(9001, 8, [15, 10, 5], 15), (2049, 16, [16, 9], 30), (4099, 8, [32, 17], 32), (601, 11, [29], 29),
                                                    (70000, 2, [24], 25), (5, 8, [12], 12), (1, 2, [18], 18)])
@pytest.mark.parametrize("alphabet", [65, 100, 129, 257, 600, 5000])
def test_gate_symbols_beyond_the_tables_of_64(n_groups, G, lens, stride, alphabet):
    """Groups in turns, with as many table rows as the largest symbol asks for, and hashed where those would not fit."""
    rng = np.random.default_rng(alphabet + G)
    lead = rng.integers(0, alphabet, size=(n_groups, 1, stride))
    acts = np.where(rng.random((n_groups, G, stride)) < 0.7, lead, rng.integers(0, alphabet, size=(n_groups, G, stride))).astype(np.int32)
    acts[0, :, -1], acts[-1, 0, :] = alphabet - 1, alphabet - 1
    s_ref, r_ref = oracle.gate_batch(acts, lens, 0.25)
    s_gpu, r_gpu = run_gpu(acts, lens, 0.25)
    assert np.array_equal(s_gpu, s_ref) and np.array_equal(r_gpu, r_ref)
