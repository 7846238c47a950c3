"""Teacher-forced log-likelihood pass and policy-gradient loss on the GPU vs the CPU checker.

The trajectories are the checker's own greedy rollout of the tiny episode; the GPU re-reads them through
sr_prefill_chunk (prompt, observations) and sr_score_chunk (action tokens).  Every per-token value
log softmax(logits)[token] differs from the fp64 checker by at most twice the logits bound (a logit and
the log-sum-exp each move by at most that bound), the per-sequence sums by that times the token count.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_05802_amd as sr
import synth
from paper_2605_05802_amd.runner import load_host_weights
from test_gpu_decoder import LOGIT_TOL, dev

pytestmark = pytest.mark.gpu

TOK_TOL = 2 * LOGIT_TOL


def oracle_rollout(shape, cfg, seed, sigma=0.02):
    w = synth.make_weights(shape, seed=0, sigma=sigma)
    conv = synth.converging_groups(cfg, seed)
    prompts = synth.prompts(cfg, shape.vocab, seed)
    obs_fn = lambda t: synth.observations(cfg, shape.vocab, seed, t, conv)
    rec = oracle.run_episode(oracle.Model(w), prompts, obs_fn, cfg.G, cfg.turns, cfg.act_len, cfg.action_mod,
                             (), cfg.threshold)                       # no gate: every trajectory runs to the end
    return w, prompts, obs_fn, rec


def oracle_scores(w, cfg, prompts, obs_fn, rec, mask_fn):
    """Per-turn per-token log-probabilities of the recorded action tokens, by the checker."""
    model = oracle.Model(w)
    n_seq = cfg.n_groups * cfg.G
    out = np.zeros((cfg.turns, n_seq, cfg.act_len))
    for r in range(n_seq):
        seq = model.new_seq(cfg.prompt_len + cfg.turns * (cfg.obs_len + cfg.act_len))
        last = seq.forward(prompts[r // cfg.G])
        for t in range(cfg.turns):
            last = seq.forward(obs_fn(t)[r])
            out[t, r], last = oracle.score(seq, last, rec["tokens"][t][:, r], mask_fn(t, r))
    return out


def gpu_scores(shape, cfg, w, prompts, obs_fn, rec, mask_fn, *, max_prefill_rows=0, page_tokens=32, rows=None):
    n_seq = cfg.n_groups * cfg.G
    rows = list(range(n_seq)) if rows is None else rows
    max_len = cfg.prompt_len + cfg.turns * (cfg.obs_len + cfg.act_len)
    ctx = sr.Context(shape, cfg.n_groups, cfg.G, cfg.threshold, page_tokens=page_tokens, max_seq_len=max_len,
                     max_turns=cfg.turns, action_mod=cfg.action_mod, max_prefill_rows=max_prefill_rows,
                     kv_pool_bytes=1 << 28)
    load_host_weights(ctx, w)
    ctx.sr_prefill_chunk(dev(prompts), True)
    out = np.zeros((cfg.turns, n_seq, cfg.act_len))
    tok_lp = torch.empty((n_seq, cfg.act_len), dtype=torch.float32, device="cuda")
    for t in range(cfg.turns):
        ctx.sr_prefill_chunk(dev(obs_fn(t)), False)
        acts = np.ascontiguousarray(rec["tokens"][t].T)               # [n_seq, act_len]
        mask = np.stack([np.asarray(mask_fn(t, r), dtype=np.uint8) for r in range(n_seq)])
        ctx.sr_score_chunk(dev(acts), dev(mask), tok_lp)
        torch.cuda.synchronize()
        out[t] = tok_lp.cpu().numpy()
    total = torch.empty(n_seq, dtype=torch.float64, device="cuda")
    ctx.sr_get_logprob(total)
    torch.cuda.synchronize()
    ctx.close()
    return out, total.cpu().numpy()


def test_tiny_episode_scores_match_the_checker():
    shape, cfg = synth.TINY, synth.TINY_EPISODE
    w, prompts, obs_fn, rec = oracle_rollout(shape, cfg, seed=0)
    rng = np.random.default_rng(0)
    masks = rng.random((cfg.turns, cfg.n_groups * cfg.G, cfg.act_len)) < 0.8
    mask_fn = lambda t, r: masks[t, r]
    ref = oracle_scores(w, cfg, prompts, obs_fn, rec, mask_fn)
    got, total = gpu_scores(shape, cfg, w, prompts, obs_fn, rec, mask_fn)
    err = np.abs(got - ref).max()
    print(f"per-token log-prob: worst error {err:.3e}; mean log-prob {ref[masks].mean():.3f}")
    assert err <= TOK_TOL
    assert (got[~masks] == 0).all()
    assert np.allclose(total, got.sum(axis=(0, 2)), rtol=0, atol=1e-4)          # the running sums are those tokens
    assert np.abs(total - ref.sum(axis=(0, 2))).max() <= TOK_TOL * masks.sum(axis=(0, 2)).max()
    # greedy tokens are the most likely ones: their log-probability beats the uniform one by a wide margin
    assert ref[masks].mean() > -np.log(shape.vocab)


def test_scoring_in_several_passes_gives_the_same_values():
    # a row cap below one chunk of the whole batch splits every call into several passes and LM-head blocks
    shape = synth.TINY
    cfg = synth.EpisodeConfig("score-long", 3, 4, 48, 2, 16, 40, 16, (), 0.3, 0.34)
    w, prompts, obs_fn, rec = oracle_rollout(shape, cfg, seed=1)
    mask_fn = lambda t, r: np.ones(cfg.act_len, dtype=bool)
    a, ta = gpu_scores(shape, cfg, w, prompts, obs_fn, rec, mask_fn)
    b, tb = gpu_scores(shape, cfg, w, prompts, obs_fn, rec, mask_fn, max_prefill_rows=256)
    assert np.abs(a - b).max() <= 1e-3 and np.abs(ta - tb).max() <= 1e-2
    ref = oracle_scores(w, cfg, prompts, obs_fn, rec, mask_fn)
    assert np.abs(a - ref).max() <= TOK_TOL and np.abs(b - ref).max() <= TOK_TOL


def test_running_sums_follow_their_sequences_through_compaction():
    shape, cfg = synth.TINY, synth.TINY_EPISODE
    w, prompts, obs_fn, rec = oracle_rollout(shape, cfg, seed=0)
    n_seq = cfg.n_groups * cfg.G
    ctx = sr.Context(shape, cfg.n_groups, cfg.G, cfg.threshold, page_tokens=32, max_seq_len=512, max_turns=cfg.turns,
                     action_mod=0, kv_pool_bytes=1 << 28)
    load_host_weights(ctx, w)
    ctx.sr_prefill_chunk(dev(prompts), True)
    ctx.sr_prefill_chunk(dev(obs_fn(0)), False)
    ctx.sr_score_chunk(dev(np.ascontiguousarray(rec["tokens"][0].T)))
    before = torch.empty(n_seq, dtype=torch.float64, device="cuda")
    ctx.sr_get_logprob(before)
    # retire the converging groups through the gate on identical / distinct action ids
    conv = synth.converging_groups(cfg, 0)
    ids = np.array([0 if conv[r // cfg.G] else r for r in range(n_seq)], dtype=np.int32)
    ctx.sr_set_actions(1, dev(ids))
    ctx.sr_gate(1)
    n_live = ctx.sr_retire_and_compact()
    keep = [r for r in range(n_seq) if not conv[r // cfg.G]]
    assert n_live * cfg.G == len(keep) and 0 < len(keep) < n_seq
    after = torch.empty(len(keep), dtype=torch.float64, device="cuda")
    ctx.sr_get_logprob(after)
    torch.cuda.synchronize()
    assert np.array_equal(after.cpu().numpy(), before.cpu().numpy()[keep])
    ctx.close()


def test_score_needs_a_context_and_rejects_bad_arguments():
    shape, cfg = synth.TINY, synth.TINY_EPISODE
    w = synth.make_weights(shape, seed=0)
    ctx = sr.Context(shape, cfg.n_groups, cfg.G, 0.3, page_tokens=32, max_seq_len=128, max_turns=4, kv_pool_bytes=1 << 27)
    load_host_weights(ctx, w)
    toks = torch.zeros((cfg.n_groups * cfg.G, 8), dtype=torch.int32, device="cuda")
    with pytest.raises(sr.SrError) as e:
        ctx.sr_score_chunk(toks)                                   # nothing predicts the first token yet
    assert e.value.status == sr.SR_E_STATE
    ctx.sr_prefill_chunk(dev(synth.prompts(cfg, shape.vocab, 0)), True)
    ctx.sr_score_chunk(toks)
    with pytest.raises(sr.SrError) as e:
        ctx.sr_score_chunk(torch.zeros((cfg.n_groups * cfg.G, 100), dtype=torch.int32, device="cuda"))
    assert e.value.status == sr.SR_E_ARG                           # beyond max_seq_len
    ctx.close()


def test_grpo_loss_matches_the_checker():
    rng = np.random.default_rng(3)
    n_groups, G = 37, 8
    lp = -rng.random(n_groups * G) * 300
    r = rng.integers(0, 2, size=n_groups * G).astype(np.float32)
    r[:3 * G] = 1.0                                                 # zero-variance groups
    r[3 * G:5 * G] = 0.0
    want_loss, want_A = oracle.grpo_loss(lp, r.astype(np.float64), G, 1e-6)
    adv = torch.empty(n_groups * G, dtype=torch.float32, device="cuda")
    scratch = torch.empty(n_groups, dtype=torch.float64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    sr.sr_grpo_loss(dev(lp), dev(r), G, 1e-6, adv, scratch, loss)
    torch.cuda.synchronize()
    A = adv.cpu().numpy()
    assert (A[:5 * G] == 0).all()                                   # exactly zero, not merely small
    assert np.allclose(A, want_A, rtol=1e-6, atol=1e-7)
    assert abs(loss.item() - want_loss) <= 1e-9 * max(1.0, abs(want_loss))


def test_scoring_a_few_hundred_rows_with_split_k_projections():
    """256 scored rows per call (64 sequences x 4 action tokens): between 129 and 1024 rows the thin projections
    are split along K, so the score path's final norm has partial sums to add; deep FFN so that the split is real."""
    shape = synth.ModelShape(1, 256, 4, 2, 64, 16896, 1024)
    cfg = synth.EpisodeConfig("score-mid", 8, 8, 16, 1, 4, 4, 16, (), 0.3, 0.4)
    w, prompts, obs_fn, rec = oracle_rollout(shape, cfg, seed=2)
    mask_fn = lambda t, r: np.ones(cfg.act_len, dtype=bool)
    ref = oracle_scores(w, cfg, prompts, obs_fn, rec, mask_fn)
    got, total = gpu_scores(shape, cfg, w, prompts, obs_fn, rec, mask_fn)
    err = np.abs(got - ref).max()
    print(f"mid-size scoring: worst per-token error {err:.3e}")
    assert err <= TOK_TOL
    assert np.abs(total - ref.sum(axis=(0, 2))).max() <= TOK_TOL * cfg.act_len


@pytest.mark.parametrize("n_groups", [1, 511, 512, 513, 2048, 2049, 6145])
def test_loss_adds_the_groups_in_index_order(n_groups):
    """One workgroup, and shares and sum in two launches (chunks of 2048 shares): every size gives the sum that adding
    the groups' shares one after the other gives, to the last bit."""
    G = 3
    rng = np.random.default_rng(n_groups)
    r = rng.integers(0, 2, size=(n_groups, G)).astype(np.float32)
    lp = -rng.uniform(5.0, 400.0, size=(n_groups, G))
    share = torch.empty(n_groups, dtype=torch.float64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    sr.sr_grpo_loss(torch.from_numpy(lp).cuda(), torch.from_numpy(r).cuda(), G, 1e-6, None, share, loss)
    torch.cuda.synchronize()
    acc = np.float64(0.0)
    for x in share.cpu().numpy():
        acc = acc + x
    assert loss.item() == -acc / (n_groups * G)
    sd = r.astype(np.float64).std(axis=1, keepdims=True)
    adv = np.where(sd > 0, (r - r.mean(axis=1, keepdims=True, dtype=np.float64)) / (sd + 1e-6), 0.0)
    assert np.allclose(share.cpu().numpy(), (adv * lp).sum(axis=1), rtol=0, atol=1e-9)


@pytest.mark.parametrize("chunk,vocab,rows_cap", [(33, 1040, 0), (40, 272, 512), (129, 528, 0), (8, 1040, 0), (1, 272, 0),
                                                  (33, 4112, 0), (40, 4112, 512), (129, 1040, 0), (64, 2048, 0), (64, 2064, 0)])
def test_scoring_without_stored_logits(plan, chunk, vocab, rows_cap):
    """Vocabularies of 1040 (at 1032 rows), 2064 and 4112 with chunks of 264 to 1032 rows: the LM head reduces its rows itself, in
    one pass and in two.  Smaller LM heads, with as many rows, and chunks of 64 and 8 rows: through stored logits in one
    block; 512 rows of 2048 and 2064 columns lie on both sides of the rule.  Vocabularies that do not fill the last tile: the
    token values agree with log softmax of the logits that the same tokens leave when they are appended one by one, and the
    logits kept behind the chunk with those of the last one."""
    rows = 8 * chunk if not rows_cap else min(8 * chunk, rows_cap // chunk * chunk)
    stored = plan.score_rows(rows, vocab, 256) >= rows
    assert stored == (rows <= 256 or (vocab <= 528) or (vocab, chunk) in ((1040, 33), (2048, 64)))
    shape = synth.ModelShape(1, 256, 4, 2, 64, 256, vocab)
    w = synth.make_weights(shape, seed=2, sigma=0.05)
    n, P = 8, 24
    mk = lambda: sr.Context(shape, 2, 4, 0.3, page_tokens=32, max_seq_len=P + chunk + 8, max_turns=1, action_mod=16,
                            max_prefill_rows=rows_cap, kv_pool_bytes=1 << 26)
    prompts = dev(synth.uniform_ids(2 * P, 0, 1, vocab).reshape(2, P))
    toks = synth.uniform_ids(n * chunk, 0, 2, vocab).reshape(n, chunk)
    mask = (np.arange(n * chunk).reshape(n, chunk) % 5 != 1).astype(np.uint8)
    a = mk()
    load_host_weights(a, w)
    a.sr_prefill_chunk(prompts, True)
    lp = torch.full((n, chunk), 7.0, dtype=torch.float32, device="cuda")
    a.sr_score_chunk(dev(toks), dev(mask), lp)
    kept = torch.empty((n, vocab), dtype=torch.float32, device="cuda")
    a.sr_get_logits(kept)
    total = torch.empty(n, dtype=torch.float64, device="cuda")
    a.sr_get_logprob(total)
    b = mk()
    load_host_weights(b, w)
    b.sr_prefill_chunk(prompts, True)
    ref = np.zeros((n, chunk))
    lg = torch.empty((n, vocab), dtype=torch.float32, device="cuda")
    for t in range(chunk):
        b.sr_get_logits(lg)
        r = torch.log_softmax(lg.double(), dim=1).cpu().numpy()
        ref[:, t] = r[np.arange(n), toks[:, t]]
        b.sr_decode_step(dev(np.ascontiguousarray(toks[:, t])))
    b.sr_get_logits(lg)
    torch.cuda.synchronize()
    got = lp.cpu().numpy()
    assert np.all(got[mask == 0] == 0.0)
    # decoded and prefilled rows round their operands apart: the bound that the logits of either carry
    assert np.abs(got - ref * mask).max() <= 2 * LOGIT_TOL
    assert np.abs(kept.cpu().numpy() - lg.cpu().numpy()).max() <= LOGIT_TOL
    assert np.abs(total.cpu().numpy() - got.astype(np.float64).sum(axis=1)).max() <= 1e-9 * chunk
    a.close()
    b.close()


@pytest.mark.parametrize("vocab", [4112, 2064])
@pytest.mark.parametrize("heavy", ["last tile", 0, 1, 2, 3])
def test_scoring_counts_every_column_of_the_last_tile(plan, vocab, heavy):
    """The vocabulary ends in a tile of 16 columns, four of which lie in each group of lanes.  Their LM-head rows are scaled by 16,
    so that without them the log-sum-exp of some row moves by far more than the bound (checked on the reference); targets
    lie among them and elsewhere."""
    assert plan.score_rows(264, vocab, 256) == 256              # 264 rows: the LM head's epilogue reduces them
    shape = synth.ModelShape(1, 256, 4, 2, 64, 256, vocab)
    w = synth.make_weights(shape, seed=2, sigma=0.05)
    cols = np.arange(vocab - 16, vocab) if heavy == "last tile" else vocab - 16 + 4 * heavy + np.arange(4)
    as_f32 = (w.lm_head[cols].astype(np.uint32) << 16).view(np.float32) * 16
    w.lm_head[cols] = (as_f32.view(np.uint32) >> 16).astype(np.uint16)          # a power of two: exact in bf16
    n, P, chunk = 8, 24, 33
    prompts = dev(synth.uniform_ids(2 * P, 0, 1, vocab).reshape(2, P))
    toks = synth.uniform_ids(n * chunk, 0, 2, vocab).reshape(n, chunk)
    toks[:, ::3] = cols[np.arange(toks[:, ::3].size).reshape(n, -1) % cols.size]
    mk = lambda: sr.Context(shape, 2, 4, 0.3, page_tokens=32, max_seq_len=P + chunk + 8, max_turns=1, action_mod=16,
                            kv_pool_bytes=1 << 26)
    a = mk()
    load_host_weights(a, w)
    a.sr_prefill_chunk(prompts, True)
    lp = torch.full((n, chunk), 7.0, dtype=torch.float32, device="cuda")
    a.sr_score_chunk(dev(toks), None, lp)
    b = mk()
    load_host_weights(b, w)
    b.sr_prefill_chunk(prompts, True)
    ref, without = np.zeros((n, chunk)), np.zeros((n, chunk))
    lg = torch.empty((n, vocab), dtype=torch.float32, device="cuda")
    for t in range(chunk):
        b.sr_get_logits(lg)
        torch.cuda.synchronize()
        x = lg.double().cpu().numpy()
        lse = np.logaddexp.reduce(x, axis=1)
        ref[:, t] = x[np.arange(n), toks[:, t]] - lse
        without[:, t] = lse - np.logaddexp.reduce(np.delete(x, cols, axis=1), axis=1)
        b.sr_decode_step(dev(np.ascontiguousarray(toks[:, t])))
    bound = 16 * 2 * LOGIT_TOL             # the logits' bound, at LM-head rows sixteen times as long, for target and log-sum-exp
    assert without[:, 1:].max() > 3 * bound
    torch.cuda.synchronize()
    assert np.abs(lp.cpu().numpy() - ref).max() <= bound
    a.close()
    b.close()


@pytest.mark.parametrize("n_groups,G", [(1, 1), (5, 3), (512, 4), (513, 4), (400, 8), (401, 8), (200, 16), (201, 16), (355, 9), (70, 33), (188, 17),
                                        (4096, 5), (8193, 2), (10000, 17)])
@pytest.mark.parametrize("equal", [0.0, 0.5, 1.0])
def test_loss_leaves_out_shares_of_zero(n_groups, G, equal):
    """Every size class of a group, on both sides of the rule for one launch, without, with some and with nothing but groups whose
    rewards are equal: advantages as in Eq. 1, the loss the shares added in index order, to the last bit."""
    rng = np.random.default_rng(n_groups + G)
    lp = -rng.uniform(1.0, 400.0, size=(n_groups, G))
    r = rng.integers(0, 3, size=(n_groups, G)).astype(np.float32)
    same = rng.random(n_groups) < equal
    r[same] = r[same, :1]
    adv = torch.full((n_groups, G), 7.0, dtype=torch.float32, device="cuda")
    share = torch.full((n_groups,), 7.0, dtype=torch.float64, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    sr.sr_grpo_loss(torch.from_numpy(lp).cuda(), torch.from_numpy(r).cuda(), G, 1e-6, adv, share, loss)
    torch.cuda.synchronize()
    shares, acc = share.cpu().numpy(), np.float64(0.0)
    for x in shares:
        acc = acc + x
    assert loss.item() == -acc / (n_groups * G)
    sd = r.astype(np.float64).std(axis=1, keepdims=True)
    want = np.where((r == r[:, :1]).all(axis=1, keepdims=True), 0.0, (r - r.mean(axis=1, keepdims=True, dtype=np.float64)) / (sd + 1e-6))
    assert (adv.cpu().numpy()[same] == 0).all() and (shares[same] == 0).all()
    assert np.allclose(adv.cpu().numpy(), want, rtol=1e-6, atol=1e-7)
    assert np.allclose(shares, (want * lp).sum(axis=1), rtol=0, atol=1e-8)
    lp[-1, 0], r[-1, 0] = np.nan, 5.0                # a share that is not a number is not left out
    sr.sr_grpo_loss(torch.from_numpy(lp).cuda(), torch.from_numpy(r).cuda(), G, 1e-6, adv, share, loss)
    assert np.isnan(loss.item())
