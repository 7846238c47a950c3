"""The work that a GRPO training program has this library do, as timed and compared cases.

Kinds of case (one entry point, or the sequence of them that a program runs, each):
  decode    sr_decode_step on a batch in the middle of an episode: one token for every live sequence.
  prefill   sr_prefill_chunk of one observation per sequence: the start of a turn.
  score     sr_score_chunk: the teacher-forced log-likelihood of one action per sequence (after the rollout).
  rollout   one whole gated rollout from fresh weights: sr_init, sr_load_weights, prompt prefill, turns of
            observation + action, members that finish early, gate, compaction, one more observation.  A context takes
            its weights once, so a training program makes one per policy update.
  gate, signals, loss   the stand-alone batch entry points on action tables and rewards.

Models: "wide" has the layer of the benchmark configuration (hidden 3584, 28 query and 4 key/value heads of 128, FFN
18944) at a few layers, because rounding differences of the 16-bit operands grow with depth until outputs of two correct
implementations no longer resemble each other to the stated tolerance; the number of layers is chosen so that a
repeatedly called case stays in the benchmark episode's range of context lengths.  "tiny" is the small
configuration of tests and smoke run (head size 64).  "mid" is the shape in between that the tests use for odd head counts.
Tokens are forced, as in a replay: a rounding difference can then move logits but not the rest of the trajectory.  The
library's own choice is still computed in every step, but not returned, because near-ties flip it.
"""
import math

import numpy as np
import torch

import paper_2605_05802_amd as sr


class Shape:
    def __init__(self, n_layers, hidden, n_q_heads, n_kv_heads, head_dim, ffn, vocab):
        self.n_layers, self.hidden, self.n_q_heads, self.n_kv_heads = n_layers, hidden, n_q_heads, n_kv_heads
        self.head_dim, self.ffn, self.vocab = head_dim, ffn, vocab
        self.rms_eps, self.rope_theta, self.qkv_bias = 1e-6, 1e6, True


# name -> hidden, query heads, kv heads, head size, FFN, vocabulary
MODELS = {"wide": (3584, 28, 4, 128, 18944, 16384), "wide-lm": (3584, 28, 4, 128, 18944, 152064),
          "mid": (512, 14, 2, 128, 8192, 16384), "tiny": (256, 4, 2, 64, 688, 1024)}
PAGE = 64


def _shape(case):
    return Shape(case["layers"], *MODELS[case["model"]])


def listed():
    return [
        # the smallest whole program: the test configuration's gated episode; launches and host calls count
        {"name": "rollout-tiny", "kind": "rollout", "model": "tiny", "layers": 2, "groups": 4, "G": 8, "prompt": 64,
         "turns": 6, "obs": 16, "act": 8, "gate": 3, "finish": 0},
        # a rollout at the benchmark's width: 16 groups of 8, a prompt that ends inside a page (members take private
        # copies), some members finishing early, the gate after the second turn
        {"name": "rollout-16x8", "kind": "rollout", "model": "wide", "layers": 2, "groups": 16, "G": 8, "prompt": 1000,
         "turns": 2, "obs": 64, "act": 8, "gate": 2, "finish": 5},
        # what is left of a batch late in an episode: one group of eight
        {"name": "decode-1x8", "kind": "decode", "model": "wide", "layers": 4, "groups": 1, "G": 8, "prompt": 1024,
         "private": 480, "temperature": 0.0},
        # the benchmark's batch in mid-episode
        {"name": "decode-16x8", "kind": "decode", "model": "wide", "layers": 4, "groups": 16, "G": 8, "prompt": 1024,
         "private": 480, "temperature": 0.0},
        # the 64-group batch after a gate: 37 groups, a row count off every tile size
        {"name": "decode-37x8", "kind": "decode", "model": "wide", "layers": 4, "groups": 37, "G": 8, "prompt": 1024,
         "private": 288, "temperature": 0.0},
        # the long-prompt configuration (32 groups of 16, prompt 4096), sampled at the paper's temperature
        {"name": "decode-32x16-long", "kind": "decode", "model": "wide", "layers": 2, "groups": 32, "G": 16,
         "prompt": 4096, "private": 192, "temperature": 0.7},
        # a turn's observations: a single group with a short ragged chunk, and the benchmark's 128 x 64
        {"name": "prefill-1x8x17", "kind": "prefill", "model": "wide", "layers": 4, "groups": 1, "G": 8, "prompt": 333,
         "private": 0, "chunk": 17},
        {"name": "prefill-16x8x64", "kind": "prefill", "model": "wide", "layers": 4, "groups": 16, "G": 8,
         "prompt": 1024, "private": 96, "chunk": 64},
        # scoring an action of 32 tokens per sequence at the benchmark's full vocabulary
        {"name": "score-16x8x32", "kind": "score", "model": "wide-lm", "layers": 2, "groups": 16, "G": 8,
         "prompt": 512, "private": 64, "chunk": 32},
        # the gate, the signals and the loss over many groups (the benchmark's gate workload; a large step's loss)
        {"name": "gate-65536x8", "kind": "gate", "groups": 65536, "G": 8, "stride": 30, "lens": "5,10,15"},
        {"name": "signals-65536x8", "kind": "signals", "groups": 65536, "G": 8, "stride": 30, "lens": "5,10,15"},
        {"name": "loss-4096x8", "kind": "loss", "groups": 4096, "G": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "score", "rollout", "gate", "signals", "loss"])
    G = rng.choice([2, 3, 4, 5, 7, 8, 8, 8, 12, 16])
    if kind in ("gate", "signals"):
        stride = rng.randint(8, 32)
        lens = ",".join(str(rng.randint(1, stride)) for _ in range(rng.randint(1, 3)))
        pairs = G * (G - 1) // 2
        # no more table cells than the largest listed case
        cells = pairs * max(int(x) for x in lens.split(",")) ** 2
        return {"kind": kind, "groups": _log_int(rng, 1, max(2, min(65536, 65536 * 28 * 225 // cells))), "G": G,
                "stride": stride, "lens": lens}
    if kind == "loss":
        return {"kind": kind, "groups": _log_int(rng, 1, 65536), "G": G}
    model = rng.choice(["wide", "wide", "wide", "mid", "tiny"])
    layers = 2
    most = max(1, (512 if kind == "decode" else 128) // G)
    case = {"kind": kind, "model": model, "layers": layers, "groups": _log_int(rng, 1, most), "G": G}
    if kind == "decode":
        case.update(prompt=_log_int(rng, 16, 2048), private=_log_int(rng, 8, 500),
                    temperature=rng.choice([0.0, 0.0, 0.7]))
    elif kind in ("prefill", "score"):
        case.update(prompt=_log_int(rng, 16, 1024), private=_log_int(rng, 8, 96),
                    chunk=_log_int(rng, 1, 64 if kind == "prefill" else 32))
    else:
        case.update(prompt=_log_int(rng, 16, 1000), turns=rng.randint(1, 2), obs=_log_int(rng, 1, 64),
                    act=rng.randint(1, 8), gate=1, finish=0)
    return case


# ----------------------------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------------------------
def _gen(seed, what):
    return torch.Generator(device="cuda").manual_seed((seed * 1000003 + what) & 0x7FFFFFFFFFFF)


def _weights(s, seed):
    """Random-init weights: matrices and biases N(0, 0.02), norm gains near 1, all bf16."""
    g = _gen(seed, 1)

    def normal(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)

    def gain():
        return (1.0 + 0.1 * torch.randn(s.hidden, device="cuda", generator=g)).bfloat16()

    qd, kd = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    layers = [{"wq": normal(qd, s.hidden), "wk": normal(kd, s.hidden), "wv": normal(kd, s.hidden),
               "wo": normal(s.hidden, qd), "wg": normal(s.ffn, s.hidden), "wu": normal(s.ffn, s.hidden),
               "wd": normal(s.hidden, s.ffn), "bq": normal(qd), "bk": normal(kd), "bv": normal(kd),
               "norm1": gain(), "norm2": gain()} for _ in range(s.n_layers)]
    return {"embed": normal(s.vocab, s.hidden), "lm_head": normal(s.vocab, s.hidden), "final_norm": gain(),
            "layers": layers}


def _tokens(seed, what, vocab, *shape):
    return torch.randint(0, vocab, shape, dtype=torch.int32, device="cuda", generator=_gen(seed, what))


def _step_tokens(case):
    """Tokens that one pass of a decode, prefill or score case appends to every sequence."""
    return 1 if case["kind"] == "decode" else case["chunk"]


def _capacity(case):
    """Longest context of a decode, prefill or score case: room for thousands of passes where the pages allow it."""
    start = case["prompt"] + case["private"]
    per_token = case["groups"] * case["G"] * 4 * MODELS[case["model"]][2] * MODELS[case["model"]][3] * case["layers"]
    room = min(16384, (8 << 30) // per_token)
    return start + max(room, 4 * _step_tokens(case))


def _kv_bytes(case, s, max_len):
    token = 4 * s.n_kv_heads * s.head_dim * s.n_layers
    pages = case["groups"] * (-(-case["prompt"] // PAGE) + 1) + \
        case["groups"] * case["G"] * (-(-(max_len - case["prompt"]) // PAGE) + 2)
    return pages * PAGE * token


def _context(case, s, max_len, w):
    ctx = sr.Context(s, case["groups"], case["G"], 0.3, page_tokens=PAGE, max_seq_len=max_len, max_turns=16,
                     action_mod=64, kv_pool_bytes=_kv_bytes(case, s, max_len), temperature=case.get("temperature", 0.0),
                     sample_seed=7)
    ctx.sr_load_weights(w["embed"], w["lm_head"], w["final_norm"], w["layers"])
    return ctx


def _start_episode(case, seed):
    """A context in the middle of an episode: the prompt, then `private` tokens per sequence."""
    s = _shape(case)
    n = case["groups"] * case["G"]
    ctx = _context(case, s, _capacity(case), _weights(s, seed))
    ctx.sr_prefill_chunk(_tokens(seed, 2, s.vocab, case["groups"], case["prompt"]), True)
    if case["private"]:
        ctx.sr_prefill_chunk(_tokens(seed, 3, s.vocab, n, case["private"]), False)
    return ctx, (_capacity(case) - case["prompt"] - case["private"]) // _step_tokens(case)


def _rollout_inputs(case, seed):
    """Tokens of a rollout.  The first 40 % of the groups converge: their members see and do the same."""
    s, ng, G = _shape(case), case["groups"], case["G"]
    n_conv = int(round(0.4 * ng))
    turns = []
    for t in range(case["turns"] + 1):
        obs = _tokens(seed, 100 + 2 * t, s.vocab, ng, G, case["obs"])
        act = _tokens(seed, 101 + 2 * t, s.vocab, case["act"], ng, G)
        obs[:n_conv] = obs[:n_conv, :1]
        act[:, :n_conv] = act[:, :n_conv, :1]
        turns.append((obs.reshape(ng * G, -1).contiguous(), act.reshape(case["act"], ng * G).contiguous()))
    # members that end after the first turn (spread over the batch, never a whole group)
    done = np.zeros(ng * G, dtype=np.uint8)
    done[[(i * (G + 1)) % (ng * G) for i in range(case["finish"])]] = 1
    return _tokens(seed, 2, s.vocab, ng, case["prompt"]), turns, done


def _rollout_len(case):
    return case["prompt"] + case["turns"] * (case["obs"] + case["act"]) + case["obs"]


def _actions(case, seed, what, modulus=64):
    """Noisy copies of a latent leader: member i keeps the leader's symbol with the group's probability."""
    ng, G, T = case["groups"], case["G"], case["stride"]
    g = _gen(seed, what)
    rnd = lambda *shape: torch.rand(shape, device="cuda", generator=g)
    p = torch.tensor([0.5, 0.8, 0.95, 1.0], device="cuda")[(rnd(ng, 1, 1) * 4).long().clamp_(max=3)]
    pick = lambda *shape: (rnd(*shape) * modulus).int().clamp_(max=modulus - 1)
    leader = pick(ng, 1, T)
    return torch.where(rnd(ng, G, T) < p, leader, pick(ng, G, T)).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "seed": seed}
    if kind in ("decode", "prefill", "score"):
        s, n = _shape(case), case["groups"] * case["G"]
        st["ctx"], st["left"] = _start_episode(case, seed)
        st["logits"] = torch.empty((n, s.vocab), dtype=torch.float32, device="cuda")
        if kind == "decode":
            st["forced"] = _tokens(seed, 4, s.vocab, n)
            st["chosen"] = torch.empty(n, dtype=torch.int32, device="cuda")
        else:
            st["chunk"] = _tokens(seed, 4, s.vocab, n, case["chunk"])
        if kind == "score":
            st["mask"] = (torch.rand((n, case["chunk"]), device="cuda", generator=_gen(seed, 5)) < 0.8).to(torch.uint8)
            st["token_lp"] = torch.empty((n, case["chunk"]), dtype=torch.float32, device="cuda")
            st["lp"] = torch.empty(n, dtype=torch.float64, device="cuda")
    elif kind == "rollout":
        s = _shape(case)
        st["shape"], st["w"] = s, _weights(s, seed)
        st["prompt"], st["turns"], st["done"] = _rollout_inputs(case, seed)
    elif kind in ("gate", "signals"):
        ng, G, T = case["groups"], case["G"], case["stride"]
        lens = [int(x) for x in case["lens"].split(",")]
        st["lens"], st["actions"] = lens, _actions(case, seed, 10)
        if kind == "gate":
            st["sums"] = torch.empty((len(lens), ng), dtype=torch.int32, device="cuda")
            st["retire"] = torch.empty((len(lens), ng), dtype=torch.uint8, device="cuda")
        else:
            # a third of the members finish early; three observation symbols
            g = _gen(seed, 11)
            st["obs"] = torch.randint(0, 3, (ng, G, T), dtype=torch.int32, device="cuda", generator=g)
            early = torch.rand((ng, G), device="cuda", generator=g) < 0.35
            step = torch.randint(1, T + 1, (ng, G), dtype=torch.int32, device="cuda", generator=g)
            st["end"] = torch.where(early, step, torch.full_like(step, 10 ** 6))
            st["out"] = torch.empty((len(lens), ng, sr.SIGNALS_BYTES), dtype=torch.uint8, device="cuda")
    else:
        st.update(_loss_inputs(case, seed))
        st["adv"] = torch.empty(case["groups"] * case["G"], dtype=torch.float32, device="cuda")
        st["scratch"] = torch.empty(case["groups"], dtype=torch.float64, device="cuda")
        st["loss"] = torch.empty(1, dtype=torch.float64, device="cuda")
    return st


def _loss_inputs(case, seed):
    """Log-likelihoods of a few hundred action tokens; success rewards, two fifths of the groups all alike."""
    ng, G = case["groups"], case["G"]
    g = _gen(seed, 12)
    lp = -300.0 * (0.5 + torch.rand(ng * G, dtype=torch.float64, device="cuda", generator=g))
    r = (torch.rand((ng, G), device="cuda", generator=g) < 0.5).float()
    same = torch.rand((ng, 1), device="cuda", generator=g) < 0.4
    return {"lp": lp, "rewards": torch.where(same, r[:, :1], r).reshape(-1).contiguous()}


# ----------------------------------------------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------------------------------------------
def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind in ("decode", "prefill", "score"):
        if st["left"] == 0:                      # the episode has reached its longest context: the next one begins
            st["ctx"].close()
            st["ctx"], st["left"] = _start_episode(case, st["seed"])
        st["left"] -= 1
        ctx = st["ctx"]
        if kind == "score":
            ctx.sr_score_chunk(st["chunk"], st["mask"], st["token_lp"])
            ctx.sr_get_logprob(st["lp"])
            return {"token_logprob": st["token_lp"], "logprob": st["lp"]}
        if kind == "decode":
            ctx.sr_decode_step(st["forced"], st["chosen"])
        else:
            ctx.sr_prefill_chunk(st["chunk"], False)
        ctx.sr_get_logits(st["logits"])
        return {"logits": st["logits"]}
    if kind == "rollout":
        return _rollout(st)
    if kind == "gate":
        sr.sr_gate_batch(st["actions"], st["lens"], 0.3, st["sums"], st["retire"])
        return {"sums": st["sums"], "retire": st["retire"]}
    if kind == "signals":
        sr.sr_signals_batch(st["actions"], st["lens"], 0.12, 0.9, st["out"], obs=st["obs"], end_step=st["end"])
        return {"signals": st["out"]}
    sr.sr_grpo_loss(st["lp"], st["rewards"], case["G"], 1e-6, st["adv"], st["scratch"], st["loss"])
    return {"advantages": st["adv"], "loss": st["loss"]}


def _rollout(st):
    case, s = st["case"], st["shape"]
    n, ng = case["groups"] * case["G"], case["groups"]
    dev = dict(device="cuda")
    ctx = _context(case, s, _rollout_len(case), st["w"])
    ctx.sr_prefill_chunk(st["prompt"], True)
    live = torch.arange(n, **dev)
    sums = torch.zeros(ng, dtype=torch.int32, **dev)
    retire = torch.zeros(ng, dtype=torch.uint8, **dev)
    logits_turn = None
    for t in range(case["turns"]):
        obs, act = st["turns"][t]
        ctx.sr_prefill_chunk(obs[live].contiguous(), False)
        for a in range(case["act"]):
            ctx.sr_decode_step(act[a][live].contiguous())
        if t == 0:
            logits_turn = torch.empty((live.numel(), s.vocab), dtype=torch.float32, **dev)
            ctx.sr_get_logits(logits_turn)
            if case["finish"]:
                ctx.sr_finish_sequences(st["done"])
                live = torch.from_numpy(ctx.sr_get_live_map().astype(np.int64)).cuda()
        if t + 1 == case["gate"]:
            ctx.sr_gate(t + 1, sums, retire)
            ctx.sr_retire_and_compact()
            live = torch.from_numpy(ctx.sr_get_live_map().astype(np.int64)).cuda()
    out = {"logits_turn": logits_turn, "sums": sums, "retire": retire, "live": live}
    if live.numel():
        ctx.sr_prefill_chunk(st["turns"][case["turns"]][0][live].contiguous(), False)
        out["logits"] = torch.empty((live.numel(), s.vocab), dtype=torch.float32, **dev)
        ctx.sr_get_logits(out["logits"])
        out["actions"] = torch.empty((live.numel(), 16), dtype=torch.int32, **dev)
        ctx.sr_get_actions(out["actions"])
    ctx.close()
    return out


# ----------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------------------------
def _layer_params(s):
    d = s.head_dim
    return s.hidden * (s.n_q_heads + 2 * s.n_kv_heads) * d + s.n_q_heads * d * s.hidden + 3 * s.hidden * s.ffn


def _forward_work(s, units, chunk, pos0, groups, shared, logit_rows):
    """One pass over `units` x `chunk` tokens at context pos0, `shared` tokens of it held once per group."""
    rows = units * chunk
    token = 4 * s.n_kv_heads * s.head_dim * s.n_layers
    w = 2 * (s.n_layers * _layer_params(s) + s.vocab * s.hidden)
    kv = token * (groups * shared + units * (pos0 - shared)) + token * rows
    flops = 2.0 * rows * s.n_layers * _layer_params(s) + 2.0 * logit_rows * s.vocab * s.hidden
    flops += 4.0 * s.n_layers * s.n_q_heads * s.head_dim * rows * (pos0 + (chunk + 1) / 2)
    return w + kv, flops


def work(case):
    kind = case["kind"]
    if kind in ("gate", "signals"):
        cells = case["groups"] * case["G"] * case["stride"] * 4
        n = len(case["lens"].split(","))
        if kind == "gate":
            return {"bytes": cells + case["groups"] * n * 5, "flops": 0}
        return {"bytes": 2 * cells + case["groups"] * (4 * case["G"] + n * 64), "flops": 0}
    if kind == "loss":
        return {"bytes": case["groups"] * case["G"] * 16 + 8, "flops": 0}
    s, ng = _shape(case), case["groups"]
    n = ng * case["G"]
    if kind == "rollout":
        b, f = _forward_work(s, ng, case["prompt"], 0, ng, 0, n)
        pos = case["prompt"]
        for t in range(case["turns"] + 1):
            rows = n if t < case["gate"] else n - int(round(0.4 * ng)) * case["G"]
            for chunk in [case["obs"]] + ([1] * case["act"] if t < case["turns"] else []):
                x, y = _forward_work(s, rows, chunk, pos, rows // case["G"], case["prompt"], rows)
                b, f, pos = b + x, f + y, pos + chunk
        return {"bytes": b + 2 * 2 * (s.n_layers * _layer_params(s) + 2 * s.vocab * s.hidden), "flops": f}
    chunk, pos = _step_tokens(case), case["prompt"] + case["private"]
    b, f = _forward_work(s, n, chunk, pos, ng, case["prompt"], n * (chunk if kind == "score" else 1))
    return {"bytes": b + (n * chunk * 9 if kind == "score" else n * s.vocab * 4), "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind in ("gate", "signals"):
        return "exact"
    if kind == "loss":
        return {"rel": 1e-6}                      # advantages are rounded to 32 bits; the loss is a 64-bit sum
    if kind == "score":
        return {"rel": 5e-3, "max": 0.05}         # log-probabilities near -ln(vocabulary); 0.001 from 64 bits, measured
    # bf16 operands: the logits measure 0.004 (tiny) to 0.014 (four wide layers) from the 64-bit evaluation, so two
    # implementations whose operands round apart are up to 1.4 times that from each other
    return {"rel": 0.03, "max": 0.3}


# ----------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------------------------------------------
class _Exact:
    """The decoder in plain torch, float64, keys and values kept as [sequence][kv head][token][d]."""

    def __init__(self, s, w):
        self.s, self.w, self.kv, self.len = s, w, [None] * s.n_layers, 0

    def expand(self, G):
        self.kv = [(k.repeat_interleave(G, 0), v.repeat_interleave(G, 0)) for k, v in self.kv]

    def keep(self, rows):
        self.kv = [(k[rows], v[rows]) for k, v in self.kv]

    def _norm(self, x, gain):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + self.s.rms_eps) * gain.double()

    def _rope(self, x, pos):
        half = self.s.head_dim // 2
        inv = self.s.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / self.s.head_dim)
        ang = pos.double()[:, None] * inv
        c, n = ang.cos()[:, None], ang.sin()[:, None]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * c - b * n, b * c + a * n], -1)

    def append(self, tokens):
        """tokens [units][chunk]; the normalised hidden states [units][chunk][hidden] after the last layer."""
        s, (U, C) = self.s, tokens.shape
        x = self.w["embed"][tokens.long()].double()
        pos = torch.arange(self.len, self.len + C, device=x.device)
        rep = s.n_q_heads // s.n_kv_heads
        for l, w in enumerate(self.w["layers"]):
            h = self._norm(x, w["norm1"])
            q, k, v = ((h @ w["w" + c].double().t() + w["b" + c].double()).reshape(U, C, -1, s.head_dim) for c in "qkv")
            q, k = self._rope(q, pos), self._rope(k, pos)
            k, v = k.transpose(1, 2), v.transpose(1, 2)
            if self.kv[l] is not None:
                k, v = torch.cat([self.kv[l][0], k], 2), torch.cat([self.kv[l][1], v], 2)
            self.kv[l] = (k, v)
            # rows of a kv head: [C][rep]
            q = q.reshape(U, C, s.n_kv_heads, rep, s.head_dim).permute(0, 2, 1, 3, 4).reshape(U, s.n_kv_heads, C * rep, -1)
            seen = torch.arange(k.shape[2], device=x.device)[None] <= pos.repeat_interleave(rep)[:, None]
            o = torch.empty_like(q)
            step = max(1, (1 << 28) // max(1, s.n_kv_heads * C * rep * k.shape[2]))
            for u in range(0, U, step):
                p = (q[u:u + step] @ k[u:u + step].transpose(-1, -2).contiguous()) / math.sqrt(s.head_dim)
                o[u:u + step] = torch.softmax(p.masked_fill_(~seen, -math.inf), -1) @ v[u:u + step]
            o = o.reshape(U, s.n_kv_heads, C, rep, s.head_dim).permute(0, 2, 1, 3, 4).reshape(U, C, -1)
            x = x + o @ w["wo"].double().t()
            h = self._norm(x, w["norm2"])
            wg, wu, wd = (w[c].double().t() for c in ("wg", "wu", "wd"))
            step = max(1, 8192 // C)
            for u in range(0, U, step):
                x[u:u + step] += (torch.nn.functional.silu(h[u:u + step] @ wg) * (h[u:u + step] @ wu)) @ wd
        self.len += C
        return self._norm(x, self.w["final_norm"])

    def logits(self, h):
        return h @ self.w["lm_head"].double().t()


def _lev(a, b):
    row = list(range(len(b) + 1))
    for i, x in enumerate(a):
        prev, row[0] = row[0], i + 1
        for j, y in enumerate(b):
            prev, row[j + 1] = row[j + 1], min(prev + (x != y), row[j] + 1, row[j + 1] + 1)
    return row[-1]


def _exact_rollout(case, seed):
    s, ng, G = _shape(case), case["groups"], case["G"]
    prompt, turns, done = _rollout_inputs(case, seed)
    m = _Exact(s, _weights(s, seed))
    m.append(prompt)
    m.expand(G)
    live, first = list(range(ng * G)), None
    ends = np.where(done != 0, 1, 1 << 30)
    acts = np.stack([(a[0] % 64).cpu().numpy() for _, a in turns], 1)
    for t in range(case["turns"]):
        obs, act = turns[t]
        h = m.append(torch.cat([obs, act.t()], 1)[live])
        if t == 0:
            first = m.logits(h[:, -1])
            if case["finish"]:
                kept = [i for i, r in enumerate(live) if not done[r]]
                m.keep(kept)
                live = [live[i] for i in kept]
        if t + 1 == case["gate"]:
            K, cut = t + 1, set()
            for g in range(ng):
                pre = [list(acts[g * G + i, :min(K, ends[g * G + i])]) for i in range(G)]
                d = sum(_lev(pre[i], pre[j]) / max(len(pre[i]), len(pre[j])) for i in range(G) for j in range(i))
                if round(d * 1e9) < round(0.3 * (G * (G - 1) // 2) * 1e9):
                    cut.add(g)
            kept = [i for i, r in enumerate(live) if r // G not in cut]
            m.keep(kept)
            live = [live[i] for i in kept]
    out = {"logits_turn": first, "sums": None, "retire": None, "live": torch.tensor(live), "actions": None}
    if live:
        out["logits"] = m.logits(m.append(turns[case["turns"]][0][live])[:, -1])
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gate", "signals"):
        return None                               # whole numbers and records compared bit for bit
    if kind == "loss":
        x = _loss_inputs(case, seed)
        r = x["rewards"].double().reshape(case["groups"], case["G"])
        sd = (r - r.mean(1, keepdim=True)).square().mean(1, keepdim=True).sqrt()
        adv = torch.where(sd > 0, (r - r.mean(1, keepdim=True)) / (sd + 1e-6), torch.zeros_like(r)).reshape(-1)
        return {"advantages": adv, "loss": -(adv * x["lp"]).sum().reshape(1) / adv.numel()}
    if kind == "rollout":
        return _exact_rollout(case, seed)
    s, n = _shape(case), case["groups"] * case["G"]
    m = _Exact(s, _weights(s, seed))
    last = m.append(_tokens(seed, 2, s.vocab, case["groups"], case["prompt"]))[:, -1].repeat_interleave(case["G"], 0)
    m.expand(case["G"])
    if case["private"]:
        last = m.append(_tokens(seed, 3, s.vocab, n, case["private"]))[:, -1]
    if kind == "decode":
        return {"logits": m.logits(m.append(_tokens(seed, 4, s.vocab, n)[:, None])[:, -1])}
    chunk = _tokens(seed, 4, s.vocab, n, case["chunk"])
    h = m.append(chunk)
    if kind == "prefill":
        return {"logits": m.logits(h[:, -1])}
    mask = torch.rand((n, case["chunk"]), device="cuda", generator=_gen(seed, 5)) < 0.8
    h = torch.cat([last[:, None], h[:, :-1]], 1)
    lp = torch.stack([torch.log_softmax(m.logits(h[u]), -1).gather(1, chunk[u].long()[:, None])[:, 0] for u in range(n)])
    lp = torch.where(mask, lp, torch.zeros_like(lp))
    return {"token_logprob": lp, "logprob": lp.sum(1)}
