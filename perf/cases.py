"""The work this library is used for, as timed cases: every stage of a Pilot-Commit sampling step through the public entry
points (shared-prefix prefill, decode steps, token sampling, reward statistics / selection / advantages, teacher-forced
scoring) and the generation loop as a whole.

A case is a plain dict.  Its kind says which stage it is:

  rollouts  prefill + generate() on the small fp32 model: the whole loop, bound by launches and host work
  decode    fork, `steps` decode steps over `prompts` x `group` sequences, release.  The tokens fed are given, so that the
            logits of the last step can be compared whatever the rounding (sampled tokens would diverge)
  prefill   pc_prefill_shared of ragged prompts, then their release
  score     pc_score of ragged sequences
  sample    pc_sample over a batch of logit rows (top_p = 1: training; below: evaluation sampling)
  allocate  pc_group_stats, pc_select_commit, pc_advantages of one sampling batch

The 16-bit decoder shapes are the 1.5B, 8B and 14B ones of the benchmark with full vocabulary and fewer layers (one case
keeps all 28 layers): a step's time is its layers' plus its head's either way.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2605_26606_amd as pc

# layers, d_model, query heads, kv heads, head_dim, d_ff, vocab, rope theta, dtype, tied embeddings
MODELS = {
    "tiny": (2, 128, 4, 2, 32, 384, 512, 1.0e4, "fp32", False),
    "1.5b": (28, 1536, 12, 2, 128, 8960, 151936, 1.0e6, "bf16", True),
    "8b": (36, 4096, 32, 8, 128, 12288, 151936, 1.0e6, "bf16", False),
    "14b": (40, 5120, 40, 8, 128, 17408, 151936, 1.0e6, "bf16", False),
}
EPS = 1e-6
MATRICES = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")


# ------------------------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the small fp32 configuration, end to end: 8 prompts x 32 tokens, 4 rollouts of 16 tokens
        dict(name="rollouts_fp32", kind="rollouts", model="tiny", layers=2, prompts=8, group=4, min_len=32, max_len=32,
             steps=16, temperature=1.0, top_p=1.0),
        # reward statistics, filter and advantages of one sampling batch: the smallest calls
        dict(name="allocate", kind="allocate", prompts=1024, pilot=8, commit=24),
        # one sampler call of the pilot pass (training: temperature 1, no truncation)
        dict(name="sample", kind="sample", rows=256, vocab=151936, temperature=1.0, top_p=1.0, eos=False),
        # one sampler call of evaluation-style sampling on the stress shape's 1024 sequences
        dict(name="sample_nucleus", kind="sample", rows=1024, vocab=151936, temperature=0.7, top_p=0.95, eos=True),
        # the benchmark's pilot pass: the whole 1.5B model, 64 prompts x 4 rollouts behind 256 shared tokens
        dict(name="decode_1.5b_whole", kind="decode", model="1.5b", layers=28, prompts=64, group=4, min_len=256,
             max_len=256, steps=16, act="f16", block=64),
        # the stress configuration: 1024 sequences
        dict(name="decode_1.5b_stress", kind="decode", model="1.5b", layers=4, prompts=128, group=8, min_len=512,
             max_len=512, steps=16, act="f16", block=64),
        # the tail of a pass with ragged stop: three sequences left, each with its own long context
        dict(name="decode_1.5b_tail", kind="decode", model="1.5b", layers=8, prompts=3, group=1, min_len=1300,
             max_len=1900, steps=32, act="f16", block=64),
        # the 8B pilot pass half way: 256 sequences, most of each context its own
        dict(name="decode_8b", kind="decode", model="8b", layers=3, prompts=256, group=1, min_len=400, max_len=900,
             steps=16, act="f16", block=64),
        # the 14B commit pass: 14 kept prompts x 12 rollouts, with bfloat16 activations
        dict(name="decode_14b_bf16", kind="decode", model="14b", layers=3, prompts=14, group=12, min_len=900,
             max_len=1100, steps=16, act="bf16", block=64),
        # the benchmark's prefill chunk
        dict(name="prefill_1.5b", kind="prefill", model="1.5b", layers=4, prompts=64, min_len=256, max_len=256, act="f16"),
        # a few ragged prompts of the 8B shape
        dict(name="prefill_8b_ragged", kind="prefill", model="8b", layers=3, prompts=11, min_len=37, max_len=1100,
             act="f16"),
        # log-probabilities of whole rollouts (prompt + completion) for the policy update
        dict(name="score_1.5b", kind="score", model="1.5b", layers=4, prompts=20, min_len=700, max_len=1280, act="f16",
             temperature=1.0),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:                                               # nothing dearer than the largest listed cases
        c = _draw(rng)
        w = work(c)
        if max(w["bytes"] / 4e12, w["flops"] / 4e14) < 0.03:
            return c


def _draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "prefill", "prefill", "score", "sample", "sample", "allocate",
                       "rollouts"))
    if kind == "allocate":
        return dict(kind=kind, prompts=_log_uniform(rng, 3, 8000), pilot=rng.randint(2, 16), commit=rng.randint(2, 32))
    if kind == "sample":
        return dict(kind=kind, rows=_log_uniform(rng, 1, 1024), vocab=rng.choice((512, 32000, 50257, 151936, 151936)),
                    temperature=rng.choice((0.6, 0.7, 1.0, 1.3)), top_p=rng.choice((1.0, 1.0, 0.8, 0.95)),
                    eos=rng.random() < 0.5)
    if kind == "rollouts":
        a = rng.randint(5, 60)
        return dict(kind=kind, model="tiny", layers=rng.randint(1, 3), prompts=rng.randint(1, 12), group=rng.randint(1, 8),
                    min_len=a, max_len=a + rng.randint(0, 40), steps=rng.randint(4, 24),
                    temperature=rng.choice((0.7, 1.0)), top_p=1.0)
    c = dict(kind=kind, model=rng.choice(("1.5b", "1.5b", "8b", "14b")), layers=rng.randint(1, 3))
    c["act"] = rng.choice(("f16", "f16", "f16", "bf16"))
    top = _log_uniform(rng, 17, 2048)
    c["max_len"] = top
    c["min_len"] = max(1, int(top * rng.uniform(0.2, 1.0)))
    if kind == "decode":
        c["group"] = rng.choice((1, 1, 4, 8, 12))
        c["prompts"] = _log_uniform(rng, 1, max(1, min(1024 // c["group"], 120000 // top)))
        c["steps"] = rng.randint(4, 16)
        c["block"] = rng.choice((32, 64, 64))
    else:
        c["prompts"] = _log_uniform(rng, 1, max(1, 16000 // top))
        if kind == "score":
            c["max_len"], c["min_len"] = max(2, c["max_len"]), max(2, c["min_len"])
            c["temperature"] = rng.choice((0.7, 1.0))
    return c


# ------------------------------------------------------------------------------------------------- inputs
def _shape(case):
    L, d, hq, hkv, hd, ff, v, theta, dt, tied = MODELS[case["model"]]
    return SimpleNamespace(n_layers=case["layers"], d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=ff, vocab=v,
                           rms_eps=EPS, rope_theta=theta, dtype=dt, tied_embeddings=tied)


def _weights(m, seed):
    """Random-init decoder weights (matrices N(0, 0.02), rounded to the storage type), on the GPU; norm gains around 1."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7 + 1)
    dt = torch.float32 if m.dtype == "fp32" else torch.bfloat16
    qd, kvd = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim

    def matrix(rows, cols):
        return torch.randn(rows, cols, generator=g, device="cuda").mul_(0.02).to(dt)

    def gain():
        return 0.9 + 0.2 * torch.rand(m.d_model, generator=g, device="cuda")

    w = {"tok_embed": matrix(m.vocab, m.d_model)}
    w["lm_head"] = w["tok_embed"] if m.tied_embeddings else matrix(m.vocab, m.d_model)
    w["final_norm"] = gain()
    shapes = dict(wq=(qd, m.d_model), wk=(kvd, m.d_model), wv=(kvd, m.d_model), wo=(m.d_model, qd),
                  w_gate=(m.d_ff, m.d_model), w_up=(m.d_ff, m.d_model), w_down=(m.d_model, m.d_ff))
    w.update({k: [] for k in MATRICES + ("attn_norm", "ffn_norm")})
    for _ in range(m.n_layers):
        for k in MATRICES:
            w[k].append(matrix(*shapes[k]))
        w["attn_norm"].append(gain())
        w["ffn_norm"].append(gain())
    return w


def _lengths(case):
    """Ragged lengths, the same for every seed of a case (output shapes follow from them)."""
    rng = np.random.default_rng([case["prompts"], case["min_len"], case["max_len"]])
    return rng.integers(case["min_len"], case["max_len"] + 1, size=case["prompts"])


def _cu(lens):
    cu = np.zeros(len(lens) + 1, np.int32)
    cu[1:] = np.cumsum(lens)
    return cu


def _tokens(n, vocab, seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7 + 2 + stream)
    return torch.randint(0, vocab, (int(n),), generator=g, device="cuda", dtype=torch.int32)


def _prompt_lens(lens):
    """Scoring: a sequence's first fifth, give or take, is its prompt."""
    rng = np.random.default_rng([len(lens), int(sum(lens))])
    return np.maximum(1, (lens * rng.uniform(0.1, 0.3, size=len(lens))).astype(np.int64)).astype(np.int32)


def _logit_rows(case, seed):
    """Logits as a decoder leaves them: a bulk of unlikely tokens and, in most rows, a few dozen likely ones."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7 + 3)
    n, v = case["rows"], case["vocab"]
    x = torch.randn(n, v, generator=g, device="cuda")
    start = torch.randint(0, v, (n, 1), generator=g, device="cuda")
    step = torch.randint(1, v // 48 + 1, (n, 1), generator=g, device="cuda")
    at = (start + step * torch.arange(48, device="cuda")) % v           # 48 different ids
    peak = 9.0 * torch.rand(n, 1, generator=g, device="cuda") + 3.0 * torch.rand(n, 48, generator=g, device="cuda")
    return x.scatter_(1, at, peak).contiguous()


def _rewards(case, seed):
    rng = np.random.default_rng([int(seed), 13])
    p_q = np.sin(0.5 * np.pi * rng.random(case["prompts"])) ** 2          # Beta(1/2, 1/2): many hopeless or solved prompts
    r = rng.random((case["prompts"], case["pilot"] + case["commit"])) < p_q[:, None]
    return r.astype(np.float32)


def _context(case, m, w, lens, group, steps, block):
    rows = max(int(max(lens)), min(int(sum(lens)), 16384), len(lens) * group)
    longest = int(max(lens)) + steps
    blocks = sum(-(-int(n) // block) for n in lens) + group * sum(-(-(int(n) + steps) // block) - int(n) // block for n in lens)
    per_block = m.n_layers * m.n_kv_heads * 2 * block * m.head_dim * (4 if m.dtype == "fp32" else 2)
    return pc.Context(m, w, block_size=block, kv_pool_bytes=(blocks + 4) * per_block, max_slots=len(lens) * (1 + group) + 4,
                      max_ctx=longest, max_batch_rows=rows, act_dtype=case.get("act", "default"))


def prepare(case, seed):
    s = SimpleNamespace(case=case, seed=int(seed), stream=torch.cuda.Stream())
    kind = case["kind"]
    if kind == "allocate":
        r = _rewards(case, seed)
        P, a, b = case["prompts"], case["pilot"], case["commit"]
        s.pilot = torch.from_numpy(np.ascontiguousarray(r[:, :a])).cuda()
        s.union = torch.from_numpy(r).cuda()
        s.pilot_off = torch.arange(P + 1, dtype=torch.int32, device="cuda") * a
        s.union_off = torch.arange(P + 1, dtype=torch.int32, device="cuda") * (a + b)
        new = lambda n, dt: torch.zeros(n, dtype=dt, device="cuda")  # noqa: E731
        s.n_pos, s.n_tot = new(P, torch.int32), new(P, torch.int32)
        s.mean, s.var, s.mu, s.sigma = (new(P, torch.float32) for _ in range(4))
        s.cls, s.evict = new(P, torch.uint8), new(P, torch.uint8)
        s.commit_idx, s.surplus_idx, s.counts = new(P, torch.int32), new(P, torch.int32), new(4, torch.int32)
        s.adv = new(P * (a + b), torch.float32)
    elif kind == "sample":
        n = case["rows"]
        s.logits = _logit_rows(case, seed)
        s.uid = torch.arange(n, dtype=torch.int64, device="cuda") * 65536 + 3
        s.tokens = torch.zeros(n, dtype=torch.int32, device="cuda")
        s.logprob = torch.zeros(n, dtype=torch.float32, device="cuda")
    else:
        m = _shape(case)
        w = _weights(m, seed)
        lens = _lengths(case)
        s.cu = _cu(lens)
        group, steps = case.get("group", 0), case.get("steps", 0)
        s.ctx = _context(case, m, w, lens, group, steps, case.get("block", 64))
        s.prompt = _tokens(s.cu[-1], m.vocab, seed, 0)
        s.last = torch.empty(len(lens), m.vocab, device="cuda")
        torch.cuda.synchronize()
        if kind == "score":
            s.prompt_len = _prompt_lens(lens)
            s.out = torch.empty(int((lens - s.prompt_len).sum()), device="cuda")
        if kind in ("decode", "rollouts"):
            s.rows = np.repeat(np.arange(len(lens), dtype=np.int32), group)
            with torch.cuda.stream(s.stream):
                s.handles = pc.pc_prefill_shared(s.ctx, s.prompt, s.cu, s.last)
            n = len(s.rows)
            s.uids = np.repeat(np.arange(len(lens), dtype=np.int64) + 100, group) * 65536 + np.tile(np.arange(group), len(lens))
            if kind == "decode":
                s.fed = _tokens(n * steps, m.vocab, seed, 1).view(steps, n)
                s.current = torch.empty(n, dtype=torch.int32, device="cuda")
                s.logits = torch.empty(n, m.vocab, device="cuda")
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------------------------------------- one pass
def run(s):
    case = s.case
    kind = case["kind"]
    with torch.cuda.stream(s.stream):
        if kind == "allocate":
            P = case["prompts"]
            pc.pc_group_stats(s.pilot, s.pilot_off, s.n_pos, s.n_tot, s.mean, s.var)
            pc.pc_select_commit(s.mean, P, 0.125, 0.75, 1.0, 0, s.cls, s.evict, s.commit_idx, s.surplus_idx, s.counts)
            pc.pc_advantages(s.union, s.union_off, 1e-6, s.adv, s.mu, s.sigma)
            return dict(n_pos=s.n_pos, n_tot=s.n_tot, mean=s.mean, var=s.var, cls=s.cls, evict=s.evict,
                        commit_idx=s.commit_idx, counts=s.counts, adv=s.adv, mu=s.mu, sigma=s.sigma)
        if kind == "sample":
            pc.pc_sample(s.logits, None, case["rows"], case["vocab"], case["temperature"], s.seed, s.uid, None, 5,
                         case["vocab"] // 3 if case["eos"] else -1, 0.5 if case["eos"] else 0.0, s.tokens, s.logprob,
                         top_p=case["top_p"])
            return dict(tokens=s.tokens, logprob=s.logprob)
        if kind == "prefill":
            handles = pc.pc_prefill_shared(s.ctx, s.prompt, s.cu, s.last)
            pc.pc_release(s.ctx, handles, 1)
            return s.last
        if kind == "score":
            pc.pc_score(s.ctx, s.prompt, s.cu, s.prompt_len, case["temperature"], s.out)
            return s.out
        if kind == "rollouts":
            handles = s.handles[s.rows]
            g = pc.generate(s.ctx, handles, s.rows, s.last, s.uids, case["steps"], case["temperature"], s.seed,
                            keep_logprobs=True, keep_logits_rows=np.arange(len(s.rows)), top_p=case["top_p"])
            return dict(tokens=g["tokens"], logprobs=g["logprobs"], logits=torch.stack(g["logits"]))
        seqs = pc.pc_fork(s.ctx, s.handles[s.rows], case["steps"])
        for t in range(case["steps"]):
            s.current.copy_(s.fed[t])
            pc.pc_decode_step(s.ctx, seqs, s.current, s.logits)
        pc.pc_release(s.ctx, seqs, 0)
        return s.logits


# ------------------------------------------------------------------------------------------------- what a pass needs
def work(case):
    kind = case["kind"]
    if kind == "allocate":
        n = case["prompts"] * (2 * case["pilot"] + 2 * case["commit"])
        return dict(bytes=4 * (n + 11 * case["prompts"]), flops=6 * n)
    if kind == "sample":
        n = case["rows"] * case["vocab"]
        return dict(bytes=4 * n, flops=4 * n)
    m = _shape(case)
    size = 4 if m.dtype == "fp32" else 2
    qd, kvd = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    body = m.n_layers * (m.d_model * (2 * qd + 2 * kvd) + 3 * m.d_model * m.d_ff)
    head = m.vocab * m.d_model
    kv = 2 * m.n_layers * kvd * size                          # cache bytes per token
    mean, P = 0.5 * (case["min_len"] + case["max_len"]), case["prompts"]
    if kind in ("decode", "rollouts"):
        n, T = P * case["group"], case["steps"]
        own = n * 0.5 * (T + 1)
        keys = n * (mean + 0.5 * (T + 1))
        return dict(bytes=T * ((body + head) * size + (P * mean + own) * kv + 4 * n * m.vocab),
                    flops=T * (2 * n * (body + head) + 4 * keys * qd * m.n_layers))
    rows = P * mean
    attention = m.n_layers * 2 * qd * P * mean * mean
    if kind == "prefill":
        return dict(bytes=(body + head) * size + rows * (kv + 4) + 4 * P * m.vocab,
                    flops=2 * rows * body + attention + 2 * P * head)
    scored = 0.8 * rows
    return dict(bytes=(body + head) * size + 4 * rows + 4 * scored,
                flops=2 * rows * body + attention + 2 * scored * head)


def tolerance(case):
    kind = case["kind"]
    if kind == "allocate":
        return dict(rel=1e-6, max=1e-5)
    if kind == "sample":
        # the sums are in double: a row differs only where its uniform falls on a rounding of the boundary
        return dict(rel=1e-6, max=1e-5, differ=0.002)
    if kind == "rollouts":
        return dict(rel=2e-6, max=1e-4, differ=0.002)
    whole = case["layers"] > 8
    unit = 8.0 if case["act"] == "bf16" else 1.0              # bfloat16 has three significand bits less than half
    if kind == "score":
        return dict(rel=3e-4 * unit, max=3e-3 * unit)         # a log-probability is the logit error over about 12
    return dict(rel=min(0.03, (8e-3 if whole else 5e-3) * unit), max=min(0.5, (8e-2 if whole else 5e-2) * unit))


# ------------------------------------------------------------------------------------------------- 64-bit values
def _uniforms(seed, uids, step):
    """Philox4x32-10 (Salmon et al., "Parallel random numbers: as easy as 1, 2, 3"), first word, top 23 bits."""
    mask = np.uint64(0xFFFFFFFF)
    uids = np.asarray(uids, np.uint64)
    c = [np.full(len(uids), step, np.uint64), uids & mask, uids >> np.uint64(32), np.zeros(len(uids), np.uint64)]
    k0, k1 = int(seed) & 0xFFFFFFFF, (int(seed) >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & mask, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return ((c[0] >> np.uint64(9)).astype(np.float64) + 0.5) / 8388608.0


def _sample64(logits, temperature, top_p, u, eos=-1, bias=0.0):
    """Inverse CDF in id order over the nucleus; the uniforms decide.  logits [n, V] -> tokens, log-probabilities."""
    tokens, logprob = [], []
    for b in range(0, len(logits), 128):
        x = logits[b:b + 128].double() / temperature
        if eos >= 0:
            x[:, eos] += bias
        x -= x.max(1, keepdim=True).values
        w = x.exp()
        if top_p < 1.0:
            order = torch.sort(x, dim=1, descending=True, stable=True).indices
            c = w.gather(1, order).cumsum(1)
            before = torch.cat([torch.zeros_like(c[:, :1]), c[:, :-1]], 1)
            keep = before < float(np.float32(top_p)) * w.sum(1, keepdim=True)
            w = w * torch.zeros_like(keep).scatter_(1, order, keep)
        c = w.cumsum(1)
        target = torch.from_numpy(u[b:b + 128]).to(x)[:, None] * c[:, -1:]
        tok = (c <= target).sum(1).clamp(max=x.shape[1] - 1)
        tokens.append(tok)
        logprob.append(x.gather(1, tok[:, None])[:, 0] - c[:, -1].log())
    return torch.cat(tokens).to(torch.int32), torch.cat(logprob)


def _forward64(m, w, prompts, cu, fed=None, group=0):
    """Normalised hidden rows of the packed prompts and of the fed tokens behind them (fed [n, T], `group` rows to a prompt)."""
    n, T = (0, 0) if fed is None else fed.shape
    lens = np.diff(cu)
    R = int(cu[-1])
    tokens = prompts.long() if fed is None else torch.cat([prompts.long(), fed.reshape(-1).long()])
    pos = np.concatenate([np.arange(k) for k in lens] + [lens[i // group] + np.arange(T) for i in range(n)])
    half = m.head_dim // 2
    angle = torch.from_numpy(pos.astype(np.float64)).cuda()[:, None] * torch.from_numpy(
        m.rope_theta ** (-2.0 * np.arange(half) / m.head_dim)).cuda()
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]

    def norm(x, g):
        return x * torch.rsqrt(x.square().mean(1, keepdim=True) + m.rms_eps) * g.double()

    def linear(x, a):
        return x @ a.double().t().contiguous()

    def rotate(x):
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    def attend(q, k, v, hidden):                                # q [h, a, hd], k, v [h or broadcast, b, hd]
        sc = torch.matmul(q, k.transpose(-1, -2).contiguous()) / math.sqrt(m.head_dim)
        return torch.matmul(torch.softmax(sc.masked_fill(hidden, -math.inf), -1), v)

    h = w["tok_embed"][tokens].double()
    rep = m.n_q_heads // m.n_kv_heads
    for l in range(m.n_layers):
        a = norm(h, w["attn_norm"][l])
        q = rotate(linear(a, w["wq"][l]).view(-1, m.n_q_heads, m.head_dim))
        k = rotate(linear(a, w["wk"][l]).view(-1, m.n_kv_heads, m.head_dim))
        v = linear(a, w["wv"][l]).view(-1, m.n_kv_heads, m.head_dim)
        out = torch.empty_like(q)
        for p in range(len(lens)):
            b, e, k_p = int(cu[p]), int(cu[p + 1]), int(lens[p])
            kp, vp = (t[b:e].transpose(0, 1).repeat_interleave(rep, 0).contiguous() for t in (k, v))
            later = torch.ones(k_p, k_p, dtype=torch.bool, device="cuda").triu(1)
            out[b:e] = attend(q[b:e].transpose(0, 1).contiguous(), kp, vp, later).transpose(0, 1)
            if group:
                rows = slice(R + p * group * T, R + (p + 1) * group * T)
                qs, ks, vs = (t[rows].view(group, T, -1, m.head_dim).transpose(1, 2) for t in (q, k, v))
                ks, vs = (torch.cat([t[None].expand(group, -1, -1, -1), own.repeat_interleave(rep, 1)], 2)
                          for t, own in ((kp, ks), (vp, vs)))
                later = torch.ones(T, k_p + T, dtype=torch.bool, device="cuda").triu(k_p + 1)
                out[rows] = attend(qs.contiguous(), ks, vs, later).transpose(1, 2).reshape(group * T, m.n_q_heads, -1)
        h = h + linear(out.reshape(len(h), -1), w["wo"][l])
        gate, up, down = (w[x][l].double().t().contiguous() for x in ("w_gate", "w_up", "w_down"))
        for b in range(0, len(h), 32768):
            a = norm(h[b:b + 32768], w["ffn_norm"][l])
            h[b:b + 32768] += (torch.nn.functional.silu(a @ gate) * (a @ up)) @ down
    return norm(h, w["final_norm"]), linear


def exact(case, seed):
    kind = case["kind"]
    if kind == "allocate":
        r = torch.from_numpy(_rewards(case, seed)).cuda().double()
        p = r[:, :case["pilot"]]
        mean, var = p.mean(1), p.var(1, unbiased=False)
        mu, sigma = r.mean(1), r.var(1, unbiased=False).sqrt()
        return dict(n_pos=None, n_tot=None, mean=mean, var=var, cls=None, evict=None, commit_idx=None, counts=None,
                    adv=((r - mu[:, None]) / (sigma[:, None] + float(np.float32(1e-6)))).reshape(-1), mu=mu, sigma=sigma)
    if kind == "sample":
        uid = np.arange(case["rows"], dtype=np.int64) * 65536 + 3
        eos = case["vocab"] // 3 if case["eos"] else -1
        tok, lp = _sample64(_logit_rows(case, seed), case["temperature"], case["top_p"], _uniforms(seed, uid, 5), eos, 0.5)
        return dict(tokens=tok, logprob=lp)
    m = _shape(case)
    w = _weights(m, seed)
    lens = _lengths(case)
    cu = _cu(lens)
    prompts = _tokens(cu[-1], m.vocab, seed, 0)
    if kind == "score":
        x, linear = _forward64(m, w, prompts, cu)
        starts = _prompt_lens(lens)
        at = torch.from_numpy(np.concatenate([np.arange(cu[i] + starts[i] - 1, cu[i + 1] - 1) for i in range(len(lens))])).cuda()
        out = []
        for b in range(0, len(at), 2048):
            rows = at[b:b + 2048]
            y = linear(x[rows], w["lm_head"]) / case["temperature"]
            out.append(y.gather(1, prompts[rows + 1].long()[:, None])[:, 0] - torch.logsumexp(y, 1))
        return torch.cat(out)
    if kind == "prefill":
        x, linear = _forward64(m, w, prompts, cu)
        return linear(x[torch.from_numpy(cu[1:].astype(np.int64) - 1).cuda()], w["lm_head"])
    group, T = case["group"], case["steps"]
    n = len(lens) * group
    if kind == "decode":
        fed = _tokens(n * T, m.vocab, seed, 1).view(T, n).t().contiguous()
        x, linear = _forward64(m, w, prompts, cu, fed, group)
        return linear(x[int(cu[-1]):].view(n, T, -1)[:, -1].contiguous(), w["lm_head"])
    uids = np.repeat(np.arange(len(lens), dtype=np.int64) + 100, group) * 65536 + np.tile(np.arange(group), len(lens))
    tokens, logprobs, logits = [], [], []
    for t in range(T):
        fed = torch.stack(tokens, 1) if tokens else None
        x, linear = _forward64(m, w, prompts, cu, fed, group if tokens else 0)
        last = (x[int(cu[-1]):].view(n, t, -1)[:, -1] if t else
                x[torch.from_numpy(cu[1:].astype(np.int64) - 1).cuda()].repeat_interleave(group, 0))
        logits.append(linear(last.contiguous(), w["lm_head"]))
        tok, lp = _sample64(logits[-1], case["temperature"], case["top_p"], _uniforms(seed, uids, t))
        tokens.append(tok)
        logprobs.append(lp)
    return dict(tokens=torch.stack(tokens, 1), logprobs=torch.stack(logprobs, 1), logits=torch.stack(logits))
