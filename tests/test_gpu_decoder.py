"""GPU parity of the decoder path (pc_prefill_shared, pc_fork, pc_decode_step,
pc_sample) against the oracle, teacher-forced: the GPU generates freely; the
oracle is fed the GPU's own token history and recomputes the logits of every
position from scratch (brute force).

Logits: max-abs error <= 1e-4 for fp32 models, <= 2e-2 for bf16 models, both
times max(1, max|logit|) (the bounds are stated for logits of order 1, which
is what the workloads' N(0, 0.02) init gives; tests that inflate the weights
to sharpen the attention scale the bound with the logit magnitude).

Tokens: a sampled token is an integer decided by floating point, so the
decision is compared in the kernel's precision: the oracle's sampler, given
the logits the GPU sampled from and the same uniform, must pick the same
token on >= 99.9 % of positions.  Sampling from the oracle's OWN logits is
checked as well: >= 99.9 % for fp32 models; for bf16 models the agreement is
bounded by the logit error itself -- a uniform lands between the two sides'
CDF boundaries with probability ~ 0.4 sqrt(V) rms(logit error) for a
near-uniform distribution over V tokens -- so there it must stay above
1 - max(1 %, 1.5 sqrt(V) rms error).
"""
import math

import numpy as np
import pytest
import torch

import workloads
from oracle import decoder, philox, sampler
from gpu_util import make_ctx, say, side_stream

pytestmark = pytest.mark.gpu

C1 = workloads.WORKLOADS["C1"]
# a small bf16 model with the head geometry of the large ones (head_dim 128, 6 query heads per kv head)
BF = workloads.scaled(C1, dtype="bf16", d_model=256, n_q_heads=12, n_kv_heads=2, head_dim=128, d_ff=640,
                      vocab=2048, n_layers=3, rope_theta=1.0e6).model
# wide enough that the feed-forward down projection takes the large-tile split-K route while decoding
BF8 = workloads.scaled(C1, dtype="bf16", d_model=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ff=8192,
                       vocab=4096, n_layers=2, rope_theta=1.0e6).model
BF4 = workloads.scaled(C1, dtype="bf16", d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ff=1024,
                       vocab=4096, n_layers=2, rope_theta=1.0e6).model
# the head geometries of the 8B and 14B shapes: 8 kv heads with 4 and with 5 query heads each
BF48 = workloads.scaled(C1, dtype="bf16", d_model=512, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ff=1024,
                        vocab=2048, n_layers=2, rope_theta=1.0e6).model
# projections as wide as the 8B model's (weights of 9 to 16 M elements per matrix, reductions of 3072 and more): the
# decode GEMMs then take 128-column tiles cut into K slices, 128- or 256-row blocks by the batch
BFW = workloads.scaled(C1, dtype="bf16", d_model=3072, n_q_heads=24, n_kv_heads=8, head_dim=128, d_ff=4096,
                       vocab=2048, n_layers=1, rope_theta=1.0e6).model
BF58 = workloads.scaled(C1, dtype="bf16", d_model=640, n_q_heads=40, n_kv_heads=8, head_dim=128, d_ff=1024,
                        vocab=2048, n_layers=2, rope_theta=1.0e6).model


def _teacher_forced(model, w, prompt, gen_tokens, gpu_logits, uid, seed, temperature, eos_id=-1, bias=0.0):
    """gpu_logits: [T, V] the logits the GPU sampled each generated token from.
    Returns (scaled max-abs error, sum of squared errors, count, agreement of the oracle's sampler on
    the GPU's logits, agreement of the oracle's sampler on its own logits)."""
    T = len(gen_tokens)
    seq = np.concatenate([prompt, gen_tokens])
    want = decoder.forward_full(model, w, seq[:-1], rows=np.arange(len(prompt) - 1, len(seq) - 1))
    # the error of a bf16 pipeline is relative to the logit magnitude: the bound is stated for
    # logits of order 1 (the workloads' N(0, 0.02) init) and scales up for inflated test weights
    diff = want - gpu_logits
    err = float(np.abs(diff).max()) / max(1.0, float(np.abs(want).max()))
    same = own = 0
    for t in range(T):
        u = philox.sampling_uniform(seed, uid, t)
        same += int(sampler.sample_token(gpu_logits[t], temperature, u, eos_id, bias)[0] == gen_tokens[t])
        own += int(sampler.sample_token(want[t], temperature, u, eos_id, bias)[0] == gen_tokens[t])
    assert np.abs(want).max() > 0.05, "degenerate logits make the comparison empty"
    return err, float((diff ** 2).sum()), diff.size, same, own


def _run_generate(model, w_cpu, prompts_list, G, T, seed, ctx_kw, opts=(), temperature=1.0, stream=True,
                  eos_id=-1, bias=0.0, poll_every=64, compact=True, expect_saturation=False):
    import paper_2605_26606_amd as pc
    ctx = make_ctx(model, w_cpu, **ctx_kw)
    for o, v in opts:
        pc.pc_set_option(ctx, o, v)
    lens = [len(p) for p in prompts_list]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = torch.from_numpy(np.concatenate(prompts_list).astype(np.int32)).cuda()
    P = len(prompts_list)
    st = side_stream() if stream else torch.cuda.current_stream()
    with torch.cuda.stream(st):
        last = torch.empty((P, model.vocab), dtype=torch.float32, device="cuda")
        handles = pc.pc_prefill_shared(ctx, toks, cu, last)
        rows = np.repeat(np.arange(P, dtype=np.int32), G)
        uids = (rows.astype(np.int64) * 65536 + np.tile(np.arange(G), P))
        n = P * G
        g = pc.generate(ctx, handles[rows], rows, last, uids, T, temperature, seed, eos_id, bias,
                        keep_logits_rows=np.arange(n), poll_every=poll_every, compact=compact, keep_logprobs=True)
        pc.pc_release(ctx, handles, 1)
    torch.cuda.synchronize()
    free, total = pc.pc_kv_blocks(ctx)
    assert free == total, "released everything, yet %d of %d blocks are free" % (free, total)
    sat = pc.pc_saturation_count(ctx)
    assert (sat > 0) == expect_saturation, "%d values were clamped to the half range" % sat
    # [steps, n, V]; rows that had left the batch (ragged stop) stay NaN
    logits = np.full((len(g["logits"]), n, model.vocab), np.nan, dtype=np.float32)
    for t, (lg, lr) in enumerate(zip(g["logits"], g["logits_rows"])):
        logits[t, lr.cpu().numpy()] = lg.cpu().numpy()
    out = dict(tokens=g["tokens"].cpu().numpy(), lengths=g["lengths"].cpu().numpy(), logits=logits,
               last=last.cpu().numpy(), uids=uids, rows=rows, steps_run=g["steps_run"],
               logprobs=g["logprobs"].cpu().numpy(),
               rows_decoded=g["rows_decoded"], saturated=sat)
    ctx.close()
    return out


def _check(model, w, prompts_list, out, seed, tol, seqs, temperature=1.0, eos_id=-1, bias=0.0):
    tot = same = own = cnt = 0
    worst = sq = 0.0
    for i in seqs:
        L = int(out["lengths"][i])
        gen = out["tokens"][i, :L]
        gl = out["logits"][:L, i]
        err, s2, c, a_same, a_own = _teacher_forced(model, w, prompts_list[out["rows"][i]], gen, gl,
                                                    int(out["uids"][i]), seed, temperature, eos_id, bias)
        # the log-probability handed on with every token (pi_theta_old of Eq. 2): log-softmax of the logits the
        # token was sampled from, at the sampled token; exactly 0 after the end
        for t in range(L):
            u = philox.sampling_uniform(seed, int(out["uids"][i]), t)
            tok, lp = sampler.sample_token(gl[t], temperature, u, eos_id, bias)
            if tok == gen[t]:
                assert abs(lp - out["logprobs"][i, t]) <= 1e-4 * max(1.0, abs(lp)), (i, t, lp, out["logprobs"][i, t])
        assert not out["logprobs"][i, L:].any()
        worst = max(worst, err)
        sq += s2
        cnt += c
        tot += L
        same += a_same
        own += a_own
    rms = math.sqrt(sq / cnt)
    say("max-abs logit error %.3g (rms %.3g) over %d positions; tokens: %d/%d from the GPU's logits, %d/%d from "
        "the oracle's own" % (worst, rms, tot, same, tot, own, tot))
    assert worst <= tol
    assert same >= math.ceil(0.999 * tot)
    if model.dtype == "fp32":
        assert own >= math.ceil(0.999 * tot)
    else:
        assert own >= math.floor((1.0 - max(0.01, 1.5 * math.sqrt(model.vocab) * rms)) * tot)


def test_fp32_c1_prefill_and_decode():
    say("fp32 C1: 8 prompts x 32, G=4, 16 new tokens")
    m = C1.model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 1), 7)
    prompts = list(workloads.make_prompts(8, 32, m.vocab, 2))
    out = _run_generate(m, w, prompts, 4, 16, 3, dict(block_size=32, kv_pool_bytes=64 << 20, max_slots=256,
                                                     max_ctx=128, max_batch_rows=512))
    # prefill logits of every prompt
    for q in range(8):
        want = decoder.forward_full(m, w, prompts[q], rows=[31])[0]
        assert np.abs(want - out["last"][q]).max() <= 1e-4
    _check(m, w, prompts, out, 3, 1e-4, range(32))


def test_fp32_ragged_prompts_partial_blocks_chunks_and_larger_weights():
    # prompt lengths that leave partially filled blocks (copy-on-fork), several prefill
    # chunks (max_batch_rows < total tokens), contexts that cross block boundaries while
    # decoding, and weights large enough that attention is far from uniform
    say("fp32 ragged prompts, std 0.15")
    m = workloads.scaled(C1, n_q_heads=6, n_kv_heads=2, d_model=96, head_dim=16, d_ff=160, vocab=300).model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 5, std=0.15), 8)
    lens = [1, 31, 32, 33, 64, 70, 5, 97]
    toks, cu = workloads.make_ragged_prompts(lens, m.vocab, 4)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    out = _run_generate(m, w, prompts, 3, 40, 11, dict(block_size=32, kv_pool_bytes=32 << 20, max_slots=64,
                                                      max_ctx=160, max_batch_rows=128), temperature=0.8)
    for q in range(len(lens)):
        want = decoder.forward_full(m, w, prompts[q], rows=[lens[q] - 1])[0]
        assert np.abs(want - out["last"][q]).max() <= 1e-4 * max(1.0, np.abs(want).max())
    _check(m, w, prompts, out, 11, 1e-4, range(0, 24, 2), temperature=0.8)


@pytest.mark.parametrize("d,hq,hkv,hd,dff,V,lens,G", [
    (104, 4, 2, 26, 96, 301, [9, 40], 3),              # reductions of 104: not whole 16s, the plain-ALU kernel
    (112, 4, 2, 32, 352, 1000, [3, 17, 70], 1),        # 7 and 22 chunks of 16 on four waves, 3 decode rows
    (512, 8, 2, 64, 1376, 5001, [150, 301, 90], 5),    # tiles of 16, 32 and 64 rows and columns
    (192, 2, 1, 96, 128, 500, [33, 64, 130], 2),       # attention over heads of 96 and of 160, caches in fragment order
    (320, 4, 2, 160, 160, 500, [1, 63, 97], 2),
])
def test_fp32_gemm_forms(d, hq, hkv, hd, dff, V, lens, G):
    # the bound of the other fp32 tests: float32 sums of up to 1376 products of order 0.02
    say("fp32 d=%d d_ff=%d V=%d" % (d, dff, V))
    m = workloads.scaled(C1, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=dff, vocab=V).model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 6), 8)
    toks, cu = workloads.make_ragged_prompts(lens, V, 4)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    out = _run_generate(m, w, prompts, G, 6, 11, dict(block_size=32, kv_pool_bytes=64 << 20, max_slots=64, max_ctx=352,
                                                     max_batch_rows=600))
    for q in range(len(lens)):
        want = decoder.forward_full(m, w, prompts[q], rows=[lens[q] - 1])[0]
        assert np.abs(want - out["last"][q]).max() <= 1e-4 * max(1.0, np.abs(want).max())
    _check(m, w, prompts, out, 11, 1e-4, range(0, len(lens) * G, 2))


@pytest.mark.parametrize("d,dff,n,scale", [
    (16, 32, 17, 1.0),          # one chunk of 16: three of a block's four waves have nothing to add up
    (48, 96, 1, 1.0),
    (272, 704, 130, 1.0),       # 17 chunks: a second round of loads with one chunk in it; 16 x 16 and 32 x 32 tiles
    (512, 1376, 700, 1.0),      # 64 x 64 tiles with a ragged last one
    (272, 704, 130, 1e-3),      # mean squares far below eps
    (272, 704, 130, 1e4),
])
def test_fp32_norm_inside_the_projection(d, dff, n, scale):
    # against the launches with a norm kernel of their own: each side rounds its normalised rows and sums at most 1376 products of
    # order 0.02 in float32, whose errors are some 2^-24 sqrt(1376) = 2e-6 of the result, a few times that behind two layers.
    # A prompt's logits are the same bits alone and among others.
    say("fp32 norm in the projection, d=%d n=%d scale=%g" % (d, n, scale))
    import paper_2605_26606_amd as pc
    m = workloads.scaled(C1, d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=16, d_ff=dff, vocab=300).model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 6), 8)
    w["tok_embed"] = w["tok_embed"] * scale
    toks, _ = workloads.make_ragged_prompts([n], m.vocab, 4)
    toks = torch.from_numpy(np.ascontiguousarray(toks, dtype=np.int32)).cuda()
    head = max(1, n // 9)

    def logits_of(fuse, cu):   # behind the prompts, and a token later
        ctx = make_ctx(m, w, block_size=32, kv_pool_bytes=64 << 20, max_slots=16, max_ctx=1024, max_batch_rows=1024)
        pc.pc_set_option(ctx, pc.PC_OPT_FUSE_DECODE, fuse)
        last = torch.empty((len(cu) - 1, m.vocab), device="cuda")
        handles = pc.pc_prefill_shared(ctx, toks[:cu[-1]], np.array(cu, np.int32), last)
        seqs = pc.pc_fork(ctx, handles, 1)
        logits = torch.empty_like(last)      # (a vocabulary of 300: the last column tile is a ragged one)
        pc.pc_decode_step(ctx, seqs, toks[:len(cu) - 1], logits)
        out = last.cpu(), logits.cpu()
        ctx.close()
        return out

    cu = [0, head, n] if n > head else [0, n]
    for a, b in zip(logits_of(1, cu), logits_of(0, cu)):
        assert torch.isfinite(a).all() and float((a - b).abs().max()) <= 1e-4 * float(b.abs().max())
    assert torch.equal(logits_of(1, [0, head])[0][0], logits_of(1, cu)[0][0])


@pytest.mark.parametrize("P,G", [(3, 1), (11, 4), (35, 4)])   # up to eight K slices; rows of 704 pieces of 16 bytes
def test_slices_of_heads_of_64(P, G):
    # norm and rotation add up the K slices of projections wide enough to be cut, in heads whose rows lie in plain order (attention on
    # the plain ALU); forks copy blocks of 32 KB with a few tokens in them
    say("heads of 64, %d rows" % (P * G))
    m = workloads.scaled(C1, dtype="bf16", d_model=2816, n_q_heads=32, n_kv_heads=8, head_dim=64, d_ff=2816, vocab=512,
                         n_layers=1, rope_theta=1.0e6).model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 3, std=0.02), 10)
    toks, cu = workloads.make_ragged_prompts([5 + 3 * i % 40 for i in range(P)], m.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(P)]
    out = _run_generate(m, w, prompts, G, 3, 21, dict(block_size=32, kv_pool_bytes=256 << 20, max_slots=P * (G + 1) + 8, max_ctx=128,
                                                     max_batch_rows=1024, act_dtype="f16"))
    _check(m, w, prompts, out, 21, 2e-2, range(0, P * G, max(1, P * G // 6)))


def test_bf16_plain_alu_path():
    say("bf16 small model, plain-ALU kernels")
    import paper_2605_26606_amd as pc
    w = workloads.perturb_norm_gains(workloads.make_weights(BF, 2), 9)
    prompts = list(workloads.make_prompts(3, 40, BF.vocab, 6))
    out = _run_generate(BF, w, prompts, 2, 12, 5, dict(block_size=32, kv_pool_bytes=64 << 20, max_slots=32,
                                                      max_ctx=128, max_batch_rows=256),
                        opts=[(pc.PC_OPT_FORCE_SIMT, 1)])
    _check(BF, w, prompts, out, 5, 2e-2, range(6))


def test_fp32_plain_alu_option():
    # the option holds for fp32 models too: within the bound of the matrix instructions, but not their sums to the last bit
    say("fp32 small model, plain-ALU kernels by option")
    import paper_2605_26606_amd as pc
    m = C1.model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 2), 9)
    prompts = list(workloads.make_prompts(3, 40, m.vocab, 6))
    kw = dict(block_size=32, kv_pool_bytes=64 << 20, max_slots=32, max_ctx=128, max_batch_rows=256)
    a = _run_generate(m, w, prompts, 2, 6, 5, kw, opts=[(pc.PC_OPT_FORCE_SIMT, 1)])
    b = _run_generate(m, w, prompts, 2, 6, 5, kw)
    _check(m, w, prompts, a, 5, 1e-4, range(6))
    assert not np.array_equal(a["last"], b["last"])


@pytest.mark.parametrize("model,lens,G,T,bs,std,act", [
    (BF, [70, 33, 128, 5, 64], 4, 24, 64, 0.02, "f16"),   # the workloads' init: absolute 2e-2 bound
    (BF, [70, 33, 128, 5, 64], 4, 24, 64, 0.02, "bf16"),  # same with bfloat16 activations
    (BF, [70, 33, 128, 5, 64], 4, 24, 64, 0.05, "f16"),   # 6 query heads per kv head, ragged, partial blocks
    (BF4, [600, 17, 520], 3, 40, 32, 0.05, "f16"),        # long contexts cut into splits, 4 heads per kv head
    (BF4, [600, 17, 520], 3, 40, 32, 0.05, "bf16"),
    (BF, [40] * 64 + [7], 4, 6, 64, 0.02, "f16"),         # 260 sequences: one split per sequence, direct output
    (BF8, [100, 31], 3, 10, 64, 0.02, "f16"),             # split-K in the large-tile GEMM
    (BF8, [100, 31], 3, 10, 64, 0.02, "bf16"),
    (BF8, [12] * 75, 4, 5, 64, 0.02, "f16"),              # 300 decode rows: two 192-row GEMM blocks, tall K slices
    (BF8, [12] * 6, 43, 3, 64, 0.02, "f16"),              # 258, 384 and 385 rows: each side of the long reductions' tile heights
    (BF8, [12] * 16, 24, 3, 64, 0.02, "f16"),
    (BF8, [12] * 11, 35, 3, 64, 0.02, "f16"),
    (BF8, [12] * 105, 4, 4, 64, 0.02, "f16"),             # 420 decode rows: gate/up on the large tiles, the rest in four 128-row blocks
    (BF8, [12] * 130, 4, 3, 64, 0.02, "f16"),             # 520 decode rows: the large-batch tiles, narrow outputs in K slices
    (BF, [70, 33, 300, 5, 256], 3, 10, 128, 0.02, "f16"), # larger KV blocks
    (BF, [70, 33, 300, 5, 256], 3, 10, 256, 0.02, "f16"), # the largest block size the cache accepts
    (BF48, [150, 9, 64, 257], 4, 12, 64, 0.02, "f16"),    # 32 query / 8 kv heads
    (BF58, [150, 9, 64, 257], 4, 12, 64, 0.02, "f16"),    # 40 query / 8 kv heads: 5 per kv head, one head per prefill wave
    (BF58, [20] * 40, 4, 5, 64, 0.02, "bf16"),            # 160 rows x 8 kv heads: the 4-wave decode blocks
    (BFW, [10] * 20 + [37], 4, 4, 64, 0.02, "f16"),       # 84 rows: 128x128 tiles in K slices
    (BFW, [10] * 40 + [37], 4, 4, 64, 0.02, "f16"),       # 164 rows: 256x128 tiles in K slices
    (BFW, [9] * 70, 4, 4, 64, 0.02, "f16"),               # 280 rows: two 256-row blocks per weight tile
])
def test_bf16_matrix_core_path(model, lens, G, T, bs, std, act):
    say("bf16 model, matrix-core path, %s activations, lens=%s G=%d T=%d std=%g" % (act, lens[:6], G, T, std))
    w = workloads.perturb_norm_gains(workloads.make_weights(model, 3, std=std), 10)
    toks, cu = workloads.make_ragged_prompts(lens, model.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    out = _run_generate(model, w, prompts, G, T, 21, dict(block_size=bs, kv_pool_bytes=512 << 20,
                                                         max_slots=len(lens) * (G + 1) + 8, max_ctx=1024,
                                                         max_batch_rows=1024, act_dtype=act))
    for q in range(len(lens)):
        want = decoder.forward_full(model, w, prompts[q], rows=[lens[q] - 1])[0]
        assert np.abs(want - out["last"][q]).max() <= 2e-2 * max(1.0, np.abs(want).max())
        if std == 0.02:
            assert np.abs(want - out["last"][q]).max() <= 2e-2
    _check(model, w, prompts, out, 21, 2e-2, range(0, len(lens) * G, max(2, len(lens) * G // 12)))


# outputs wide enough for unsplit tiles: 8192 and 12992 columns of 128-wide tiles, and 34816 and 33024 columns, for which
# 128-wide tiles would need a second round of blocks and 192-wide ones do not
WIDE1 = workloads.scaled(C1, dtype="bf16", d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=6400, vocab=12992,
                         n_layers=1, rope_theta=1.0e6).model
WIDE2 = workloads.scaled(C1, dtype="bf16", d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=17408, vocab=33024,
                         n_layers=1, rope_theta=1.0e6).model


@pytest.mark.parametrize("model,P,G,act", [(WIDE1, 3, 1, "f16"), (WIDE1, 11, 3, "f16"), (WIDE1, 13, 5, "f16"),
                                           (WIDE1, 43, 3, "f16"), (WIDE1, 49, 4, "f16"), (WIDE1, 64, 4, "bf16"),
                                           (WIDE2, 1, 1, "f16"), (WIDE2, 8, 4, "f16"), (WIDE2, 16, 4, "bf16"),
                                           (WIDE2, 32, 4, "f16"), (WIDE2, 64, 3, "f16"), (WIDE2, 65, 3, "f16"),
                                           (WIDE1, 65, 4, "f16"), (WIDE2, 77, 5, "bf16")])
def test_wide_tiles_by_row_count(model, P, G, act):
    # decode batches of 3, 33, 65, 129, 196, 256, 260 and of 1, 32, 64, 128, 192, 195, 385 rows: each side of the tiles' heights
    say("wide tiles, d_ff %d, %d rows" % (model.d_ff, P * G))
    w = workloads.perturb_norm_gains(workloads.make_weights(model, 3), 10)
    rng = np.random.default_rng(P)
    lens = rng.integers(1, 9, P).tolist()
    toks, cu = workloads.make_ragged_prompts(lens, model.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(P)]
    out = _run_generate(model, w, prompts, G, 3, 21, dict(block_size=32, kv_pool_bytes=256 << 20,
                                                         max_slots=P * (G + 1) + 8, max_ctx=64, max_batch_rows=600,
                                                         act_dtype=act))
    _check(model, w, prompts, out, 21, 2e-2, range(0, P * G, max(1, P * G // 6)))


# a vocabulary of 513 column blocks: the head of a decode step on the large tiles; its gate/up, without and with the norm scale
VOC1 = workloads.scaled(C1, dtype="bf16", d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=6400, vocab=65552,
                        n_layers=1, rope_theta=1.0e6).model
VOC2 = workloads.scaled(C1, dtype="bf16", d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=20512, vocab=512,
                        n_layers=2, rope_theta=1.0e6).model
# (those two with reductions too short for the large tiles up to 512 rows, these with longer ones)
VOC3 = workloads.scaled(C1, dtype="bf16", d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=640, vocab=65552,
                        n_layers=1, rope_theta=1.0e6).model
VOC4 = workloads.scaled(C1, dtype="bf16", d_model=384, n_q_heads=3, n_kv_heads=1, head_dim=128, d_ff=20512, vocab=512,
                        n_layers=2, rope_theta=1.0e6).model


@pytest.mark.parametrize("model,P,G,act", [(VOC1, 48, 4, "f16"), (VOC1, 193, 1, "f16"), (VOC1, 64, 4, "bf16"), (VOC1, 257, 1, "f16"),
                                           (VOC1, 96, 4, "f16"), (VOC1, 77, 5, "f16"), (VOC1, 128, 4, "bf16"), (VOC1, 171, 3, "f16"),
                                           (VOC2, 64, 3, "f16"), (VOC2, 193, 1, "f16"), (VOC2, 64, 4, "f16"), (VOC2, 77, 5, "f16"),
                                           (VOC2, 128, 4, "bf16"), (VOC2, 128, 4, "f16"), (WIDE1, 128, 4, "f16"), (WIDE1, 96, 4, "f16"),
                                           (VOC3, 48, 4, "f16"), (VOC3, 193, 1, "f16"), (VOC3, 64, 4, "bf16"), (VOC3, 257, 1, "f16"),
                                           (VOC3, 96, 4, "f16"), (VOC3, 77, 5, "f16"), (VOC3, 128, 4, "bf16"), (VOC3, 171, 3, "f16"),
                                           (VOC4, 64, 3, "f16"), (VOC4, 96, 4, "f16"), (VOC4, 77, 5, "f16"), (VOC4, 128, 4, "bf16"),
                                           (VOC4, 171, 3, "f16")])
def test_large_tiles_of_decode_batches(model, P, G, act):
    # 192, 193, 256, 257, 384, 385, 512 and 513 rows: each side of the rules that send a step's projections to the large tiles;
    # gate/up of 41024 columns runs several tiles per block, each with row scales of its own
    say("large tiles in decode, d_ff %d, vocabulary %d, %d rows" % (model.d_ff, model.vocab, P * G))
    w = workloads.perturb_norm_gains(workloads.make_weights(model, 3), 10)
    lens = np.random.default_rng(P).integers(1, 9, P).tolist()
    toks, cu = workloads.make_ragged_prompts(lens, model.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(P)]
    out = _run_generate(model, w, prompts, G, 2, 21, dict(block_size=32, kv_pool_bytes=256 << 20,
                                                         max_slots=P * (G + 1) + 8, max_ctx=64, max_batch_rows=1400,
                                                         act_dtype=act))
    _check(model, w, prompts, out, 21, 2e-2, list(range(0, P * G, max(1, P * G // 6))) + [P * G - 1])


@pytest.mark.parametrize("hq,hkv,lens,bs,act,d", [
    (8, 2, [201, 3, 190, 128, 90], 32, "f16", 128),             # 612 rows x 1536 columns: 64 x 128 tiles, eight waves
    (8, 2, [333, 201, 3, 300, 66, 400, 201], 32, "f16", 128),   # 1504 x 1536: 128 x 128
    (32, 8, [201, 3, 190, 128, 178], 64, "bf16", 128),          # 700 x 6144: 256 x 128
    (48, 8, [201, 3, 190, 128, 38], 32, "f16", 128),            # 560 x 8192: rotation in a kernel of its own
    (48, 8, [201, 3, 190, 128, 78], 32, "f16", 128),            # 600 x 8192: 256 x 128
    (48, 8, [333, 1, 300, 65, 301], 64, "f16", 128),            # 1000 x 8192: the same, one full round
    (48, 8, [700, 9, 650, 800, 777, 640, 555], 64, "f16", 128),   # 4131 x 8192: 192 x 128 on four waves, a row tile with 99 rows
    (48, 8, [700, 9, 650, 800, 777, 640, 555], 128, "bf16", 128),
    (48, 8, [333, 1, 300, 65, 601], 64, "f16", 1024),           # 1300 x 8192 x 1024: 192 x 256
    (32, 8, [700, 9, 650, 800, 777, 640, 555], 64, "f16", 1024),  # 4131 x 6144 x 1024: 256 x 256, a row tile with 35 rows
])
def test_projection_that_rotates_and_appends(hq, hkv, lens, bs, act, d):
    # prefill chunks of more than 512 rows: q, k and v leave the projection rotated and filed; sequences start anywhere in a
    # tile and in a KV block, and two decode steps read the cache back
    say("q/k/v projection with rotary positions, %d rows x %d columns" % (sum(lens), (hq + 2 * hkv) * 128))
    m = workloads.scaled(C1, dtype="bf16", d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ff=128, vocab=512,
                         n_layers=2, rope_theta=1.0e6).model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 3, std=0.05 if d == 128 else 0.02), 10)
    toks, cu = workloads.make_ragged_prompts(lens, m.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    out = _run_generate(m, w, prompts, 2, 3, 21, dict(block_size=bs, kv_pool_bytes=256 << 20, max_slots=40, max_ctx=900,
                                                     max_batch_rows=4200, act_dtype=act))
    for q in range(len(lens)):
        want = decoder.forward_full(m, w, prompts[q], rows=[lens[q] - 1])[0]
        assert np.abs(want - out["last"][q]).max() <= 2e-2 * max(1.0, np.abs(want).max())
    _check(m, w, prompts, out, 21, 2e-2, range(0, len(lens) * 2, 3))


@pytest.mark.parametrize("d,dff,vocab,lens,act", [
    (192, 6400, 528, [700, 9, 650, 800, 777, 640, 555], "f16"),   # 4131 rows: several tiles per block, 3 steps of 64 to a tile
    (192, 6400, 528, [700, 9, 650, 800, 777, 640, 555], "bf16"),
    (320, 320, 8208, [513], "f16"),                               # one row beyond the small batches, 5 steps
    (128, 1184, 8208, [190] * 70 + [257], "f16"),                 # two steps to a tile; 13557 rows in chunks; 80 last rows
    (2048, 384, 528, [333, 201, 300], "f16"),                     # 834 rows of a wide model: residual projections in 128 x 64 tiles
    (2048, 2112, 528, [333, 201, 300], "f16"),                    # down just beyond those: K slices in the large tiles
    (208, 320, 528, [513], "f16"),                                # 64 x 64 tiles: one row and 16 columns in the last ones
    (960, 2048, 528, [700, 9, 650, 577], "bf16"),                 # 1936 rows in 240 blocks of 128 x 64; their longest reduction
    (2560, 256, 528, [190, 323], "f16"),                          # 513 rows x 2560: 360 blocks of 64 x 64, 200 of 128 x 64
    # short reductions, eight waves: gate/up (K = 64) in 256 x 256 tiles, q/k/v in 128 x 128 two to a CU; down (K = 128) in 256 x 256
    (64, 6400, 528, [700, 9, 650, 800, 777, 640, 555], "f16"),
    (8192, 128, 528, [700, 9, 650, 800, 777, 640, 555], "f16"),
])
def test_many_rows(d, dff, vocab, lens, act):
    # batches of more than 512 rows: runs of tiles, remainders in rows and columns, odd numbers of steps between two tiles
    say("%d rows, d_model %d, d_ff %d, %s" % (sum(lens), d, dff, act))
    m = workloads.scaled(C1, dtype="bf16", d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=dff, vocab=vocab,
                         n_layers=2, rope_theta=1.0e6).model
    # (The logits' spread is std sqrt(d).  The bound on the oracle's own tokens, 1.5 sqrt(V) rms misses, is for near-uniform
    # distributions; in general a uniform falls between the two sides' boundaries with a chance of about V rms sqrt(sum p^2) / 2, and
    # sum p^2 is exp(spread^2) / V.  At a spread of 1.8 and an rms of 0.0046 that is 27 % against a bound of 16 %; at half of both,
    # the spread of the 2048-wide model, 4 % against 8 %.)
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 3, std=0.02 if d <= 2048 else 0.01), 10)
    toks, cu = workloads.make_ragged_prompts(lens, m.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    out = _run_generate(m, w, prompts, 1, 2, 21, dict(block_size=64, kv_pool_bytes=512 << 20, max_slots=160, max_ctx=900,
                                                     max_batch_rows=4200, act_dtype=act))
    for q in range(0, len(lens), max(1, len(lens) // 9)):
        want = decoder.forward_full(m, w, prompts[q], rows=[lens[q] - 1])[0]
        assert np.abs(want - out["last"][q]).max() <= 2e-2 * max(1.0, np.abs(want).max())
    _check(m, w, prompts, out, 21, 2e-2, range(0, len(lens), max(1, len(lens) // 9)))


@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_many_rows_of_a_64_wide_model(act):
    # every reduction but the down projection's is a single step of 64: prefill and decode of more than 512 rows
    say("64-wide model, %s" % act)
    m = workloads.scaled(C1, dtype="bf16", d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=1184, vocab=65552,
                         n_layers=2, rope_theta=1.0e6).model
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 3, std=0.05), 10)
    lens = np.random.default_rng(4).integers(1, 9, 173).tolist()
    toks, cu = workloads.make_ragged_prompts(lens, m.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    out = _run_generate(m, w, prompts, 3, 2, 21, dict(block_size=32, kv_pool_bytes=256 << 20, max_slots=720, max_ctx=64,
                                                     max_batch_rows=1400, act_dtype=act))
    _check(m, w, prompts, out, 21, 2e-2, [0, 100, 259, 400, 518])


def test_output_projection_and_logits_off_16_byte_boundaries():
    # an lm_head two bytes into an allocation (a view into a flat buffer of parameters), logits one float into theirs: the same
    # bits as from aligned ones, for prefill, decode and scoring of few and of many rows; the misaligned head is copied by
    # pc_create, its memory may change afterwards
    import paper_2605_26606_amd as pc
    say("lm_head and logits off 16-byte boundaries")
    m = workloads.scaled(C1, dtype="bf16", d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=256, vocab=65552,
                         n_layers=1, rope_theta=1.0e6).model
    w = workloads.weights_to(workloads.perturb_norm_gains(workloads.make_weights(m, 3), 10), "cuda")
    rng = np.random.default_rng(5)
    results = []
    for off in (0, 1):
        wd = dict(w)
        flat = torch.empty(m.vocab * m.d_model + 8, dtype=torch.bfloat16, device="cuda")
        wd["lm_head"] = flat[off:off + m.vocab * m.d_model].view(m.vocab, m.d_model)
        wd["lm_head"].copy_(w["lm_head"])
        ctx = pc.Context(m, wd, block_size=32, kv_pool_bytes=256 << 20, max_slots=1400, max_ctx=64, max_batch_rows=1400, act_dtype="bf16")
        if off:
            flat.zero_()
        got = []
        for P in (3, 200, 600):
            toks = torch.from_numpy(np.random.default_rng(P).integers(0, m.vocab, 2 * P).astype(np.int32)).cuda()
            cu = (np.arange(P + 1) * 2).astype(np.int32)
            last = torch.empty(P * m.vocab + 4, device="cuda")[off:off + P * m.vocab].view(P, m.vocab)
            logits = torch.empty(P * m.vocab + 4, device="cuda")[off:off + P * m.vocab].view(P, m.vocab)
            handles = pc.pc_prefill_shared(ctx, toks, cu, last)
            seqs = pc.pc_fork(ctx, handles, 4)
            pc.pc_decode_step(ctx, seqs, toks[:P], logits)
            pc.pc_release(ctx, seqs, 0)
            pc.pc_release(ctx, handles, 1)
            score = torch.empty(P, device="cuda")
            pc.pc_score(ctx, toks, cu, np.ones(P, np.int32), 1.0, score)
            got += [last.clone(), logits.clone(), score]
        torch.cuda.synchronize()
        ctx.close()
        results.append(got)
    assert float(results[0][0].abs().max()) > 0.05
    for a, b in zip(*results):
        assert torch.equal(a, b)


def test_attention_keeps_the_largest_probability_exact():
    # One key holds nearly all of a head's weight, in a later tile than the largest score before it.  Its probability is 1 and
    # must not round: weighted values and weights are then summed alike and the output is the value itself.  (Taken relative to
    # the earlier score it would be 2^2 .. 2^7.3 here, picked so that half rounds it by 2e-4 to 4e-4 of itself, up in every
    # other head.)  Scores are sums of +-1 times the query weights, exact in half, and the dims in use have rotary angles of
    # zero.  Logit h is the sum of head h's outputs over 128 dims: their own rounding averages to 2^-12 / sqrt(3 * 128) =
    # 1.2e-5, twice (attention output, normalised row); three standard deviations of both and an equal share for the weights
    # below the largest: 6e-5.
    m = workloads.scaled(C1, dtype="bf16", d_model=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ff=64, vocab=512,
                         n_layers=1, rope_theta=1.0e30).model
    say("largest probability exact")
    w = workloads.make_weights(m, 1)
    for k in ("wq", "wk", "wv", "wo", "w_down"):
        w[k][0].zero_()
    sign = torch.randint(0, 2, (m.vocab, m.d_model), generator=torch.Generator().manual_seed(2)) * 2.0 - 1.0
    sign[:, 0] = 1.0                                      # query and value source
    sign[:, 1:3] = -1.0                                   # token 1: the largest score of the first tile, token 2: the peak
    sign[1, 1] = sign[2, 1] = sign[2, 2] = 1.0
    w["tok_embed"].copy_(sign)
    dims = torch.arange(32, 64), torch.arange(96, 128)
    for h, second in enumerate((192, 158, 164, 227, 223, 220, 95, 161)):
        w["wq"][0][128 * h + dims[0], 0] = 2.5
        w["wq"][0][128 * h + dims[1], 0] = second / 256.0
        w["wo"][0][128 * h + torch.arange(128), 128 * h + torch.arange(128)] = 1.0
    for g in range(2):
        w["wk"][0][128 * g + dims[0], 1] = 1.0
        w["wk"][0][128 * g + dims[1], 2] = 1.0
        w["wv"][0][128 * g + torch.arange(128), 0] = (1.0 + torch.arange(128) / 128.0).to(torch.bfloat16)
    w["lm_head"].zero_()
    for h in range(8):
        w["lm_head"][h, 128 * h:128 * (h + 1)] = 1.0
    prompt = np.zeros(300, dtype=np.int64)
    prompt[5], prompt[260] = 1, 2                         # (decode: eight waves take every eighth tile of 32)
    want = decoder.forward_full(m, w, np.append(prompt, 0), rows=[299, 300])[:, :8]
    import paper_2605_26606_amd as pc
    ctx = make_ctx(m, w, block_size=32, kv_pool_bytes=64 << 20, max_slots=130, max_ctx=320, max_batch_rows=512, act_dtype="f16")
    last = torch.empty(1, m.vocab, device="cuda")
    handle = pc.pc_prefill_shared(ctx, torch.from_numpy(prompt.astype(np.int32)).cuda(), np.array([0, 300], np.int32), last)
    seqs = pc.pc_fork(ctx, np.repeat(handle, 100), 4)     # 200 (row, kv head) pairs: contexts are not split
    logits = torch.empty(100, m.vocab, device="cuda")
    pc.pc_decode_step(ctx, seqs, torch.zeros(100, dtype=torch.int32, device="cuda"), logits)
    torch.cuda.synchronize()
    for name, got, ref in (("prefill", last[0, :8], want[0]), ("decode", logits[99, :8], want[1])):
        err = np.abs(got.cpu().numpy() / ref - 1.0)
        say("%s: relative errors %s" % (name, " ".join("%.1e" % e for e in err)))
        assert err.max() <= 6e-5
    ctx.close()


def test_graph_replay_equals_eager_and_is_deterministic():
    say("graph vs eager, bf16")
    import paper_2605_26606_amd as pc
    w = workloads.make_weights(BF, 4, std=0.05)
    prompts = list(workloads.make_prompts(4, 100, BF.vocab, 12))
    kw = dict(block_size=64, kv_pool_bytes=128 << 20, max_slots=64, max_ctx=1024, max_batch_rows=512)
    a = _run_generate(BF, w, prompts, 4, 30, 2, kw, opts=[(pc.PC_OPT_USE_GRAPH, 1)])
    b = _run_generate(BF, w, prompts, 4, 30, 2, kw, opts=[(pc.PC_OPT_USE_GRAPH, 0)])
    c = _run_generate(BF, w, prompts, 4, 30, 2, kw, opts=[(pc.PC_OPT_USE_GRAPH, 1)])
    assert np.array_equal(a["tokens"], b["tokens"]) and np.array_equal(a["logits"], b["logits"])
    assert np.array_equal(a["tokens"], c["tokens"]) and np.array_equal(a["logits"], c["logits"])


def test_captured_step_replays_for_other_lists():
    # one context, stream and pair of buffers; lists of the same length and grouping over other slots and lengths, a list over
    # released and reused slots, a permuted one, and one of another grouping in between: every step equals the eager one
    import paper_2605_26606_amd as pc
    say("captured step with other lists")
    w = workloads.make_weights(BF, 4, std=0.05)
    toks, cu = workloads.make_ragged_prompts([100, 7, 260, 33, 64, 190], BF.vocab, 8)
    feed = torch.from_numpy(np.random.default_rng(5).integers(0, BF.vocab, (14, 6)).astype(np.int32)).cuda()
    runs = []
    for graph in (1, 0):
        ctx = make_ctx(BF, w, block_size=64, kv_pool_bytes=128 << 20, max_slots=64, max_ctx=512, max_batch_rows=800)
        pc.pc_set_option(ctx, pc.PC_OPT_USE_GRAPH, graph)
        out = []
        with torch.cuda.stream(side_stream()):
            last = torch.empty(6, BF.vocab, device="cuda")
            h = pc.pc_prefill_shared(ctx, torch.from_numpy(toks.astype(np.int32)).cuda(), cu.astype(np.int32), last)
            tokens, logits = torch.empty(6, dtype=torch.int32, device="cuda"), torch.empty(6, BF.vocab, device="cuda")

            def steps(seqs, n):
                for _ in range(n):
                    tokens.copy_(feed[len(out)])
                    pc.pc_decode_step(ctx, seqs, tokens, logits)
                    out.append(logits.clone())

            a = pc.pc_fork(ctx, np.repeat(h[:3], 2), 16)
            b = pc.pc_fork(ctx, np.repeat(h[3:], 2), 16)
            steps(a, 2)
            steps(b, 2)
            steps(a[[4, 5, 0, 1, 2, 3]], 2)              # the same sequences, prompts in another order
            pc.pc_release(ctx, b[:4], 0)
            c = pc.pc_fork(ctx, np.repeat(h[[0, 5]], 2), 16)
            steps(np.concatenate([c, a[2:4]]), 2)         # reused slots beside sequences that have decoded
            steps(np.concatenate([a[::2], b[4:5], c[::2]]), 2)   # single sequences: another grouping
            steps(a, 2)
            steps(np.concatenate([b[4:], c]), 2)
        torch.cuda.synchronize()
        runs.append(out)
        ctx.close()
    assert len(runs[0]) == 14
    for t, (x, y) in enumerate(zip(*runs)):
        assert torch.equal(x, y), "step %d" % t


def test_eos_stops_sequences_fp32():
    say("fp32 C1 with a biased EOS id")
    m = C1.model
    w = workloads.make_weights(m, 1)
    prompts = list(workloads.make_prompts(4, 20, m.vocab, 2))
    eos = workloads.make_eos_id(m.vocab, 4)
    bias = math.log(m.vocab / 6.0)
    out = _run_generate(m, w, prompts, 4, 24, 3, dict(block_size=32, kv_pool_bytes=32 << 20, max_slots=64,
                                                     max_ctx=64, max_batch_rows=128), eos_id=eos, bias=bias)
    lens = out["lengths"]
    assert (lens < 24).any()
    for i in range(16):
        L = int(lens[i])
        assert (out["tokens"][i, :L - 1] != eos).all()
        if L < 24:
            assert out["tokens"][i, L - 1] == eos and (out["tokens"][i, L:] == eos).all()
    _check(m, w, prompts, out, 3, 1e-4, range(16), eos_id=eos, bias=bias)


@pytest.mark.parametrize("name", ["fp32", "f16"])
def test_ragged_stop_shrinks_the_batch(name):
    # sequences that hit EOS leave the decode batch at the next poll; what the others generate is unchanged
    m = C1.model if name == "fp32" else BF
    say("ragged stop, %s: 4 prompts x 8 rollouts, 72 new tokens, poll every 8 steps" % name)
    w = workloads.perturb_norm_gains(workloads.make_weights(m, 1), 7)
    prompts = list(workloads.make_prompts(4, 20, m.vocab, 2))
    eos = workloads.make_eos_id(m.vocab, 4)
    bias = math.log(m.vocab / 12.0)             # hazard about 1/12 per step
    kw = dict(block_size=32, kv_pool_bytes=64 << 20, max_slots=96, max_ctx=128, max_batch_rows=128)
    a = _run_generate(m, w, prompts, 8, 72, 3, kw, eos_id=eos, bias=bias, poll_every=8, compact=True)
    b = _run_generate(m, w, prompts, 8, 72, 3, kw, eos_id=eos, bias=bias, poll_every=8, compact=False)
    lens = a["lengths"]
    say("lengths %s; batch rows decoded %d with compaction, %d without" % (sorted(lens.tolist()), a["rows_decoded"],
                                                                        b["rows_decoded"]))
    assert (lens < 72).sum() >= 16 and a["rows_decoded"] < b["rows_decoded"]
    for i in range(32):
        L = int(lens[i])
        assert (a["tokens"][i, :L - 1] != eos).all()
        if L < 72:
            assert a["tokens"][i, L - 1] == eos and (a["tokens"][i, L:] == eos).all()
        assert not np.isnan(a["logits"][:L, i]).any()      # every token was sampled from recorded logits
    if name == "fp32":   # the plain-ALU kernels treat a row the same whatever else is in the batch
        assert np.array_equal(a["tokens"], b["tokens"]) and np.array_equal(lens, b["lengths"])
    _check(m, w, prompts, a, 3, 1e-4 if name == "fp32" else 2e-2, range(0, 32, 3), eos_id=eos, bias=bias)


@pytest.mark.parametrize("kept", [[2, 0], [-1, 0, 2, 2], [[0, 1], [5, -2]], []])
def test_kept_logits_of_any_index_form(kept):
    import paper_2605_26606_amd as pc
    w = workloads.make_weights(C1.model, 3)
    ctx = make_ctx(C1.model, w, block_size=32, kv_pool_bytes=16 << 20, max_slots=32, max_ctx=64, max_batch_rows=64)
    rows = np.repeat(np.arange(2, dtype=np.int32), 3)
    toks = torch.arange(24, dtype=torch.int32, device="cuda")
    got = []
    with torch.cuda.stream(side_stream()):
        last = torch.empty((2, C1.model.vocab), device="cuda")
        handles = pc.pc_prefill_shared(ctx, toks, np.array([0, 9, 24], np.int32), last)
        for keep in (np.arange(6), np.array(kept, np.int64)):
            g = pc.generate(ctx, handles[rows], rows, last, rows.astype(np.int64) * 65536 + np.arange(6), 4, 1.0, 5, keep_logits_rows=keep)
            got.append(g)
    torch.cuda.synchronize()
    at = torch.as_tensor(kept, dtype=torch.long)
    assert torch.equal(got[0]["tokens"], got[1]["tokens"])
    for t in range(4):
        assert torch.equal(got[1]["logits_rows"][t].cpu(), at)
        assert torch.equal(got[1]["logits"][t].cpu(), got[0]["logits"][t].cpu()[at])
    ctx.close()


def test_error_paths_leave_state_unchanged():
    import paper_2605_26606_amd as pc
    m = C1.model
    w = workloads.make_weights(m, 1)
    ctx = make_ctx(m, w, block_size=32, kv_pool_bytes=2 * 2 * 2 * 32 * 32 * 4 * 6, max_slots=8, max_ctx=96,
                   max_batch_rows=64)
    free0, total = pc.pc_kv_blocks(ctx)
    assert total == 6
    toks = torch.zeros(200, dtype=torch.int32, device="cuda")
    last = torch.empty((1, m.vocab), device="cuda")
    with pytest.raises(pc.PcError) as e:          # prompt longer than max_batch_rows
        pc.pc_prefill_shared(ctx, toks, [0, 65], last)
    assert e.value.code == -1
    with pytest.raises(pc.PcError) as e:          # empty prompt
        pc.pc_prefill_shared(ctx, toks, [0, 0], last)
    assert e.value.code == -1
    last7 = torch.empty((7, m.vocab), device="cuda")
    with pytest.raises(pc.PcError) as e:          # 7 prompts x 1 block > 6 blocks
        pc.pc_prefill_shared(ctx, toks, np.arange(8) * 8, last7)
    assert e.value.code == -2
    assert pc.pc_kv_blocks(ctx)[0] == free0
    h = pc.pc_prefill_shared(ctx, toks, [0, 40], last)
    assert pc.pc_kv_blocks(ctx)[0] == free0 - 2
    with pytest.raises(pc.PcError) as e:          # 3 forks x (1 private + ...) blocks do not fit
        pc.pc_fork(ctx, [h[0]] * 5, 20)
    assert e.value.code == -2
    assert pc.pc_kv_blocks(ctx)[0] == free0 - 2
    with pytest.raises(pc.PcError):               # beyond max_ctx
        pc.pc_fork(ctx, [h[0]], 100)
    with pytest.raises(pc.PcError):               # not a prompt handle
        pc.pc_fork(ctx, [7], 4)
    s = pc.pc_fork(ctx, [h[0], h[0]], 2)
    cur = torch.zeros(2, dtype=torch.int32, device="cuda")
    lg = torch.empty((2, m.vocab), device="cuda")
    with pytest.raises(pc.PcError):               # repeated sequence
        pc.pc_decode_step(ctx, [s[0], s[0]], cur, lg)
    with pytest.raises(pc.PcError):               # a prompt handle is not a sequence
        pc.pc_decode_step(ctx, [h[0]], cur, lg)
    for _ in range(2):                            # 40 prompt tokens + the 2 reserved new ones
        pc.pc_decode_step(ctx, s, cur, lg)
    with pytest.raises(pc.PcError) as e:          # the reservation is used up, although the last block has room
        pc.pc_decode_step(ctx, s, cur, lg)
    assert e.value.code == -1
    pc.pc_release(ctx, s, 0)
    with pytest.raises(pc.PcError):
        pc.pc_release(ctx, s, 0)                  # already released
    pc.pc_release(ctx, h, 1)
    torch.cuda.synchronize()
    assert pc.pc_kv_blocks(ctx)[0] == total
    ctx.close()


def test_decode_stops_at_the_reservation_and_at_max_ctx():
    # max_ctx is not a multiple of the block size: the last block could hold tokens beyond max_ctx (and beyond
    # the rotary tables); the step that would write them is refused on the host
    import paper_2605_26606_amd as pc
    m = C1.model
    w = workloads.make_weights(m, 1)
    ctx = make_ctx(m, w, block_size=64, kv_pool_bytes=64 << 20, max_slots=8, max_ctx=100, max_batch_rows=128)
    toks = torch.zeros(96, dtype=torch.int32, device="cuda")
    last = torch.empty((1, m.vocab), device="cuda")
    h = pc.pc_prefill_shared(ctx, toks, [0, 96], last)
    with pytest.raises(pc.PcError):               # 96 + 5 > max_ctx
        pc.pc_fork(ctx, [h[0]], 5)
    s = pc.pc_fork(ctx, [h[0]], 4)                # up to position 99 = max_ctx - 1
    cur = torch.zeros(1, dtype=torch.int32, device="cuda")
    lg = torch.empty((1, m.vocab), device="cuda")
    for _ in range(4):
        pc.pc_decode_step(ctx, s, cur, lg)
    free_before = pc.pc_kv_blocks(ctx)[0]
    with pytest.raises(pc.PcError) as e:          # the block has 28 more places, the reservation has none
        pc.pc_decode_step(ctx, s, cur, lg)
    assert e.value.code == -1 and pc.pc_kv_blocks(ctx)[0] == free_before
    torch.cuda.synchronize()
    assert torch.isfinite(lg).all()
    pc.pc_release(ctx, s, 0)
    pc.pc_release(ctx, h, 1)
    assert pc.pc_kv_blocks(ctx)[0] == pc.pc_kv_blocks(ctx)[1]
    ctx.close()


@pytest.mark.parametrize("act,floor", [("f16", 0.99), ("bf16", 0.97)])
def test_peaked_distributions_token_agreement(act, floor):
    # The ">= 99 % of sampled tokens" criterion where it means something: at temperature 0.01 the top token holds
    # most of the mass, so a logit error of the 16-bit pipeline only matters when the uniform lands next to one of
    # the few heavy CDF boundaries.  Tokens sampled from the oracle's OWN logits (teacher-forced, same uniform)
    # must agree with the GPU's on >= 99 % of positions for half activations (the acceptance type); bfloat16
    # activations carry eight times the rounding error and are held to 97 %.
    say("peaked next-token distributions (temperature 0.01), %s activations" % act)
    w = workloads.perturb_norm_gains(workloads.make_weights(BF, 3, std=0.02), 10)
    lens = [70, 33, 128, 5, 64]
    toks, cu = workloads.make_ragged_prompts(lens, BF.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    G, T, temp = 4, 24, 0.01
    out = _run_generate(BF, w, prompts, G, T, 21, dict(block_size=64, kv_pool_bytes=256 << 20, max_slots=64, max_ctx=512,
                                                      max_batch_rows=512, act_dtype=act), temperature=temp)
    tot = own = same = 0
    top = []
    for i in range(len(lens) * G):
        gen = out["tokens"][i]
        seq = np.concatenate([prompts[out["rows"][i]], gen])
        Lp = len(seq) - T
        want = decoder.forward_full(BF, w, seq[:-1], rows=np.arange(Lp - 1, len(seq) - 1))
        for t in range(T):
            u = philox.sampling_uniform(21, int(out["uids"][i]), t)
            own += int(sampler.sample_token(want[t], temp, u)[0] == gen[t])
            same += int(sampler.sample_token(out["logits"][t, i], temp, u)[0] == gen[t])
            tot += 1
        top.append(np.array([sampler.softmax_probs(want[t], temp).max() for t in range(T)]))
    top = np.concatenate(top)
    say("%d/%d tokens from the oracle's own logits, %d/%d from the GPU's; mean mass of the top token %.2f"
        % (own, tot, same, tot, top.mean()))
    assert top.mean() > 0.7                          # the distributions are peaked indeed
    assert len(set(out["tokens"].reshape(-1).tolist())) >= 10         # ... and still not one constant token
    assert same == tot
    assert own >= math.ceil(floor * tot)


def test_saturation_count_is_that_of_the_stored_values():
    # Normalised rows are +-1 (+1 in the first 16 places), so a weight row of 8192 in those places gives 131072, beyond half,
    # and all other values stay far inside: three key dims and ten gate/up outputs saturate in every row, and three query dims
    # in the second run (dims 40 and 104 are rotary partners, with an angle of zero at this theta).  Row tiles of 128 and more end in rows that do not exist; the copies standing in for them must not be counted.
    m = workloads.scaled(C1, dtype="bf16", d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ff=224, vocab=512,
                         n_layers=1, rope_theta=1.0e30).model
    w = workloads.make_weights(m, 1)
    w["tok_embed"].copy_(torch.randint(0, 2, (m.vocab, m.d_model), generator=torch.Generator().manual_seed(2)) * 2.0 - 1.0)
    w["tok_embed"][:, :16] = 1.0
    w["wo"][0].zero_()
    w["w_down"][0].zero_()
    for name, rows in (("wk", (40, 104, 128 + 41)), ("w_gate", range(0, 220, 22)), ("w_up", range(0, 220, 22))):
        w[name][0][list(rows), :16] = 8192.0
    per_row = 3 + 10
    import paper_2605_26606_amd as pc
    lens = [201, 3, 190, 128, 90]                         # 612 rows: 128-row tiles end in 28 that do not exist
    rng = np.random.default_rng(1)
    prompts = [rng.integers(0, m.vocab, n) for n in lens]
    toks = torch.from_numpy(np.concatenate(prompts).astype(np.int32)).cuda()
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    for query in (False, True):
        if query:
            w["wq"][0][[40, 104, 128 * 7 + 41], :16] = 8192.0
        want = per_row + (3 if query else 0)
        for max_rows in (700, 256):                       # one chunk, and several
            ctx = make_ctx(m, w, block_size=32, kv_pool_bytes=64 << 20, max_slots=40, max_ctx=256, max_batch_rows=max_rows,
                           act_dtype="f16")
            last = torch.empty(len(lens), m.vocab, device="cuda")
            handles = pc.pc_prefill_shared(ctx, toks, cu, last)
            count = pc.pc_saturation_count(ctx, True)
            say("saturated: %d (max rows %d)" % (count, max_rows))
            assert count == want * sum(lens)
            for n in (3, 20):                             # decode tiles of 16, 32 and 128 rows
                seqs = pc.pc_fork(ctx, np.repeat(handles[:1], n), 2)
                pc.pc_decode_step(ctx, seqs, torch.zeros(n, dtype=torch.int32, device="cuda"), torch.empty(n, m.vocab, device="cuda"))
                assert pc.pc_saturation_count(ctx, True) == want * n
                pc.pc_release(ctx, seqs, 0)
            ctx.close()


def test_half_range_saturation_is_clamped_and_counted():
    # A model whose feed-forward product leaves the IEEE-half range (gate and up projections inflated): the
    # stores clamp to +-65504 instead of producing inf/NaN, every clamp is counted, and the logits stay finite.
    # The same model with bfloat16 activations needs no clamp.
    say("activations beyond the half range")
    w = workloads.make_weights(BF, 3, std=0.02)
    big = {k: v for k, v in w.items()}
    big["w_gate"] = [(t.float() * 2000.0).to(t.dtype) for t in w["w_gate"]]
    big["w_up"] = [(t.float() * 2000.0).to(t.dtype) for t in w["w_up"]]
    prompts = list(workloads.make_prompts(3, 40, BF.vocab, 6))
    kw = dict(block_size=64, kv_pool_bytes=128 << 20, max_slots=32, max_ctx=128, max_batch_rows=256)
    a = _run_generate(BF, big, prompts, 2, 6, 5, dict(kw, act_dtype="f16"), expect_saturation=True)
    assert a["saturated"] > 0
    assert np.isfinite(a["logits"]).all() and np.isfinite(a["last"]).all()
    b = _run_generate(BF, big, prompts, 2, 6, 5, dict(kw, act_dtype="bf16"))
    assert b["saturated"] == 0 and np.isfinite(b["logits"]).all()


@pytest.mark.parametrize("model,lens", [(BF, [70, 33, 128, 5, 64]), (BF8, [100, 31])])
def test_one_kernel_per_operation_decode_path(model, lens):
    # PC_OPT_FUSE_DECODE = 0 keeps the unfused layer (projection, RoPE + append, RMSNorm as kernels of their own) for
    # decode batches; it must match the oracle like the fused default, and the two must agree closely
    import paper_2605_26606_amd as pc
    say("decode layer with one kernel per operation, lens=%s" % lens)
    w = workloads.perturb_norm_gains(workloads.make_weights(model, 3), 10)
    toks, cu = workloads.make_ragged_prompts(lens, model.vocab, 8)
    prompts = [toks[cu[i]:cu[i + 1]] for i in range(len(lens))]
    kw = dict(block_size=64, kv_pool_bytes=512 << 20, max_slots=64, max_ctx=1024, max_batch_rows=1024)
    a = _run_generate(model, w, prompts, 3, 12, 21, kw, opts=[(pc.PC_OPT_FUSE_DECODE, 0)])
    _check(model, w, prompts, a, 21, 2e-2, range(0, len(lens) * 3, 2))
    b = _run_generate(model, w, prompts, 3, 12, 21, kw)
    # step 1 feeds both paths the same token wherever the first tokens agree (they come from the same prefill)
    same0 = a["tokens"][:, 0] == b["tokens"][:, 0]
    assert same0.all()
    assert np.abs(a["logits"][1] - b["logits"][1]).max() <= 5e-3
