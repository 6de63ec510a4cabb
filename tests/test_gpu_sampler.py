"""GPU parity: pc_sample against the oracle's in-order double-precision
inverse CDF with the same Philox uniform.  One token is correct per (logits,
u); the two sides may differ only when u*Z falls within summation rounding of
a CDF boundary, so exact agreement is required on >= 99.9 % of draws (in
practice all of them)."""
import math

import numpy as np
import pytest
import torch

from oracle import philox, sampler
from gpu_util import say

pytestmark = pytest.mark.gpu


def _run(logits, n, V, T, seed, uids, step_base, eos_id=-1, bias=0.0, rows=None, steps=None, finished=None,
         want_lp=True):
    import paper_2605_26606_amd as pc
    d = "cuda"
    ld = torch.from_numpy(logits).to(d)
    tok = torch.full((n,), -5, dtype=torch.int32, device=d)
    lp = torch.zeros(n, device=d) if want_lp else None
    pc.pc_sample(ld, None if rows is None else torch.from_numpy(rows).to(d), n, V, T, seed,
                 torch.from_numpy(uids).to(d), None if steps is None else torch.from_numpy(steps).to(d), step_base,
                 eos_id, bias, tok, lp, finished)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), None if lp is None else lp.cpu().numpy()


@pytest.mark.parametrize("V,n,T,scale", [(512, 64, 1.0, 1.0), (151936, 24, 1.0, 0.8), (151936, 8, 0.7, 3.0),
                                         (1001, 40, 1.3, 2.0), (2, 50, 1.0, 1.0), (65, 33, 1.0, 5.0),
                                         (16384 + 4, 16, 1.0, 1.0)])
def test_tokens_and_logprobs(V, n, T, scale):
    say("sample V=%d n=%d T=%g" % (V, n, T))
    rng = np.random.default_rng(V + n)
    logits = (scale * rng.standard_normal((n, V))).astype(np.float32)
    uids = (rng.integers(0, 2 ** 40, n)).astype(np.int64)
    seed = 0x1234_5678_9ABC
    agree = 0
    for step_base in (0, 17):
        tok, lp = _run(logits, n, V, T, seed, uids, step_base)
        for i in range(n):
            u = philox.sampling_uniform(seed, int(uids[i]), step_base)
            wt, wlp = sampler.sample_token(logits[i], T, u)
            agree += int(tok[i] == wt)
            if tok[i] == wt:
                assert abs(lp[i] - wlp) < 2e-5 * max(1.0, abs(wlp))
            assert 0 <= tok[i] < V
    assert agree >= math.ceil(0.999 * 2 * n)


def test_row_map_steps_eos_and_finished():
    import paper_2605_26606_amd as pc
    V, P, G = 3000, 5, 4
    n = P * G
    rng = np.random.default_rng(3)
    logits = rng.standard_normal((P, V)).astype(np.float32)
    rows = np.repeat(np.arange(P, dtype=np.int32), G)
    uids = (np.repeat(np.arange(P), G) * 65536 + np.tile(np.arange(G), P)).astype(np.int64)
    steps = rng.integers(0, 100, n).astype(np.int32)
    eos, bias = 77, math.log(V / 3.0)
    fin = torch.zeros(n, dtype=torch.uint8, device="cuda")
    fin[3] = 1
    tok, lp = _run(logits, n, V, 1.0, 9, uids, 5, eos, bias, rows, steps, fin)
    f = fin.cpu().numpy()
    n_eos = 0
    for i in range(n):
        if i == 3:
            assert tok[i] == eos and lp[i] == 0.0 and f[i] == 1
            continue
        u = philox.sampling_uniform(9, int(uids[i]), 5 + int(steps[i]))
        wt, wlp = sampler.sample_token(logits[rows[i]], 1.0, u, eos, bias)
        assert tok[i] == wt and abs(lp[i] - wlp) < 2e-5
        assert f[i] == (1 if wt == eos else 0)
        n_eos += wt == eos
    assert n_eos >= 1          # the bias makes EOS likely enough that the flag path is exercised
    # rollouts of one prompt draw different uniforms from the same row
    assert len(set(tok[4:8])) > 1


def test_distribution_over_many_steps():
    # chi-square of 20000 GPU draws from one row against its softmax
    V, n = 40, 20000
    rng = np.random.default_rng(11)
    logits = rng.standard_normal((1, V)).astype(np.float32)
    rows = np.zeros(n, np.int32)
    uids = np.arange(n, dtype=np.int64) + 1000
    tok, _ = _run(logits, n, V, 1.0, 5, uids, 0, rows=rows, want_lp=False)
    p = sampler.softmax_probs(logits[0])
    counts = np.bincount(tok, minlength=V)
    chi2 = float(((counts - n * p) ** 2 / (n * p)).sum())
    assert chi2 < 100.0            # 39 dof


def test_history_destinations():
    # the token and its log-probability also go to a second place, at a caller-given index (the [step][sequence]
    # history of a decode batch that has shrunk); rows finished on entry file eos_id / 0 there too
    import paper_2605_26606_amd as pc
    V, n, n_orig = 700, 9, 20
    rng = np.random.default_rng(5)
    logits = torch.from_numpy(rng.standard_normal((n, V)).astype(np.float32)).cuda()
    uids = torch.arange(n, dtype=torch.int64, device="cuda") + 50
    index = torch.from_numpy(rng.permutation(n_orig)[:n].astype(np.int32)).cuda()
    fin = torch.zeros(n, dtype=torch.uint8, device="cuda")
    fin[2] = 1
    tok = torch.zeros(n, dtype=torch.int32, device="cuda")
    lp = torch.zeros(n, device="cuda")
    ht = torch.full((n_orig,), -9, dtype=torch.int32, device="cuda")
    hl = torch.full((n_orig,), 7.0, device="cuda")
    pc.pc_sample(logits, None, n, V, 1.0, 3, uids, None, 4, 11, 0.0, tok, lp, fin, hist_tokens=ht, hist_logprob=hl,
                 hist_index=index)
    torch.cuda.synchronize()
    idx = index.long()
    assert torch.equal(ht[idx], tok) and torch.equal(hl[idx], lp) and tok[2] == 11 and lp[2] == 0
    untouched = torch.ones(n_orig, dtype=torch.bool, device="cuda")
    untouched[idx] = False
    assert (ht[untouched] == -9).all() and (hl[untouched] == 7.0).all()
    # without an index: row i
    ht2 = torch.full((n,), -9, dtype=torch.int32, device="cuda")
    pc.pc_sample(logits, None, n, V, 1.0, 3, uids, None, 4, 11, 0.0, tok, None, None, hist_tokens=ht2)
    torch.cuda.synchronize()
    assert torch.equal(ht2, tok)


# ---------------------------------------------------------------- nucleus (top-p) sampling

def _run_top_p(logits, T, top_p, seed, uids, step_base, eos_id=-1, bias=0.0):
    import paper_2605_26606_amd as pc
    n, V = logits.shape
    ld = torch.from_numpy(logits).cuda()
    tok = torch.full((n,), -5, dtype=torch.int32, device="cuda")
    lp = torch.zeros(n, device="cuda")
    pc.pc_sample(ld, None, n, V, T, seed, torch.from_numpy(uids).cuda(), None, step_base, eos_id, bias, tok, lp, None,
                 top_p=top_p)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), lp.cpu().numpy()


def test_top_p_worked_example_and_ties():
    # probabilities (0.5, 0.3, 0.2) and (0.2, 0.5, 0.3): top_p = 0.7 keeps two tokens, renormalised to (0.625, 0.375)
    n = 400
    uids = np.arange(n, dtype=np.int64) + 7
    for probs, kept in (((0.5, 0.3, 0.2), (0, 1)), ((0.2, 0.5, 0.3), (1, 2))):
        logits = np.tile(np.log(np.array(probs, np.float64)).astype(np.float32), (n, 1))
        tok, lp = _run_top_p(logits, 1.0, 0.7, 11, uids, 3)
        for i in range(n):
            u = philox.sampling_uniform(11, int(uids[i]), 3)
            wt, wlp = sampler.sample_token(logits[i], 1.0, u, top_p=0.7)
            assert tok[i] == wt and tok[i] in kept and abs(lp[i] - wlp) < 1e-5
        assert abs((tok == kept[0]).mean() - 0.625) < 0.08
    # all logits equal: exactly the first half of the ids stays at top_p = 0.5 (ties: lower id first)
    V = 1000
    logits = np.zeros((n, V), np.float32)
    tok, lp = _run_top_p(logits, 1.0, 0.5, 5, uids, 0)
    assert tok.max() == 499 or tok.max() < 500
    assert tok.max() < 500 and tok.min() >= 0 and len(set(tok.tolist())) > 100
    assert np.allclose(lp, -math.log(500.0), atol=1e-5)
    for i in range(0, n, 7):
        u = philox.sampling_uniform(5, int(uids[i]), 0)
        assert tok[i] == sampler.sample_token(logits[i], 1.0, u, top_p=0.5)[0]
    # four equal heavy tokens among light ones, top_p reached in the middle of the tie
    logits = np.full((n, 64), -3.0, np.float32)
    logits[:, [5, 9, 33, 60]] = 2.0
    tok, _ = _run_top_p(logits, 1.0, 0.45, 5, uids, 0)
    assert set(tok.tolist()) == {5, 9}


@pytest.mark.parametrize("V,n,T,top_p,scale", [(512, 64, 0.7, 0.9, 1.0), (151936, 16, 0.7, 0.95, 1.0),
                                               (151936, 8, 0.7, 0.5, 3.0), (1001, 40, 1.0, 0.8, 2.0),
                                               (4096, 32, 0.7, 0.999, 1.0), (65, 33, 1.3, 0.3, 5.0)])
def test_top_p_tokens_and_logprobs(V, n, T, top_p, scale):
    # One nucleus is correct per (logits, top_p), and one token per (nucleus, u).  The GPU takes the cut-off decision on
    # float32 weights summed in double per radix bucket, the oracle on float64 weights in sorted order; they can differ
    # by the one token at the cut when the cumulative mass lands within rounding of top_p Z, which then moves the
    # sampled token with probability ~1/2.  Measured: no difference; required: >= 99.5 % of draws equal.
    say("top-p V=%d n=%d T=%g top_p=%g" % (V, n, T, top_p))
    rng = np.random.default_rng(V + n)
    logits = (scale * rng.standard_normal((n, V))).astype(np.float32)
    uids = (rng.integers(0, 2 ** 40, n)).astype(np.int64)
    eos = 17
    agree = tot = 0
    for step_base, bias in ((0, 0.0), (9, 1.5)):
        tok, lp = _run_top_p(logits, T, top_p, 77, uids, step_base, eos, bias)
        for i in range(n):
            u = philox.sampling_uniform(77, int(uids[i]), step_base)
            wt, wlp = sampler.sample_token(logits[i], T, u, eos, bias, top_p=top_p)
            agree += int(tok[i] == wt)
            tot += 1
            if tok[i] == wt:
                assert abs(lp[i] - wlp) < 3e-5 * max(1.0, abs(wlp))
            # whatever the uniform, the token lies inside the oracle's nucleus
            x = logits[i].astype(np.float64) / T
            x[eos] += bias
            keep = sampler.nucleus(np.exp(x - x.max()), top_p)
            assert keep[tok[i]]
    assert agree >= math.ceil(0.995 * tot)


def _nucleus_form(form, V, rng):
    x = rng.standard_normal(V).astype(np.float32)
    if form == "ties":               # a row on a few values: at 30000 tokens more alike than the list of the cut's bin holds
        x = np.round(x) + np.float32(0.0)   # (no negative zeros: their order beside zero is the key's)
    elif form == "some_ties":        # a few dozen alike at the cut: the lowest ids of them stay
        x = (np.round(x * 200.0) / 200.0).astype(np.float32) + np.float32(0.0)
    elif form == "flat":             # a whole row in one or two bins, more than the list holds at 30000
        x *= np.float32(0.004)
    elif form == "hidden_peak":      # one token 50 above all others
        x[V // 2 + 1] = 50.0
    elif form == "masked":           # most of the vocabulary at minus infinity
        x[rng.random(V) < 0.9] = -np.inf
    elif form == "lowest":           # masked with the type's lowest value, and all the rest far from zero
        x = x + np.float32(3000.0)
        x[rng.random(V) < 0.5] = np.finfo(np.float32).min
    elif form == "far":              # scaled logits beyond the range of the bins' edges
        x = x + np.float32(3.0e5)
    elif form == "one":              # one token holds all the mass
        x[V // 3] = 200.0
    if not np.isfinite(x[V // 3]) or x[V // 3] < -1e30:
        x[V // 3] = 0.5              # some token has weight
    return x


@pytest.mark.parametrize("form", ["normal", "ties", "some_ties", "flat", "hidden_peak", "masked", "lowest", "far", "one"])
@pytest.mark.parametrize("V", [3, 512, 1023, 5124, 30000])   # (512: most waves have no tokens of their own)
def test_top_p_forms(V, form):
    # rows on either side of every rule that picks the way to the cut.  A token is right if the oracle draws it; where the
    # mass lands within rounding (1e-6 relative: float32 weights) of top_p Z the cut may move by one token, hence 98 %.
    rng = np.random.default_rng(V)
    n, T = 4, 0.8
    logits = np.stack([_nucleus_form(form, V, rng) for _ in range(n)])
    uids = np.arange(n, dtype=np.int64) + 11
    same = tot = 0
    for top_p in (1e-6, 0.3, 0.9, 0.999999):
        tok, lp = _run_top_p(logits, T, top_p, 21, uids, 2, V // 2, 0.75)
        for i in range(n):
            u = philox.sampling_uniform(21, int(uids[i]), 2)
            # fp32 scaled logits, as the kernel forms them (far from zero their rounding is the distribution)
            with np.errstate(over="ignore"):
                x = logits[i] * np.float32(1.0 / np.float32(T))
            want, wlp = sampler.sample_token(x, 1.0, u, V // 2, 0.75, top_p=top_p)
            tot += 1
            if tok[i] == want:
                same += 1
                assert abs(lp[i] - wlp) <= 3e-5 * max(1.0, abs(wlp)) + 1e-6 * np.abs(x[np.isfinite(x) & (x > -1e30)]).max()
    say("top-p form %s V=%d: %d of %d" % (form, V, same, tot))
    assert same >= math.floor(0.98 * tot)


def test_weights_are_those_of_expf():
    # every 73rd float from -0 to -210 and the ends of the range: the same bits
    import ctypes
    import paper_2605_26606_amd as pc
    lo, hi = np.float32(-0.0).view(np.uint32), np.float32(-210.0).view(np.uint32)
    bits = np.concatenate([np.arange(int(lo), int(hi), 73, dtype=np.uint32),
                           np.array([0.0, -103.97, -104.0, -3.4e38, -np.inf], np.float32).view(np.uint32)])
    d = torch.from_numpy(bits.view(np.float32)).cuda()
    a, b = torch.empty_like(d), torch.empty_like(d)
    f = pc.library().pc_internal_exp_weight
    f.argtypes, f.restype = [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_void_p], None
    f(d.data_ptr(), a.data_ptr(), b.data_ptr(), len(bits), torch.cuda.current_stream().cuda_stream or None)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("form", ["late", "edges", "few"])
@pytest.mark.parametrize("V", [4100, 20484, 66571])   # (odd: one token per lane and load)
def test_top_p_granules(V, form):
    # late: the first tokens of every wave's segment are masked with a large negative number, so that the bins' ring goes
    # round; edges: likely tokens at either end of granules of 256 tokens and of the row, the others too far behind to be kept;
    # few: likely tokens here and there, others just behind the cut.  (Tolerances: test_top_p_forms.)
    rng = np.random.default_rng(V + len(form))
    n, T = 6, 0.9
    x = rng.standard_normal((n, V)).astype(np.float32)
    if form == "late":
        seg = -(-(-(-V // 16)) // 256) * 256
        x[:, np.arange(V) % seg < seg // 2] = -1e9
    elif form == "edges":
        at = np.arange(V) % 256
        x[:, (at == 0) | (at == 255) | (np.arange(V) == V - 1)] += 14.0
    else:
        x[:, 3::577] += 9.0
    uids = np.arange(n, dtype=np.int64) + 51
    same = tot = 0
    for top_p in (0.2, 0.9, 0.99):
        tok, lp = _run_top_p(x, T, top_p, 5, uids, 1, V // 2, 0.25)
        for i in range(n):
            u = philox.sampling_uniform(5, int(uids[i]), 1)
            want, wlp = sampler.sample_token(x[i] * np.float32(1.0 / np.float32(T)), 1.0, u, V // 2, 0.25, top_p=top_p)
            tot += 1
            if tok[i] == want:
                same += 1
                assert abs(lp[i] - wlp) <= 3e-5 * max(1.0, abs(wlp))
    say("top-p granules %s V=%d: %d of %d" % (form, V, same, tot))
    assert same >= math.floor(0.98 * tot)


@pytest.mark.parametrize("V,T,top_p,eos,bias", [(32000, 0.7, 0.95, 9, 0.5), (30001, 1.0, 0.8, -1, 0.0), (700, 1.3, 0.3, -1, 0.0)])
def test_top_p_draws_as_the_plain_sampler_on_the_kept_tokens(V, T, top_p, eos, bias):
    # Nothing but the cut distinguishes the two: with the other tokens masked, plain sampling gives the same token and the same
    # log-probability to the last bit.  (The float64 cut may lie one token off, see above: each row equals one of three.)
    rng = np.random.default_rng(V)
    n = 300
    logits = rng.standard_normal((n, V)).astype(np.float32)
    uids = np.arange(n, dtype=np.int64) + 17
    tok, lp = _run_top_p(logits, T, top_p, 33, uids, 6, eos, bias)
    x = logits.astype(np.float64) / T
    if eos >= 0:
        x[:, eos] += bias
    order = np.argsort(-x, axis=1, kind="stable")
    size = np.array([sampler.nucleus(np.exp(r - r.max()), top_p).sum() for r in x])
    matched = np.zeros(n, dtype=bool)
    for d in (0, -1, 1):
        masked = logits.copy()
        for i in range(n):
            masked[i, order[i, max(1, size[i] + d):]] = -np.inf
        t1, l1 = _run(masked, n, V, T, 33, uids, 6, eos, bias)
        matched |= (t1 == tok) & (l1 == lp)
    assert matched.all(), "rows %s" % np.nonzero(~matched)[0]


@pytest.mark.parametrize("V", [700, 5001])
@pytest.mark.parametrize("share", [0.5, 0.99])
def test_masked_rows(V, share):
    # top_p = 1 over rows with most of the vocabulary at minus infinity, whole stretches of it
    rng = np.random.default_rng(V)
    n = 40
    logits = rng.standard_normal((n, V)).astype(np.float32)
    logits[rng.random((n, V)) < share] = -np.inf
    logits[:, :V // 3] = -np.inf
    logits[:, V // 2] = 0.25
    uids = np.arange(n, dtype=np.int64) + 7
    tok, lp = _run(logits, n, V, 0.9, 12, uids, 3)
    for i in range(n):
        want, wlp = sampler.sample_token(logits[i], 0.9, philox.sampling_uniform(12, int(uids[i]), 3))
        assert tok[i] == want and abs(lp[i] - wlp) < 3e-5 * max(1.0, abs(wlp))


@pytest.mark.parametrize("V", [512, 5000])
@pytest.mark.parametrize("gap", [40.0, 94.0, 96.0, 97.0, 110.0, 280.0])
def test_top_p_with_the_largest_logit_suppressed(V, gap):
    # the EOS id is far above every other token and its bias takes it far below them: nucleus and log-probabilities are
    # those of the others.  A token may differ where the mass lands within rounding of top_p Z or of u Z (1e-6 relative).
    rng = np.random.default_rng(V + int(gap))
    n, T, eos = 16, 1.0, V // 2          # (an id that the sampled tokens include, at both sizes)
    logits = (2.0 * rng.standard_normal((n, V))).astype(np.float32)
    logits[:, eos] = logits.max(axis=1) + np.float32(gap)
    uids = np.arange(n, dtype=np.int64) + 31
    for bias in (-300.0, -np.inf):
        tok, lp = _run_top_p(logits, T, 0.97, 8, uids, 4, eos, bias)
        same = 0
        for i in range(n):
            want, wlp = sampler.sample_token(logits[i], T, philox.sampling_uniform(8, int(uids[i]), 4), eos, bias, top_p=0.97)
            if tok[i] == want:
                same += 1
                assert abs(lp[i] - wlp) <= 3e-5 * max(1.0, abs(wlp))
        assert same >= n - 1


@pytest.mark.parametrize("top_p", [1.0, 0.9])
@pytest.mark.parametrize("fill", [-np.inf, np.nan])
def test_rows_without_weight(fill, top_p):
    # nothing to draw from: the call still answers with a token of the vocabulary, and the rows beside are untouched
    V = 2053
    logits = np.random.default_rng(4).standard_normal((3, V)).astype(np.float32)
    logits[1] = fill
    uids = np.arange(3, dtype=np.int64) + 5
    tok, lp = _run_top_p(logits, 1.0, top_p, 9, uids, 1)
    assert 0 <= tok[1] < V
    for i in (0, 2):
        want, wlp = sampler.sample_token(logits[i], 1.0, philox.sampling_uniform(9, int(uids[i]), 1), top_p=top_p)
        assert tok[i] == want and abs(lp[i] - wlp) < 3e-5 * max(1.0, abs(wlp))
