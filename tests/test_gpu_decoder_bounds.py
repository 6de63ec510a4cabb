"""Two tests of test_gpu_decoder further: the fp32 norm inside the projection within what its roundings explain, and the kept logits of a
single row given as a number."""
import numpy as np
import pytest
import torch

import test_gpu_decoder
import workloads
from gpu_util import make_ctx, say

pytestmark = pytest.mark.gpu

C1 = workloads.WORKLOADS["C1"]


@pytest.mark.parametrize("d,dff,n,scale", [
    (16, 32, 17, 1.0),          # one chunk of 16: three of a block's four waves have nothing to add up
    (48, 96, 1, 1.0),
    (272, 704, 130, 1.0),       # 17 chunks: a second round of loads with one chunk in it; 16 x 16 and 32 x 32 tiles
    (512, 1376, 700, 1.0),      # 64 x 64 tiles with a ragged last one
    (272, 704, 130, 1e-3),      # mean squares far below eps
    (272, 704, 130, 1e4),
])
def test_fp32_norm_inside_the_projection_within_its_roundings(d, dff, n, scale):
    # against the launches with a norm kernel of their own: each side rounds its normalised rows and sums at most 1376 products of
    # order 0.02 in float32, whose errors are some 2^-24 sqrt(1376) = 2e-6 of the result, a few times that behind two layers: 1e-5.
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
        assert torch.isfinite(a).all() and float((a - b).abs().max()) <= 1e-5 * float(b.abs().max())
    assert torch.equal(logits_of(1, [0, head])[0][0], logits_of(1, cu)[0][0])


@pytest.mark.parametrize("kept", [2, -1])
def test_kept_logits_of_a_single_row(kept):
    test_gpu_decoder.test_kept_logits_of_any_index_form(kept)
