"""What the generation loop keeps of each step's logits, with the library's calls replaced by stand-ins on the CPU: a decode step
overwrites the one logit buffer of the pass with its own number."""
import numpy as np
import pytest
import torch

from paper_2605_26606_amd import rollout

N, V, T = 6, 5, 5


@pytest.fixture
def loop(monkeypatch):
    steps = []

    def fork(ctx, handles, new_tokens, stream):
        return np.arange(len(handles), dtype=np.int32)

    def decode(ctx, seqs, tokens, logits, stream):
        steps.append(len(seqs))
        logits.copy_(100.0 * len(steps) + torch.arange(len(logits))[:, None])

    monkeypatch.setattr(rollout.B, "pc_fork", fork)
    monkeypatch.setattr(rollout.B, "pc_decode_step", decode)
    monkeypatch.setattr(rollout.B, "pc_sample", lambda *a, **k: None)
    monkeypatch.setattr(rollout.B, "pc_release", lambda *a, **k: None)
    monkeypatch.setattr(rollout, "_upload", lambda t, dev, stream: t.to(dev))      # (no GPU to pin memory for)
    return steps


def _generate(keep, **kw):
    class Context:
        vocab = V
    first = torch.arange(N, dtype=torch.float32)[:, None].repeat(1, V)
    out = rollout.generate_wave(Context, np.arange(N, dtype=np.int32), np.arange(N, dtype=np.int32), first, np.arange(N), T, 1.0, 0,
                                keep_logits_rows=keep, **kw)
    first.fill_(-1.0)      # the caller's buffer is its own again
    return out


@pytest.mark.parametrize("keep", [2, np.array(2), torch.tensor(-1), np.array([2]), [3, 0], [-1, 2, 2], [[0, 1], [5, -2]], []])
def test_every_step_keeps_its_own_rows(loop, keep):
    out = _generate(keep)
    at = torch.as_tensor(keep, dtype=torch.long)
    want = torch.arange(N, dtype=torch.float32)[:, None].repeat(1, V)
    assert len(out["logits"]) == len(out["logits_rows"]) == T
    for t in range(T):
        assert torch.equal(out["logits"][t], (100.0 * t + want)[at])
        assert torch.equal(out["logits_rows"][t], at)


def test_only_kept_steps_take_memory(loop):
    # one step of a long pass: nothing is allocated for the steps that keep nothing
    out = _generate(np.arange(N), keep_logits_steps=[3])
    assert out["logits_steps"] == [3] and len(out["logits"]) == 1
    rows = out["logits_rows"][0]
    assert torch.equal(rows, torch.arange(N)) and rows.untyped_storage().nbytes() == N * 8
