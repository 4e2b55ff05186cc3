"""A sequence's states are the same bits whichever kernel computes them: the stage kernel row by row, siblings together (from 256
parents on), or the first stage inside the head's launch (which a call with debug outputs does not use)."""
import pytest
import torch

from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu


def _inputs(D, V, tree, batch, seed):
    wl = W.Workload("states", 128, D, V, len(tree), tree, 2, batch, "bf16", "f32", 0.5, seed=seed, emb_std=1.0)
    gen = W.make_generator(seed, "cuda")
    w = W.make_speculator(wl, gen, device="cuda", ln_affine="random")
    return wl, w, W.make_draft_inputs(wl, gen, device="cuda")


@pytest.mark.parametrize("D,k", [(576, 2), (1088, 5), (2112, 4), (4160, 8)])
def test_one_parent_more(D, k):
    tables = []
    for batch in (255, 256):
        wl, w, (state, last) = _inputs(D, 700, (k, 2), 256, seed=k)
        step = Step(W.replace(wl, batch=batch), w, debug=True)
        step.draft(state[:batch].contiguous(), last[:batch].contiguous())
        torch.cuda.synchronize()
        tables.append(step.debug_tables())
        step.close()
    for stage, rows in ((0, 255), (1, 255 * k)):
        for what in ("states", "tok", "lse"):
            a, b = (t[what][stage][:rows] for t in tables)
            assert torch.equal(a, b), "stage %d: %d of %d %s differ" % (stage, int((a != b).sum()), a.numel(), what)


@pytest.mark.parametrize("batch", [1, 2])
def test_with_and_without_debug_outputs(batch):
    wl, w, (state, last) = _inputs(4096, 1500, (4, 2), 48, seed=3)
    steps = [Step(W.replace(wl, batch=batch), w, debug=debug) for debug in (True, False)]
    for at in range(0, 48, batch):
        for step in steps:
            step.draft(state[at:at + batch].contiguous(), last[at:at + batch].contiguous())
        torch.cuda.synchronize()
        for what in ("cand_tokens", "cand_leaf", "cand_scores"):
            assert torch.equal(getattr(steps[0], what), getattr(steps[1], what)), "sequences %d: %s differ" % (at, what)
    for step in steps:
        step.close()
