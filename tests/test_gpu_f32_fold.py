"""float32 stages computed inside the head's launch (a call with debug outputs does not) are the stage kernel's, bit for bit: on
both sides of 16 rows, one and two chunks per lane and one too many, 64 parts and one more, with trees per sequence as well."""
import math

import pytest
import torch

from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu

# E, D, V, tree, batch
CASES = [(8, 8, 9, (8, 2), 1), (33, 264, 700, (4, 4, 1), 1), (64, 512, 4096, (1, 1, 1), 16), (64, 520, 4097, (2, 1, 2), 8),
         (64, 1024, 1000, (5, 3, 2), 1), (64, 1032, 300, (2, 2), 3), (64, 256, 2000, (6, 1, 1, 1), 3), (130, 72, 65, (7, 1), 2)]


def _steps(case, seed=19):
    E, D, V, tree, batch = case
    wl = W.Workload("fold32", E, D, V, len(tree), tree, min(2, math.prod(tree)), batch, "f32", "f32", 0.5, seed=seed,
                    emb_std=1.0)
    gen = W.make_generator(seed, "cuda")
    w = W.make_speculator(wl, gen, device="cuda", ln_affine="random")
    return wl, [Step(wl, w, debug=debug) for debug in (True, False)], gen


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)).replace(" ", "") for c in CASES])
def test_with_and_without_debug_outputs(case):
    wl, steps, gen = _steps(case)
    for _ in range(4):   # (each pass finds what the one before left in the workspace)
        state, last = W.make_draft_inputs(wl, gen, device="cuda")
        for step in steps:
            step.draft(state, last)
        torch.cuda.synchronize()
        for what in ("cand_tokens", "cand_leaf", "cand_scores"):
            assert torch.equal(getattr(steps[0], what), getattr(steps[1], what)), what
    for step in steps:
        step.close()


def test_trees_per_sequence():
    wl, steps, gen = _steps((64, 256, 1500, (4, 2, 2), 6))
    trees, counts = [[4, 2, 2], [1, 1, 1], [1, 1, 1], [3, 1, 2], [2, 2, 1], [1, 1, 1]], [8, 0, 1, 6, 4, 1]
    state, last = W.make_draft_inputs(wl, gen, device="cuda")
    rows, kw, _ = B.dynamic_rows(trees, counts)
    lse = torch.zeros((sum(rows),), device="cuda")
    got = []
    for step, dbg in zip(steps, ({"row_lse": lse}, None)):
        out = [torch.zeros((6, 8, 3), dtype=torch.int32, device="cuda"), torch.zeros((6, 8), device="cuda"),
               torch.zeros((6, 8), dtype=torch.int32, device="cuda"), torch.zeros((6,), dtype=torch.int32, device="cuda")]
        B.spec_draft_dynamic(step.model, state, last, trees, counts, *out, dbg=dbg)
        torch.cuda.synchronize()
        got.append(out)
    assert all(torch.equal(a, b) for a, b in zip(*got))
    for step in steps:
        step.close()


# what a head holds: rows whose logits overflow to -inf (most of a part, all but two of the vocabulary, all of it), or are NaN
@pytest.mark.parametrize("what", ["part", "all_but_two", "all", "nan_first", "nan_last", "nan_state"])
@pytest.mark.parametrize("case", [(64, 64, 9, (8, 1, 1), 2), (64, 264, 700, (4, 2, 2), 2), (128, 1024, 4093, (2, 2, 1), 3)],
                         ids=["V9", "V700", "V4093"])
def test_logits_that_are_not_finite(case, what):
    """The folded stage takes its parents' partial results as the stage kernel does: same candidates, same scores, NaN where that
    has NaN; in every stage, so that the next one's fold reads them, and with tokens that name no row of the embedding."""
    E, D, V, tree, batch = case
    wl = W.Workload("fold32", E, D, V, len(tree), tree, min(4, math.prod(tree)), batch, "f32", "f32", 0.5, seed=23, emb_std=1.0)
    gen = W.make_generator(23, "cuda")
    w = W.make_speculator(wl, gen, device="cuda", ln_affine="random")
    for i in range(len(tree)):
        w["ln_beta"][i] += 1.0   # the sum of a state is far above 0: a head row of -3e38 gives -inf
        head = w["head"][i]
        if what == "part":
            head[:V // 2] = -3.0e38
        elif what == "all_but_two":
            head[:V // 3] = -3.0e38
            head[V // 3 + 2:] = -3.0e38
        elif what == "all":
            head[:] = -3.0e38
        elif what != "nan_state":
            head[0 if what == "nan_first" else -1] = float("nan")
    steps = [Step(wl, w, debug=debug) for debug in (True, False)]
    state, last = W.make_draft_inputs(wl, gen, device="cuda")
    if what == "nan_state":
        state[1] = float("nan")
    for _ in range(2):   # (the second pass finds what the first left in the workspace)
        for step in steps:
            step.draft(state, last)
        torch.cuda.synchronize()
        t = steps[0].debug_tables()
        lse = torch.cat([x.reshape(-1) for x in t["lse"]])
        assert bool(torch.isnan(lse).any()) == what.startswith("nan")
        assert bool(torch.isinf(lse).any()) == (what == "all")
        a, b = steps[0].cand_scores, steps[1].cand_scores
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(a[~torch.isnan(a)], b[~torch.isnan(b)])
        assert torch.equal(steps[0].cand_tokens, steps[1].cand_tokens) and torch.equal(steps[0].cand_leaf, steps[1].cand_leaf)
    for step in steps:
        step.close()
