"""The top-k lists of the wide dense kernel: exact ties (smaller vocabulary index first) between logits of either sign,
for every list length and block height."""
import numpy as np
import pytest
import torch

from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu

CLASSES = 5


# batch, k: 64-, 96-, 128- and 160-row blocks, lists of 2, 3, 4, 6 and 8 entries, short and full tiles
@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("batch,k,V", [(40, 2, 33003), (64, 4, 33003), (40, 6, 33003), (33, 8, 33003), (70, 2, 2051),
                                       (96, 3, 33003), (70, 4, 2051), (70, 5, 2051), (96, 8, 33003), (310, 2, 20300),
                                       (310, 3, 20300), (310, 4, 36000), (465, 2, 16500), (465, 4, 16500)])
def test_exact_ties_go_to_the_smaller_index(batch, k, V, sign):
    D = 128
    wl = W.Workload("ties", D, D, V, 1, (k,), k, batch, "bf16", "f32", 0.5, seed=41, emb_std=0.3)
    assert B.spec_plan_contraction(batch, D, V, k, 0)["kernel"] >= 1000
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    # every head row is one of five: all logits of a class are equal, and of the given sign
    distinct = sign * torch.rand((CLASSES, D), generator=gen).to(torch.bfloat16).abs()
    of = torch.randint(0, CLASSES, (V,), generator=gen)
    w["head"][0] = distinct[of].contiguous()
    w["ln_beta"][0] += 1.0     # states around 1: the sums keep the rows' sign
    state, last = W.make_draft_inputs(wl, gen)
    step = Step(wl, {key: [t.cuda() for t in v] for key, v in w.items()}, debug=True)
    step.draft(state.cuda(), last.cuda())
    torch.cuda.synchronize()
    s = step.debug_tables()["states"][0].float().cpu()
    logits = s.double() @ distinct.double().t()
    assert bool((logits * sign > 0).all())
    best = logits.argmax(1)
    two = logits.topk(2, dim=1)[0]
    assert float((two[:, 0] - two[:, 1]).min()) > 1e-3   # classes are told apart far above float32 rounding
    want = np.stack([np.flatnonzero(of.numpy() == int(c))[:k] for c in best])
    assert np.array_equal(step.cand_tokens.cpu().numpy()[:, :, 0], want)
    step.close()


@pytest.mark.parametrize("batch,k,V", [(40, 2, 33003), (64, 4, 33003), (40, 6, 33003), (33, 8, 33003), (96, 3, 33003),
                                       (310, 2, 20300), (465, 4, 16500)])
def test_logits_of_exactly_zero_tie_by_index(batch, k, V):
    """Head rows of zeros above all others: the float64 keys of their logits are denormal numbers, told apart by the
    index alone."""
    D = 128
    wl = W.Workload("ties", D, D, V, 1, (k,), k, batch, "bf16", "f32", 0.5, seed=47, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    zero = torch.rand(V, generator=gen) < 0.2
    zero[-1] = True
    w["head"][0] = -(torch.rand((V, D), generator=gen) + 0.1).to(torch.bfloat16)
    w["head"][0][zero] = 0
    w["ln_beta"][0] += 1.0     # states around 1: the other rows' logits are negative
    state, last = W.make_draft_inputs(wl, gen)
    step = Step(wl, {key: [t.cuda() for t in v] for key, v in w.items()}, debug=True)
    step.draft(state.cuda(), last.cuda())
    torch.cuda.synchronize()
    s = step.debug_tables()["states"][0].float().cpu()
    assert float((s @ w["head"][0][~zero][:500].float().t()).max()) < -1e-3
    want = np.flatnonzero(zero.numpy())[:k]
    assert (step.cand_tokens.cpu().numpy()[:, :, 0] == want).all()
    step.close()
