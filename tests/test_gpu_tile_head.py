"""The tile kernel of many rows at the edges of its tiles: a last weight tile of one row, of less than half and whole; a last
row block of one row and whole; ranges of one and of several tiles; the shortest K."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as O
from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,D,V,k,block", [(513, 128, 33003, 4, 192), (513, 384, 20300, 1, 192), (192, 128, 33024, 3, 192),
                                              (900, 128, 12289, 2, 192), (577, 384, 20300, 2, 256), (1000, 128, 12289, 3, 256),
                                              (640, 128, 20300, 1, 256)])
def test_tables_against_the_oracle(rows, D, V, k, block):
    plan = B.spec_plan_head(rows, D, V, k)
    assert 100 <= plan["kernel"] < 1000 and plan["block_rows"] == block
    wl = W.Workload("tiles", D, D, V, 1, (k,), k, rows, "bf16", "f32", 0.5, seed=53, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    w["head"][0] *= 10.0     # logits of a few units
    w["head"][0][-1] *= 3.0  # the last row of the vocabulary is among the best of some rows
    state, last = W.make_draft_inputs(wl, gen)
    step = Step(wl, {key: [t.cuda() for t in v] for key, v in w.items()}, debug=True)
    for _ in range(2):       # (the second pass finds what the first left in the workspace)
        step.draft(state.cuda(), last.cuda())
    torch.cuda.synchronize()
    t = step.debug_tables()
    tok, logp, lse, s = (t[key][0].float().cpu().numpy() for key in ("tok", "logp", "lse", "states"))
    step.close()
    want_logp, want_lse = O.log_softmax(O.head_logits(s, W.to_numpy_f32(w["head"][0])))
    tok = tok.astype(np.int64)
    at = np.arange(rows)[:, None]
    # float32 sums of K products of both signs against float64, K 2^-24 of their magnitudes: below 1e-4
    assert np.abs(lse - want_lse).max() < 1e-4
    assert np.abs(logp - want_logp[at, tok]).max() < 1e-4
    assert tok.min() >= 0 and tok.max() < V and all(len(set(r)) == k for r in tok)
    best = -np.sort(-want_logp, axis=1)[:, :k]
    assert np.abs(want_logp[at, tok] - best).max() < 1e-4   # in order, up to ties within that
