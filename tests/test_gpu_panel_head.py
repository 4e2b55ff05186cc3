"""The panel kernel at the edges of its fragments, tiles and slabs, against the oracle: one row past a fragment and all of the
last, a K of two steps, of one group of steps and one slab more, of groups and a remainder; a last tile of one row of the
vocabulary, tiles of nine fragments and of one, the projection's tiles behind the head's, several tiles per range."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as O
from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step
from tests.gpu_common import run_workload

pytestmark = pytest.mark.gpu

# D, V, top_k, batch, fragments of the first stage
CASES = [(64, 17, (1, 1), 33, 3), (64, 2305, (2, 1), 48, 3), (192, 4097, (8, 1), 49, 4), (256, 36352, (5, 1), 64, 4),
         (320, 20001, (3, 1), 65, 5), (448, 9000, (4, 1), 81, 6), (1024, 5003, (6, 1), 96, 6), (576, 16500, (7, 1), 113, 8),
         (128, 3000, (1, 2), 128, 8), (2112, 16401, (2, 1), 40, 3)]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)).replace(" ", "") for c in CASES])
def test_drafts(case):
    D, V, top_k, batch, mf = case
    plan = B.spec_plan_panel(batch, D, V, top_k[0], D)
    assert 300 <= plan["kernel"] < 1000 and plan["block_rows"] == 16 * mf
    wl = W.Workload("panel", 64, D, V, 2, top_k, top_k[0], batch, "bf16", "f32", 0.6, seed=61, emb_std=0.3)
    rep, step, od, ov = run_workload(wl, ln_affine="random", gen_device="cpu", check_verify=False)
    assert rep.rows_checked + rep.rows_skipped_below_exempt == sum(wl.rows())
    assert rep.rows_exempt <= 1


@pytest.mark.parametrize("rows,D,V,k", [(20, 128, 70000, 3), (32, 4160, 36900, 2), (17, 320, 65600, 8)])
def test_ranges_of_several_tiles(rows, D, V, k):
    """Of a head alone, twice on one workspace: what a row carries from tile to tile."""
    plan = B.spec_plan_panel(rows, D, V, k, 0)
    assert 300 <= plan["kernel"] < 1000 and plan["tiles"] > plan["ranges"]
    wl = W.Workload("panels", D, D, V, 1, (k,), k, rows, "bf16", "f32", 0.5, seed=62, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    w["head"][0] *= 10.0     # logits of a few units
    w["head"][0][-1] *= 3.0  # the last row of the vocabulary is among the best of some rows
    state, last = W.make_draft_inputs(wl, gen)
    step = Step(wl, {key: [t.cuda() for t in v] for key, v in w.items()}, debug=True)
    for _ in range(2):
        step.draft(state.cuda(), last.cuda())
    torch.cuda.synchronize()
    t = step.debug_tables()
    tok, logp, lse, s = (t[key][0].float().cpu().numpy() for key in ("tok", "logp", "lse", "states"))
    tok = t["tok"][0].cpu().numpy().astype(np.int64)
    step.close()
    want_logp, want_lse = O.log_softmax(O.head_logits(s, W.to_numpy_f32(w["head"][0])))
    at = np.arange(rows)[:, None]
    # float32 sums of K products of both signs against float64, K 2^-24 of their magnitudes: below 1e-3 up to K = 4160
    assert np.abs(lse - want_lse).max() < 1e-3
    assert np.abs(logp - want_logp[at, tok]).max() < 1e-3
    assert tok.min() >= 0 and tok.max() < V and all(len(set(r)) == k for r in tok)
    best = -np.sort(-want_logp, axis=1)[:, :k]
    assert np.abs(want_logp[at, tok] - best).max() < 1e-3   # in order, up to ties within that


# D, V, top_k, rows; head tiles and tiles of the range that holds both matrices
@pytest.mark.parametrize("D,V,top_k,rows,mixed", [(320, 70001, (3, 1), 20, (1, 1)), (448, 75001, (6, 1), 31, (2, 1))])
def test_ranges_of_head_and_projection(D, V, top_k, rows, mixed):
    """One range closes its last head tiles and then stores tiles of the projection, which the second stage's states show."""
    plan = B.spec_plan_panel(rows, D, V, top_k[0], D)
    assert 300 <= plan["kernel"] < 400 and plan["tiles"] > plan["ranges"]
    head, at = -(-V // plan["tile_rows"]), [r * plan["tiles"] // plan["ranges"] for r in range(plan["ranges"] + 1)]
    assert [(head - a, b - head) for a, b in zip(at, at[1:]) if a < head < b] == [mixed]
    wl = W.Workload("mixed", 64, D, V, 2, top_k, top_k[0], rows, "bf16", "f32", 0.6, seed=73, emb_std=0.3)
    rep, step, od, ov = run_workload(wl, ln_affine="random", gen_device="cpu", check_verify=False)
    assert rep.rows_checked + rep.rows_skipped_below_exempt == sum(wl.rows())
    assert rep.rows_exempt <= 1
