"""Logits that are not finite: one of -inf takes nothing from the rest of its row, one that is NaN shows."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as O
from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu

BIG = 3.0e38   # a head row of it: the logit of a state around 1 overflows


def _first_stage(dtype, V, batch, k, edit, D=128, stages=1):
    """The tables of the first stage of a draft (by default its only one), and its states and head."""
    top_k = (k,) + (1,) * (stages - 1)
    wl = W.Workload("nonfinite", 128, D, V, stages, top_k, k, batch, dtype, "f32", 0.5, seed=43, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    w["ln_beta"][0] += 1.0
    edit(w["head"][0])
    state, last = W.make_draft_inputs(wl, gen)
    step = Step(wl, {key: [t.cuda() for t in v] for key, v in w.items()}, debug=True)
    step.draft(state.cuda(), last.cuda())
    torch.cuda.synchronize()
    t = step.debug_tables()
    got = {key: t[key][0].float().cpu().numpy() for key in ("tok", "logp", "lse", "states")}
    step.close()
    return got, W.to_numpy_f32(w["head"][0])


# up to 16 and 17 to 32 rows (streaming kernels), float32: two tiles of weight rows and more per workgroup, so that finite logits
# follow in the same thread
STREAM = [("bf16", 20500, 20, 3), ("bf16", 20500, 3, 3), ("f32", 20500, 5, 3),
          ("bf16", 3001, 50, 3), ("bf16", 20500, 50, 3), ("bf16", 20500, 100, 3)]   # and the two dense kernels


@pytest.mark.parametrize("dtype,V,batch,k", STREAM)
def test_logits_of_minus_infinity_count_nothing(dtype, V, batch, k):
    low = np.zeros(V, bool)
    low[:min(4096, V // 2)] = True      # the first tiles of every workgroup
    low[V // 4::7] = True

    def edit(head):
        head[torch.from_numpy(low)] = -BIG

    got, head = _first_stage(dtype, V, batch, k, edit)
    logits = O.head_logits(got["states"], head)
    assert (got["states"].sum(1) > 2).all()   # so these logits are below the smallest float32
    logits[:, low] = -np.inf
    logp, lse = O.log_softmax(logits)
    # float32 sums of 128 products against float64: the bound of the other float32 shapes
    assert np.abs(got["lse"] - lse).max() < 1e-3
    for r in range(batch):
        want = O.topk_desc(logits[r].astype(np.float32), k)
        assert np.array_equal(got["tok"][r], want)
        assert np.abs(got["logp"][r] - logp[r, want]).max() < 1e-3


@pytest.mark.parametrize("at", [0, -1], ids=["first", "last"])
@pytest.mark.parametrize("dtype,V,batch,k", [("bf16", 4097, 20, 2), ("bf16", 9, 32, 3), ("bf16", 20500, 17, 2),
                                             ("f32", 65, 3, 3), ("f32", 1024, 17, 2), ("f32", 20500, 2, 2),
                                             ("bf16", 4097, 3, 2), ("bf16", 9, 16, 3), ("bf16", 3004, 50, 2),
                                             ("bf16", 20500, 50, 2), ("bf16", 20500, 100, 2)])
def test_a_logit_that_is_nan_shows_in_its_rows_sum(dtype, V, batch, k, at):
    """Also where it is the only logit of its thread, or (the last row of a ragged tile) of its workgroup."""
    def edit(head):
        head[at] = float("nan")

    got, head = _first_stage(dtype, V, batch, k, edit)
    assert np.isnan(got["lse"]).all() and np.isnan(got["logp"]).all()
    logits = O.head_logits(got["states"], head)
    logits[:, at] = -np.inf   # and takes no place among the row's best
    for r in range(batch):
        assert np.array_equal(got["tok"][r], O.topk_desc(logits[r].astype(np.float32), k))


@pytest.mark.parametrize("dtype,V,batch", [("bf16", 3001, 3), ("bf16", 3001, 20), ("bf16", 3001, 50), ("f32", 300, 3)])
def test_a_row_without_an_order_names_no_made_up_token(dtype, V, batch):
    """All logits NaN: every entry of the row is a token of the vocabulary or the mark of none (2^31 - 1)."""
    k = 5
    wl = W.Workload("nonfinite", 128, 128, V, 2, (k, 2), 2 * k, batch, dtype, "f32", 0.5, seed=44, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    state, last = W.make_draft_inputs(wl, gen)
    state[1] = float("nan")
    step = Step(wl, {key: [t.cuda() for t in v] for key, v in w.items()}, debug=True)
    step.draft(state.cuda(), last.cuda())
    torch.cuda.synchronize()
    tok = step.debug_tables()["tok"][0].cpu().numpy()
    assert (tok[[0, 2]] < V).all() and (tok[[0, 2]] >= 0).all()
    assert (((tok[1] >= 0) & (tok[1] < V)) | (tok[1] == 2**31 - 1)).all()
    cand = step.cand_tokens.cpu().numpy()
    assert (((cand >= 0) & (cand < V)) | (cand == 2**31 - 1)).all()
    step.close()


# the tile kernel of many rows, by blocks of 192 and of 256 rows: its last weight tile has one row of the vocabulary, or 235
TILES = [(1000, 24577, 3, 256), (1000, 24577, 1, 256), (513, 33003, 4, 192), (900, 12289, 2, 192)]


def _tile_plan(batch, V, k, block):
    plan = B.spec_plan_head(batch, 128, V, k)
    assert 100 <= plan["kernel"] < 1000 and plan["block_rows"] == block
    return plan


@pytest.mark.parametrize("batch,V,k,block", TILES)
def test_tile_kernel_logits_of_minus_infinity(batch, V, k, block):
    """The first tile of every other range whole (of a range with one tile: nothing finite), and rows all over the others."""
    plan = _tile_plan(batch, V, k, block)
    low = np.zeros(V, bool)
    low[V // 4::7] = True
    for t0 in (r * plan["tiles"] // plan["ranges"] for r in range(0, plan["ranges"], 2)):
        low[256 * t0:256 * (t0 + 1)] = True
    assert not low.all()

    def edit(head):
        head[torch.from_numpy(low)] = -BIG

    got, head = _first_stage("bf16", V, batch, k, edit)
    assert (got["states"].sum(1) > 2).all()
    logits = O.head_logits(got["states"], head)
    logits[:, low] = -np.inf
    logp, lse = O.log_softmax(logits)
    assert np.abs(got["lse"] - lse).max() < 1e-3
    for r in range(batch):
        want = O.topk_desc(logits[r].astype(np.float32), k)
        assert np.array_equal(got["tok"][r], want)
        assert np.abs(got["logp"][r] - logp[r, want]).max() < 1e-3


@pytest.mark.parametrize("at", [0, -1], ids=["first", "last"])
@pytest.mark.parametrize("batch,V,k,block", TILES)
def test_tile_kernel_logit_that_is_nan(batch, V, k, block, at):
    """In the first row of the vocabulary, and in the last, behind which the tile goes on."""
    _tile_plan(batch, V, k, block)

    def edit(head):
        head[at] = float("nan")

    got, head = _first_stage("bf16", V, batch, k, edit)
    assert np.isnan(got["lse"]).all() and np.isnan(got["logp"]).all()
    logits = O.head_logits(got["states"], head)
    logits[:, at] = -np.inf
    for r in range(batch):
        assert np.array_equal(got["tok"][r], O.topk_desc(logits[r].astype(np.float32), k))


@pytest.mark.parametrize("batch,V,k,block", TILES)
def test_tile_kernel_rows_of_nan_only(batch, V, k, block):
    """A row without one finite logit: NaN in its sum, tokens of the vocabulary or the mark of none; the others as they were."""
    _tile_plan(batch, V, k, block)
    wl = W.Workload("nonfinite", 128, 128, V, 1, (k,), k, batch, "bf16", "f32", 0.5, seed=45, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    state, last = W.make_draft_inputs(wl, gen)
    odd = torch.tensor([0, 17, 200, batch - 1])
    step = Step(wl, {key: [t.cuda() for t in v] for key, v in w.items()}, debug=True)
    tables = []
    for _ in range(2):
        step.draft(state.cuda(), last.cuda())
        torch.cuda.synchronize()
        t = step.debug_tables()
        tables.append({key: t[key][0].cpu() for key in ("tok", "lse", "logp")})
        state[odd] = float("nan")
    step.close()
    keep = torch.ones(batch, dtype=torch.bool)
    keep[odd] = False
    for key in ("tok", "lse", "logp"):
        assert torch.equal(tables[0][key][keep], tables[1][key][keep])
    assert torch.isnan(tables[1]["lse"][odd]).all()
    tok = tables[1]["tok"][odd]
    assert (((tok >= 0) & (tok < V)) | (tok == 2**31 - 1)).all()


# the panel kernel's ranges of one and of two tiles, and head and projection in one round: finite logits follow in the same tile
PANELS = [(70, 3001, 3, 128, 1, 300), (17, 70001, 2, 128, 1, 300), (140, 33601, 2, 256, 2, 400)]


@pytest.mark.parametrize("batch,V,k,D,stages,kernel", PANELS)
def test_panel_kernel(batch, V, k, D, stages, kernel):
    """Logits of -inf count nothing; one that is NaN, first or last of the vocabulary, shows in the sum and takes no place."""
    assert kernel <= B.spec_plan_panel(batch, D, V, k, D if stages > 1 else 0)["kernel"] < kernel + 100
    low = np.zeros(V, bool)
    low[:V // 3] = True
    low[V // 2::7] = True

    def edit(head):
        head[torch.from_numpy(low)] = -BIG

    got, head = _first_stage("bf16", V, batch, k, edit, D, stages)
    assert (got["states"].sum(1) > 2).all()
    logits = O.head_logits(got["states"], head)
    logits[:, low] = -np.inf
    logp, lse = O.log_softmax(logits)
    assert np.abs(got["lse"] - lse).max() < 1e-3
    for r in range(batch):
        assert np.array_equal(got["tok"][r], O.topk_desc(logits[r].astype(np.float32), k))
    for at in (0, -1):
        def nan(head):
            head[at] = float("nan")

        got, head = _first_stage("bf16", V, batch, k, nan, D, stages)
        assert np.isnan(got["lse"]).all() and np.isnan(got["logp"]).all()
        logits = O.head_logits(got["states"], head)
        logits[:, at] = -np.inf
        for r in range(batch):
            assert np.array_equal(got["tok"][r], O.topk_desc(logits[r].astype(np.float32), k))
