"""A head, with the next projection or alone, in one round of tiles, at the edges: one row past a wave's fragments and all of the last, a last tile of
one row of the vocabulary, all CUs busy, one group of K-steps and several; against the oracle, the projection through the second
stage's states."""
import pytest

from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from tests.gpu_common import run_workload

pytestmark = pytest.mark.gpu

# D, V, top_k, batch, rows of a block, rows of a tile (one stage: the head alone)
CASES = [(256, 33601, (1, 1), 129, 192, 160), (256, 40640, (4, 1), 192, 192, 160), (768, 32161, (2, 1), 193, 256, 160),
         (512, 40001, (3, 1), 256, 256, 160), (256, 32513, (2, 1), 257, 320, 160), (1024, 39801, (3, 1), 320, 320, 160),
         (256, 21249, (2, 1), 129, 192, 128), (512, 32256, (4, 1), 192, 192, 128), (3072, 18433, (3, 1), 256, 256, 128),
         (256, 24577, (2,), 129, 192, 128), (512, 25001, (3,), 192, 192, 128), (256, 32768, (4,), 256, 256, 128),
         (256, 32769, (3,), 193, 256, 160), (320, 33001, (1, 1), 320, 320, 160), (448, 40000, (2, 1), 200, 256, 160),
         (704, 24577, (3,), 150, 192, 128), (832, 31001, (2,), 256, 256, 128), (256, 40960, (4,), 320, 320, 160),
         (2112, 20001, (2, 1), 200, 256, 128)]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)).replace(" ", "") for c in CASES])
def test_drafts(case):
    D, V, top_k, batch, block, tile = case
    plan = B.spec_plan_panel(batch, D, V, top_k[0], D if len(top_k) > 1 else 0)
    assert 400 <= plan["kernel"] < 1000 and plan["block_rows"] == block and plan["tile_rows"] == tile
    wl = W.Workload("once", 64, D, V, len(top_k), top_k, top_k[0], batch, "bf16", "f32", 0.6, seed=63, emb_std=0.3)
    seqs = sorted({0, 1, 15, 16, 79, 80, batch // 2, batch - 17, batch - 16, batch - 1})
    rep, step, od, ov = run_workload(wl, ln_affine="random", gen_device="cpu", sample_seqs=seqs, check_verify=False)
    assert rep.rows_checked + rep.rows_skipped_below_exempt == len(seqs) * (1 + (top_k[0] if len(top_k) > 1 else 0))
    assert rep.rows_exempt <= 1
