"""The float32 contraction at the edges of its tiles, K parts and row blocks, against the oracle."""
import pytest

from paper_2404_19124_amd import workloads as W
from tests.gpu_common import run_workload

pytestmark = pytest.mark.gpu

F32 = [
    # E, D, V, top_k, B, batch
    (7, 8, 9, (8, 3), 24, 1),            # less than one K step and one tile, rows off the 16-byte boundary
    (33, 72, 64, (2, 2), 4, 8),          # 8 and 16 rows, exactly one block of weight rows
    (64, 136, 65, (5, 3, 2), 16, 3),     # 3, 15, 45 rows: several row tiles, one weight row in the second block
    (130, 256, 1023, (1, 1, 1), 1, 17),  # chains, ragged everything
    (128, 128, 16385, (6, 1), 6, 2),     # one block more than there are parts: two blocks per workgroup
]


@pytest.mark.parametrize("case", F32, ids=["x".join(map(str, c)).replace(" ", "") for c in F32])
def test_float32_contraction_edges(case):
    E, D, V, top_k, Bc, batch = case
    wl = W.Workload("f32_edge", E, D, V, len(top_k), top_k, Bc, batch, "f32", "f32", 0.6, seed=29, emb_std=0.3)
    rep, step, od, ov = run_workload(wl, ln_affine="random", gen_device="cpu")
    assert rep.rows_exempt == 0
    assert rep.max_state_rel < 1e-4 and rep.max_logp_abs < 1e-3   # as the other float32 shapes
