"""33 to 64 state rows on either side of the line between the two dense kernels, against the oracle."""
import pytest

from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from tests.gpu_common import run_workload

pytestmark = pytest.mark.gpu

# E, D, V, top_k, B, batch, wide at the first stage: 64 * 256 weight rows (head and next projection) and one more
CASES = [(64, 64, 16321, (2, 1), 2, 40, True), (64, 64, 16320, (2, 1), 2, 40, False),
         (64, 64, 16384, (3, 1), 3, 64, True), (64, 128, 17003, (8, 1), 8, 33, True)]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)).replace(" ", "") for c in CASES])
def test_33_to_64_rows_around_the_rule(case):
    E, D, V, top_k, Bc, batch, wide = case
    wl = W.Workload("rule", E, D, V, len(top_k), top_k, Bc, batch, "bf16", "f32", 0.6, seed=37, emb_std=0.3)
    assert (B.spec_plan_contraction(batch, D, V, top_k[0], D)["kernel"] >= 1000) == wide
    rep, step, od, ov = run_workload(wl, ln_affine="random", gen_device="cpu")
    assert rep.rows_checked + rep.rows_skipped_below_exempt == sum(wl.rows())
    assert rep.rows_exempt <= 1
