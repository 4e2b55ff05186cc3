"""Trees whose last head has more rows per sequence than the tree kernel merges in one pass: every width of the lists, up to
and past 256 leaves, and the largest tree that is merged in one pass."""
import pytest

from paper_2404_19124_amd import workloads as W
from tests.gpu_common import run_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tree,batch", [((5, 4, 1), 3), ((3, 6, 2), 5), ((4, 6, 3), 16), ((8, 3, 4), 2), ((5, 5, 5), 3),
                                        ((6, 3, 6), 1), ((4, 5, 7), 2), ((8, 8, 4), 2), ((8, 4, 8), 3), ((8, 8, 8, 2), 1),
                                        ((4, 4, 2), 3)])
def test_candidates_against_the_oracle(tree, batch):
    wl = W.Workload("rows", 128, 256, 900, len(tree), tree, 24 if tree[-1] > 1 else 16, batch, "bf16", "f32", 0.5,
                    seed=7 * sum(tree) + batch, emb_std=0.3)
    rep, step, _, _ = run_workload(wl, ln_affine="random", check_verify=False)
    assert rep.seqs == batch
    step.close()
