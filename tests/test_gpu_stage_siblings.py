"""Siblings that share a workgroup of the stage kernel (256 parents and more): every width of the lists, parents that end
within a group of tiles, rows of less than a workgroup's elements, of one and of two elements' chunks per thread."""
import pytest

from paper_2404_19124_amd import workloads as W
from tests.gpu_common import run_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,k,batch", [(128, 2, 256), (640, 3, 257), (2176, 4, 263), (2048, 5, 271), (4224, 5, 259),
                                       (4096, 6, 258), (384, 7, 300), (4224, 8, 257)])
def test_drafts_against_the_oracle(D, k, batch):
    wl = W.Workload("siblings", 128, D, 700, 2, (k, 2), 2 * k, batch, "bf16", "f32", 0.5, seed=11 * k + batch, emb_std=0.3)
    rep, step, _, _ = run_workload(wl, ln_affine="random", check_verify=False)
    assert rep.seqs == batch
    step.close()
