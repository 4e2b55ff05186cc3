"""The packed copy of the weights takes what the weights take: for narrow models too."""
import pytest
import torch

from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,V", [(64, 300000), (256, 200000), (1024, 60000), (2048, 32000), (3072, 32000), (4096, 32000)])
def test_device_memory_of_a_model(D, V):
    wl = W.Workload("memory", 64, D, V, 1, (2,), 2, 1, "bf16", "f32", 0.5, seed=61)
    w = W.make_speculator(wl, W.make_generator(61, "cuda"), device="cuda")
    Step(wl, w).close()   # (what the first model of a process allocates once)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    step = Step(wl, w)
    torch.cuda.synchronize()
    taken = before - torch.cuda.mem_get_info()[0]
    step.close()
    # 1/16 for tiles apart, 16 MiB for the workspace of 16384 partial results and the allocations' granularity
    assert taken <= (1 + 1 / 16) * 2 * V * D + 2**24, "%.1f MB for %.1f MB of weights" % (taken / 1e6, 2 * V * D / 1e6)
