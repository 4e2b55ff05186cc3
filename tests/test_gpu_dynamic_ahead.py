"""Drafts with trees per sequence enqueued behind work that holds the stream: the fifth call waits until the first one's row maps
have been read, and every call's candidates are its own; 300 sequences: several workgroups fetch."""
import pytest
import torch

from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [2, 300])
def test_a_caller_that_runs_ahead(batch):
    wl = W.Workload("ahead", 64, 64, 300, 2, (3, 2), 4, batch, "bf16", "f32", 0.6, seed=59, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    state, last = (t.cuda() for t in W.make_draft_inputs(wl, gen))
    step = Step(wl, {k: [t.cuda() for t in v] for k, v in w.items()}, max_batch=batch, max_top_k=wl.top_k)
    calls = [([[1 + (c + q) % 3, 1 + (c * q) % 2] for q in range(batch)], [(c + q) % 2 for q in range(batch)]) for c in range(9)]

    def run(trees, counts):
        i32 = dict(dtype=torch.int32, device="cuda")
        out = [torch.empty((batch, 4, 2), **i32), torch.empty((batch, 4), device="cuda"), torch.empty((batch, 4), **i32),
               torch.empty((batch,), **i32)]
        B.spec_draft_dynamic(step.model, state, last, trees, counts, *out)
        return out

    alone = []
    for c in calls:
        alone.append(run(*c))
        torch.cuda.synchronize()
    torch.cuda._sleep(50_000_000)   # some 20 ms
    for got, want in zip([run(*c) for c in calls], alone):
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    step.close()
