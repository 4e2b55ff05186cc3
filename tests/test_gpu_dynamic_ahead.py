"""Drafts with trees per sequence enqueued behind work that holds the stream: the fifth call waits until the first one's row maps
have been read, and every call's candidates are its own; 300 sequences: several workgroups fetch.  Recorded into a graph, every
call keeps its trees."""
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


def test_a_captured_call_is_waited_for_by_nobody():
    """Eager calls between the replays of a captured one, and after a capture that was never replayed, are their own."""
    wl = W.Workload("captured", 64, 64, 300, 2, (3, 2), 4, 3, "bf16", "f32", 0.6, seed=61, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    state, last = (t.cuda() for t in W.make_draft_inputs(wl, gen))
    step = Step(wl, {k: [t.cuda() for t in v] for k, v in w.items()}, max_batch=3, max_top_k=wl.top_k)
    calls = [([[3, 2], [1, 1], [2, 1]], [4, 0, 2]), ([[1, 2], [3, 2], [2, 2]], [1, 4, 3]), ([[1, 1], [1, 1], [3, 1]], [1, 1, 0])]
    i32 = dict(dtype=torch.int32, device="cuda")

    def buffers():
        return [torch.empty((3, 4, 2), **i32), torch.empty((3, 4), device="cuda"), torch.empty((3, 4), **i32),
                torch.empty((3,), **i32)]

    def run(call, out, stream=None):
        B.spec_draft_dynamic(step.model, state, last, *call, *out, stream=stream)
        return out

    want = [run(c, buffers()) for c in calls]
    torch.cuda.synchronize()
    captured, eager = buffers(), buffers()
    for replays in (3, 0):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run(calls[0], captured)
        for rep in range(replays):   # (the graph holds its maps itself)
            for t in captured:
                t.fill_(-7)
            graph.replay()
            run(calls[1 + rep % 2], eager)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(captured, want[0])), rep
            assert all(torch.equal(a, b) for a, b in zip(eager, want[1 + rep % 2])), rep
        for n in range(9):
            run(calls[n % 3], eager)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(eager, want[n % 3])), (replays, n)
    step.close()


# 300 sequences: the maps of a call are several launches
@pytest.mark.parametrize("batch", [3, 300])
def test_more_recorded_calls_than_slots(batch):
    """Six calls in one graph, replayed after and between eager calls that have used every slot several times: each its own."""
    wl = W.Workload("recorded", 64, 64, 300, 2, (3, 2), 4, batch, "bf16", "f32", 0.6, seed=67, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    state, last = (t.cuda() for t in W.make_draft_inputs(wl, gen))
    step = Step(wl, {k: [t.cuda() for t in v] for k, v in w.items()}, max_batch=batch, max_top_k=wl.top_k)
    calls = [([[1 + (c + q) % 3, 1 + (c * q) % 2] for q in range(batch)], [(c + q) % 2 for q in range(batch)]) for c in range(9)]

    def buffers():
        i32 = dict(dtype=torch.int32, device="cuda")
        return [torch.empty((batch, 4, 2), **i32), torch.empty((batch, 4), device="cuda"), torch.empty((batch, 4), **i32),
                torch.empty((batch,), **i32)]

    def run(call, out):
        B.spec_draft_dynamic(step.model, state, last, *call, *out)
        return out

    want = [run(c, buffers()) for c in calls]
    torch.cuda.synchronize()
    recorded, eager = [buffers() for _ in range(6)], buffers()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for call, out in zip(calls, recorded):
            run(call, out)
    for rep in range(3):
        for n in range(9):
            run(calls[(n + rep) % 9], eager)
            assert all(torch.equal(a, b) for a, b in zip(eager, want[(n + rep) % 9])), (rep, n)
        for out in recorded:
            for t in out:
                t.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        for c, out in enumerate(recorded):
            assert all(torch.equal(a, b) for a, b in zip(out, want[c])), (rep, c)
    step.close()


def test_a_caller_that_runs_ahead_waits_for_its_own_stream():
    """The fifth call behind 2 s of work on its stream comes back when that is done, not 5 s of another stream's work."""
    wl = W.Workload("ahead", 64, 64, 300, 2, (3, 2), 4, 2, "bf16", "f32", 0.6, seed=71, emb_std=0.3)
    gen = W.make_generator(wl.seed)
    w = W.make_speculator(wl, gen)
    state, last = (t.cuda() for t in W.make_draft_inputs(wl, gen))
    step = Step(wl, {k: [t.cuda() for t in v] for k, v in w.items()}, max_batch=2, max_top_k=wl.top_k)
    i32 = dict(dtype=torch.int32, device="cuda")
    outs = [[torch.empty((2, 4, 2), **i32), torch.empty((2, 4), device="cuda"), torch.empty((2, 4), **i32),
             torch.empty((2,), **i32)] for _ in range(5)]
    own, other = torch.cuda.Stream(), torch.cuda.Stream()

    def busy(stream, cycles):
        with torch.cuda.stream(stream):
            torch.cuda._sleep(cycles)

    t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    busy(own, 1000)
    t0.record(own)
    busy(own, 10_000_000)
    t1.record(own)
    torch.cuda.synchronize()
    second = int(1e10 / t0.elapsed_time(t1))   # of _sleep's cycles
    busy(own, 2 * second)
    busy(other, 5 * second)
    for out in outs:   # the fifth takes the first one's slot
        B.spec_draft_dynamic(step.model, state, last, [[3, 2], [2, 1]], [4, 2], *out, stream=own)
    assert not other.query()
    torch.cuda.synchronize()
    for out in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out, outs[0]))
    step.close()
