"""What the plan queries answer is what a draft launches: spec_plan_panel first, then spec_plan_contraction and, for a head alone,
spec_plan_head; compared with the launches that the library records."""
import pytest
import torch

from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step

pytestmark = pytest.mark.gpu


def expected(batch, E, D, V, tree):
    launches, rows = [B.spec_plan_contraction(batch, E, 0, 0, D)["kernel"]], batch
    for i, k in enumerate(tree):
        proj = D if i + 1 < len(tree) else 0
        plan, first = B.spec_plan_contraction(rows, D, V, k, proj), B.spec_plan_panel(rows, D, V, k, proj)
        if 300 <= first["kernel"] < 1000:
            launches.append(first["kernel"])
        elif plan["proj_apart"]:
            launches += [B.spec_plan_head(rows, D, V, k)["kernel"], B.spec_plan_contraction(rows, D, 0, 0, D)["kernel"]]
        else:
            launches.append(plan["kernel"] if proj else B.spec_plan_head(rows, D, V, k)["kernel"])
        rows *= k
    return launches


# D, V, tree, batch, families of kernels among the launches (the id's hundreds; 10: 1000 and more)
@pytest.mark.parametrize("D,V,tree,batch,families", [
    (256, 9000, (2, 1), 5, {0}), (256, 33000, (3, 2, 1), 20, {0, 3}), (256, 33000, (2, 2, 2), 40, {0, 3, 4}),
    (256, 33000, (3, 3, 1), 130, {1, 4, 10}), (1024, 65000, (5, 2, 2), 31, {0, 10}), (3072, 18500, (1, 1), 200, {5, 10}),
    (2048, 18500, (1, 1), 200, {10})])
def test_a_draft_launches_what_the_queries_answer(D, V, tree, batch, families):
    wl = W.Workload("plans", 64, D, V, len(tree), tree, 1, batch, "bf16", "f32", 0.5, seed=79, emb_std=0.3)
    gen = W.make_generator(wl.seed, "cuda")
    w = W.make_speculator(wl, gen, device="cuda")
    state, last = W.make_draft_inputs(wl, gen, device="cuda")
    step = Step(wl, w)
    B.spec_profile_enable(step.model, 64)
    step.draft(state, last)
    got = [r["kernel"] for r in B.spec_profile_read(step.model)]
    B.spec_profile_enable(step.model, 0)
    step.close()
    assert got == expected(batch, 64, D, V, tree)
    assert {min(k // 100, 10) for k in got} == families
