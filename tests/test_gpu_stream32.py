"""The streaming head kernel of 17 to 32 state rows, at the sizes where its tiling can go wrong, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as O
from paper_2404_19124_amd import binding as B
from paper_2404_19124_amd import workloads as W
from paper_2404_19124_amd.runner import Step
from tests.gpu_common import run_workload

pytestmark = pytest.mark.gpu

CASES = [
    # E, D, V, top_k, B, batch: rows per stage; the K slices of the 16 waves; tiles per workgroup of 256
    (64, 64, 9, (1, 1), 1, 17),           # 17, 17: two K-steps for 16 waves, one ragged tile
    (64, 1984, 4100, (2, 1), 2, 16),      # 16, 32: 62 steps, the last slice shorter
    (128, 2048, 16400, (8, 1), 8, 24),    # 24, 192: three tiles in flight, a last round that is not whole
    (128, 3072, 8200, (8, 1), 4, 31),     # 31 rows, widest lists, two tiles in flight
    (192, 4032, 4097, (3, 1), 3, 25),     # 126 steps: the last slice is two steps short
    (128, 4096, 4097, (5, 1), 5, 32),     # full slices, ragged vocabulary, projection behind the head
    (64, 768, 65536, (2, 1), 2, 20),      # the longest head: 16 tiles per workgroup
]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)).replace(" ", "") for c in CASES])
def test_17_to_32_rows(case):
    E, D, V, top_k, Bc, batch = case
    wl = W.Workload("stream32", E, D, V, len(top_k), top_k, Bc, batch, "bf16", "f32", 0.6, seed=23, emb_std=0.3)
    rows = [r for r in wl.rows() if 16 < r <= 32]
    assert B.spec_plan_contraction(20, 768, 65537, 1, 768)["kernel"] == 1   # longer heads: the dense kernel
    assert rows and all(B.spec_plan_contraction(r, D, V, 1, D)["kernel"] == 2 for r in rows)
    rep, step, od, ov = run_workload(wl, ln_affine="random", gen_device="cpu")
    assert rep.rows_checked + rep.rows_skipped_below_exempt == sum(wl.rows())
    assert rep.rows_exempt <= 1


@pytest.mark.parametrize("D,V", [(1536, 16400), (1600, 8200), (2560, 8209), (2624, 4100)])
def test_rings_on_either_side_of_a_slice_length(D, V):
    """Slices of 3, 4, 5 and 6 K-steps: the rings of three, two, two and one tile."""
    wl = W.Workload("rings32", 64, D, V, 2, (1, 2), 2, 29, "bf16", "f32", 0.6, seed=29, emb_std=0.3)
    assert B.spec_plan_contraction(29, D, V, 1, D)["kernel"] == 2
    run_workload(wl, ln_affine="random", gen_device="cpu", check_verify=False)


@pytest.mark.parametrize("rows,D,V", [(17, 64, 33), (32, 4096, 4111)])
def test_store_epilogue_of_row_major_states(rows, D, V):
    wl = W.Workload("logp32", 64, D, V, 1, (2,), 2, 32, "bf16", "f32", 0.6, seed=24)
    gen = W.make_generator(24)
    w = W.make_speculator(wl, gen)
    step = Step(wl, {k: [t.cuda() for t in v] for k, v in w.items()})
    s = torch.randn(rows, D, generator=gen).to(torch.bfloat16)
    out = torch.empty((rows, V), dtype=torch.float32, device="cuda")
    B.spec_head_logp(step.model, 0, s.cuda(), out)
    torch.cuda.synchronize()
    want, _ = O.log_softmax(O.head_logits(s.float().numpy(), W.to_numpy_f32(w["head"][0])))
    # float32 sums of K products of size |s| |h| / K against float64: 1e-3 is the bound the other rows are held to
    assert np.abs(out.cpu().numpy().astype(np.float64) - want).max() < 1e-3
    step.close()
