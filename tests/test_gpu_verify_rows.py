"""The row scan of the verify on rows that start anywhere, against numpy's first maximum."""
import numpy as np
import pytest
import torch

from paper_2404_19124_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [1, 3, 7, 8, 9, 1025, 2048, 2051, 4097, 8195, 16389, 33001])
@pytest.mark.parametrize("rows", [6, 1026])
def test_first_maximum_of_rows_that_start_anywhere(dtype, V, rows):
    """Both workgroup sizes (rows), every offset of a row from its 16-byte boundary, the maximum at each edge of the
    vector part, planted twice (the first one counts), rows of one value and of -inf only."""
    n1 = 2
    b = rows // n1
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(V * rows)
    x = torch.randn((rows, V), generator=g).to(dt)
    for r in range(rows):
        at = [0, V - 1, V // 2, min(V - 1, 7), max(0, V - 9), (r * 37) % V][r % 6]
        x[r, at] = 50.0
        x[r, (at + 1 + r) % V] = 50.0
    x[1] = -float("inf")
    x[2] = 0.5
    for off in ((0, 1, 3) if rows == 6 else (1,)):
        buf = torch.zeros(rows * V + 8, dtype=dt, device="cuda")
        logits = buf[off:off + rows * V].view(b, 1, n1, V)
        logits.copy_(x.view(b, 1, n1, V))
        i32 = dict(dtype=torch.int32, device="cuda")
        greedy = torch.full((b, 1, n1), -7, **i32)
        cand = torch.zeros((b, 1, n1 - 1), **i32)
        B.spec_verify(logits, cand, greedy, torch.empty(b, **i32), torch.empty(b, **i32), torch.empty((b, n1), **i32),
                      torch.empty(b, **i32))
        torch.cuda.synchronize()
        want = np.argmax(x.float().numpy(), axis=1)
        assert np.array_equal(greedy.cpu().numpy().reshape(-1), want)
