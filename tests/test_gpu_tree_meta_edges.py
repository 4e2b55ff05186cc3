"""Token-tree metadata at the edges of its scan and of its mask's 16-byte words, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import spec_oracle as O
from tests.test_gpu_next_rows import _device_metadata

pytestmark = pytest.mark.gpu

# b, B, n, V: odd mask sizes for several sequences (rows of the mask start anywhere), more candidates than threads,
# items across the chunks of the scan, all candidates equal, padding candidates, chains
CASES = [(3, 67, 5, 2), (2, 300, 1, 2), (1, 4096, 1, 3000), (5, 3, 3, 2), (2, 257, 3, 6), (2, 40, 7, 1),
         (24, 1, 7, 3), (1, 1, 1, 3), (3, 2, 5, 1), (2, 64, 8, 3), (2, 65, 8, 3)]


@pytest.mark.parametrize("b,Bc,n,V", CASES)
def test_tree_metadata_edges(b, Bc, n, V):
    rng = np.random.default_rng(b * 1000 + Bc)
    cand = rng.integers(0, V, (b, Bc, n)).astype(np.int32)
    cand[:, Bc - Bc // 4:] = -1
    want = O.tree_metadata(cand)
    got = _device_metadata(torch.from_numpy(cand).cuda(), with_mask=Bc < 1000)
    for key, w in want.items():
        if key != "mask" or got["mask"] is not None:
            assert np.array_equal(got[key].cpu().numpy(), w), key
