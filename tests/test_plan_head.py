"""Host logic of the plan for a head launched alone (no GPU): what the tile kernel takes is covered whole, fits the CU's LDS
and the partial-result workspace, and is asked for by a kernel instance; everything else keeps the general plan."""
import random

import pytest

from paper_2404_19124_amd import binding as B


def check(rows, k, n_head, k_top, n_cu):
    p = B.spec_plan_head(rows, k, n_head, k_top, n_cu)
    what = "rows=%d k=%d n_head=%d k_top=%d n_cu=%d -> %s" % (rows, k, n_head, k_top, n_cu, p)
    if not 100 <= p["kernel"] < 1000:
        assert p == B.spec_plan_contraction(rows, k, n_head, k_top, 0, n_cu), what
        return p
    assert rows > 64 and k % 128 == 0 and k_top <= 4, what
    mb, kt = divmod(p["kernel"] - 100, 20)
    assert (mb, kt) in ((3, 2), (3, 3), (3, 4), (4, 2), (4, 3)) and kt >= k_top, what
    assert p["block_rows"] == 64 * mb and p["tile_rows"] == 256, what
    assert p["row_blocks"] * p["block_rows"] >= rows > (p["row_blocks"] - 1) * p["block_rows"], what
    assert p["tiles"] * 256 >= n_head > (p["tiles"] - 1) * 256, what
    assert 1 <= p["ranges"] <= p["tiles"] and p["parts"] == p["ranges"], what
    assert p["workgroups"] == p["row_blocks"] * p["ranges"] <= max(n_cu, p["row_blocks"]), what
    assert rows * p["parts"] <= rows * n_cu and 0 < p["lds_bytes"] <= 160 * 1024, what
    return p


def test_invariants_over_random_shapes():
    rnd = random.Random(20241203)
    taken = 0
    for _ in range(4000):
        rows = rnd.choice([rnd.randint(1, 100), rnd.randint(65, 1200), rnd.randint(500, 200000)])
        p = check(rows, rnd.choice([64, 128, 128, 128]) * rnd.randint(1, 64), rnd.choice([rnd.randint(1, 3000), rnd.randint(3000, 200000)]),
                  rnd.choice([1, 2, 3, 4, 5, 8]), rnd.choice([256, 256, 304, 128, 40, 7]))
        taken += 100 <= p["kernel"] < 1000
    assert taken > 200


# the launches whose times the rule rests on, and shapes it has to leave alone
@pytest.mark.parametrize("args,block", [((384, 4096, 32000, 3), 192), ((960, 4096, 32000, 2), 256), ((192, 3072, 128256, 4), 192),
                                        ((768, 3072, 128256, 3), 256), ((2304, 3072, 128256, 2), 256),
                                        ((320, 4096, 32000, 3), 0), ((96, 4096, 32000, 4), 0), ((75, 4096, 32000, 2), 0),
                                        ((960, 4096, 32000, 5), 0), ((960, 4160, 32000, 2), 0), ((64, 4096, 32000, 2), 0)])
def test_who_takes_which_head(args, block):
    p = check(*args, 256)
    assert (p["block_rows"] if 100 <= p["kernel"] < 1000 else 0) == block


@pytest.mark.parametrize("args", [(0, 4096, 32000, 2, 256), (400, 100, 32000, 2, 256), (400, 4096, 0, 2, 256),
                                  (400, 4096, 32000, 9, 256), (400, 4096, 32000, 0, 256), (400, 4096, 32000, 2, 0)])
def test_bad_arguments(args):
    with pytest.raises(B.SpecError) as e:
        B.spec_plan_head(*args)
    assert e.value.status == B.SPEC_EINVAL
