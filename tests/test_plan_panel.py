"""Host logic of the panel kernel's plan (no GPU): what it takes is covered whole, fits the CU's LDS and the partial-result
workspace, and no range of the projection alone counts as a part; everything else keeps the general plan."""
import random

import pytest

from paper_2404_19124_amd import binding as B


def check(rows, k, n_head, k_top, n_proj, n_cu):
    p = B.spec_plan_panel(rows, k, n_head, k_top, n_proj, n_cu)
    what = "rows=%d k=%d n_head=%d k_top=%d n_proj=%d n_cu=%d -> %s" % (rows, k, n_head, k_top, n_proj, n_cu, p)
    if 400 <= p["kernel"] < 1000:   # one round of tiles of both matrices, all state rows in a block
        tile = 128 if p["kernel"] >= 500 else 160
        mb, kt = divmod(p["kernel"] % 100, 10)
        assert mb in (3, 4, 5) and kt in (2, 3, 4) and kt >= k_top and k >= 256, what
        assert p["block_rows"] == 64 * mb >= rows > 128 and p["row_blocks"] == 1 and p["tile_rows"] == tile, what
        assert p["tiles"] == -(-n_head // tile) + -(-n_proj // tile) == p["workgroups"] <= n_cu, what
        assert p["parts"] == -(-n_head // tile) and 0 < p["lds_bytes"] <= 160 * 1024, what
        return p
    if not 300 <= p["kernel"] < 1000:
        assert p == B.spec_plan_contraction(rows, k, n_head, k_top, n_proj, n_cu), what
        return p
    mf, kt = divmod(p["kernel"] - 300, 10)
    assert 16 < rows <= 128 and mf in (2, 3, 4, 5, 6, 8) and kt in (2, 3, 4, 6, 8) and kt >= k_top, what
    assert p["block_rows"] == 16 * mf >= rows and p["row_blocks"] == 1, what
    head = -(-n_head // p["tile_rows"])
    assert 16 <= p["tile_rows"] <= 144 and p["tiles"] == head + -(-n_proj // p["tile_rows"]), what
    starts = [r * p["tiles"] // p["ranges"] for r in range(p["ranges"])]
    assert p["workgroups"] == p["ranges"] <= min(n_cu, p["tiles"]) and len(set(starts)) == len(starts), what
    assert p["parts"] == sum(s < head for s in starts) >= 1, what
    assert rows * p["parts"] <= max(128, rows) * n_cu and 0 < p["lds_bytes"] <= 160 * 1024, what
    return p


def test_invariants_over_random_shapes():
    rnd = random.Random(20241204)
    taken = once = 0
    for _ in range(500):   # around one round of tiles of both matrices
        n_cu = rnd.choice([256, 304, 40])
        k = 64 * rnd.randint(1, 64)
        p = check(rnd.randint(100, 330), k, max(1, rnd.randint(80, 170) * n_cu - rnd.choice([k, 64])), rnd.randint(1, 5),
                  rnd.choice([k, 64, 0]), n_cu)
        once += 400 <= p["kernel"] < 1000
    for _ in range(4000):
        n_head = rnd.choice([rnd.randint(1, 3000), rnd.randint(3000, 200000)])
        p = check(rnd.choice([rnd.randint(1, 400), rnd.randint(17, 128)]), 64 * rnd.randint(1, 128), n_head, rnd.randint(1, 8),
                  rnd.choice([0, 64 * rnd.randint(1, 128)]), rnd.choice([256, 256, 304, 128, 40, 7]))
        taken += 300 <= p["kernel"] < 400
    assert taken > 200 and once > 10


# the lines of the rule, and launches whose times it rests on: state fragments, or 0 where another kernel stays
@pytest.mark.parametrize("args,block", [((64, 4096, 32000, 5, 4096), 4), ((96, 4096, 32000, 4, 4096), 6), ((75, 4096, 32000, 2, 0), 5),
                                        ((33, 4096, 32000, 3, 4096), 3), ((128, 4096, 32000, 3, 0), 8), ((129, 4096, 32000, 3, 0), 0),
                                        ((32, 3072, 128256, 6, 3072), 2), ((32, 4096, 32000, 5, 4096), 0), ((16, 4096, 32000, 5, 4096), 0),
                                        ((33, 3072, 128256, 6, 3072), 0), ((48, 4096, 49152, 1, 0), 0), ((64, 4096, 16384, 2, 0), 0),
                                        ((64, 4096, 16385, 2, 0), 4), ((64, 1024, 2000, 2, 0), 4), ((64, 1088, 2000, 2, 0), 0),
                                        ((65, 4096, 2000, 2, 0), 5), ((64, 4096, 36864, 2, 0), 4), ((64, 4096, 36865, 2, 0), 0)])
def test_who_takes_which_launch(args, block):
    p = check(*args, 256)
    assert (p["block_rows"] // 16 if 300 <= p["kernel"] < 400 else 0) == block


# the lines of the rule: (state rows of a block, weight rows of a tile), or None where another kernel stays
@pytest.mark.parametrize("args,block", [((320, 4096, 32000, 3, 4096), (320, 160)), ((321, 4096, 32000, 3, 4096), None),
                                        ((129, 4096, 32000, 3, 4096), (192, 160)), ((128, 4096, 32000, 3, 4096), None),
                                        ((256, 4096, 28672, 3, 4096), (256, 128)), ((257, 4096, 28672, 3, 4096), None),
                                        ((257, 4096, 28673, 3, 4096), (320, 160)), ((200, 4096, 36800, 4, 4096), (256, 160)),
                                        ((200, 4096, 36801, 4, 4096), None), ((200, 4096, 32000, 5, 4096), None),
                                        ((200, 4160, 32000, 3, 4160), (256, 160)), ((200, 192, 33000, 3, 192), None), ((320, 2048, 32000, 3, 2048), (320, 160)),
                                        ((192, 2048, 30720, 3, 2048), (192, 128)), ((193, 2048, 30720, 3, 2048), None),
                                        ((192, 8192, 18000, 3, 8192), (192, 128)), ((193, 8192, 18000, 3, 8192), None),
                                        ((160, 4096, 17408, 2, 4096), None), ((160, 4096, 17409, 2, 4096), (192, 128)),
                                        ((192, 4096, 24576, 3, 0), None), ((192, 4096, 24577, 3, 0), (192, 128)),
                                        ((193, 4096, 30720, 3, 0), None), ((256, 4096, 30721, 3, 0), (256, 128)),
                                        ((257, 4096, 32768, 3, 0), None), ((257, 4096, 32769, 3, 0), (320, 160)),
                                        ((320, 4096, 40960, 3, 0), (320, 160)), ((320, 4096, 40961, 3, 0), None)])
def test_who_takes_one_round(args, block):
    p = check(*args, 256)
    assert ((p["block_rows"], p["tile_rows"]) if 400 <= p["kernel"] < 1000 else None) == block


# 193 to 256 rows beside a projection: above K = 2048, where weight tiles do not lie a whole number of 64 KiB apart
@pytest.mark.parametrize("k,taken", [(1536, False), (2048, False), (2112, True), (2560, True), (3072, True), (4096, True), (6080, True),
                                     (6144, False), (6208, True), (7168, True), (8128, True), (8192, False), (10240, False)])
@pytest.mark.parametrize("rows", [193, 256])
def test_tiles_of_128_rows_beside_a_projection(rows, k, taken):
    p = check(rows, k, 30000 - k, 2, k, 256)
    assert (500 <= p["kernel"] < 1000) == taken
    assert 500 <= check(192, k, 30000 - k, 2, k, 256)["kernel"] < 1000


@pytest.mark.parametrize("args", [(0, 4096, 32000, 2, 0, 256), (64, 100, 32000, 2, 0, 256), (64, 4096, 32000, 9, 0, 256),
                                  (64, 4096, 32000, 0, 0, 256), (64, 4096, 0, 0, 0, 256), (64, 4096, 32000, 2, 0, 0)])
def test_bad_arguments(args):
    with pytest.raises(B.SpecError) as e:
        B.spec_plan_panel(*args)
    assert e.value.status == B.SPEC_EINVAL
