"""GPU: the launch shapes that a column's size picks, and columns at any item
alignment.  Neither shows in a result bit: every function at the sizes where
the shape changes, from aligned and unaligned addresses, filtered and not,
equals the oracle, and the bits of a plan with other launch parameters."""
import numpy as np
import pytest

import datagen
import oracle
from aggcheck import check, same_bits

pytestmark = pytest.mark.gpu

SEG = 16 * 1024
T = {"i32": 4, "i64": 8, "f32": 4}


@pytest.fixture(scope="module")
def agg():
    import torch
    import paper_2606_10030_amd as agg
    assert torch.cuda.is_available()
    return agg


@pytest.mark.parametrize("dtype", ["i32", "i64", "f32"])
@pytest.mark.parametrize("segs", [1, 64, 65, 256, 257, 512, 513, 1023, 1024, 1025, 8192, 8193, 16385])
def test_shapes_by_size(agg, dtype, segs):
    import torch
    n = segs * SEG // T[dtype] - 3          # the last segment is short
    x = datagen.column(n + 1, dtype, "uniform", seed=segs)
    d = torch.from_numpy(x).to("cuda")
    tune = agg.make_tune(waves_per_block=4, blocks_per_cu=1, unroll=4)
    big = agg.Plan(dtype, "sum", max_n=1 << 28)       # its size picks another shape than a run's
    for op in ("sum", "min", "max", "avg"):
        for off in (0, 1):
            col, ref = d[off:off + n], x[off:off + n]
            got = agg.Plan(dtype, op, max_n=n).run(col)
            check(ref, dtype, op, "neumaier", got, ctx=f"{dtype} {op} segs={segs} off={off}")
            assert same_bits(got, agg.Plan(dtype, op, max_n=n, tune=tune).run(col))
            if op == "sum":
                assert same_bits(got, big.run(col))
    # filtered: a third of the items, from one column aligned and the other not
    y = datagen.column(n + 1, "i32", "uniform", seed=segs + 1)
    dy = torch.from_numpy(y).to("cuda")
    for off in (0, 1):
        mask = y[1 - off:1 - off + n] < -350_000
        f = agg.make_filter(dy[1 - off:1 - off + n], None, -350_000, hi_inclusive=False)
        got = agg.Plan(dtype, "max", max_n=n).run_filtered(d[off:off + n], f)
        sel = x[off:off + n][mask]
        assert got["count"] == sel.size
        assert got["value"] == (None if sel.size == 0 else oracle.value(sel, "max"))


@pytest.mark.parametrize("dtype", ["i32", "i64", "f32"])
@pytest.mark.parametrize("segs", [2048, 2559, 2560, 2561, 4095, 4096, 4097])
def test_one_launch_or_two(agg, dtype, segs):
    """Where the scan's last workgroup merges, and where a launch of its own does:
    the bits of both, call after call (the counter is clear again)."""
    import torch
    n = segs * SEG // T[dtype] - 3
    x = datagen.column(n, dtype, "uniform", seed=segs)
    d = torch.from_numpy(x).to("cuda")
    for op in ("sum", "min"):
        two = agg.Plan(dtype, op, max_n=n, tune=agg.make_tune(waves_per_block=4, blocks_per_cu=2)).run(d)
        check(x, dtype, op, "neumaier", two, ctx=f"{dtype} {op} segs={segs}")
        for plan in (agg.Plan(dtype, op, max_n=n),
                     agg.Plan(dtype, op, max_n=n, tune=agg.make_tune(waves_per_block=8, blocks_per_cu=1))):
            for _ in range(3):
                assert same_bits(plan.run(d), two), f"{dtype} {op} segs={segs}"
