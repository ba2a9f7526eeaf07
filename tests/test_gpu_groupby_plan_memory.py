"""GPU: the regions for merged tables in a group-by plan's memory, one per
workgroup that a run of the plan's size can have, and runs at that size."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16 * 16384, 16 * 16384 + 1, 1_000_000])
def test_merge_regions_by_rows(agg, n):
    import torch
    groups = 8000
    keys = np.random.default_rng(n).integers(0, groups, size=n).astype(np.int32)
    vals = make_vals(n, "i64", seed=n)
    dk, dv = torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()
    warm = agg.GroupBy("i32", "i64", "sum", max_n=n, max_groups=groups)
    warm.run(dk, dv)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plans = [agg.GroupBy("i32", "i64", "sum", max_n=n, max_groups=groups) for _ in range(8)]
    held = (before - torch.cuda.mem_get_info()[0]) / 8
    # two regions (hash halves) per 16384 rows, each of 5064 records of 16 bytes; the table and rounding 4 MB
    bound = -(-n // 16384) * 2 * 5064 * 16 + (4 << 20)
    assert held <= bound, f"{held} bytes a plan, {bound}"
    for p in plans[:2]:
        for m in (n, n - 1, n // 2):
            compare(p.run(dk[:m], dv[:m]), oracle.groupby(keys[:m], vals[:m], "sum"), f"{m} of {n} rows")
