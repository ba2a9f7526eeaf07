"""GPU: group-by of two codes packed in one int64 key, against the oracle.

The few-groups, direct, merged, two-pass and partitioned paths.  All results are
exact."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,b", [(5, 6), (10, 10), (45, 45), (64, 64), (300, 300), (1000, 1000)])
@pytest.mark.parametrize("vdt,op", [("i64", "sum"), ("f32", "sum"), ("i32", "count")])
def test_packed_pairs(agg, a, b, vdt, op):
    import torch
    r = np.random.default_rng(a)
    for n in (30_011, 700_001):
        for shift, off in ((32, 0), (32, 1001), (20, -3)):
            keys = ((r.integers(0, a, size=n) + off) << shift) + r.integers(0, b, size=n)
            vals = make_vals(n, vdt, seed=n)
            g = agg.GroupBy("i64", vdt, op, max_n=n, max_groups=a * b)
            compare(g.run(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()), oracle.groupby(keys, vals, op),
                    f"{a} x {b} << {shift} from {off} {vdt} {op} n={n}")
            g.close()
