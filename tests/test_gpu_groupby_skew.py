"""GPU: group-by columns most of whose rows have one key, against the oracle.

A partition that is mostly one key's gives each lane of a wave an entry of its
own for that key.  The hot key's share runs from a few rows of a wave to all of
them; the hot key itself may be the one whose bits mark an empty slot, or 0;
the rows cover less and more than one tile of every workgroup, and the tiles'
remainders.  All results are exact."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu

GROUPS = 40_000


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("i64", "min"), ("i64", "max"), ("f32", "sum"), ("f32", "max"),
                                    ("i32", "count")])
def test_hot_keys(agg, kdt, vdt, op):
    import torch
    dt = np.int32 if kdt == "i32" else np.int64
    low = np.iinfo(dt).min
    r = np.random.default_rng(5)
    for n in (40_961, 400_003, 2_500_001):
        vals = make_vals(n, vdt, seed=n)
        dv = torch.from_numpy(vals).cuda()
        for hot, share in ((12345, 0.02), (12345, 0.6), (0, 0.97), (low, 0.9), (-1, 1.0)):
            pool = r.integers(low, -(low + 1), size=GROUPS // 2, dtype=np.int64)
            keys = np.where(r.random(n) < share, hot, pool[r.integers(0, pool.size, size=n)]).astype(dt)
            g = agg.GroupBy(kdt, vdt, op, max_n=n, max_groups=GROUPS)
            compare(g.run(torch.from_numpy(keys).cuda(), dv), oracle.groupby(keys, vals, op),
                    f"{kdt}/{vdt} {op} n={n} hot={hot} share={share}")
            g.close()
