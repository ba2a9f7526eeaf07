"""GPU: the direct path's merged tables, against the oracle.

With many workgroups and groups the tables of the direct path are written out by
sections of the key's hash and merged by a second launch.  Sizes either side of
that line; few keys and as many as the plan allows, in one pass and in two;
the key that marks an empty slot; more keys than the plan allows; float columns
whose rows leave the table or take several passes.  All results are exact."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("i64", "min"), ("f32", "sum"), ("i32", "count")])
@pytest.mark.parametrize("groups", [33, 1500, 8192])
def test_merged_tables(agg, kdt, vdt, op, groups):
    import torch
    dt = np.int32 if kdt == "i32" else np.int64
    low = np.iinfo(dt).min
    r = np.random.default_rng(groups)
    top = 65 * 16384  # 17 workgroups are the fewest
    g = agg.GroupBy(kdt, vdt, op, max_n=2 * top, max_groups=groups)

    def run(n, keys, vals, what):
        got = g.run(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda())
        if np.unique(keys).size > groups:
            assert got is None, what
        else:
            compare(got, oracle.groupby(keys, vals, op), f"{kdt}/{vdt} {op} groups={groups} n={n} {what}")

    for n in (16 * 16384, 16 * 16384 + 1, top + 4097):
        pool = np.unique(r.integers(low, -(low + 1), size=groups, dtype=np.int64))
        pool[0] = low
        keys = pool[r.integers(0, pool.size, size=n)].astype(dt)
        vals = make_vals(n, vdt, seed=n)
        run(n, keys, vals, "random")
        if vdt == "f32" and n > top:
            far = vals.copy()
            far[::4999] = np.float32(1e30)
            far[7::50_021] = -np.inf
            run(n, keys, far, "some far floats")
            run(n, keys, np.exp2(r.integers(-120, 120, size=n)).astype(np.float32), "all exponents")
    run(n, np.full(n, low, dt), vals, "one key")
    over = (np.arange(n) % (groups + 1)).astype(dt)
    run(n, over, vals, "one key too many")
    run(n, (np.arange(n) % (40 * groups)).astype(dt), vals, "far too many keys")
    run(n, keys, vals, "afterwards")
    g.close()
