"""GPU: partitions whose groups leave from one workgroup's table, against the
oracle: as many partitions as workgroups and more, with shares whose ends meet
partition starts and shares whose ends do not (few keys, skewed keys), with
tables that sent rows to the global one (floats outside the windows), and more
groups than the plan allows.  All results are exact."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("i64", "min"), ("f32", "avg"), ("f32", "max"), ("i32", "count")])
def test_whole_partitions(agg, kdt, vdt, op):
    import torch
    dt = np.int32 if kdt == "i32" else np.int64
    low = np.iinfo(dt).min
    groups = 1 << 17
    r = np.random.default_rng(11)
    g = agg.GroupBy(kdt, vdt, op, max_n=1_000_000, max_groups=groups)
    for n, keys_of in ((1, 1), (5000, 5000), (300_000, 120_000), (1_000_000, 131_072), (1_000_000, 300)):
        pool = np.unique(r.integers(low, -(low + 1), size=keys_of, dtype=np.int64))
        pool[0] = low
        keys = pool[r.integers(0, pool.size, size=n)].astype(dt)
        keys[: n // 3] = np.where(r.random(n // 3) < 0.5, pool[-1], keys[: n // 3])
        vals = make_vals(n, vdt, seed=n)
        if vdt == "f32":  # outside any window that the others' exponents place, and non-finite
            vals[:: 997] = np.float32(1e30)
            vals[5 :: 1999] = np.float32(1e-30)
            vals[7 :: 50_021] = np.inf
        got = g.run(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda())
        compare(got, oracle.groupby(keys, vals, op), f"{kdt}/{vdt} {op} n={n} keys={keys_of}")
    over = np.arange(groups + 1000).astype(dt)
    vals = make_vals(over.size, vdt, seed=2)
    assert g.run(torch.from_numpy(over).cuda(), torch.from_numpy(vals).cuda()) is None
    over = over[:groups]
    compare(g.run(torch.from_numpy(over).cuda(), torch.from_numpy(vals[:groups]).cuda()),
            oracle.groupby(over, vals[:groups], op), f"{kdt}/{vdt} {op} full")
    g.close()
