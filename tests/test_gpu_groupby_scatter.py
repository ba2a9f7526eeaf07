"""GPU: the scatter of keys only (COUNT) into more partitions than carry rows
between tiles (1024 of int32 keys, 2048), several tiles a workgroup, against
torch's whole-number counts per key; and the fewest partitions, against the
oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("declared", [4_200_000, 9_000_000])
def test_key_only_tiles(agg, kdt, declared):
    import torch
    n, card = 35_000_011, 19_997  # 512 workgroups of 68 360 rows: 5 or 6 tiles and a partial one
    idx = torch.arange(n, dtype=torch.int64, device="cuda")
    spread = (idx * 2654435761) % card
    g = agg.GroupBy(kdt, "i32", "count", max_n=n, max_groups=declared)
    out = torch.empty(declared, 4, dtype=torch.int64, device="cuda")
    ng = torch.zeros(1, dtype=torch.int64, device="cuda")
    for keys in (spread, torch.where(idx % 10 != 0, 77, spread % 3000)):
        for m in (n, n - 68_360 * 3 - 1, 40_000):
            k = keys[:m].to(torch.int32 if kdt == "i32" else torch.int64)
            count = torch.bincount(keys[:m], minlength=card)
            g.enqueue(k, k if kdt == "i32" else k.to(torch.int32), out, ng)
            got = out[:int(ng.item())]
            got = got[torch.argsort(got[:, 0])]
            seen = torch.nonzero(count).flatten()
            ctx = f"{kdt} declared={declared} {m} rows"
            assert torch.equal(got[:, 0], seen), ctx
            assert torch.equal(got[:, 3], count[seen]) and torch.equal(got[:, 1], count[seen]), ctx
    g.close()


@pytest.mark.parametrize("groups", [2049, 4096, 4097, 8193, 16_385])
@pytest.mark.parametrize("kdt,vdt,op", [("i32", "f32", "sum"), ("i64", "f32", "avg"), ("i64", "i64", "sum"),
                                        ("i32", "i32", "count")])
def test_few_partitions(agg, kdt, vdt, op, groups):
    """Plans of 2^21 rows and one fewer: 32, 64 and 128 partitions (and the direct
    path where the table holds the groups)."""
    import torch
    low = np.iinfo(np.int32 if kdt == "i32" else np.int64).min
    r = np.random.default_rng(groups)
    pool = np.unique(r.integers(low, -(low + 1), size=groups, dtype=np.int64))
    pool[0] = low
    for max_n in ((1 << 21) - 1, 1 << 21):
        g = agg.GroupBy(kdt, vdt, op, max_n=max_n, max_groups=groups)
        for n in (1, 5000, 400_003):
            keys = pool[r.integers(0, pool.size, size=n)].astype(np.int32 if kdt == "i32" else np.int64)
            vals = make_vals(n, vdt, seed=n)
            compare(g.run(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()), oracle.groupby(keys, vals, op),
                    f"{kdt}/{vdt} {op} max_n={max_n} groups={groups} n={n}")
        g.close()
