"""GPU: the scatter of keys only (COUNT) into more partitions than carry rows
between tiles (1024 of int32 keys, 2048), several tiles a workgroup, against
torch's whole-number counts per key."""
import pytest

from test_gpu_groupby import agg  # noqa: F401

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
