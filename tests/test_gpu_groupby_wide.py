"""GPU: group-by float sums of columns with many exponents, against the oracle.

Tables of 3, 7 and 16 windows of 16 exponents, chosen by a sample of the column:
either side of each line, through the few-groups, direct, merged and partitioned
paths, with as many groups as a table takes in one pass and in several; and
columns whose sampled rows show none of the exponents that most rows have.  (2^27
rows of int64 keys: the direct path's two passes.)  All results are exact."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare  # noqa: F401

pytestmark = pytest.mark.gpu


def sampled_rows(n, threads=1024):
    """The rows that the kernels sample of a column of n."""
    t = np.arange(threads, dtype=np.uint64)
    probe = (t * np.uint64(0x85EBCA6B) + np.uint64(0x7FEB352D)) % np.uint64(2**32)
    return (np.uint64(n) * t // np.uint64(threads) + (probe * np.uint64(n // threads) >> np.uint64(32))).astype(np.int64)


def spread(r, n, lo, hi):
    v = (r.integers(0, 2, size=n) * 2 - 1) * np.ldexp(1 + r.random(n), r.integers(lo, hi + 1, size=n))
    return np.clip(v, -3.4e38, 3.4e38).astype(np.float32)


@pytest.mark.parametrize("kdt,groups,max_n", [
    ("i32", 3, 0), ("i64", 32, 0), ("i32", 33, 0), ("i32", 512, 0), ("i64", 1024, 0), ("i32", 1025, 0), ("i64", 2048, 0),
    ("i32", 2049, 0), ("i64", 4096, 1 << 27), ("i64", 40_000, 0), ("i32", 250_000, 0), ("i64", 2_000_000, 0)])
def test_many_exponents(agg, kdt, groups, max_n):
    import torch
    r = np.random.default_rng(groups)
    top = 17 * 16384 + 4099  # 18 workgroups: merged from about 900 groups on
    g = agg.GroupBy(kdt, "f32", "sum", max_n=max(top, max_n), max_groups=groups)
    low = np.iinfo(np.int32 if kdt == "i32" else np.int64).min
    pool = np.unique(r.integers(low, -(low + 1), size=groups, dtype=np.int64))
    pool[0] = low

    def run(keys, vals, what):
        with np.errstate(all="ignore"):
            compare(g.run(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()),
                    oracle.groupby(keys, vals, "sum"), f"{kdt} groups={groups} n={keys.size} {what}")

    for n in (1, 40_003, top):
        keys = pool[r.integers(0, pool.size, size=n)].astype(np.int32 if kdt == "i32" else np.int64)
        for lo, hi in ((-20, 27), (-20, 28), (-60, 51), (-60, 52), (-127, 127)):
            run(keys, spread(r, n, lo, hi), f"2^{lo}..2^{hi}")
        some = spread(r, n, -100, 100)
        some[::7], some[::101], some[::997], some[::499] = 0.0, np.float32(1e-44), np.nan, np.inf
        run(keys, some, "zeros, subnormal and non-finite rows among them")
        for far in (1e30, 1e-30):  # the sampled rows are near 1, every second other row is not
            vals = np.where(r.random(n) < 0.5, spread(r, n, -3, 3), np.float32(far) * spread(r, n, -3, 3)).astype(np.float32)
            rows = sampled_rows(n)
            vals[rows] = spread(r, rows.size, -3, 3)
            run(keys, vals, f"rows near {far} that the sample misses")
            vals[:n // 2] = spread(r, n // 2, -3, 3)
            run(keys, vals, f"rows near {far} in the second half only")
        # the sample sees zeros only: windows at 1, then where the rows are, then all
        vals = spread(r, n, 60, 70)
        vals[sampled_rows(n)] = 0.0
        run(keys, vals, "the sample sees zeros only")
        vals[n // 3:] *= np.float32(2.0**-130)
        vals[sampled_rows(n)] = 0.0
        run(keys, vals, "and the rows change on the way")
        vals[2 * n // 3:] = spread(r, n - 2 * n // 3, 100, 120)
        run(keys, vals, "twice")
        vals[::3] = np.float32(3e-40)
        vals[sampled_rows(n)] = 1.0
        run(keys, vals, "with subnormal rows")
        run(keys, spread(r, n, 0, 3), "few exponents")
    g.close()


def test_many_exponents_take_one_pass(agg):
    """A column of 60 exponents and few groups is read once, like one of few
    exponents: half as much time again at most (two readings took three times)."""
    import torch
    n = 1 << 26
    gen = torch.Generator(device="cuda").manual_seed(1)
    keys = torch.randint(0, 5, (n,), dtype=torch.int32, device="cuda", generator=gen)
    few = torch.rand(n, device="cuda", generator=gen) + 1
    many = few * torch.exp2(torch.randint(-30, 30, (n,), device="cuda", generator=gen).to(torch.float32))
    g = agg.GroupBy("i32", "f32", "sum", max_n=n, max_groups=5)
    out = torch.empty(5 * agg.GROUP_BYTES, dtype=torch.uint8, device="cuda")
    ng = torch.zeros(1, dtype=torch.int64, device="cuda")

    def best(vals):
        ms = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                g.enqueue(keys, vals, out, ng)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        return min(ms)
    t_few, t_many = best(few), best(many)
    assert t_many <= 1.5 * t_few, f"{t_many} ms against {t_few}"
    g.close()
