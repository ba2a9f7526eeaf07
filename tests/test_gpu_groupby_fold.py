"""GPU: the group-by fold's tiles and its hash, against the oracle.

Rows are folded in tiles of 4096 or 8192 per workgroup, read as vectors of 2 or
4 items; the last tile is partial.  Keys are placed by one multiplicative
hash, so regular key sets (strides, keys that differ in one word only) are the
ones that could crowd a partition or a table.  All results are exact."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu

NP = {"i32": np.int32, "i64": np.int64}


def run(agg, keys, vals, op, max_groups, ctx, offset=0):
    """Group-by of device columns that start `offset` items into their allocations."""
    import torch
    kdt = "i32" if keys.dtype == np.int32 else "i64"
    vdt = {"int32": "i32", "int64": "i64", "float32": "f32"}[vals.dtype.name]

    def dev(x):
        d = torch.zeros(x.size + offset, dtype=torch.from_numpy(x[:0]).dtype, device="cuda")
        d[offset:].copy_(torch.from_numpy(x))
        return d[offset:]
    g = agg.GroupBy(kdt, vdt, op, max_n=max(1, keys.size), max_groups=max_groups)
    compare(g.run(dev(keys), dev(vals)), oracle.groupby(keys, vals, op), ctx)
    g.close()


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("i64", "min"), ("f32", "avg"), ("i32", "count")])
def test_fold_tile_edges(agg, kdt, vdt, op):
    """One row, and one row either side of one and of several tiles, through the
    few-groups, direct, two-pass and partitioned paths, from aligned columns and
    from columns that start one item further on."""
    r = np.random.default_rng(3)
    for groups in (3, 700, 6000, 40_000):
        for n in (1, 3, 4095, 4097, 8191, 8193, 3 * 8192, 40_961):
            keys = r.integers(0, min(groups, n), size=n).astype(NP[kdt])
            vals = make_vals(n, vdt, seed=n)
            for offset in (0, 1):
                run(agg, keys, vals, op, groups, f"{kdt}/{vdt} {op} n={n} groups={groups} offset={offset}", offset)


@pytest.mark.parametrize("kdt,first,stride", [
    ("i32", 0, 1), ("i32", -5000, 1), ("i32", 7, 1 << 12), ("i32", 0, 75_025), ("i32", -2**31, 2**32 // 10_000),
    ("i64", 0, 1), ("i64", 10**12, 86_400), ("i64", 0, 1 << 32), ("i64", -2**63, (1 << 32) + 1), ("i64", 5, 1 << 50)])
def test_regular_key_sets(agg, kdt, first, stride):
    """Arithmetic key sequences (dense codes, powers of two, other strides,
    keys that differ in their high words only) through the direct, two-pass,
    partitioned and sub-partition paths."""
    n = 100_003
    bits = 32 if kdt == "i32" else 64
    pool = [first + i * stride for i in range(10_000)]
    pool = np.array([(p + 2**(bits - 1)) % 2**bits - 2**(bits - 1) for p in pool], dtype=NP[kdt])
    r = np.random.default_rng(stride % 1000)
    for groups in (20, 1000, 10_000):
        keys = pool[r.integers(0, groups, size=n)]
        for vdt, op in (("i64", "sum"), ("f32", "sum"), ("i32", "count")):
            for declared in (groups, 3_000_000):
                run(agg, keys, make_vals(n, vdt, seed=groups), op, declared,
                    f"{kdt} {first}+{stride}i groups={groups} declared={declared} {vdt} {op}")


def window_values(kind, n, r):
    """Float columns that place an LDS table's windows differently (48 exponents
    a pass, placed by a sample of the column)."""
    def spread(lo, hi):
        return (np.where(r.random(n) < 0.5, -1.0, 1.0) * np.ldexp(1.0 + r.random(n), r.integers(lo, hi + 1, size=n)))
    v = {
        "one exponent": lambda: 1.0 + r.random(n),
        "48 exponents": lambda: spread(-20, 27),
        "49 exponents": lambda: spread(-20, 28),
        "five passes": lambda: spread(-120, 100),
        "top": lambda: spread(120, 127),
        "bottom": lambda: spread(-126, -120),
        "subnormal": lambda: r.integers(-1000, 1000, size=n) * 2.0**-149,
        "zeros": lambda: np.where(r.random(n) < 0.5, 0.0, -0.0),
        "mostly zeros": lambda: np.where(r.random(n) < 0.9, 0.0, r.standard_normal(n)),
        "non-finite": lambda: np.where(r.random(n) < 0.1, r.choice([np.nan, np.inf, -np.inf], size=n), r.standard_normal(n)),
        # most of these are not among the 1024 rows that place the windows
        "rare outliers": lambda: np.where(np.arange(n) % 9973 == 17, r.choice([1e38, -1e-38, 1e-44], size=n), r.random(n)),
        "ascending": lambda: np.sort(np.abs(spread(-60, 60))),
    }[kind]()
    with np.errstate(over="ignore"):
        x = v.astype(np.float32)
    return x if kind == "non-finite" else np.where(np.isfinite(x), x, np.float32(3.4e38))


@pytest.mark.parametrize("kind", ["one exponent", "48 exponents", "49 exponents", "five passes", "top", "bottom",
                                  "subnormal", "zeros", "mostly zeros", "non-finite", "rare outliers", "ascending"])
def test_float_windows(agg, kind):
    """Float sums of every spread of exponents, exact through every path."""
    n = 150_001
    r = np.random.default_rng(len(kind))
    vals = window_values(kind, n, r)
    for kdt, groups in (("i32", 3), ("i64", 20), ("i32", 1500), ("i64", 3000), ("i32", 20_000)):
        keys = r.integers(0, groups, size=n).astype(NP[kdt])
        for op, declared in (("sum", groups), ("avg", groups), ("sum", 6_000_000)):
            run(agg, keys, vals, op, declared, f"{kind} {kdt} groups={groups} declared={declared} {op}")


@pytest.mark.parametrize("kdt,vdt,op", [("i32", "i32", "count"), ("i64", "i32", "count"), ("i32", "f32", "sum"),
                                        ("i32", "i64", "sum"), ("i64", "i32", "sum"), ("i64", "i64", "sum")])
def test_scatter_carries_rows_between_tiles(agg, kdt, vdt, op):
    """Partitioned plans whose workgroups scatter several tiles each (and a
    partial last one), with partition counts on both sides of the tile forms
    (64 to 2048; keys only to 1024), uniform and skewed keys (a partition with nearly all rows,
    and empty ones), against torch's whole-number sums per key."""
    import torch
    n, card = 35_000_011, 19_997
    idx = torch.arange(n, dtype=torch.int64, device="cuda")
    spread = (idx * 2654435761) % card
    vals = (idx % 1001 - 500).to({"i32": torch.int32, "i64": torch.int64, "f32": torch.float32}[vdt])
    for keys in (spread, torch.where(idx % 10 != 0, 77, spread % 3000)):
        count = torch.bincount(keys, minlength=card)
        want = count if op == "count" else torch.zeros(card, dtype=torch.int64, device="cuda").index_add_(0, keys, vals.long())
        k = keys.to(torch.int32 if kdt == "i32" else torch.int64)
        for declared in (20_000, 300_000, 900_000, 1_900_000, 3_500_000):
            g = agg.GroupBy(kdt, vdt, op, max_n=n, max_groups=declared)
            out = torch.empty(declared, 4, dtype=torch.int64, device="cuda")
            ng = torch.zeros(1, dtype=torch.int64, device="cuda")
            g.enqueue(k, vals, out, ng)
            got = out[:int(ng.item())]
            got = got[torch.argsort(got[:, 0])]
            seen = torch.nonzero(count).flatten()
            ctx = f"{kdt}/{vdt} {op} declared={declared}"
            assert torch.equal(got[:, 0], seen), ctx
            assert torch.equal(got[:, 3], count[seen]), ctx
            assert torch.equal(got.view(torch.float64)[:, 2], want[seen].to(torch.float64)), ctx
            g.close()


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("i64", "max"), ("f32", "sum"), ("i32", "count")])
def test_few_keys_that_meet(agg, kdt, vdt, op):
    """Up to 32 random keys in the small table: several sets, so that keys meet at
    home and at their second and third slots, the marker key and key 0 among them."""
    low = np.iinfo(NP[kdt]).min
    r = np.random.default_rng(17)
    for groups in (2, 20, 32, 32, 32, 32):
        pool = r.integers(low, -(low + 1), size=groups, dtype=np.int64)
        pool[:2] = (low, 0)
        for n in (8191, 120_001):
            keys = pool[r.integers(0, groups, size=n)].astype(NP[kdt])
            run(agg, keys, make_vals(n, vdt, seed=n), op, 32, f"{kdt}/{vdt} {op} n={n} groups={groups}")
