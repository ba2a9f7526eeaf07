"""GPU: a group-by plan's calls one after another, against the oracle.

A call leaves the plan's table clean for the next (the emission clears the
slots it reads), so each kind of call is followed by others on the same plan:
no rows, more keys than the plan allows, a call recorded into a graph and
replayed.  Table sizes either side of the one-launch limit and the partitioned
path.  All results are exact."""
import numpy as np
import pytest

import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", [3, 30, 200, 1000, 3000, 40_000])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("f32", "sum"), ("i64", "max"), ("f32", "min"), ("i32", "count")])
def test_calls_of_one_plan(agg, groups, vdt, op):
    import torch
    r = np.random.default_rng(groups)
    n = 60_000
    g = agg.GroupBy("i32", vdt, op, max_n=4 * n, max_groups=groups)

    def call(m, keyset, seed):
        keys = r.choice(keyset, size=m).astype(np.int32)
        keys[:min(m, 1)] = np.iinfo(np.int32).min
        vals = make_vals(m, vdt, seed=seed)
        return keys, vals, torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()

    def check(m, keyset, seed, what):
        keys, vals, dk, dv = call(m, keyset, seed)
        compare(g.run(dk, dv), oracle.groupby(keys, vals, op), f"{what} {vdt} {op} groups={groups}")

    a = r.integers(-2**31, 2**31, size=max(1, groups // 2), dtype=np.int64)
    b = r.integers(-2**31, 2**31, size=max(1, groups // 3), dtype=np.int64)
    many = np.arange(min(4 * n, 3 * groups + 100), dtype=np.int32)  # more than the plan allows
    dk, dv = torch.from_numpy(many).cuda(), torch.from_numpy(make_vals(many.size, vdt, seed=9)).cuda()
    check(n, a, 1, "first")
    check(n, b, 2, "second")
    assert g.run(dk[:0], dv[:0]) == []
    check(1, b, 3, "one row")
    assert g.run(dk, dv) is None
    check(n, a, 4, "after too many keys")

    # recorded and replayed: by a plan that has run, and by one whose first call is the recorded one
    for fresh in (False, True):
        if fresh:
            g.close()
            g = agg.GroupBy("i32", vdt, op, max_n=4 * n, max_groups=groups)
        out = torch.empty(groups * agg.GROUP_BYTES, dtype=torch.uint8, device="cuda")
        ng = torch.zeros(1, dtype=torch.int64, device="cuda")
        _, _, sk, sv = call(n, a, 5)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            g.enqueue(sk, sv, out, ng, stream=s)
        for rep in range(3):
            keys, vals, tk, tv = call(n, b if rep == 1 else a, 6 + rep)
            sk.copy_(tk)
            sv.copy_(tv)
            graph.replay()
            torch.cuda.synchronize()
            m = int(ng.item())
            raw = out[:m * agg.GROUP_BYTES].cpu().numpy().tobytes()
            gs = [agg.Group.from_buffer_copy(raw, i * agg.GROUP_BYTES) for i in range(m)]
            got = sorted(((x.key, x.i64, x.f64, x.count) for x in gs), key=lambda t: t[0])
            compare(got, oracle.groupby(keys, vals, op), f"replay {rep} fresh={fresh} {vdt} {op} groups={groups}")
            check(n, b, 20 + rep, "between replays")
    g.close()


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("f32", "sum"), ("i32", "count")])
def test_plan_for_many_rows_run_on_few(agg, kdt, vdt, op):
    """A plan for 2^25 rows has fewer partitions than one for the rows it is run
    on; from one row to a few partitions' worth, its workgroups get parts of
    one partition, one, or several."""
    import torch
    groups = 30_000
    g = agg.GroupBy(kdt, vdt, op, max_n=1 << 25, max_groups=groups)
    r = np.random.default_rng(7)
    for n in (1, 63, 65, 4097, 70_001, 700_001):
        keys = r.integers(-groups // 2, groups // 2, size=n).astype(np.int32 if kdt == "i32" else np.int64)
        vals = make_vals(n, vdt, seed=n)
        compare(g.run(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()), oracle.groupby(keys, vals, op),
                f"{kdt}/{vdt} {op} n={n}")
    g.close()


@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("op", ["sum", "avg"])
def test_two_pass_float_plan(agg, kdt, op):
    """Float sums by as many groups as take two passes of the direct path, which
    plans for 2^27 rows and more do (smaller ones partition): few rows, flushed,
    and more, merged, with rows outside the windows and without."""
    import torch
    groups = 4000
    r = np.random.default_rng(23)
    for max_n in ((1 << 27) - 1, 1 << 27):
        g = agg.GroupBy(kdt, "f32", op, max_n=max_n, max_groups=groups)
        for n in (1, 4097, 200_003, 600_001):
            keys = (r.integers(-groups // 2, groups // 2, size=n) * 7919).astype(np.int32 if kdt == "i32" else np.int64)
            vals = make_vals(n, "f32", seed=n)
            for far in (False, True):
                if far:
                    vals[::1009] = np.float32(-1e33)
                compare(g.run(torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()),
                        oracle.groupby(keys, vals, op), f"{kdt} {op} max_n={max_n} n={n} far={far}")
        g.close()
