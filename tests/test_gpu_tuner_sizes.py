"""GPU: what a tuned size does to plans of that size and of others."""
import json

import pytest

pytestmark = pytest.mark.gpu

FIELDS = ("waves_per_block", "blocks_per_cu", "unroll", "nontemporal")


@pytest.fixture
def agg():
    import torch
    import paper_2606_10030_amd as agg
    assert torch.cuda.is_available()
    agg.tune_clear()
    yield agg
    agg.tune_clear()


def shape(t):
    return tuple(getattr(t, k) for k in FIELDS)


def test_a_tuned_size_leaves_others_alone(agg):
    """int32 MIN, whose best shapes differ from size to size: tuned at 1 GiB."""
    import torch
    n = 1 << 28
    sizes = (1 << 20, 12_000_000, 1 << 25)
    before = [shape(agg.default_tune("i32", "min", m)) for m in sizes]
    runs = [shape(agg.Plan("i32", "min", max_n=n).info(m)[1]) for m in sizes]
    col = torch.randint(-1000, 1000, (n,), dtype=torch.int32, device="cuda")
    t, _ = agg.autotune("i32", "min", col)
    assert shape(agg.default_tune("i32", "min", n)) == shape(t)
    assert shape(agg.default_tune("i32", "min", n // 2)) == shape(t)
    assert [shape(agg.default_tune("i32", "min", m)) for m in sizes] == before
    plan = agg.Plan("i32", "min", max_n=n)
    assert [shape(plan.info(m)[1]) for m in sizes] == runs
    assert shape(plan.info(n)[1]) == shape(t)
    for m in sizes + (n,):
        assert plan.run(col[:m])["i64"] == col[:m].min().item()


def test_the_untuned_shape_is_a_candidate(agg):
    """Compensated float SUM of 48 MB, whose built-in shape (16 waves, 1, 8) is not in
    the tuner's grid of others: the tuned one is at least about as fast."""
    import torch
    col = torch.rand(12_000_000, device="cuda")
    plain = agg.Plan("f32", "sum", max_n=col.numel())
    out = torch.zeros(4, dtype=torch.int64, device="cuda")

    def best(plan):
        ms = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                plan.enqueue(col, out)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        return min(ms)
    agg.autotune("f32", "sum", col)
    assert best(agg.Plan("f32", "sum", max_n=col.numel())) <= 1.15 * best(plain)


def test_tuned_page_locked_columns(agg, tmp_path):
    """A plan takes what was fastest, reading over the link or staging, also from a
    saved file; files from before the two were told apart stage."""
    import torch
    n = 1 << 25
    host = torch.arange(n, dtype=torch.int32).pin_memory()
    t, gbs = agg.autotune("i32", "sum", host, src="pinned_host")
    assert gbs > 1
    path = tmp_path / "tune.json"
    agg.tune_save(str(path))
    doc = json.load(open(path))
    (entry,) = doc["entries"]
    link = shape(agg.Plan("i32", "sum", max_n=n, src="zerocopy").info(n)[1])

    def taken():
        plan = agg.Plan("i32", "sum", max_n=n, src="pinned_host")
        assert plan.run(host)["i64"] == n * (n - 1) // 2
        return shape(plan.info(n)[1])
    assert taken() == (link if entry["link"] else shape(t))
    for flag, want in ((1, link), (0, shape(t)), (None, shape(t))):
        e = {k: v for k, v in entry.items() if k != "link"}
        if flag is not None:
            e["link"] = flag
        path.write_text(json.dumps({**doc, "entries": [e]}))
        agg.tune_clear()
        agg.tune_load(str(path))
        assert taken() == want
    path.write_text(json.dumps({**doc, "entries": [{**entry, "link": 2}]}))
    with pytest.raises(agg.AggError):
        agg.tune_load(str(path))
