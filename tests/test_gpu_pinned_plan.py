"""GPU: plans for page-locked columns whose runs read the column over the link:
what they report and what they hold, and the same for plans that stage."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,op", [("i32", "sum"), ("i64", "max"), ("f32", "sum")])
def test_pinned_plan_reports_what_its_runs_take(dtype, op):
    import torch
    import paper_2606_10030_amd as agg
    assert torch.cuda.is_available()
    agg.tune_clear()
    n = 1 << 26
    fields = ("waves_per_block", "blocks_per_cu", "unroll", "nontemporal")

    def of(plan, m):
        t = plan.info(m)[1]
        return {k: getattr(t, k) for k in fields}
    # what the first streams, kernels and copies of a process allocate is not a plan's
    warm = [agg.Plan(dtype, op, max_n=n, src="pinned_host") for _ in range(5)]
    host = torch.zeros(n, dtype={"i32": torch.int32, "i64": torch.int64, "f32": torch.float32}[dtype], pin_memory=True)
    for w in warm:
        w.run(host)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plans = [agg.Plan(dtype, op, max_n=n, src="pinned_host") for _ in range(4)]
    held = before - torch.cuda.mem_get_info()[0]
    assert held <= 4 * (16 << 20), f"four plans hold {held >> 20} MiB"
    link = agg.Plan(dtype, op, max_n=n, src="zerocopy")
    for m in (1, 1000, 1 << 20, n):
        assert of(plans[0], m) == of(link, m)
    given = agg.make_tune(chunk_bytes=16 << 20, staging_depth=3)
    assert of(agg.Plan(dtype, op, max_n=n, src="pinned_host", tune=given), n) == {k: getattr(given, k) for k in fields}
