"""GPU: the filtered scan's launch shapes by column length, one launch and two,
against torch (integers, counts) and a plan that is given another shape (bits)."""
import pytest

from aggcheck import same_bits

pytestmark = pytest.mark.gpu

SEG = 16 * 1024


@pytest.mark.parametrize("dtype", ["i32", "i64", "f32"])
@pytest.mark.parametrize("fdtype", ["i32", "i64", "f32"])
def test_filtered_lengths(dtype, fdtype):
    import torch
    assert torch.cuda.is_available()
    import paper_2606_10030_amd as agg
    T = {"i32": torch.int32, "i64": torch.int64, "f32": torch.float32}
    width = 8 if dtype == "i64" else 4
    top = 1026 * SEG // width
    gen = torch.Generator(device="cuda").manual_seed(3)
    col = torch.randint(-1000, 1000, (top,), dtype=torch.int32, device="cuda", generator=gen).to(T[dtype])
    key = torch.randint(0, 1000, (top,), dtype=torch.int32, device="cuda", generator=gen).to(T[fdtype])
    for op in ("sum", "max", "count"):
        plan = agg.Plan(dtype, op, max_n=top)
        given = agg.Plan(dtype, op, max_n=top, tune=agg.make_tune(waves_per_block=1, blocks_per_cu=4))
        for nseg in (256, 257, 512, 513, 640, 641, 1024, 1025):
            for n in (nseg * SEG // width, nseg * SEG // width - 1):
                f = agg.make_filter(key[:n], 100, 700)
                got = plan.run_filtered(col[:n], f)
                hit = (key[:n] >= 100) & (key[:n] <= 700)
                picked = col[:n][hit].to(torch.int64)
                want = {"sum": picked.sum(), "max": picked.max(), "count": hit.sum()}[op].item()
                ctx = f"{dtype} WHERE {fdtype} {op} n={n}"
                assert got["count"] == hit.sum().item(), ctx
                assert (got["f64"] if dtype == "f32" and op != "count" else got["i64"]) == want, ctx  # sums of whole numbers below 2^24 a lane: exact
                assert same_bits(got, given.run_filtered(col[:n], f)), ctx
