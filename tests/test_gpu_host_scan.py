"""GPU: columns in page-locked host memory, read over the link by the scan
(plans without given launch parameters) and staged in chunks (with them).

The result bits do not depend on the source, so both equal the device column's,
at sizes either side of a 16-byte vector, a segment, one launch and two, and
from the first item of the allocation and from one further on."""
import numpy as np
import pytest

from test_gpu_parity import agg, check, column, same_bits  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,op,prec", [("i32", "sum", "neumaier"), ("i64", "min", "neumaier"),
                                           ("f32", "sum", "neumaier"), ("f32", "avg", "f32")])
@pytest.mark.parametrize("offset", [0, 1])
def test_read_or_staged(agg, dtype, op, prec, offset):
    import torch
    width = 8 if dtype == "i64" else 4
    seg = 16384 // width
    for n in (1, 5, seg - 1, seg + 1, 1024 * seg, 1024 * seg + 3):
        x = column(dtype, n + offset, seed=n % 1000, kind="wide")[offset:]
        host = torch.empty(n + offset, dtype=torch.from_numpy(x[:0]).dtype, pin_memory=True)[offset:]
        host.copy_(torch.from_numpy(np.ascontiguousarray(x)))
        want = agg.Plan(dtype, op, max_n=n, prec=prec).run(host.to("cuda"))
        check(x, dtype, op, prec, want, ctx=f"device {dtype} {op} n={n}")
        for tune in (None, agg.make_tune(chunk_bytes=1 << 20, staging_depth=2)):
            plan = agg.Plan(dtype, op, max_n=n, prec=prec, src="pinned_host", tune=tune)
            for _ in range(2):
                assert same_bits(plan.run(host), want), f"{dtype} {op} {prec} n={n} offset={offset} tune={tune}"
            plan.close()
