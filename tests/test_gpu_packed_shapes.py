"""GPU: packed columns at the block counts where the launch form changes (one
launch up to 1024 blocks, 8 or 16 waves per CU past it, headers read 64 at a
time per wave), at narrow, wide and mixed bit widths.  Results are exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 7, 8, 9, 64, 1023, 1024, 1025, 4097, 140_001])
@pytest.mark.parametrize("bits", [0, 5, 14, 27, 28, 32, "mixed"])
def test_packed_shapes(blocks, bits):
    import torch
    import paper_2606_10030_amd as agg
    if blocks > 5000 and bits not in (5, 27):
        pytest.skip("one narrow and one wide column of this size")
    r = np.random.default_rng(blocks)
    n = blocks * agg.PACK_BLOCK - 5          # the last block is short
    if bits == "mixed":
        width = np.repeat(r.integers(1, 33, size=blocks), agg.PACK_BLOCK)[:n]
        x = (r.integers(0, 2**32, size=n, dtype=np.int64) >> (32 - width)).astype(np.uint32).view(np.int32)
    else:
        x = r.integers(0, 1 << bits, size=n, dtype=np.int64).astype(np.uint32).view(np.int32)
    col = agg.pack_i32(x).to("cuda")
    for op in ("sum", "min", "max", "avg", "count"):
        p = agg.Plan("i32", op, max_n=n)
        for _ in range(2):                    # the second call finds the counter at zero again
            got = p.run_packed(col)
            assert got["value"] == oracle.value(x, op) and got["count"] == n, f"{blocks} blocks of {bits} bits {op}"
        p.close()


def test_corrupt_header_in_one_launch_and_in_two():
    import torch
    import paper_2606_10030_amd as agg
    for blocks in (3, 5000):
        x = np.arange(blocks * agg.PACK_BLOCK, dtype=np.int32)
        good = agg.pack_i32(x)
        bad = agg.pack_i32(x)
        bad.blocks["word_off"][blocks // 2] = 1 << 62
        p = agg.Plan("i32", "sum", max_n=x.size)
        with pytest.raises(agg.AggError):
            p.run_packed(bad.to("cuda"))
        assert p.run_packed(good.to("cuda"))["i64"] == oracle.value(x, "sum")   # the flag is clear again
        p.close()
