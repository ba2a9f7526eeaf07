"""GPU: merged tables of the direct path with crowded sections, against the oracle.

The merge adds up each 1/128 of the hash in a table of 512 slots.  Keys that all
find a slot in the fold's larger table but crowd a few sections go to the global
table from the merge itself, while the other sections write their groups
straight to the output.  All results are exact."""
import numpy as np
import pytest

import hash_model
import oracle
from test_gpu_groupby import agg, compare, make_vals  # noqa: F401

NP = {"i32": np.int32, "i64": np.int64}


def crowd(kdt, sections, each, spread, seed):
    """`each` random keys in each of `sections` and `spread` anywhere."""
    low = np.iinfo(NP[kdt]).min
    pool = np.unique(np.random.default_rng(seed).integers(low, -(low + 1), size=1 << 20, dtype=np.int64)).astype(NP[kdt])
    pool = np.random.default_rng(seed + 1).permutation(pool)
    sec = hash_model.hashes(pool) >> 25
    return np.unique(np.concatenate([pool[sec == s][:each] for s in sections] + [pool[:spread]]))


@pytest.mark.gpu
@pytest.mark.parametrize("kdt", ["i32", "i64"])
@pytest.mark.parametrize("vdt,op", [("i32", "sum"), ("i64", "min"), ("f32", "sum"), ("i32", "count")])
def test_merge_sections_overflow(agg, kdt, vdt, op):
    import torch
    n = 41 * 16384 + 5
    sets = [crowd(kdt, [5], 1500, 0, 1), crowd(kdt, [0, 127], 700, 100, 2),
            np.arange(2000, dtype=NP[kdt]) * 46423, np.arange(4096, dtype=NP[kdt]) * 15867]
    if kdt == "i32" and vdt != "f32":  # two passes over the rows (COUNT: one)
        sets.append(crowd(kdt, [3, 60, 64, 100], 1000, 1500, 3))
    for i, pool in enumerate(sets):
        g = agg.GroupBy(kdt, vdt, op, max_n=n, max_groups=pool.size)
        other = np.arange(pool.size, dtype=NP[kdt])
        for rep in range(3):
            for keys in (pool, other, pool[:40], pool):
                k = keys[np.random.default_rng(rep).integers(0, keys.size, size=n)]
                vals = make_vals(n, vdt, seed=rep)
                compare(g.run(torch.from_numpy(k).cuda(), torch.from_numpy(vals).cuda()), oracle.groupby(k, vals, op),
                        f"{kdt}/{vdt} {op} set {i} rep {rep} keys={keys.size}")
        g.close()


def test_crowded_sets_overflow_in_the_merge_only():
    """The sets above are what they are for: every key has a slot in the fold's
    table, and a section of the merge has too many."""
    for kdt, slots in (("i32", 8192), ("i64", 4096)):
        for pool in (crowd(kdt, [5], 1500, 0, 1), crowd(kdt, [0, 127], 700, 100, 2)):
            assert hash_model.fill(pool, slots)[0] == 0
            assert max(hash_model.fill(pool[hash_model.hashes(pool) >> 25 == s], 512, 7)[0] for s in range(128)) > 0
