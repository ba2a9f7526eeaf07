"""The group-by's key hash (csrc/agg_hash.hpp) on the key sets that programs have:
dense codes, strides, timestamps, doubles, two codes packed in one key, random keys.

Bounds, from what random keys do.  At most half full, a table whose every probe
lands anew takes (1/a) ln(1/(1-a)) = 1.39 probes a key; a key set may take up to 2
and leaves no key without a slot (random keys: 2^-32 each).  m of 2^20 random keys
share a 32-bit hash with probability 2^20 / m! * 2^(-12 (m - 1)): 8 never do.  The
merge's sections and the partitions hold 128 sections' or P partitions' shares:
none may have more keys than its table has slots, and none more than twice its
share and eight standard deviations."""
import math

import numpy as np
import pytest

import hash_model

I32, I64 = np.int32, np.int64


def seq(n, stride, start=0, dt=I64):
    bits = 8 * dt().itemsize
    v = np.arange(n, dtype=np.uint64) * np.uint64(stride % 2**64) + np.uint64(start % 2**64)
    return v.astype(np.uint32 if bits == 32 else np.uint64).view(dt)


def pairs(a, b, shift, dt=I64, a0=0, b0=0):
    x = (np.arange(a, dtype=I64) + a0)[:, None] << shift
    return (x + np.arange(b, dtype=I64) + b0).ravel().astype(dt)


def key_sets(dt):
    r = np.random.default_rng(5)
    for n in (25, 300, 2000, 50_000, 200_000, 1 << 20):
        yield f"dense {n}", seq(n, 1, dt=dt), 1.1
        yield f"dense {n} from 1000003", seq(n, 1, 1_000_003, dt), 1.1
        yield f"dense {n} about 0", seq(n, 1, -n // 2, dt), 1.1
        low = np.iinfo(dt).min
        yield f"random {n}", np.unique(r.integers(low, -(low + 1), size=n, dtype=I64).astype(dt)), 2
    strides = [2, 3, 5, 7, 8, 10, 12, 16, 60, 100, 128, 1000, 1024, 3600, 4096, 86_400, 10**6, 1 << 16, 1 << 20,
               15_867, 46_423, 63_468, 109_891, 173_359, 283_250, 75_025, 832_040]
    if dt is I64:
        strides += [10**9, 86_400 * 10**3, 86_400 * 10**6, 86_400 * 10**9, 1 << 31, 1 << 32, (1 << 32) + 1, (1 << 32) - 1,
                    (1 << 33) + 2, 1 << 40, 1 << 44]
    for s in strides:
        for n in (25, 300, 2000, 50_000, 200_000):
            if n * s < 2**(8 * dt().itemsize):
                yield f"{n} by {s}", seq(n, s, dt=dt), 2
                yield f"{n} by {s} from afar", seq(n, s, 1_700_000_000 // s * s, dt), 2
    for shift in (8, 10, 12, 16) + ((20, 24, 32, 40, 48) if dt is I64 else ()):
        for a, b in ((5, 6), (10, 10), (45, 45), (64, 64), (200, 250)) + (((1000, 1000),) if shift >= 20 else ()):
            yield f"pairs {a} x {b} << {shift}", pairs(a, b, shift, dt), 2
            yield f"pairs {a} x {b} << {shift} from afar", pairs(a, b, shift, dt, 1001, 77), 2
    for n in (25, 300, 2000, 50_000, 200_000):
        yield f"floats {n}", np.arange(n, dtype=np.float32).view(I32).astype(dt), 2
        if dt is I64:
            yield f"doubles {n}", np.arange(n, dtype=np.float64).view(I64), 2
            yield f"cents {n}", (np.arange(n) * 0.01).view(I64), 2
            yield f"equal words {n}", seq(n, (1 << 32) + 1), 2


@pytest.mark.parametrize("dt", [I32, I64])
def test_key_sets_spread(dt):
    half = 4096 if dt is I32 else 2048  # half of the LDS table of an integer sum
    for name, keys, most_probes in key_sets(dt):
        n = np.unique(keys).size
        keys = np.random.default_rng(1).permutation(np.unique(keys))
        h = hash_model.hashes(keys)
        _, mult = np.unique(h, return_counts=True)
        assert mult.max() <= (1 if dt is I32 else 7), f"{name}: {mult.max()} keys with one hash"
        if n <= half:
            slots, bits = (256 if n <= 32 else 2 * half), 7
            missed, probes = hash_model.fill(keys, slots)
            assert missed == 0 and probes <= most_probes, f"{name}: {missed} without a slot, {probes} probes"
            if n <= 32:
                continue  # the table of few groups is neither merged nor partitioned
        else:
            bits = max(math.ceil(math.log2(n / half)), 8 if n >= 1 << 17 else 7)
        share = np.bincount(h >> (32 - bits), minlength=1 << bits)
        mean = n / 2**bits
        assert share.max() <= 2 * mean + 8 * math.sqrt(mean), f"{name}: {share.max()} of {mean} keys in a share"
        slots = 512 if n <= half else 2 * half
        order = np.argsort(h >> (32 - bits), kind="stable")
        parts = [hash_model.fill(p, slots, bits) for p in np.split(keys[order], np.cumsum(share)[:-1]) if p.size]
        assert sum(m for m, _ in parts) == 0, f"{name}: keys without a slot in their share's table"
        if n > half:
            probes = sum(q * s for (_, q), s in zip(parts, share[share > 0])) / n
            assert probes <= most_probes, f"{name}: {probes} probes"
