"""The group-by's key hash and probe sequence (csrc/agg_hash.hpp), compiled for
the host, and the LDS table's slots as the kernels take them."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_10030_amd", "csrc")

SRC = r"""
#define __host__
#define __device__
#include <vector>
#include "agg_hash.hpp"
using namespace agg::gb;
static uint32_t hash(int64_t k, int wide) { return wide ? key_hash_of(k) : key_hash_of((int32_t)k); }
extern "C" void hashes(const int64_t* k, int64_t n, int wide, uint32_t* out) {
  for (int64_t i = 0; i < n; ++i) out[i] = hash(k[i], wide);
}
// Distinct keys put into a table of 2^log2l slots one after another: returns the
// keys that found none, and the probes that all of them took.
extern "C" int64_t fill(const int64_t* k, int64_t n, int wide, int log2l, int skip, int64_t* probes) {
  const uint32_t mask = (1u << log2l) - 1;
  std::vector<char> used(mask + 1);
  const int64_t mark = wide ? INT64_MIN : INT32_MIN;
  int64_t missed = 0;
  *probes = 0;
  for (int64_t i = 0; i < n; ++i) {
    if (k[i] == mark) continue;  // has a slot of its own
    uint32_t h = hash(k[i], wide), s = (h >> (32 - log2l - skip)) & mask;
    int p = 0;
    for (; p < kLdsProbes && used[s]; ++p) {
      h = next_probe(h);
      s = h >> (32 - log2l);
    }
    *probes += p + 1;
    if (p == kLdsProbes) ++missed;
    else used[s] = 1;
  }
  return missed;
}
"""

_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "h.cpp"), os.path.join(d, "h.so")
            with open(src, "w") as f:
                f.write(SRC)
            subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", CSRC, src, "-o", so])
            _lib = ctypes.CDLL(so)
        _lib.fill.restype = ctypes.c_int64
    return _lib


def _args(keys):
    k = np.ascontiguousarray(keys, dtype=np.int64)
    return k, k.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(k.size), int(keys.dtype == np.int64)


def hashes(keys):
    k, p, n, wide = _args(keys)
    out = np.empty(k.size, dtype=np.uint32)
    lib().hashes(p, n, wide, out.ctypes.data_as(ctypes.c_void_p))
    return out


def fill(keys, slots, skip=0):
    """(keys without a slot, probes per key) of a table of `slots` slots whose
    keys agree in the top `skip` bits of their hash."""
    k, p, n, wide = _args(keys)
    probes = ctypes.c_int64()
    missed = lib().fill(p, n, wide, slots.bit_length() - 1, skip, ctypes.byref(probes))
    return missed, probes.value / max(1, k.size)
