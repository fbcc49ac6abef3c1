"""Bucket limits of the near-far SSSP rounds (grb_bucket.h), compiled for the host:
the limit taken from a distance lies above it, so a round always takes the vertex
it was taken from, also where (bucket + 1) * delta in float32 does not."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1908_01407_amd", "csrc")
SRC = """#include "grb_bucket.h"
extern "C" void ends(const float *d, const float *delta, float *e, int *b, int n) {
  for (int i = 0; i < n; ++i) {
    e[i] = grb::bucket_end(d[i], delta[i]);
    b[i] = grb::bucket_of(d[i], delta[i]);
  }
}
"""


@pytest.fixture(scope="module")
def ends(tmp_path_factory):
    d = tmp_path_factory.mktemp("bucket")
    src, so = d / "ends.cpp", d / "ends.so"
    src.write_text(SRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", CSRC, str(src), "-o", str(so)], check=True, timeout=110)
    lib = ctypes.CDLL(str(so))

    def run(dist, delta):
        dist, delta = np.broadcast_arrays(np.float32(dist), np.float32(delta))
        dist, delta = np.ascontiguousarray(dist).ravel(), np.ascontiguousarray(delta).ravel()
        e, b = np.empty(dist.size, np.float32), np.empty(dist.size, np.int32)
        p = [x.ctypes.data_as(ctypes.c_void_p) for x in (dist, delta, e, b)]
        lib.ends(*p, dist.size)
        return dist, delta, e, b

    return run


def test_limits_that_plain_rounding_misses(ends):
    d, delta, e, b = ends([1.2269344, 200.0, 3e9, 1e30, 2.0**25], [0.17527635, 1e-5, 1.0, 1e-3, 1.0])
    with np.errstate(over="ignore"):
        plain = (np.floor(d / delta) + np.float32(1)) * delta
    assert np.all(plain <= d)  # no round would take these vertices
    assert np.array_equal(e, np.nextafter(d, np.float32(np.inf)))
    assert b.tolist() == [6, 20000000, 2**31 - 1, 2**31 - 1, 2**25]


def test_limits_above_their_distance(ends):
    rng = np.random.default_rng(5)
    d = np.exp(rng.uniform(np.log(1e-30), np.log(1e30), 400000)).astype(np.float32)
    delta = np.exp(rng.uniform(np.log(1e-30), np.log(1e30), 400000)).astype(np.float32)
    k = rng.integers(1, 3000, 200000)  # multiples of the width, where the quotient rounds
    w = rng.uniform(0.01, 900, 200000).astype(np.float32)
    d = np.concatenate([d, (w * k).astype(np.float32), np.zeros(100, np.float32)])
    delta = np.concatenate([delta, w, rng.uniform(0.01, 9, 100).astype(np.float32)])
    d, delta, e, b = ends(d, delta)
    assert np.all(d < e)
    with np.errstate(over="ignore", divide="ignore"):
        q = np.floor(d / delta)
        plain = (q + np.float32(1)) * delta
    ok = plain > d
    assert np.array_equal(e[ok], plain[ok]) and (~ok).sum() > 1000
    small = q < 2**31
    assert np.array_equal(b[small], q[small].astype(np.int64))
