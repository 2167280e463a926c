"""The map from a slab point's time to its bucket (csrc/common.h, bucket_of_time), compiled for
the CPU: it follows the (key, index) order, and no bucket is so full that its placement
leaves the LDS path, for half-widths from the smallest double to just below pi/2."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import workloads as W
from paper_1805_04463_amd import build as hip_build

MEAN, CAP = 64, 2048   # kBucketMean, kBucketCap


@pytest.fixture(scope="module")
def bucket(tmp_path_factory):
    d = tmp_path_factory.mktemp("buckets")
    src = d / "buckets.hip"
    src.write_text(f'#include "{hip_build.CSRC}/common.h"\n' + """
extern "C" void buckets(const double* x, double X, uint64_t n, uint64_t B, uint64_t* out) {
  for (uint64_t g = 0; g < n; ++g) {
    const uint64_t b = cs::bucket_of_time(x[g], X, g, n, B);
    out[g] = b < B ? b : B - 1;
  }
}
""")
    lib = str(d / "buckets.so")
    subprocess.run([hip_build.HIPCC, "-O1", "-std=c++17", "-ffp-contract=off", "--offload-host-only",
                    "-shared", "-fPIC", str(src), "-o", lib], check=True, capture_output=True)
    f = ctypes.CDLL(lib).buckets
    f.argtypes = [ctypes.c_void_p, ctypes.c_double, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_void_p]

    def run(x, X):
        n = len(x)
        B = (n + MEAN - 1) // MEAN
        out = np.empty(n, np.uint64)
        f(x.ctypes.data, X, n, B, out.ctypes.data)
        return out, B
    return run


def slab_times(region, X, n, seed):
    u = np.random.default_rng(seed).integers(0, 2**53, n) * 2.0**-53
    if region == W.DS2_SLAB:
        return (2.0 * u - 1.0) * X
    y = (2.0 * u - 1.0) * (X + X * X * X / 3.0)
    return 2.0 * np.sinh(np.arcsinh(1.5 * y) / 3.0)


SMALLEST = 5e-324
HALF_WIDTHS = [SMALLEST * k for k in (1, 2, 3, 7, 20, 1000)] + [
    1e-315, 2.3e-308, 1e-306, 2.0**-901, np.nextafter(2.0**-900, 0.0), 2.0**-900, 1e-100, 1e-3, 0.5,
    1.2, 1.57, np.nextafter(np.pi / 2, 0.0)]


@pytest.mark.parametrize("n", [8193, 30001, 200003])
@pytest.mark.parametrize("region", [W.DS2_SLAB, W.DS4_SLAB])
def test_buckets_follow_the_order(bucket, region, n):
    for k, eta0 in enumerate(HALF_WIDTHS):
        X = float(np.tan(eta0))
        x = slab_times(region, X, n, 10 * n + k)
        b, B = bucket(x, X)
        bits = x.view(np.uint64)  # the key: the numeric order, and -0 before 0
        key = np.where(bits >> np.uint64(63), ~bits, bits | np.uint64(1 << 63))
        order = np.lexsort((np.arange(n), key))
        assert np.all(np.diff(b[order].astype(np.int64)) >= 0), eta0
        assert np.bincount(b.astype(np.int64), minlength=B).max() <= CAP // 4, eta0
