"""The order in which 128-row histogram tiles leave their queue above 11777 points
(csrc/common.h, scatter_step, compiled for the CPU): every tile once, and the tiles in flight
together spread over the distances from the diagonal.  Tiles of one distance can add to the
same bins of the global histogram, all at once if they run at once."""
import ctypes
import math
import subprocess

import numpy as np
import pytest

from paper_1805_04463_amd import build as hip_build

IN_FLIGHT = 512


@pytest.fixture(scope="module")
def scatter_step(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    src = d / "order.hip"
    src.write_text(f'#include "{hip_build.CSRC}/common.h"\n'
                   'extern "C" int64_t step(int64_t m) { return cs::scatter_step(m); }\n')
    lib = str(d / "order.so")
    subprocess.run([hip_build.HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-shared", "-fPIC",
                    str(src), "-o", lib], check=True, capture_output=True)
    f = ctypes.CDLL(lib).step
    f.argtypes, f.restype = [ctypes.c_int64], ctypes.c_int64
    return f


@pytest.mark.parametrize("T", [93, 94, 128, 141, 157, 187, 188])
def test_tiles_scatter(scatter_step, T):
    tiles = T * (T + 1) // 2
    spread = tiles * 3 // 4
    step = scatter_step(spread)
    assert math.gcd(step, spread) == 1
    order = np.arange(spread) * step % spread
    assert len(np.unique(order)) == spread
    # tile t lies at distance T - 1 - e, e (e + 1) / 2 <= t
    e = ((np.sqrt(8.0 * order + 1.0) - 1.0) / 2.0 + 1e-9).astype(int)
    for at in range(0, spread - IN_FLIGHT, 97):
        assert np.bincount(e[at:at + IN_FLIGHT]).max() <= 2 * IN_FLIGHT * T // spread + 2


def test_every_length(scatter_step):
    for m in range(1, 3000):
        assert math.gcd(scatter_step(m), m) == 1
