"""GPU parity of the matrix counters and the d'Alembertian where one instance changes from
128-row tiles (a workgroup per tile, bins for every count, up to 8193 points) to 256-row
ones, and at the edges of their tiles, against the oracle; a total order makes the counts
reach the last bin."""
import numpy as np
import pytest

import workloads as W
from test_gpu_dalembertian import check, cs  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("counter", [1, 2], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [129, 3969, 4097, 8065, 8192, 8193, 8194, 8449])
def test_histogram_sizes(cs, orc, n, counter):  # noqa: F811
    coords = orc.sprinkle(W.MINK3_DIAMOND, n, 3 * n)
    bits = orc.causal_matrix(W.MINK3_DIAMOND, coords)
    b = torch.from_numpy(bits.view(np.int64)).cuda()
    got = cs.cs_interval_histogram(b, n, counter).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, orc.histogram_fast(bits, n)[0]), n


@pytest.mark.parametrize("counter", [1, 2], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [4096, 8193, 8194])
def test_total_order(cs, n, counter):  # noqa: F811
    """N_m = n - 1 - m for m = 0 .. n - 2."""
    u = torch.arange(n, dtype=torch.float64, device="cuda") / n
    b = cs.cs_causal_matrix(W.MINK2_DIAMOND, torch.stack([u, u]).contiguous())
    got = cs.cs_interval_histogram(b, n, counter)
    want = torch.arange(n - 1, 0, -1, dtype=torch.int64, device="cuda")
    assert torch.equal(got, want)


@pytest.mark.parametrize("counter", [1, 2], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [8193, 8194])
def test_dalembertian_sizes(cs, orc, n, counter):  # noqa: F811
    check(cs, orc, W.MINK2_DIAMOND, 2, n, 5 + n, counter)
