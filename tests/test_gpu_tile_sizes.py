"""GPU parity of the matrix counters and the d'Alembertian where one instance changes its
form, and at the edges of the tiles, against the oracle: a workgroup per 128-row tile up to
8193 points, resident workgroups above, bins for every count up to 11777 points, 256-row
tiles above 11777 (int8) and 24000 (fp4), for the d'Alembertian above 15000 and 32768.  A
total order makes the counts reach the last bin."""
import numpy as np
import pytest

import workloads as W
from test_gpu_dalembertian import check, cs  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("counter", [1, 2], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [129, 3969, 4097, 8065, 8192, 8193, 8320, 8321, 8449, 11777, 11778,
                               12000])
def test_histogram_sizes(cs, orc, n, counter):  # noqa: F811
    coords = orc.sprinkle(W.MINK3_DIAMOND, n, 3 * n)
    bits = orc.causal_matrix(W.MINK3_DIAMOND, coords)
    b = torch.from_numpy(bits.view(np.int64)).cuda()
    got = cs.cs_interval_histogram(b, n, counter).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, orc.histogram_fast(bits, n)[0]), n


@pytest.mark.parametrize("counter", [1, 2], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [4096, 8193, 8321, 11777, 11778, 11841, 24000, 24001])
def test_total_order(cs, n, counter):  # noqa: F811
    """N_m = n - 1 - m for m = 0 .. n - 2."""
    u = torch.arange(n, dtype=torch.float64, device="cuda") / n
    b = cs.cs_causal_matrix(W.MINK2_DIAMOND, torch.stack([u, u]).contiguous())
    got = cs.cs_interval_histogram(b, n, counter)
    want = torch.arange(n - 1, 0, -1, dtype=torch.int64, device="cuda")
    assert torch.equal(got, want)


@pytest.mark.parametrize("counter", [1, 2], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [8193, 15000, 15001])
def test_dalembertian_sizes(cs, orc, n, counter):  # noqa: F811
    check(cs, orc, W.MINK2_DIAMOND, 2, n, 5 + n, counter)


@pytest.mark.parametrize("n", [32768, 32769])
def test_dalembertian_large_total_order(cs, n):  # noqa: F811
    """phi = 1 on a total order: L_m(j) holds one element for m <= j, so 2 (-1 + 2 - 4 + 2)
    = -2 from j = 3 on, and the first elements lack the layers below them."""
    u = torch.arange(n, dtype=torch.float64, device="cuda") / n
    b = cs.cs_causal_matrix(W.MINK2_DIAMOND, torch.stack([u, u]).contiguous())
    phi = torch.ones(n, dtype=torch.float64, device="cuda")
    got = cs.cs_dalembertian(b, n, 2, 1.0, phi).cpu().numpy()
    want = np.full(n, -2.0)
    want[:3] = [-2.0, 2.0, -6.0]
    assert np.array_equal(got, want)


@pytest.mark.parametrize("counter", [1, 2], ids=["mfma", "mfma_fp4"])
@pytest.mark.parametrize("n", [2, 128, 129, 4100, 15000, 15001, 32768, 32769])
def test_dalembertian_workspaces(cs, n, counter):  # noqa: F811
    """The smallest workspace (one accumulator per element) and the queried one (a second,
    with whatever it held before) give the same bits for whole phi and coefficients, whose
    sums are exact in any order; one byte less than the smallest is refused."""
    b = cs.cs_causal_matrix(W.MINK4_DIAMOND, cs.cs_sprinkle(W.MINK4_DIAMOND, n, n))
    g = torch.Generator(device="cuda").manual_seed(n)
    phi = torch.randint(-8, 9, (n,), device="cuda", generator=g).double()
    small = torch.full((256,), 255, dtype=torch.uint8, device="cuda")
    full = torch.full((cs.lib().cs_dalembertian_workspace_bytes(n, counter),), 255,
                      dtype=torch.uint8, device="cuda")
    one = cs.cs_dalembertian(b, n, 4, 1.0, phi, counter=counter, workspace=small)
    two = cs.cs_dalembertian(b, n, 4, 1.0, phi, counter=counter, workspace=full)
    assert torch.equal(one, two)
    with pytest.raises(RuntimeError):
        cs.cs_dalembertian(b, n, 4, 1.0, phi, counter=counter, workspace=small[:255])
