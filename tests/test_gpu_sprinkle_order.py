"""GPU time order of sets placed by buckets, against the oracle's qsort: every region, sizes
off the bucket mean, a slab so deep that its points crowd at the ends, and the rank
placement just below."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_04463_amd as cs
    cs.lib()
    return cs


@pytest.mark.parametrize("n", [4096, 4097, 8192, 8193, 30001, 131072, 200003])
@pytest.mark.parametrize("region,eta0", [(W.MINK2_DIAMOND, 1.2), (W.MINK3_DIAMOND, 1.2),
                                         (W.MINK4_DIAMOND, 1.2), (W.DS2_SLAB, 0.5),
                                         (W.DS2_SLAB, 1.57), (W.DS4_SLAB, 1.2), (W.DS4_SLAB, 1.57)])
def test_time_order(cs, orc, region, eta0, n):
    got = cs.cs_sprinkle(region, n, 5 * n + region, eta0).cpu().numpy()
    want = orc.sprinkle(region, n, 5 * n + region, eta0)
    if region == W.DS2_SLAB:  # atan may differ by an ulp; the key and the angle are exact
        np.testing.assert_array_equal(got[[0, 2]], want[[0, 2]])
        np.testing.assert_array_max_ulp(got[1], want[1], 2)
    elif region == W.DS4_SLAB:  # the S^3 directions are exact and show the order by themselves
        np.testing.assert_array_equal(got[3:].view(np.uint64), want[3:].view(np.uint64))
        assert np.all(np.diff(got[0]) >= 0)
    else:
        np.testing.assert_array_equal(got.view(np.uint64), want.view(np.uint64))
