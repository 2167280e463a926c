"""GPU time order of slabs so thin that many points share a time, or that twice the half-width's
reciprocal overflows, placed by buckets and (4000 points) by ranks: the times of the 1+1
slab and their ties by generation index are exact; in the 3+1 slab the S^3 directions are,
and do not depend on the width."""
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


@pytest.mark.parametrize("eta0", [5e-324, 1e-322, 1e-310, 1e-306, 2.0**-901, 1e-200])
@pytest.mark.parametrize("n", [4000, 9001, 30001])
def test_thin_slabs(cs, orc, n, eta0):
    got = cs.cs_sprinkle(W.DS2_SLAB, n, n, eta0).cpu().numpy()
    want = orc.sprinkle(W.DS2_SLAB, n, n, eta0)
    np.testing.assert_array_equal(got[[0, 2]], want[[0, 2]])
    got = cs.cs_sprinkle(W.DS4_SLAB, n, n, eta0).cpu().numpy()
    want = orc.sprinkle(W.DS4_SLAB, n, n, eta0)
    assert np.all(np.diff(got[0]) >= 0)
    by_direction = [np.lexsort(c[3:]) for c in (got, want)]
    np.testing.assert_array_equal(got[3:, by_direction[0]], want[3:, by_direction[1]])
