"""GPU smeared action where the walk over the bins ends before the histogram does: counts up
to 2^62 in every bin, the far ones included, against the oracle's quad-precision sum over
all of them.  The bound is the double-double sum's: 2^-96 of the absolute summands (2^-104
per operation, a few hundred of them), and the one rounding to fp64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("n,eps", [(40000, 0.5), (40000, 0.1), (40000, 0.02), (3000, 0.9), (3000, 0.1)])
def test_far_bins(orc, n, eps, dim):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_04463_amd as cs
    rng = np.random.default_rng(n + dim)
    hist = rng.integers(0, 2**62, size=n - 1, dtype=np.int64)
    hist[n // 2:] = 2**62 - 1
    got = cs.cs_action(torch.from_numpy(hist).cuda(), n, dim, eps).item()
    want, kappa = orc.action(hist.view(np.uint64), n, dim, eps)[:2]
    assert abs(got - want) <= (2.0**-96 * kappa + 2.0**-52) * abs(want), (got, want, kappa)
