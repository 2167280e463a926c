"""GPU causal matrix of the de Sitter slabs where the builder's block test of the times can go
wrong: time-ordered points, ties of the time across the edges of the 64-point blocks, one
late point among early ones, reversed and shuffled points, and times that are not numbers.
Bit-exact against the oracle, which compares the times of every pair."""
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


@pytest.mark.parametrize("form", ["sorted", "ties", "swap", "reversed", "shuffled", "nan"])
@pytest.mark.parametrize("n", [64, 200, 577, 1100])
@pytest.mark.parametrize("region", [W.DS2_SLAB, W.DS4_SLAB])
def test_slab_orders(cs, orc, region, n, form):
    c = orc.sprinkle(region, n, seed=n)
    rng = np.random.default_rng(n)
    if form == "ties":  # the last points of a block share the time of the next one's first
        for e in range(64, n, 64):
            c[0, e - 2:e + 1] = c[0, e]
    elif form == "swap":  # a late point in the first block, an early one in the last
        c[:, [min(63, n // 2), n - 1]] = c[:, [n - 1, min(63, n // 2)]]
    elif form == "reversed":
        c = c[:, ::-1]
    elif form == "shuffled":
        c = c[:, rng.permutation(n)]
    elif form == "nan":
        c[0, rng.choice(n, 3, replace=False)] = np.nan
    c = np.ascontiguousarray(c)
    want = orc.causal_matrix(region, c)
    got = cs.cs_causal_matrix(region, torch.from_numpy(c).cuda()).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, want)
