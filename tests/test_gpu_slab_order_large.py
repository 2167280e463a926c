"""The orders of test_gpu_slab_order.py above 3072 points, where a wavefront of the builder takes
four row blocks and its block test of the times looks at all of them: time-ordered points,
ties across block edges, one late point among early ones in each of the four row blocks,
reversed and shuffled points, times that are not numbers, and a run of equal times longer than
the four blocks.  Bit-exact against the oracle."""
import numpy as np
import pytest

import workloads as W
from test_gpu_slab_order import cs  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("form", ["sorted", "ties", "run", "swap0", "swap1", "swap2", "swap3", "reversed",
                                  "shuffled", "nan"])
@pytest.mark.parametrize("n", [3073, 3333, 4224])
@pytest.mark.parametrize("region", [W.DS2_SLAB, W.DS4_SLAB])
def test_slab_orders_of_four_row_blocks(cs, orc, region, n, form):  # noqa: F811
    c = orc.sprinkle(region, n, seed=n)
    rng = np.random.default_rng(n)
    # the time that the relation compares: x = tan(eta) in the 3+1 slab, eta in the 1+1 slab
    time = 0 if region == W.DS4_SLAB else 1
    if form == "ties":
        for e in range(64, n, 64):
            c[time, e - 2:e + 1] = c[time, e]
    elif form == "run":
        c[time, 1000:1400] = c[time, 1400]
    elif form.startswith("swap"):  # in row block 0 .. 3 of a group of four
        k = 64 * int(form[-1]) + 17
        c[:, [k, n - 1]] = c[:, [n - 1, k]]
    elif form == "reversed":
        c = c[:, ::-1]
    elif form == "shuffled":
        c = c[:, rng.permutation(n)]
    elif form == "nan":
        c[time, rng.choice(n, 5, replace=False)] = np.nan
    c = np.ascontiguousarray(c)
    want = orc.causal_matrix(region, c)
    got = cs.cs_causal_matrix(region, torch.from_numpy(c).cuda()).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, want)
