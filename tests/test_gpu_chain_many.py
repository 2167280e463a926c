"""GPU longest chains of many pairs of small sets: more than 256 pairs, whose members are
surveyed by a wavefront per pair, in both forms of the rounds and with every number of
threads per word, against the oracle and against the same pairs in calls of 200."""
import numpy as np
import pytest

import workloads as W
from test_gpu_chain_forms import cs, rectangle_heights  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,count", [(65, 257), (65, 2000), (65, 40000), (500, 257), (1000, 3000),
                                     (1025, 300), (4096, 700), (4097, 700), (33000, 300)])
def test_many_pairs(cs, n, count):  # noqa: F811
    coords = cs.cs_sprinkle(W.MINK2_DIAMOND, n, n + count)
    bits = cs.cs_causal_matrix(W.MINK2_DIAMOND, coords)
    u, v = coords.cpu().numpy()
    rng = np.random.default_rng(n)
    ends = np.sort(rng.integers(0, n, size=(2, count)), axis=0)
    lo, hi = ends[0] - 1, ends[1] + 1
    lo[count // 2], hi[count // 2] = -1, n
    length, height = cs.cs_longest_chain(bits, n, lo, hi, heights=True)
    for s in range(0, min(count, 4000), 200):
        some, theirs = cs.cs_longest_chain(bits, n, lo[s:s + 200], hi[s:s + 200], heights=True)
        assert torch.equal(length[s:s + 200], some) and torch.equal(height[s:s + 200], theirs), s
    for s in [*range(0, count, 1 + count // 8), count // 2, count - 1]:
        want_length, want = rectangle_heights(u, v, int(lo[s]), int(hi[s]))
        if hi[s] < n and lo[s] >= 0 and not (u[hi[s]] > u[lo[s]] and v[hi[s]] > v[lo[s]]):
            want_length, want = 0, np.zeros(n, np.int32)
        assert int(length[s]) == want_length, (s, lo[s], hi[s])
        assert np.array_equal(height[s].cpu().numpy(), want), (s, lo[s], hi[s])
