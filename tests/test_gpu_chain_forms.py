"""GPU longest chains at the sizes where the call changes form: one workgroup per pair with
the set in LDS (up to 32768 elements, 16-bit indices) against a launch per round, few pairs
(16 wavefronts per word) against many (4), and the blind first batch (up to 4096 words in
all).  1+1 diamonds, where the height of an element above lo is the longest increasing
subsequence of v in u order inside the rectangle of the pair."""
import bisect

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


def rectangle_heights(u, v, lo, hi):
    n = len(u)
    inside = np.ones(n, bool)
    if lo >= 0:
        inside &= (u > u[lo]) & (v > v[lo])
    if hi < n:
        inside &= ((u < u[hi]) & (v < v[hi])) | (np.arange(n) == hi)
    height = np.zeros(n, np.int32)
    members = np.flatnonzero(inside)
    tails = []
    for k in members[np.lexsort((-v[members], u[members]))]:
        p = bisect.bisect_left(tails, v[k])
        tails[p:p + 1] = [v[k]]
        height[k] = p + 1
    length = height[hi] if hi < n else len(tails) + 1
    return length, height


@pytest.mark.parametrize("n,count", [(65, 1), (700, 300), (4096, 64), (4097, 70), (16385, 17),
                                     (32767, 2), (32768, 3), (32769, 3)])
def test_chain_forms(cs, n, count):
    coords = cs.cs_sprinkle(W.MINK2_DIAMOND, n, 7 * n + count)
    bits = cs.cs_causal_matrix(W.MINK2_DIAMOND, coords)
    u, v = coords.cpu().numpy()
    rng = np.random.default_rng(n)
    ends = np.sort(rng.integers(0, n, size=(2, count)), axis=0)
    lo, hi = ends[0] - 1, ends[1] + 1  # lo < hi, virtual ends among them
    lo[0], hi[0] = -1, n
    length, height = cs.cs_longest_chain(bits, n, lo, hi, heights=True)
    torch.cuda.synchronize()
    length, height = length.cpu().numpy(), height.cpu().numpy()
    for s in range(0, count, 1 + count // 12):
        want_length, want = rectangle_heights(u, v, int(lo[s]), int(hi[s]))
        if hi[s] < n and want[hi[s]] and lo[s] >= 0 and not (u[hi[s]] > u[lo[s]] and v[hi[s]] > v[lo[s]]):
            want_length, want = 0, np.zeros(n, np.int32)
        assert np.array_equal(height[s], want), (n, s, lo[s], hi[s])
        assert length[s] == want_length, (n, s, lo[s], hi[s])
