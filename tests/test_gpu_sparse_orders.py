"""GPU counts and d'Alembertian of orders whose matrices have whole tiles without a related pair:
an antichain, and clusters of related points that are unrelated to each other, so that full and
empty tiles alternate in a workgroup.  128-row tiles end an empty one after its first stage."""
import numpy as np
import pytest

import workloads as W
from test_gpu_dalembertian import K, cs  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def clusters(n, size, seed):
    """1+1 points, cluster after cluster: u grows and v falls from one to the next."""
    rng = np.random.default_rng(seed)
    k = np.arange(n) // size
    u, v = rng.random(n), rng.random(n)
    m = k[-1] + 1
    order = np.lexsort((u + v, k))          # time order within each: a linear extension
    return np.ascontiguousarray(np.stack([(k + u) / m, (m - 1 - k + v) / m])[:, order])


@pytest.mark.parametrize("counter", [0, 1, 2], ids=["bitset", "mfma", "mfma_fp4"])
@pytest.mark.parametrize("n,size", [(900, 1), (4097, 300), (5000, 1), (8320, 1000), (9000, 700),
                                    (12000, 1), (12000, 130), (12000, 2500)])
def test_empty_tiles(cs, orc, n, size, counter):  # noqa: F811
    coords = clusters(n, size, n + size)
    bits = orc.causal_matrix(W.MINK2_DIAMOND, coords)
    b = cs.cs_causal_matrix(W.MINK2_DIAMOND, torch.from_numpy(coords).cuda())
    assert np.array_equal(b.cpu().numpy().view(np.uint64), bits)
    got = cs.cs_interval_histogram(b, n, counter).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, orc.histogram_fast(bits, n)[0])
    if counter == 0:
        return
    phi = np.random.default_rng(n).normal(size=n)
    want, terms, mag = orc.dalembertian(bits, n, 2, 0.05, phi)
    out = cs.cs_dalembertian(b, n, 2, 0.05, torch.from_numpy(phi).cuda(), counter=counter).cpu().numpy()
    bound = K[2] / 0.05 ** 2 * (terms + 2) * 2.0 ** -52 * mag + 8 * 2.0 ** -52 * np.abs(want)
    assert np.all(np.abs(out - want) <= bound)
