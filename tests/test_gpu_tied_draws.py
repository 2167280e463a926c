"""GPU ensembles with two points of exactly equal u, or of equal v: unrelated whatever their
other coordinate, so the places that the rank counter and the builder work from must take
opposite orders in u and v.

A pair of equal 53-bit draws is rare (n^2 / 2^54 per instance), but seeds that hold one can be
written down: the finalizer of SplitMix64 and the seeding are bijections, so from two 64-bit
states with equal leading output bits whose difference is an even multiple d of the generator's
increment, a seed follows that makes them draws c and c + d of an instance's stream, for any c:
the u (c even) or the v (c odd) of points c / 2 and (c + d) / 2."""
import numpy as np
import pytest

import workloads as W
from test_gpu_batch import EPS, check_instances, cs, forced_cache  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GOLDEN, MASK = 0x9E3779B97F4A7C15, 2**64 - 1
STATE, D = 0x78398C82C5FEE9C6, 7486    # found by a search over 2^29 leading values


def unmix(z):
    """Inverse of SplitMix64's finalizer."""
    z ^= z >> 31 ^ z >> 62
    z = z * pow(0x94D049BB133111EB, -1, 2**64) & MASK
    z ^= z >> 27 ^ z >> 54
    z = z * pow(0xBF58476D1CE4E5B9, -1, 2**64) & MASK
    return z ^ z >> 30 ^ z >> 60


def seed_with_tie(c):
    """Seed of a 1+1 diamond whose draws c and c + D share their 53 bits."""
    key = (STATE - (c + 1) * GOLDEN) & MASK          # the stream key
    return (unmix((unmix(key) - GOLDEN) & MASK) - GOLDEN) & MASK


DRAWS = [0, 1, 2, 3, 10, 11, 700, 701, 702, 703]
SIZES = [D // 2 + 1 + c // 2 for c in DRAWS[:2]] + [4097, 5000, 8192, 8192, 4096 + 64, 6000, 8191, 7000]


def test_seeds_hold_ties(orc):
    for c, n in zip(DRAWS, SIZES):
        tied = orc.sprinkle(W.MINK2_DIAMOND, n, seed_with_tie(c))[c % 2]
        assert len(np.unique(tied)) == n - 1
    assert {c % 2 for c in DRAWS} == {0, 1}


@pytest.mark.parametrize("counter,tiles", [(2, False), (2, True), (1, True), (0, True)],
                         ids=["ranks", "fp4", "int8", "bitset"])
def test_tied_draws(cs, orc, tmp_path, counter, tiles):  # noqa: F811
    seeds = [seed_with_tie(c) for c in DRAWS]
    choice = (0, 2, 2304) if counter == 0 else (2, 2, 0)
    cache = forced_cache(tmp_path / "tune.json", counter, choice) if tiles else None
    plan = cs.BatchPlan(SIZES, counter=counter, eps=EPS, tune_cache=cache)
    dev = torch.device("cuda")
    s = torch.from_numpy(np.asarray(seeds, dtype=np.uint64).view(np.int64)).to(dev)
    hist = torch.empty(plan.hist_len, dtype=torch.int64, device=dev)
    acts = torch.empty(len(SIZES) * len(EPS), dtype=torch.float64, device=dev)
    ws = torch.empty(plan.ws_bytes, dtype=torch.uint8, device=dev)
    plan.run(s, hist, acts, ws)
    torch.cuda.synchronize()
    host = ws.cpu().numpy()
    for k, (n, seed) in enumerate(zip(SIZES, seeds)):
        want = orc.sprinkle(W.MINK2_DIAMOND, n, seed)
        co, bo, ld = plan.coords_offsets[k], plan.bits_offsets[k], cs.cs_ld_words(n)
        got = host[co:co + 16 * n].view(np.float64).reshape(2, n)
        assert np.array_equal(got.view(np.uint64), want.view(np.uint64)), (k, n)
        bits = host[bo:bo + 8 * n * ld].view(np.uint64).reshape(n, ld)
        assert np.array_equal(bits, orc.causal_matrix(W.MINK2_DIAMOND, want, ld=ld)), (k, n)
    check_instances(orc, plan, hist.cpu().numpy().view(np.uint64), acts.cpu().numpy(), SIZES, seeds,
                    range(len(SIZES)))
