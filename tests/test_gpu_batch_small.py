"""GPU parity of ensembles whose small diamonds (up to 512 points) run in launches of their
own, because there are at least 512 of them or none has more than 192 points: sizes at the
edges of the forms, with and without larger diamonds beside them, counted by ranks or, from a
cache, on tiles; coordinates and matrices bit for bit, and replays of the graph."""
import numpy as np
import pytest

import workloads as W
from test_gpu_batch import EPS, check_instances, cs, forced_cache, run_batch  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGES = [2, 3, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 319, 320, 321,
         383, 385, 447, 448, 449, 511, 512]
LARGE = [513, 577, 1024, 3000, 8192]


def ensemble(form):
    if form == "tiny":
        return [n for n in EDGES if n <= 192]
    if form == "one":
        return [192]
    if form == "few small":
        return EDGES
    if form == "many":
        return EDGES * 20
    sizes = EDGES * 19 + LARGE          # 513 small ones
    if form == "too few":
        sizes = sizes[2:]               # 511
    return [sizes[k] for k in np.random.default_rng(4).permutation(len(sizes))]


@pytest.mark.parametrize("counter", [0, 1, 2], ids=["bitset", "mfma", "mfma_fp4"])
@pytest.mark.parametrize("form", ["tiny", "one", "few small", "many", "mixed", "too few"])
@pytest.mark.parametrize("tiles", [False, True], ids=["ranks", "tiles"])
def test_small_instances(cs, orc, tmp_path, form, counter, tiles):  # noqa: F811
    sizes = ensemble(form)
    seeds = [700 + 13 * k for k in range(len(sizes))]
    choice = (0, 2, 2304) if counter == 0 else (2, 2, 0)
    cache = forced_cache(tmp_path / "tune.json", counter, choice) if tiles else None
    plan, hist, acts = run_batch(cs, sizes, seeds, counter, tune_cache=cache)
    check_instances(orc, plan, hist, acts, sizes, seeds,
                    [k for k in range(len(sizes)) if sizes[k] < 4000 or counter == 2])


@pytest.mark.parametrize("form", ["tiny", "mixed"])
def test_small_workspace_and_graph(cs, orc, form):  # noqa: F811
    sizes = ensemble(form)
    seeds = [40 + 7 * k for k in range(len(sizes))]
    dev = torch.device("cuda")
    plan = cs.BatchPlan(sizes, counter=2, eps=EPS)
    s = torch.from_numpy(np.asarray(seeds, dtype=np.uint64).view(np.int64)).to(dev)
    hist = torch.empty(plan.hist_len, dtype=torch.int64, device=dev)
    acts = torch.empty(len(sizes) * len(EPS), dtype=torch.float64, device=dev)
    ws = torch.full((plan.ws_bytes,), 255, dtype=torch.uint8, device=dev)
    plan.run(s, hist, acts, ws)
    torch.cuda.synchronize()
    host = ws.cpu().numpy()
    for k, (n, seed) in enumerate(zip(sizes, seeds)):
        want_c = orc.sprinkle(W.MINK2_DIAMOND, n, seed)
        co, bo, ld = plan.coords_offsets[k], plan.bits_offsets[k], cs.cs_ld_words(n)
        got_c = host[co:co + 16 * n].view(np.float64).reshape(2, n)
        assert np.array_equal(got_c.view(np.uint64), want_c.view(np.uint64)), (k, n)
        got_b = host[bo:bo + 8 * n * ld].view(np.uint64).reshape(n, ld)
        assert np.array_equal(got_b, orc.causal_matrix(W.MINK2_DIAMOND, want_c, ld=ld)), (k, n)
    h0, a0 = hist.clone(), acts.clone()
    g = plan.graph(s, hist, acts, ws)
    for rep in range(3):
        hist.fill_(-1)
        acts.fill_(float("nan"))
        x = torch.randn(1024, device=dev).sum()  # eager work between replays
        g.launch()
        torch.cuda.synchronize()
        assert torch.equal(hist, h0) and torch.equal(acts, a0), rep
        del x
