"""GPU ensembles counted on the counters' tiles, which a plan takes only from a tuner cache (without
one every counter's instances are counted by ranks): the 256-instance workload on the bitset,
int8 and fp4 tiles against the rank counter, every bin and action, and replays of the graph on
every tile configuration."""
import numpy as np
import pytest

import workloads as W
from test_gpu_batch import (BITSET_CHOICES, EPS, MFMA_CHOICES, check_instances, cs,  # noqa: F401
                            forced_cache, run_batch)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CHOICES = [(c, m) for c in (1, 2) for m in MFMA_CHOICES] + [(0, m) for m in BITSET_CHOICES]


def test_workload_256_ranks_and_tiles(cs, orc, tmp_path):  # noqa: F811
    cfg = W.WORKLOADS["batch_mink2_256"]
    sizes, seeds = W.batch_instances(cfg["seed"], cfg["count"], cfg["nmin"], cfg["nmax"])
    plan, hist, acts = run_batch(cs, sizes, seeds, cs.CS_COUNT_MFMA_FP4)
    assert int(hist.sum()) > 0
    for counter, choice in ((0, (0, 2, 2304)), (1, (2, 2, 0)), (2, (2, 2, 0)), (2, (4, 1, 0))):
        cache = forced_cache(tmp_path / f"tune{counter}{choice[0]}.json", counter, choice)
        tiles, h, a = run_batch(cs, sizes, seeds, counter, tune_cache=cache)
        assert tiles.ws_bytes < plan.ws_bytes      # no rank tables: the tiles did the counting
        assert np.array_equal(h, hist), (counter, choice)
        assert np.array_equal(a, acts), (counter, choice)


@pytest.mark.parametrize("counter,choice", CHOICES)
def test_graph_replays_on_tiles(cs, orc, tmp_path, counter, choice):  # noqa: F811
    sizes, seeds = [300, 1500, 4200, 6000, 999], [5, 6, 7, 8, 9]
    dev = torch.device("cuda")
    plan = cs.BatchPlan(sizes, counter=counter, eps=EPS,
                        tune_cache=forced_cache(tmp_path / "tune.json", counter, choice))
    s = torch.from_numpy(np.asarray(seeds, dtype=np.uint64).view(np.int64)).to(dev)
    hist = torch.empty(plan.hist_len, dtype=torch.int64, device=dev)
    acts = torch.empty(len(sizes) * len(EPS), dtype=torch.float64, device=dev)
    ws = torch.empty(plan.ws_bytes, dtype=torch.uint8, device=dev)
    plan.run(s, hist, acts, ws)
    torch.cuda.synchronize()
    h0, a0 = hist.clone(), acts.clone()
    check_instances(orc, plan, h0.cpu().numpy().view(np.uint64), a0.cpu().numpy(), sizes, seeds,
                    range(len(sizes)))
    g = plan.graph(s, hist, acts, ws)
    for rep in range(3):
        hist.fill_(-1)
        acts.fill_(float("nan"))
        x = torch.randn(1024, device=dev).sum()  # eager work between replays
        g.launch()
        torch.cuda.synchronize()
        assert torch.equal(hist, h0) and torch.equal(acts, a0), rep
        del x
