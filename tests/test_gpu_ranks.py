"""GPU parity of the ensembles' rank counter against the oracle, bit for bit: sizes at the
edges of its 64-point blocks and 256-row units, and plans that mix ranks and tiles."""
import json

import numpy as np
import pytest

from test_gpu_batch import BUCKETS, NAMES, check_instances, cs, run_batch  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = [2, 3, 63, 64, 65, 127, 128, 129, 255, 256, 257, 319, 320, 321, 511, 512, 513, 575, 576,
         1023, 1025, 2049, 4097, 8129, 8191, 8192]


@pytest.mark.parametrize("sizes", [EDGES, [2], [8192], [5] * 300], ids=["edges", "one", "largest",
                                                                         "many"])
def test_rank_counter_sizes(cs, orc, sizes):  # noqa: F811
    seeds = [9000 + 31 * k for k in range(len(sizes))]
    plan, hist, acts = run_batch(cs, sizes, seeds, cs.CS_COUNT_MFMA_FP4)
    check_instances(orc, plan, hist, acts, sizes, seeds, range(0, len(sizes), 1 + len(sizes) // 40))


@pytest.mark.parametrize("counter", [0, 1, 2], ids=["bitset", "mfma", "mfma_fp4"])
def test_rank_counter_beside_tiles(cs, orc, tmp_path, counter):  # noqa: F811
    """A cache entry keeps its tiles unless it shows a faster rank count: here the first
    bucket has no entry, the second a faster rank count, the third a slower one, the fourth
    none (a file of the earlier format)."""
    mode, per_cu, pair_max = (0, 2, 2304) if counter == 0 else (2, 2, 0)
    entries = [{"counter": NAMES[counter], "n_lo": lo, "n_hi": hi, "mode": mode, "tile": 128,
                "per_cu": per_cu, "pair_max": pair_max, "ms": 1.0} for lo, hi in BUCKETS[1:]]
    entries[0]["rank_ms"], entries[1]["rank_ms"] = 0.5, 2.0
    path = tmp_path / "tune.json"
    path.write_text("{\n  \"entries\": [\n" + ",\n".join(json.dumps(e) for e in entries) + "\n  ]\n}\n")
    sizes = [900, 65, 1500, 1024, 3000, 2111, 6000, 4096]
    seeds = [40 + k for k in range(len(sizes))]
    plan, hist, acts = run_batch(cs, sizes, seeds, counter, tune_cache=str(path))
    check_instances(orc, plan, hist, acts, sizes, seeds, range(len(sizes)))
    ranked = cs.BatchPlan([900, 65, 1500, 1024], counter=counter)
    tiles = cs.BatchPlan([3000, 2111, 6000, 4096], counter=counter, tune_cache=str(path))
    matrices = sum(8 * n * cs.cs_ld_words(n) for n in sizes)
    # only the instances counted by ranks have rank tables in the workspace
    assert matrices < plan.ws_bytes < ranked.ws_bytes + tiles.ws_bytes
    assert np.asarray(hist).sum() > 0
