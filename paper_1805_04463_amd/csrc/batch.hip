// Ensembles of independent 1+1 diamonds: plan, run, HIP-graph capture and the tile
// autotuner.  (The thesis averages its action measurements over ensembles of
// causal sets; here the ensemble is one pipeline of five launches.)
//
// Plan: per-instance offsets into three concatenated buffers (coordinates, matrices,
// histograms), the builder's work lists (groups of 512 columns, per XCD) and
// the counters' work lists (one item per row panel I of output tiles, i.e. all tiles
// (I, J >= I) of an instance, so a workgroup keeps one instance's histogram in LDS for
// a whole panel), dealt to one queue per XCD: whole instances, largest first to the
// least loaded queue, so the queues balance instances of very different sizes while the
// workgroups of one XCD work through one instance at a time and share its panels in that
// XCD's L2 (a workgroup that runs out of its own queue takes from the others).  Against
// one queue of row panels sorted by cost across all instances, this fetches 2.5x fewer
// bytes from HBM per launch.  These tables live in device memory owned
// by the plan, uploaded once at plan time, so a run only enqueues kernels: sprinkle,
// build, rank tables, count (one persistent launch per configuration in use), action.
//
// Counting configuration per instance: by ranks (ranks.hip), the default, or the
// counter's tiles for the instance's size bucket.  The candidates are, for the MFMA
// counters, 128x128 tiles with one or two workgroups per CU and 256x256 tiles (one per
// CU); for the bitset counter, the dense
// product on every tile or the related-pair tiles with two thresholds, two workgroups
// per CU, and the related-pair tiles with one.  cs_autotune times every candidate on
// the device per (counter, bucket) and stores the fastest in a JSON cache, one entry per
// line, with the time of the rank counter on the same ensemble; cs_batch_plan reads its
// counter's entries from that file when given its path and takes the tiles of an entry
// that shows no faster rank count (a file written without that field keeps its tiles).
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "common.h"

using namespace cs;

namespace {

constexpr int kMaxSlots = 8;  // distinct tile configurations in one plan
constexpr int kSmallUnits = 12;  // counting units of 512 points: an item holds a small instance

// Size buckets of the tuner: [lo, hi] and the centre of the sizes timed for each.
constexpr int kBuckets = 4;
constexpr int64_t kBucketLo[kBuckets] = {2, 1024, 2048, 4096};
constexpr int64_t kBucketHi[kBuckets] = {1023, 2047, 4095, kBatchMaxN};
constexpr int64_t kBucketProbe[kBuckets] = {768, 1536, 3072, 6144};

int bucket_of(int64_t n) {
  for (int b = 0; b < kBuckets; ++b)
    if (n <= kBucketHi[b]) return b;
  return kBuckets - 1;
}

// Counter slots of the cache: 0 bitset, 1 int8 MFMA, 2 fp4 MFMA.
constexpr const char* kCounterName[3] = {"bitset", "mfma", "mfma_fp4"};

bool same_tile(const BatchTile& a, const BatchTile& b) {
  return a.mode == b.mode && a.per_cu == b.per_cu && a.pair_max == b.pair_max;
}

// Candidates the tuner times per counter family.
const BatchTile kMfmaCandidates[] = {{2, 2, 0}, {2, 1, 0}, {4, 1, 0}};
const BatchTile kBitsetCandidates[] = {{0, 2, -1}, {0, 2, 1152}, {0, 2, 2304}, {0, 1, 2304}};

// Counting by ranks is one more configuration (mode 1), the same for every counter: O(N^2)
// operations per instance where the tiles take O(N^3), the same exact counts.
// Small instances in launches of their own (kSmallN) have eight workgroups per CU.
const BatchTile kRankTile = {1, 2, 0}, kSmallRankTile = {1, 32 / kSmallWaves, 0};

struct TuneTable {
  bool have[3][kBuckets] = {};
  BatchTile cfg[3][kBuckets] = {};
  double ms[3][kBuckets] = {};
  int64_t reps[3][kBuckets] = {};  // instances of the probe ensemble
  double rank_ms[3][kBuckets] = {};  // the rank counter on the same ensemble (0: not timed)
  // The configuration of an instance of bucket b: the faster of the entry's tiles and the
  // rank counter, which also serves the buckets without an entry.
  BatchTile choice(int c, int b) const {
    const bool tiles = have[c][b] && !(rank_ms[c][b] > 0.0 && rank_ms[c][b] < ms[c][b]);
    return tiles ? cfg[c][b] : kRankTile;
  }
};

int counter_slot(int counter) {
  return counter == CS_COUNT_BITSET ? 0 : (counter == CS_COUNT_MFMA ? 1 : 2);
}

long long field_ll(const char* entry, const char* end, const char* key, bool* ok) {
  const char* k = strstr(entry, key);
  if (!k || k > end) {
    *ok = false;
    return 0;
  }
  const char* colon = strchr(k, ':');
  if (!colon || colon > end) {
    *ok = false;
    return 0;
  }
  return atoll(colon + 1);
}

// Reads the entries {"counter": ..., "n_lo": ..., "mode": ..., "per_cu": ..., "pair_max":
// ..., "ms": ...} of a cache written by cs_autotune; unknown or malformed entries are
// skipped, a missing file gives an empty table.
TuneTable read_tune(const char* path) {
  TuneTable t;
  if (!path || !*path) return t;
  FILE* f = fopen(path, "r");
  if (!f) return t;
  std::string text;
  char buf[4096];
  size_t got;
  while ((got = fread(buf, 1, sizeof(buf), f)) > 0) text.append(buf, got);
  fclose(f);
  const char* p = text.c_str();
  while ((p = strstr(p, "{\"counter\": \"")) != nullptr) {
    const char* name = p + strlen("{\"counter\": \"");
    const char* end = strchr(name, '}');
    if (!end) break;
    int c = -1;
    for (int q = 0; q < 3; ++q) {
      const size_t L = strlen(kCounterName[q]);
      if (strncmp(name, kCounterName[q], L) == 0 && name[L] == '"') c = q;
    }
    bool ok = c >= 0;
    const long long lo = field_ll(name, end, "\"n_lo\"", &ok);
    const long long mode = field_ll(name, end, "\"mode\"", &ok);
    const long long per_cu = field_ll(name, end, "\"per_cu\"", &ok);
    const long long pmax = field_ll(name, end, "\"pair_max\"", &ok);
    const char* msk = strstr(name, "\"ms\"");
    const double ms = (msk && msk < end) ? atof(strchr(msk, ':') + 1) : 0.0;
    const char* rk = strstr(name, "\"rank_ms\"");
    const double rank_ms = (rk && rk < end) ? atof(strchr(rk, ':') + 1) : 0.0;
    int b = -1;
    for (int q = 0; q < kBuckets; ++q)
      if (kBucketLo[q] == lo) b = q;
    const bool mode_ok = c == 0 ? mode == 0 : (mode == 2 || mode == 4);
    if (ok && b >= 0 && mode_ok && (per_cu == 1 || per_cu == 2) && !(mode == 4 && per_cu != 1)) {
      bool has_reps = true;
      const long long reps = field_ll(name, end, "\"probe_instances\"", &has_reps);
      t.have[c][b] = true;
      t.cfg[c][b] = {(int)mode, (int)per_cu, (int)pmax};
      t.ms[c][b] = ms;
      t.rank_ms[c][b] = rank_ms;
      t.reps[c][b] = has_reps ? reps : 0;
    }
    p = end;
  }
  return t;
}

bool write_tune(const char* path, const TuneTable& t) {
  FILE* f = fopen(path, "w");
  if (!f) return false;
  fprintf(f, "{\n  \"format\": \"causal-batch-tune-2\",\n  \"entries\": [");
  bool first = true;
  for (int c = 0; c < 3; ++c)
    for (int b = 0; b < kBuckets; ++b) {
      if (!t.have[c][b]) continue;
      const BatchTile& x = t.cfg[c][b];
      fprintf(f, "%s\n    {\"counter\": \"%s\", \"n_lo\": %lld, \"n_hi\": %lld, \"mode\": %d, "
                 "\"tile\": %d, \"per_cu\": %d, \"pair_max\": %d, \"ms\": %.5f, "
                 "\"rank_ms\": %.5f, \"probe_n\": %lld, \"probe_instances\": %lld}",
              first ? "" : ",", kCounterName[c], (long long)kBucketLo[b],
              (long long)kBucketHi[b], x.mode, x.mode == 4 ? 256 : 128, x.per_cu, x.pair_max,
              t.ms[c][b], t.rank_ms[c][b], (long long)kBucketProbe[b], (long long)t.reps[c][b]);
      first = false;
    }
  fprintf(f, "\n  ]\n}\n");
  return fclose(f) == 0;
}

}  // namespace

struct cs_batch_plan_t {
  int64_t count = 0;
  int counter = CS_COUNT_MFMA;
  int n_eps = 0;
  std::vector<BatchInst> inst;
  int64_t coords_len = 0, bits_len = 0, hist_len = 0;
  int nslots = 0;
  BatchTile slot_cfg[kMaxSlots] = {};
  int64_t n_items[kMaxSlots] = {};
  BatchQueues queues[kMaxSlots] = {};
  size_t ws_bytes = 0, off_coords = 0, off_bits = 0, off_uv = 0, off_rank = 0;
  int rank_units = kRankWaves;      // counting units per item (small instances: kSmallUnits)
  void* dev = nullptr;              // device tables
  BatchInst* d_inst = nullptr;
  RankInst* d_rank = nullptr;
  double* d_eps = nullptr;
  uint32_t* d_items[kMaxSlots] = {};
  // Per class, small instances first: its instances (ids null: all of the plan), and the work
  // items of the builder and of the rank tables.
  struct Class {
    int64_t count = 0, n_build = 0, n_tab = 0;
    uint32_t *ids = nullptr, *build = nullptr, *tab = nullptr;
  } cls[2];
  int device = 0;
};

namespace {

size_t take(size_t* off, size_t bytes) {
  size_t o = *off;
  *off = align_up(*off + bytes, 256);
  return o;
}

// tune: the cache's choices; force: if not null, every instance takes this configuration
// (the tuner's candidates).
cs_status build_plan(int64_t count, const int64_t* n, int counter, int n_eps, const double* eps,
                     const TuneTable& tune, const BatchTile* force, cs_batch_plan_t* p) {
  p->count = count;
  p->counter = counter;
  p->n_eps = n_eps;
  p->inst.resize(count);
  struct Item {
    uint32_t packed;
    int64_t cost;
  };
  std::vector<Item> items[kMaxSlots];
  const int cslot = counter_slot(counter);
  std::vector<RankInst> rank(count);  // n = 0: counted by tiles
  const int64_t nsmall = std::count_if(n, n + count, [](int64_t m) { return m <= kSmallN; });
  const bool tiny = *std::max_element(n, n + count) <= kTinyN;
  const bool split = tiny || nsmall >= kSmallMany;  // small instances by themselves
  auto class_of = [&](int64_t m) { return split && m <= kSmallN ? 0 : 1; };
  std::vector<uint32_t> ids[2], build[2], tab[2];
  int64_t roff = 0, units = 0;
  int64_t coff = 0, boff = 0, hoff = 0;
  for (int64_t k = 0; k < count; ++k) {
    BatchInst& d = p->inst[k];
    d.n = n[k];
    d.ld = ld_words(d.n);
    d.coord_off = coff;
    d.bits_off = boff;
    d.hist_off = hoff;
    coff += 2 * d.n;
    boff += d.n * d.ld;
    hoff += d.n - 1;
    const int64_t nb = ceil_div(d.n, 64);
    const int b = bucket_of(d.n);
    const int cl = class_of(d.n);
    ids[cl].push_back((uint32_t)k);
    BatchTile cfg = force ? *force : tune.choice(cslot, b);
    if (cl == 0 && same_tile(cfg, kRankTile)) cfg = kSmallRankTile;
    int slot = -1;
    for (int q = 0; q < p->nslots; ++q)
      if (same_tile(p->slot_cfg[q], cfg)) slot = q;
    if (slot < 0) {
      if (p->nslots == kMaxSlots) return CS_ERR_UNSUPPORTED;
      slot = p->nslots++;
      p->slot_cfg[slot] = cfg;
    }
    if (cfg.mode == kRankTile.mode) {
      RankInst& r = rank[k];
      r.base = roff;
      r.hist_off = d.hist_off;
      r.n = (int32_t)d.n;
      r.nb = (int32_t)nb;
      roff = (int64_t)align_up((size_t)r.end(), 256);
      if (cl == 1) units += r.units();
      for (int64_t g = 0; g * (cl ? kTabBlocks : kSmallWaves) < nb; ++g)
        tab[cl].push_back((uint32_t)(k << 16 | g));
      continue;
    }
    const int64_t BM = cfg.mode == 4 ? 256 : 128;
    const int64_t T = ceil_div(d.n, BM);
    for (int64_t I = 0; I < T; ++I)  // row panel I: tiles (I, J) for J = I .. T-1
      items[slot].push_back({(uint32_t)(k << 16 | I << 8), (T - I) * (T - I + 1) / 2 * BM * BM * BM});
  }
  p->coords_len = coff;
  p->bits_len = boff;
  p->hist_len = hoff;
  // Builder lists, one per XCD: whole instances dealt largest first to the least loaded
  // list, so that every line of a matrix is written from one L2 (partial lines written
  // back from several XCDs multiplied the builder's HBM writes).  Workgroup b takes entry
  // b div 8 of list b mod 8 (the XCD that the dispatcher gives it): a group of 512 columns
  // of an instance.  Lists are padded with kNoBuildItem to one length.
  for (int cl = 0; cl < 2; ++cl) {
    std::vector<uint32_t> order = ids[cl];
    std::stable_sort(order.begin(), order.end(),
                     [&](uint32_t a, uint32_t b) { return p->inst[a].n > p->inst[b].n; });
    std::vector<uint32_t> lists[kBatchQueues];
    int64_t load[kBatchQueues] = {};
    for (uint32_t k : order) {
      const BatchInst& d = p->inst[k];
      const int best = (int)(std::min_element(load, load + kBatchQueues) - load);
      load[best] += d.n * d.ld;
      for (int64_t g = 0; g < d.ld / 8; ++g) lists[best].push_back((uint32_t)(k << 16 | g));
    }
    size_t len = 0;
    for (auto& l : lists) len = std::max(len, l.size());
    build[cl].assign(len * kBatchQueues, kNoBuildItem);
    for (int x = 0; x < kBatchQueues; ++x)
      std::copy(lists[x].begin(), lists[x].end(), build[cl].begin() + x * len);
    p->cls[cl].count = (int64_t)ids[cl].size();
    p->cls[cl].n_build = (int64_t)build[cl].size();
    p->cls[cl].n_tab = (int64_t)tab[cl].size();
  }
  for (int s = 0; s < p->nslots; ++s) {
    if (same_tile(p->slot_cfg[s], kSmallRankTile)) {  // an item per instance, largest first
      std::vector<uint32_t> order;
      for (uint32_t k : ids[0])
        if (rank[k].n) order.push_back(k);
      std::stable_sort(order.begin(), order.end(),
                       [&](uint32_t a, uint32_t b) { return rank[a].n > rank[b].n; });
      for (uint32_t k : order) items[s].push_back({k << 16, 0});
      p->n_items[s] = (int64_t)items[s].size();
      continue;
    }
    if (same_tile(p->slot_cfg[s], kRankTile)) {
      // Units in items of one instance, largest instances first.  An item's histogram is
      // flushed when the workgroup moves to another instance, so items are long, down to
      // about four per resident workgroup (two per CU), and at least a unit per wavefront.
      const int64_t per = units / (4 * 2 * (int64_t)device_cu_count()) / kRankWaves * kRankWaves;
      p->rank_units = (int)std::min<int64_t>(std::max<int64_t>(per, kRankWaves), 8 * kRankWaves);
      std::vector<uint32_t> order;
      for (uint32_t k : ids[1])
        if (rank[k].n) order.push_back(k);
      std::stable_sort(order.begin(), order.end(),
                       [&](uint32_t a, uint32_t b) { return rank[a].n > rank[b].n; });
      for (uint32_t k : order)
        for (int64_t c = 0; c * p->rank_units < rank[k].units(); ++c)
          items[s].push_back({(uint32_t)(k << 16 | c), 0});
      p->n_items[s] = (int64_t)items[s].size();
      continue;
    }
    // One queue per XCD holding whole instances, dealt largest first to the least loaded
    // queue; a queue runs its instances one after another (largest first), each
    // instance's row panels longest first, so the workgroups of one XCD work on the same
    // matrix at the same time and share its panels through that XCD's L2.
    std::vector<int64_t> work(count, 0);
    std::vector<std::vector<Item>> per(count);
    for (const Item& it : items[s]) {
      work[it.packed >> 16] += it.cost;
      per[it.packed >> 16].push_back(it);
    }
    std::vector<int64_t> order;
    for (int64_t k = 0; k < count; ++k)
      if (!per[k].empty()) order.push_back(k);
    std::stable_sort(order.begin(), order.end(),
                     [&](int64_t a, int64_t b) { return work[a] > work[b]; });
    std::vector<int> queue_of(count, 0);
    int64_t load[kBatchQueues] = {};
    for (int64_t k : order) {
      int best = 0;
      for (int x = 1; x < kBatchQueues; ++x)
        if (load[x] < load[best]) best = x;
      queue_of[k] = best;
      load[best] += work[k];
    }
    std::vector<Item> sorted;
    sorted.reserve(items[s].size());
    for (int x = 0; x < kBatchQueues; ++x) {
      p->queues[s].off[x] = (uint32_t)sorted.size();
      for (int64_t k : order)
        if (queue_of[k] == x) {
          std::stable_sort(per[k].begin(), per[k].end(),
                           [](const Item& a, const Item& b) { return a.cost > b.cost; });
          sorted.insert(sorted.end(), per[k].begin(), per[k].end());
        }
    }
    p->queues[s].off[kBatchQueues] = (uint32_t)sorted.size();
    items[s].swap(sorted);
    p->n_items[s] = (int64_t)items[s].size();
  }

  // Caller workspace: [work counters, per slot][coordinates][matrices][u and v places][rank
  // tables].
  size_t off = 0;
  static_assert(sizeof(unsigned int) * kMaxSlots * kBatchQueues == 256, "work counters");
  take(&off, 256);
  p->off_coords = take(&off, sizeof(double) * (size_t)coff);
  p->off_bits = take(&off, sizeof(uint64_t) * (size_t)boff);
  p->off_uv = take(&off, sizeof(uint32_t) * (size_t)(coff / 2));
  p->off_rank = take(&off, (size_t)roff);
  p->ws_bytes = off;

  // Device tables owned by the plan.
  size_t doff = 0;
  size_t o_inst = take(&doff, sizeof(BatchInst) * count);
  size_t o_rank = take(&doff, sizeof(RankInst) * count);
  size_t o_eps = take(&doff, sizeof(double) * (n_eps > 0 ? n_eps : 1));
  size_t o_ids[2], o_build[2], o_tab[2];
  for (int cl = 0; cl < 2; ++cl) {
    o_ids[cl] = take(&doff, sizeof(uint32_t) * ids[cl].size());
    o_build[cl] = take(&doff, sizeof(uint32_t) * build[cl].size());
    o_tab[cl] = take(&doff, sizeof(uint32_t) * tab[cl].size());
  }
  size_t o_items[kMaxSlots];
  for (int s = 0; s < p->nslots; ++s) o_items[s] = take(&doff, sizeof(uint32_t) * items[s].size());
  CS_HIP_CHECK(hipGetDevice(&p->device));
  CS_HIP_CHECK(hipMalloc(&p->dev, doff));
  char* b = (char*)p->dev;
  p->d_inst = (BatchInst*)(b + o_inst);
  p->d_rank = (RankInst*)(b + o_rank);
  p->d_eps = (double*)(b + o_eps);
  std::vector<char> host(doff, 0);
  memcpy(host.data() + o_inst, p->inst.data(), sizeof(BatchInst) * count);
  memcpy(host.data() + o_rank, rank.data(), sizeof(RankInst) * count);
  if (n_eps > 0) memcpy(host.data() + o_eps, eps, sizeof(double) * n_eps);
  for (int cl = 0; cl < 2; ++cl) {
    auto put = [&](const std::vector<uint32_t>& v, size_t at) {
      std::copy(v.begin(), v.end(), (uint32_t*)(host.data() + at));
      return (uint32_t*)(b + at);
    };
    uint32_t* all = put(ids[cl], o_ids[cl]);
    p->cls[cl].ids = p->cls[cl].count == count ? nullptr : all;
    p->cls[cl].build = put(build[cl], o_build[cl]);
    p->cls[cl].tab = put(tab[cl], o_tab[cl]);
  }
  for (int s = 0; s < p->nslots; ++s) {
    p->d_items[s] = (uint32_t*)(b + o_items[s]);
    uint32_t* dst = (uint32_t*)(host.data() + o_items[s]);
    for (size_t q = 0; q < items[s].size(); ++q) dst[q] = items[s][q].packed;
  }
  CS_HIP_CHECK(hipMemcpy(p->dev, host.data(), doff, hipMemcpyHostToDevice));
  return CS_OK;
}

cs_status run_counts(cs_batch_plan_t* p, char* ws, uint64_t* hist, hipStream_t st) {
  unsigned int* ctr = (unsigned int*)ws;
  const uint64_t* bits = (const uint64_t*)(ws + p->off_bits);
  char* rank_base = ws + p->off_rank;
  for (int s = 0; s < p->nslots; ++s) {
    if (!p->n_items[s]) continue;
    if (p->slot_cfg[s].mode == kRankTile.mode) {
      const bool small = same_tile(p->slot_cfg[s], kSmallRankTile);
      const cs_batch_plan_t::Class& c = p->cls[small ? 0 : 1];
      cs_status r = launch_rank_tables(small, p->d_rank, c.tab, c.n_tab, rank_base, st);
      if (r != CS_OK) return r;
      r = launch_count_ranks(small, p->d_rank, p->d_items[s], p->n_items[s],
                             small ? kSmallUnits : p->rank_units, rank_base, hist,
                             ctr + s * kBatchQueues, st);
      if (r != CS_OK) return r;
      continue;
    }
    cs_status r = launch_count_batch(p->slot_cfg[s], p->counter == CS_COUNT_MFMA_FP4, bits,
                                     p->d_inst, p->d_items[s], p->queues[s], hist,
                                     ctr + s * kBatchQueues, st);
    if (r != CS_OK) return r;
  }
  return CS_OK;
}

}  // namespace

extern "C" {

cs_status cs_batch_plan(int64_t count, const int64_t* n, int counter, int n_eps, const double* eps,
                        const char* tune_cache, cs_batch_plan_handle* plan) {
  if (!plan) return CS_ERR_INVALID_ARG;
  *plan = nullptr;
  if (counter != CS_COUNT_BITSET && counter != CS_COUNT_MFMA && counter != CS_COUNT_MFMA_FP4)
    return CS_ERR_UNSUPPORTED;
  if (count < 1 || count > 65535 || !n || n_eps < 0 || (n_eps > 0 && !eps))
    return CS_ERR_INVALID_ARG;
  for (int64_t k = 0; k < count; ++k)
    if (n[k] < 2 || n[k] > kBatchMaxN) return CS_ERR_INVALID_ARG;
  for (int e = 0; e < n_eps; ++e)
    if (!(eps[e] >= 0.0 && eps[e] <= 1.0)) return CS_ERR_INVALID_ARG;
  cs_batch_plan_t* p = new (std::nothrow) cs_batch_plan_t();
  if (!p) return CS_ERR_HIP;
  cs_status s = build_plan(count, n, counter, n_eps, eps, read_tune(tune_cache), nullptr, p);
  if (s != CS_OK) {
    if (p->dev) (void)hipFree(p->dev);
    delete p;
    return s;
  }
  *plan = p;
  return CS_OK;
}

size_t cs_batch_workspace_bytes(cs_batch_plan_handle plan) { return plan ? plan->ws_bytes : 0; }

int64_t cs_batch_hist_len(cs_batch_plan_handle plan) { return plan ? plan->hist_len : -1; }

int64_t cs_batch_hist_offset(cs_batch_plan_handle plan, int64_t k) {
  if (!plan || k < 0 || k >= plan->count) return -1;
  return plan->inst[k].hist_off;
}

int64_t cs_batch_coords_offset(cs_batch_plan_handle plan, int64_t k) {
  if (!plan || k < 0 || k >= plan->count) return -1;
  return (int64_t)plan->off_coords + (int64_t)sizeof(double) * plan->inst[k].coord_off;
}

int64_t cs_batch_bits_offset(cs_batch_plan_handle plan, int64_t k) {
  if (!plan || k < 0 || k >= plan->count) return -1;
  return (int64_t)plan->off_bits + (int64_t)sizeof(uint64_t) * plan->inst[k].bits_off;
}

cs_status cs_batch_run(cs_batch_plan_handle plan, const uint64_t* seeds, uint64_t* hist,
                       double* actions, void* workspace, size_t workspace_bytes, void* stream) {
  if (!plan || !seeds || !hist || !workspace || (plan->n_eps > 0 && !actions))
    return CS_ERR_INVALID_ARG;
  if (workspace_bytes < plan->ws_bytes) return CS_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  unsigned int* ctr = (unsigned int*)ws;
  double* coords = (double*)(ws + plan->off_coords);
  uint64_t* bits = (uint64_t*)(ws + plan->off_bits);
  uint32_t* uv = (uint32_t*)(ws + plan->off_uv);
  cs_status s;
  // the sprinkle kernel also clears the histograms and the work counters
  bool cleared = false;
  for (int cl = 0; cl < 2; ++cl) {
    const cs_batch_plan_t::Class& c = plan->cls[cl];
    if (!c.count) continue;
    if ((s = launch_sprinkle_batch(cl == 0, seeds, plan->d_inst, plan->d_rank, c.ids, c.count, coords,
                                   uv, ws + plan->off_rank, hist, (uint64_t*)ctr,
                                   cleared ? 0 : kMaxSlots * kBatchQueues / 2, st)) != CS_OK)
      return s;
    cleared = true;
  }
  for (int cl = 0; cl < 2; ++cl) {
    const cs_batch_plan_t::Class& c = plan->cls[cl];
    if ((s = launch_build_batch(cl == 0, uv, plan->d_inst, c.build, c.n_build, bits, st)) != CS_OK)
      return s;
  }
  if ((s = run_counts(plan, ws, hist, st)) != CS_OK) return s;
  return launch_action_batch(hist, plan->d_inst, plan->count, 2, plan->d_eps, plan->n_eps, actions,
                             st);
}

cs_status cs_batch_free(cs_batch_plan_handle plan) {
  if (!plan) return CS_OK;
  hipError_t e = plan->dev ? hipFree(plan->dev) : hipSuccess;
  delete plan;
  return e == hipSuccess ? CS_OK : CS_ERR_HIP;
}

cs_status cs_batch_graph_create(cs_batch_plan_handle plan, const uint64_t* seeds, uint64_t* hist,
                                double* actions, void* workspace, size_t workspace_bytes,
                                void** graph_exec) {
  if (!graph_exec) return CS_ERR_INVALID_ARG;
  *graph_exec = nullptr;
  hipStream_t cap;
  CS_HIP_CHECK(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
  hipGraph_t g = nullptr;
  cs_status s = CS_OK;
  if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    (void)hipStreamDestroy(cap);
    return CS_ERR_HIP;
  }
  s = cs_batch_run(plan, seeds, hist, actions, workspace, workspace_bytes, cap);
  hipError_t e = hipStreamEndCapture(cap, &g);
  (void)hipStreamDestroy(cap);
  if (s != CS_OK) {
    if (g) (void)hipGraphDestroy(g);
    return s;
  }
  if (e != hipSuccess) return CS_ERR_HIP;
  hipGraphExec_t ex = nullptr;
  e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return CS_ERR_HIP;
  *graph_exec = (void*)ex;
  return CS_OK;
}

cs_status cs_batch_graph_launch(void* graph_exec, void* stream) {
  if (!graph_exec) return CS_ERR_INVALID_ARG;
  CS_HIP_CHECK(hipGraphLaunch((hipGraphExec_t)graph_exec, (hipStream_t)stream));
  return CS_OK;
}

cs_status cs_batch_graph_destroy(void* graph_exec) {
  if (!graph_exec) return CS_OK;
  CS_HIP_CHECK(hipGraphExecDestroy((hipGraphExec_t)graph_exec));
  return CS_OK;
}

// For each requested (counter, bucket): an ensemble of `reps` diamonds of the bucket's
// probe size, every tile configuration of the counter's candidates forced on all of them,
// the counting launches timed (best of five, HIP events), and the rank counter's; the
// fastest tiles are stored with both times.
cs_status cs_autotune(const char* cache_path, int64_t n_bucket, int counter, void* stream) {
  if (!cache_path) return CS_ERR_INVALID_ARG;
  if (counter != -1 && counter != CS_COUNT_BITSET && counter != CS_COUNT_MFMA &&
      counter != CS_COUNT_MFMA_FP4)
    return CS_ERR_UNSUPPORTED;
  if (n_bucket != 0 && (n_bucket < 2 || n_bucket > kBatchMaxN)) return CS_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  TuneTable table = read_tune(cache_path);
  const int cus = device_cu_count();
  hipEvent_t e0, e1;
  CS_HIP_CHECK(hipEventCreate(&e0));
  CS_HIP_CHECK(hipEventCreate(&e1));
  cs_status status = CS_OK;
  const int counters[3] = {CS_COUNT_BITSET, CS_COUNT_MFMA, CS_COUNT_MFMA_FP4};
  for (int ci = 0; ci < 3 && status == CS_OK; ++ci) {
    const int c = counters[ci];
    if (counter != -1 && counter != c) continue;
    const BatchTile* cand = c == CS_COUNT_BITSET ? kBitsetCandidates : kMfmaCandidates;
    const int ncand = c == CS_COUNT_BITSET
                          ? (int)(sizeof(kBitsetCandidates) / sizeof(kBitsetCandidates[0]))
                          : (int)(sizeof(kMfmaCandidates) / sizeof(kMfmaCandidates[0]));
    for (int b = 0; b < kBuckets && status == CS_OK; ++b) {
      if (n_bucket != 0 && bucket_of(n_bucket) != b) continue;
      // Enough instances that the row-panel items of 128-row tiles fill every CU sixteen
      // times over, as in a full ensemble (a handful of instances would leave most CUs
      // idle and favour the wrong occupancy; eight times over left candidates within the
      // timing noise of each other that differ by 8 % in a full ensemble).
      const int64_t reps = std::max<int64_t>(16, ceil_div(16 * (int64_t)cus,
                                                          ceil_div(kBucketProbe[b], 128)));
      // Sizes spread evenly over the bucket, centred on its probe size, as in an ensemble
      // of uneven instances (identical ones would all end at once and favour other tiles).
      const int64_t plo = 2 * kBucketProbe[b] - kBucketHi[b], phi = kBucketHi[b];
      std::vector<int64_t> sizes(reps);
      for (int64_t k = 0; k < reps; ++k) sizes[k] = plo + (phi - plo) * k / (reps - 1);
      double best_ms = 1e30, rank_ms = 0.0;
      int best = -1;
      for (int v = 0; v <= ncand && status == CS_OK; ++v) {
        cs_batch_plan_t q;
        status = build_plan(reps, sizes.data(), c, 0, nullptr, TuneTable{},
                            v < ncand ? &cand[v] : &kRankTile, &q);
        void* ws = nullptr;
        uint64_t* hist = nullptr;
        uint64_t* seeds = nullptr;
        double ms_v = 1e30;
        if (status == CS_OK &&
            (hipMalloc(&ws, q.ws_bytes) != hipSuccess ||
             hipMalloc((void**)&hist, sizeof(uint64_t) * q.hist_len) != hipSuccess ||
             hipMalloc((void**)&seeds, sizeof(uint64_t) * reps) != hipSuccess))
          status = CS_ERR_HIP;
        if (status == CS_OK) {
          std::vector<uint64_t> hs(reps);
          for (int64_t k = 0; k < reps; ++k) hs[k] = 0x5EEDull + 7919ull * k + 104729ull * b;
          if (hipMemcpy(seeds, hs.data(), sizeof(uint64_t) * reps, hipMemcpyHostToDevice) !=
              hipSuccess)
            status = CS_ERR_HIP;
          if (status == CS_OK) status = cs_batch_run(&q, seeds, hist, nullptr, ws, q.ws_bytes, st);
          for (int it = 0; it < 5 && status == CS_OK; ++it) {
            unsigned int* ctr = (unsigned int*)ws;
            status = launch_fill_u64((uint64_t*)ctr, kMaxSlots * kBatchQueues / 2, 0, st);
            if (status == CS_OK) status = launch_fill_u64(hist, q.hist_len, 0, st);
            if (status != CS_OK) break;
            (void)hipEventRecord(e0, st);
            status = run_counts(&q, (char*)ws, hist, st);
            (void)hipEventRecord(e1, st);
            if (hipEventSynchronize(e1) != hipSuccess) status = CS_ERR_HIP;
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            ms_v = std::min(ms_v, (double)ms);
          }
        }
        if (ws) (void)hipFree(ws);
        if (hist) (void)hipFree(hist);
        if (seeds) (void)hipFree(seeds);
        if (q.dev) (void)hipFree(q.dev);
        q.dev = nullptr;
        if (status == CS_OK && v == ncand) {
          rank_ms = ms_v;
        } else if (status == CS_OK && ms_v < best_ms) {
          best_ms = ms_v;
          best = v;
        }
      }
      if (status == CS_OK && best >= 0) {
        const int cs_ = counter_slot(c);
        table.have[cs_][b] = true;
        table.cfg[cs_][b] = cand[best];
        table.ms[cs_][b] = best_ms;
        table.rank_ms[cs_][b] = rank_ms;
        table.reps[cs_][b] = reps;
      }
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (status != CS_OK) return status;
  return write_tune(cache_path, table) ? CS_OK : CS_ERR_INVALID_ARG;
}

}  // extern "C"
