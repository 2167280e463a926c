// Sprinkling and time ordering on the GPU (App. A "Causal Set Sprinklings";
// Sec. 3.2 "Pairwise Relations": label elements so that no later index precedes
// an earlier one).
//
// Pipeline per call: generate raw SoA coordinates, a 64-bit time key and a bucket per point
// -> scan the bucket counts -> scatter the points to their buckets -> place each bucket's
// points in (key, generation index) order straight into the coordinate planes.  Sets of
// at most kRankMaxN points skip the buckets: each point's rank is counted over all keys and
// its planes are written there.
// The 3+1 diamond is sampled by rejection: candidates are flagged, counted per
// block, scanned, and the first n accepted are scattered in candidate order.
#include "common.h"

namespace cs {
namespace {

constexpr int kBlock = 256;
constexpr int kBucketMean = 64;     // points per bucket on average; at most five times as many
                                    // expected anywhere (the densities below; the thinnest slabs)
constexpr int kBucketCap = 2048;    // points of a bucket placed through LDS: six times the most
                                    // expected, 96 standard deviations above
constexpr int kBucketPad = 16;      // counters 64 bytes apart: adds to one line queue up (30001
                                    // points of the 3+1 diamond: 45 us with counters side by side)
constexpr int kPlaceThreads = 512;
constexpr int kPlaceSplit = 4;      // lanes that share a point's comparisons

// Candidate budget of the rejection samplers of the diamonds of height 1: the
// acceptance probability is the diamond's volume in the unit box, pi/24 (3+1) or
// pi/12 (2+1); the budget covers the mean plus 12 standard deviations, and a
// one-workgroup tail kernel handles any shortfall.
bool is_rejection(int region) { return region == CS_MINK4_DIAMOND || region == CS_MINK3_DIAMOND; }

int64_t mink_candidates(int region, int64_t n) {
  const double p = region == CS_MINK3_DIAMOND ? 0.26179938779914941   // pi / 12
                                              : 0.13089969389957471;  // pi / 24
  double m = (double)n / p + 12.0 * sqrt((double)n * (1.0 - p)) / p + 4096.0;
  return align_up((size_t)m, kBlock);
}

int64_t buckets_of(int64_t n) { return ceil_div(n, kBucketMean); }

struct SprinkleWs {
  double* raw;
  uint64_t* keys;
  uint32_t* arrive;      // arrival number of each point in its bucket
  uint32_t* slots;       // points by bucket
  uint32_t* bkt_of;      // bucket of each point
  uint32_t* bkt_count;   // points per bucket, kBucketPad apart, zeroed before the draws
  uint64_t* bkt_start;   // their exclusive scan, plus [buckets] = n
  uint32_t* blk_count;   // rejection samplers only
  uint64_t* blk_offset;  // rejection samplers only (exclusive scan), plus [nblk] = total
};

size_t layout(int region, int64_t n, void* base, SprinkleWs* w) {
  const int planes = coord_planes(region);
  const int64_t B = buckets_of(n);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  size_t o_raw = take(sizeof(double) * planes * n);
  size_t o_keys = take(sizeof(uint64_t) * n);
  size_t o_arrive = take(sizeof(uint32_t) * n);
  size_t o_slots = take(sizeof(uint32_t) * n);
  size_t o_bof = take(sizeof(uint32_t) * n);
  size_t o_bcnt = take(sizeof(uint32_t) * B * kBucketPad);
  size_t o_bstart = take(sizeof(uint64_t) * (B + 1));
  size_t o_cnt = 0, o_off = 0;
  if (is_rejection(region)) {
    int64_t nblk = mink_candidates(region, n) / kBlock;
    o_cnt = take(sizeof(uint32_t) * nblk);
    o_off = take(sizeof(uint64_t) * (nblk + 1));
  }
  if (w) {
    char* b = (char*)base;
    w->raw = (double*)(b + o_raw);
    w->keys = (uint64_t*)(b + o_keys);
    w->arrive = (uint32_t*)(b + o_arrive);
    w->slots = (uint32_t*)(b + o_slots);
    w->bkt_of = (uint32_t*)(b + o_bof);
    w->bkt_count = (uint32_t*)(b + o_bcnt);
    w->bkt_start = (uint64_t*)(b + o_bstart);
    w->blk_count = is_rejection(region) ? (uint32_t*)(b + o_cnt) : nullptr;
    w->blk_offset = is_rejection(region) ? (uint64_t*)(b + o_off) : nullptr;
  }
  return off;
}

// Where the samplers put a point's time key and, for sets that are placed by buckets (B >
// 0), its bucket: a monotone map of the key onto [0, B), under which no bucket holds more
// than five times the mean.  (Densities of the key: 2 at the middle of the u + v triangle,
// 3 and 4 at the waists of the 2+1 and 3+1 diamonds, 1 in tan(eta) on the 1+1 slab, up to
// 3 at the ends of the 3+1 slab, up to 5 in slabs a few steps of the smallest double wide.)
struct KeyOut {
  uint64_t* keys;
  uint32_t *bkt_of, *arrive, *bkt_count;
  uint64_t B;
};
__device__ inline void put_key(const KeyOut& o, int64_t g, uint64_t key, uint64_t bucket) {
  o.keys[g] = key;
  if (o.B == 0) return;
  const uint32_t b = (uint32_t)(bucket < o.B ? bucket : o.B - 1);
  o.bkt_of[g] = b;
  o.arrive[g] = atomicAdd(&o.bkt_count[(uint64_t)b * kBucketPad], 1u);
}
// Integer keys of `bits` bits; the slabs' real keys take bucket_of_time.
__device__ inline uint64_t bucket_of_bits(uint64_t key, int bits, uint64_t B) {
  return __umul64hi(key << (64 - bits), B);
}

// ---------------------------------------------------------------------------
// 1+1 diamond: u = U(2g), v = U(2g+1); key = exact integer (u + v) * 2^53.
// ---------------------------------------------------------------------------
__global__ void k_sprinkle_mink2(uint64_t skey, int64_t n, double* __restrict__ raw, KeyOut out) {
  int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  uint64_t ku = sm_output(skey, 2 * (uint64_t)g) >> 11;
  uint64_t kv = sm_output(skey, 2 * (uint64_t)g + 1) >> 11;
  raw[g] = (double)ku * 0x1.0p-53;
  raw[n + g] = (double)kv * 0x1.0p-53;
  put_key(out, g, ku + kv, bucket_of_bits(ku + kv, 54, out.B));
}

// ---------------------------------------------------------------------------
// D-dimensional diamond of height 1 (D = 3 or 4) by rejection from [0,1) x
// [-1/2,1/2)^(D-1): candidate c takes draws D c .. D c + D-1 of the stream.
// ---------------------------------------------------------------------------
struct Cand {
  double t, x, y, z;
  uint64_t kt;
  bool ok;
};

template <int D>
__device__ inline Cand mink_candidate(uint64_t skey, uint64_t c) {
  Cand r;
  r.kt = sm_output(skey, D * c) >> 11;
  r.t = (double)r.kt * 0x1.0p-53;
  r.x = unit53(sm_output(skey, D * c + 1)) - 0.5;
  r.y = unit53(sm_output(skey, D * c + 2)) - 0.5;
  r.z = D == 4 ? unit53(sm_output(skey, D * c + 3)) - 0.5 : 0.0;
  double one_t = 1.0 - r.t;
  double rad = r.t < one_t ? r.t : one_t;
  double rr = __dadd_rn(__dmul_rn(r.x, r.x), __dmul_rn(r.y, r.y));
  if (D == 4) rr = __dadd_rn(rr, __dmul_rn(r.z, r.z));
  r.ok = rr < __dmul_rn(rad, rad);
  return r;
}

// Block-wide exclusive rank of `flag` among the block's threads, and the block total.
__device__ inline uint32_t block_rank(bool flag, uint32_t* total, uint32_t* s_wave) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  uint64_t m = __ballot(flag);
  uint32_t below = __popcll(m & ((1ull << lane) - 1ull));
  if (lane == 0) s_wave[wave] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    if (w < wave) base += s_wave[w];
    tot += s_wave[w];
  }
  __syncthreads();
  *total = tot;
  return base + below;
}

template <int D>
__global__ void k_mink_count(uint64_t skey, uint32_t* __restrict__ blk_count) {
  __shared__ uint32_t s_wave[kBlock / 64];
  uint64_t c = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  Cand r = mink_candidate<D>(skey, c);
  uint32_t tot;
  block_rank(r.ok, &tot, s_wave);
  if (threadIdx.x == 0) blk_count[blockIdx.x] = tot;
}

// Exclusive scan of nblk counts, `stride` apart, by one workgroup of 1024 threads, eight counts per thread
// and step: lane exchanges within the waves, their sums through LDS.
constexpr int kScanPer = 8;
__global__ __launch_bounds__(1024) void k_scan_counts(const uint32_t* __restrict__ cnt, int stride,
                                                      int64_t nblk, uint64_t* __restrict__ off) {
  __shared__ uint64_t wave_sum[2][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t carry = 0;
  int buf = 0;
  for (int64_t base = 0; base < nblk; base += 1024 * kScanPer, buf ^= 1) {
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanPer;
    uint32_t v[kScanPer];
    uint64_t sum = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      v[q] = i0 + q < nblk ? cnt[(i0 + q) * stride] : 0u;
      sum += v[q];
    }
    uint64_t x = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t y = __shfl_up((unsigned long long)x, d);
      if (lane >= d) x += y;
    }
    if (lane == 63) wave_sum[buf][wave] = x;
    __syncthreads();
    uint64_t at = carry + x - sum, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const uint64_t s = wave_sum[buf][w];
      at += w < wave ? s : 0ull;
      total += s;
    }
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      if (i0 + q < nblk) off[i0 + q] = at;
      at += v[q];
    }
    carry += total;
  }
  if (threadIdx.x == 0) off[nblk] = carry;
}

template <int D>
__device__ inline void put(const Cand& r, uint64_t rank, int64_t n, double* raw, const KeyOut& out) {
  raw[rank] = r.t;
  raw[n + rank] = r.x;
  raw[2 * n + rank] = r.y;
  if (D == 4) raw[3 * n + rank] = r.z;
  put_key(out, (int64_t)rank, r.kt, bucket_of_bits(r.kt, 53, out.B));
}

template <int D>
__global__ void k_mink_scatter(uint64_t skey, int64_t n, const uint64_t* __restrict__ blk_off,
                                double* __restrict__ raw, KeyOut out) {
  __shared__ uint32_t s_wave[kBlock / 64];
  uint64_t c = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  Cand r = mink_candidate<D>(skey, c);
  uint32_t tot;
  uint32_t local = block_rank(r.ok, &tot, s_wave);
  uint64_t rank = blk_off[blockIdx.x] + local;
  if (r.ok && rank < (uint64_t)n) put<D>(r, rank, n, raw, out);
}

// Continues candidates after the budget if (improbably) fewer than n were accepted.
// One workgroup; bounded number of rounds.
template <int D>
__global__ void k_mink_tail(uint64_t skey, int64_t n, int64_t M, const uint64_t* __restrict__ total,
                             double* __restrict__ raw, KeyOut out) {
  __shared__ uint32_t s_wave[kBlock / 64];
  uint64_t have = *total;
  const int64_t kMaxRounds = 1ll << 22;
  for (int64_t round = 0; have < (uint64_t)n && round < kMaxRounds; ++round) {
    uint64_t c = (uint64_t)M + (uint64_t)round * kBlock + threadIdx.x;
    Cand r = mink_candidate<D>(skey, c);
    uint32_t tot;
    uint32_t local = block_rank(r.ok, &tot, s_wave);
    uint64_t rank = have + local;
    if (r.ok && rank < (uint64_t)n) put<D>(r, rank, n, raw, out);
    have += tot;
  }
}

// ---------------------------------------------------------------------------
// 1+1 de Sitter slab: the density sec^2(eta) = d tan(eta)/d eta makes x = tan(eta)
// uniform, x = (2u - 1) tan(eta0) (one rounding); eta = atan(x); theta = 2 pi w.
// Sorted by x, which orders the points by eta.
// ---------------------------------------------------------------------------
__global__ void k_sprinkle_ds2(uint64_t skey, double X, int64_t n, double* __restrict__ raw,
                               KeyOut out) {
  int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const double two_pi = 2.0 * 3.141592653589793;  // twice the double nearest pi (exact)
  double u = unit53(sm_output(skey, 2 * (uint64_t)g));
  double w = unit53(sm_output(skey, 2 * (uint64_t)g + 1));
  double x = __dmul_rn(__dsub_rn(__dmul_rn(2.0, u), 1.0), X);
  raw[g] = x;
  raw[n + g] = atan(x);
  raw[2 * n + g] = __dmul_rn(two_pi, w);
  put_key(out, g, order_bits(x), bucket_of_time(x, X, (uint64_t)g, (uint64_t)n, out.B));
}

// ---------------------------------------------------------------------------
// 3+1 de Sitter slab: x = tan(eta) from the inverse CDF of (1 + x^2) dx,
// x = 2 sinh(asinh(3y/2)/3); direction on S^3 by cube rejection, normalised.
// ---------------------------------------------------------------------------
__global__ void k_sprinkle_ds4(uint64_t skey_t, uint64_t skey_s, double X, int64_t n,
                               double* __restrict__ raw, KeyOut out) {
  int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  double Y = __dadd_rn(X, __ddiv_rn(__dmul_rn(__dmul_rn(X, X), X), 3.0));
  double u = unit53(sm_output(skey_t, (uint64_t)g));
  double y = __dmul_rn(__dsub_rn(__dmul_rn(2.0, u), 1.0), Y);
  double x = __dmul_rn(2.0, sinh(__ddiv_rn(asinh(__dmul_rn(1.5, y)), 3.0)));
  double ce = __ddiv_rn(1.0, __dsqrt_rn(__dadd_rn(1.0, __dmul_rn(x, x))));
  double se = __dmul_rn(x, ce);
  uint64_t ps = sm_output(skey_s, (uint64_t)g);
  double a0 = 1.0, a1 = 0.0, a2 = 0.0, a3 = 0.0, r2 = 1.0;
  for (int k = 0; k < kSphereTries; ++k) {
    double b0 = __dsub_rn(__dmul_rn(2.0, unit53(sm_output(ps, 4 * (uint64_t)k + 0))), 1.0);
    double b1 = __dsub_rn(__dmul_rn(2.0, unit53(sm_output(ps, 4 * (uint64_t)k + 1))), 1.0);
    double b2 = __dsub_rn(__dmul_rn(2.0, unit53(sm_output(ps, 4 * (uint64_t)k + 2))), 1.0);
    double b3 = __dsub_rn(__dmul_rn(2.0, unit53(sm_output(ps, 4 * (uint64_t)k + 3))), 1.0);
    double q = __dadd_rn(__dmul_rn(b0, b0), __dmul_rn(b1, b1));
    q = __dadd_rn(q, __dmul_rn(b2, b2));
    q = __dadd_rn(q, __dmul_rn(b3, b3));
    if (q < 1.0 && q > 0x1.0p-40) {
      a0 = b0; a1 = b1; a2 = b2; a3 = b3; r2 = q;
      break;
    }
  }
  double r = __dsqrt_rn(r2);
  raw[g] = x;
  raw[n + g] = ce;
  raw[2 * n + g] = se;
  raw[3 * n + g] = __ddiv_rn(a0, r);
  raw[4 * n + g] = __ddiv_rn(a1, r);
  raw[5 * n + g] = __ddiv_rn(a2, r);
  raw[6 * n + g] = __ddiv_rn(a3, r);
  put_key(out, g, order_bits(x), bucket_of_time(x, X, (uint64_t)g, (uint64_t)n, out.B));
}

// ---------------------------------------------------------------------------
// Time order by buckets.  The points of a bucket are brought together (k_bucket_scatter), and
// a workgroup per bucket counts each one's rank among them and writes its planes to the
// bucket's start plus the rank.  Four launches that pass over the points once each, bound
// by launches and latency, where a bitonic network took 10 to 30 launches: the whole call for
// a 3+1 diamond of 30001 points 35 us against 83, of 131072 points 49 against 133.  A bucket
// of more than kBucketCap points (none arises from these densities) is ranked from memory.
// ---------------------------------------------------------------------------
__global__ void k_bucket_scatter(int64_t n, const uint32_t* __restrict__ bkt_of,
                                 const uint32_t* __restrict__ arrive,
                                 const uint64_t* __restrict__ start, uint32_t* __restrict__ slots) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) slots[start[bkt_of[g]] + arrive[g]] = (uint32_t)g;
}

__global__ __launch_bounds__(kPlaceThreads) void k_bucket_place(
    const uint64_t* __restrict__ keys, const uint32_t* __restrict__ slots,
    const uint64_t* __restrict__ start, int64_t B, const double* __restrict__ raw, int planes,
    int64_t n, double* __restrict__ coords) {
  __shared__ uint64_t sk[kBucketCap];
  __shared__ uint32_t sg[kBucketCap];
  const int64_t b = group_index();
  if (b >= B) return;  // the whole workgroup
  const int64_t lo = (int64_t)start[b], m = (int64_t)start[b + 1] - lo;
  const bool lds = m <= kBucketCap;
  if (lds) {
    for (int i = threadIdx.x; i < m; i += kPlaceThreads) {
      const uint32_t g = slots[lo + i];
      sg[i] = g;
      sk[i] = keys[g];
    }
    __syncthreads();
  }
  const int s = threadIdx.x % kPlaceSplit;
  for (int64_t i = threadIdx.x / kPlaceSplit; i < m; i += kPlaceThreads / kPlaceSplit) {
    const uint32_t g = lds ? sg[i] : slots[lo + i];
    const uint64_t k = lds ? sk[i] : keys[g];
    uint32_t rank = 0;
    if (lds) {
#pragma unroll 8
      for (int j = s; j < (int)m; j += kPlaceSplit) rank += key_less(sk[j], sg[j], k, g) ? 1u : 0u;
    } else {
      for (int64_t j = s; j < m; j += kPlaceSplit) {
        const uint32_t h = slots[lo + j];
        rank += key_less(keys[h], h, k, g) ? 1u : 0u;
      }
    }
#pragma unroll
    for (int off = kPlaceSplit / 2; off > 0; off >>= 1) rank += __shfl_xor(rank, off);
    for (int p = s; p < planes; p += kPlaceSplit)
      coords[(int64_t)p * n + lo + rank] = raw[(int64_t)p * n + g];
  }
}

// ---------------------------------------------------------------------------
// Small sets: the time order by ranks.  Element g's place is the number of elements
// before it in (key, index) order, the order of the buckets above 8192 points; the place is
// counted over every key and the coordinates are written straight there, in one launch.
// Sixteen lanes share an element, each comparing against every sixteenth key of a chunk
// staged in LDS (consecutive lanes read consecutive words, so a wave's reads hit distinct
// banks); the partial counts are summed by lane exchanges.  Each comparison is the order
// itself, key first and index on equal keys, so equal keys need no separate pass.
// ---------------------------------------------------------------------------
constexpr int kRankThreads = 256;
constexpr int kRankSplit = 16;                       // lanes per element
constexpr int kRankPer = kRankThreads / kRankSplit;  // elements per workgroup
constexpr int kRankChunk = 2048;                     // keys staged per pass
// n^2 comparisons: small sets only.  The line was drawn against a sorting network; buckets take,
// by ranks / by buckets, us, the whole call: 1+1 diamond 2000 points 6.6 / 16.0, 4001 10.9 / 17.5,
// 6000 18.0 / 17.2, 8192 23.4 / 17.5; 1+1 slab 9.9 / 14.3, 15.6 / 15.2, 21.8 / 14.4, 27.4 / 15.5; 3+1
// diamond 17.6 / 28.4, 23.4 / 30.0, 29.3 / 31.9, 35.8 / 32.8; 3+1 slab 18.6 / 25.9, 24.4 / 25.9, 30.9 /
// 26.0, 37.0 / 27.1.  So buckets are ahead from 4000 points on in slabs and 6000 to 8000 in diamonds.
constexpr int64_t kRankMaxN = 8192;

__device__ inline uint32_t rank_lane_sum(uint32_t v) {
#pragma unroll
  for (int off = kRankSplit / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

__global__ __launch_bounds__(kRankThreads) void k_rank_place(const uint64_t* __restrict__ keys,
                                                             const double* __restrict__ raw,
                                                             int planes, int64_t n,
                                                             double* __restrict__ coords) {
  __shared__ uint64_t sk[kRankChunk];
  const int s = threadIdx.x & (kRankSplit - 1);
  const int64_t g = (int64_t)blockIdx.x * kRankPer + threadIdx.x / kRankSplit;
  const bool live = g < n;
  const uint64_t kg = live ? keys[g] : 0ull;
  uint32_t before = 0;  // elements h with (key_h, h) < (key_g, g)
  for (int64_t base = 0; base < n; base += kRankChunk) {
    const int m = (int)(n - base < kRankChunk ? n - base : kRankChunk);
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += kRankThreads) sk[i] = keys[base + i];
    __syncthreads();
    const int gi = (int)(g - base);  // g's index within the chunk (any value if outside)
#pragma unroll 8
    for (int i = s; i < m; i += kRankSplit) {
      const uint64_t kh = sk[i];
      before += (kh < kg || (kh == kg && i < gi)) ? 1u : 0u;
    }
  }
  const uint32_t lt = rank_lane_sum(before);
  if (live)
    for (int p = s; p < planes; p += kRankSplit) coords[(int64_t)p * n + lt] = raw[(int64_t)p * n + g];
}

// The 1+1 diamond's time key of draw g (see k_sprinkle_mink2).
__device__ inline uint64_t mink2_key(uint64_t skey, uint64_t g) {
  return (sm_output(skey, 2 * g) >> 11) + (sm_output(skey, 2 * g + 1) >> 11);
}

// 1+1 diamonds up to kRankMaxN points: k_rank_place with the keys and coordinates taken
// straight from the counter-based generator, so the draws, the ranks and the placement
// are one launch.
__global__ __launch_bounds__(kRankThreads) void k_rank_place_mink2(uint64_t skey, int64_t n,
                                                                   double* __restrict__ coords) {
  __shared__ uint64_t sk[kRankChunk];
  const int s = threadIdx.x & (kRankSplit - 1);
  const int64_t g = (int64_t)blockIdx.x * kRankPer + threadIdx.x / kRankSplit;
  const bool live = g < n;
  const uint64_t ku = live ? sm_output(skey, 2 * (uint64_t)g) >> 11 : 0ull;
  const uint64_t kv = live ? sm_output(skey, 2 * (uint64_t)g + 1) >> 11 : 0ull;
  const uint64_t kg = ku + kv;
  uint32_t before = 0;  // elements h with (key_h, h) < (key_g, g)
  for (int64_t base = 0; base < n; base += kRankChunk) {
    const int m = (int)(n - base < kRankChunk ? n - base : kRankChunk);
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += kRankThreads) sk[i] = mink2_key(skey, (uint64_t)(base + i));
    __syncthreads();
    const int gi = (int)(g - base);  // g's index within the chunk (any value if outside)
#pragma unroll 8
    for (int i = s; i < m; i += kRankSplit) {
      const uint64_t kh = sk[i];
      before += (kh < kg || (kh == kg && i < gi)) ? 1u : 0u;
    }
  }
  const uint32_t lt = rank_lane_sum(before);
  if (live && s < 2) coords[(int64_t)s * n + lt] = (double)(s == 0 ? ku : kv) * 0x1.0p-53;
}

// ---------------------------------------------------------------------------
// Ensemble of 1+1 diamonds: one workgroup per instance (n <= 8192).  Each of a point's
// three places -- in time order (key u + v, then draw index), in u and in v -- comes from a
// bucket sort in LDS: the keys are draws of known density (uniform, or the triangle of
// u + v), so with a bucket per power of two at least n a bucket holds a few points.  A
// point takes an arrival slot of its bucket (LDS atomic), the bucket counts are scanned,
// and its place is its bucket's start plus the points of the bucket that precede it.
// The bucket's leading key bits being equal, the remaining ones and the index fit one
// 64-bit word, so a comparison is exact.  Bound by its barriers and LDS latency (one
// workgroup per CU, the largest instance ends last; sixteen of the form for small instances:
// 30000 diamonds of 64 points 61 us, 926 in the large form).
// ---------------------------------------------------------------------------
template <int CAP>
constexpr int kSortThreads = CAP == kBatchMaxN ? 1024 : 128;  // for up to CAP points
template <int CAP>
constexpr int kSortPer = CAP / kSortThreads<CAP>;             // points per thread

template <int CAP>
struct BucketLds {
  uint64_t word[CAP];       // rest of the key << lg | index, by bucket slot
  uint32_t start[CAP + 4];  // bucket counts, then starts; start[buckets] = n
  uint32_t wsum[kSortThreads<CAP> / 64];
};

// place[e] = number of points before point threadIdx.x + threads e in (key, index) order; keys
// below 2^KB, 2^lg >= n buckets.  tie(g, h): for equal keys, whether g comes first.
template <int KB, int CAP, typename Tie>
__device__ inline void bucket_places(const uint64_t (&key)[kSortPer<CAP>], int n, int lg,
                                     BucketLds<CAP>& L, uint32_t (&place)[kSortPer<CAP>], Tie&& tie) {
  constexpr int kThreads = kSortThreads<CAP>, kPer = kSortPer<CAP>;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int P = 1 << lg, sh = KB - lg;
  __syncthreads();  // the last use of the buffers is over
  for (int b = t; b < P; b += kThreads) L.start[b] = 0;
  __syncthreads();
  uint32_t at[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e)
    if (t + e * kThreads < n) at[e] = atomicAdd(&L.start[key[e] >> sh], 1u);
  __syncthreads();
  {  // exclusive scan of the counts: m consecutive buckets per thread
    const int m = P > kThreads ? P / kThreads : 1;
    uint32_t c[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      if (q < m && t * m + q < P) {
        c[q] = L.start[t * m + q];
        sum += c[q];
      }
    uint32_t x = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d);
      if (lane >= d) x += y;
    }
    if (lane == 63) L.wsum[wave] = x;
    __syncthreads();
    uint32_t off = x - sum;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) off += w < wave ? L.wsum[w] : 0u;
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      if (q < m && t * m + q < P) {
        L.start[t * m + q] = off;
        off += c[q];
      }
    if (t == 0) L.start[P] = (uint32_t)n;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const uint32_t g = t + e * kThreads;
    if ((int)g < n)
      L.word[L.start[key[e] >> sh] + at[e]] = (key[e] & ((1ull << sh) - 1)) << lg | g;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const uint32_t g = t + e * kThreads;
    if ((int)g < n) {
      const uint64_t b = key[e] >> sh;
      const uint64_t w = (key[e] & ((1ull << sh) - 1)) << lg | g;
      const uint32_t lo = L.start[b], hi = L.start[b + 1];
      uint32_t r = lo;
      for (uint32_t s = lo; s < hi; ++s) {
        const uint64_t o = L.word[s];
        bool before = o < w;
        if ((o >> lg) == (w >> lg) && o != w) before = tie((uint32_t)o & (P - 1u), g);
        r += before ? 1u : 0u;
      }
      place[e] = r;
    }
  }
}

// Also clears the instance's histogram and (workgroup 0) the work counters, which the
// later launches accumulate into.  uv: each point's places in u and v, in time order, for
// the builder.  Instances counted by ranks (rank[k].n != 0) also get their u order:
// sigma[x] is the u place of the point at v place x, pi its inverse.  Equal coordinates
// are unrelated, so ties take opposite orders in u and v: equal u by v descending, equal
// v by u descending, equal points by index one way and the other.
template <int CAP>
__global__ __launch_bounds__(kSortThreads<CAP>) void k_sprinkle_mink2_batch(
    const uint64_t* __restrict__ seeds, const BatchInst* __restrict__ inst,
    const RankInst* __restrict__ rank, const uint32_t* __restrict__ ids, double* __restrict__ coords,
    uint32_t* __restrict__ uv, char* __restrict__ rank_base, uint64_t* __restrict__ hist,
    uint64_t* __restrict__ zero, int nzero) {
  constexpr int kThreads = kSortThreads<CAP>, kPer = kSortPer<CAP>;
  __shared__ BucketLds<CAP> L;
  const uint32_t inst_id = ids ? ids[blockIdx.x] : blockIdx.x;
  const BatchInst d = inst[inst_id];
  const int n = (int)d.n, t = threadIdx.x;
  for (int m = t; m < n - 1; m += kThreads) hist[d.hist_off + m] = 0;
  if (blockIdx.x == 0)
    for (int w = t; w < nzero; w += kThreads) zero[w] = 0;
  int lg = 1;
  while ((1 << lg) < n) ++lg;
  const uint64_t skey = sm_stream_key(seeds[inst_id], kStreamMink2);
  uint64_t ku[kPer], kv[kPer], key[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int g = t + e * kThreads;
    ku[e] = kv[e] = key[e] = 0;
    if (g < n) {
      ku[e] = sm_output(skey, 2 * (uint64_t)g) >> 11;
      kv[e] = sm_output(skey, 2 * (uint64_t)g + 1) >> 11;
      key[e] = ku[e] + kv[e];
    }
  }
  uint32_t place[kPer];
  bucket_places<54, CAP>(key, n, lg, L, place, [](uint32_t a, uint32_t b) { return a < b; });
  double* cu = coords + d.coord_off;
  double* cv = cu + n;
#pragma unroll
  for (int e = 0; e < kPer; ++e)
    if (t + e * kThreads < n) {
      cu[place[e]] = (double)ku[e] * 0x1.0p-53;
      cv[place[e]] = (double)kv[e] * 0x1.0p-53;
    }
  auto draw = [&](uint32_t g, int axis) { return sm_output(skey, 2 * (uint64_t)g + axis) >> 11; };
  uint32_t pu[kPer], pv[kPer];
  bucket_places<53, CAP>(ku, n, lg, L, pu, [&](uint32_t a, uint32_t b) {
    const uint64_t va = draw(a, 1), vb = draw(b, 1);
    return va > vb || (va == vb && a < b);
  });
  bucket_places<53, CAP>(kv, n, lg, L, pv, [&](uint32_t a, uint32_t b) {
    const uint64_t ua = draw(a, 0), ub = draw(b, 0);
    return ua > ub || (ua == ub && a > b);
  });
  uint32_t* place_uv = uv + d.coord_off / 2;
#pragma unroll
  for (int e = 0; e < kPer; ++e)
    if (t + e * kThreads < n) place_uv[place[e]] = pu[e] << 16 | pv[e];
  const RankInst r = rank[inst_id];
  if (r.n == 0) return;
  // Both permutations leave through LDS, in whole lines.
  uint16_t* perm = (uint16_t*)L.word;  // sigma, then pi
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPer; ++e)
    if (t + e * kThreads < n) {
      perm[pv[e]] = (uint16_t)pu[e];
      perm[CAP + pu[e]] = (uint16_t)pv[e];
    }
  __syncthreads();
  uint16_t* sigma = (uint16_t*)(rank_base + r.sigma_off());
  uint16_t* pi = (uint16_t*)(rank_base + r.pi_off());
  for (int i = t; i < 64 * r.nb; i += kThreads) {
    sigma[i] = i < n ? perm[i] : (uint16_t)0xFFFFu;
    pi[i] = i < n ? perm[CAP + i] : (uint16_t)0u;
  }
}

}  // namespace

size_t sprinkle_ws_bytes(int region, int64_t n) { return layout(region, n, nullptr, nullptr); }

cs_status launch_sprinkle(int region, double eta0, uint64_t seed, int64_t n, double* coords,
                          void* ws, hipStream_t st) {
  SprinkleWs w;
  layout(region, n, ws, &w);
  const int planes = coord_planes(region);
  const unsigned grid = (unsigned)ceil_div(n, kBlock);
  if (region == CS_MINK2_DIAMOND && n <= kRankMaxN) {
    hipLaunchKernelGGL(k_rank_place_mink2, dim3((unsigned)ceil_div(n, kRankPer)), dim3(kRankThreads),
                       0, st, sm_stream_key(seed, kStreamMink2), n, coords);
    CS_LAUNCH_CHECK();
    return CS_OK;
  }
  const int64_t B = n <= kRankMaxN ? 0 : buckets_of(n);
  const KeyOut out{w.keys, w.bkt_of, w.arrive, w.bkt_count, (uint64_t)B};
  if (B > 0) {
    cs_status s = launch_fill_u64((uint64_t*)w.bkt_count, B * kBucketPad / 2, 0, st);
    if (s != CS_OK) return s;
  }
  if (region == CS_MINK2_DIAMOND) {
    hipLaunchKernelGGL(k_sprinkle_mink2, dim3(grid), dim3(kBlock), 0, st,
                       sm_stream_key(seed, kStreamMink2), n, w.raw, out);
    CS_LAUNCH_CHECK();
  } else if (is_rejection(region)) {
    const bool d4 = region == CS_MINK4_DIAMOND;
    const int64_t M = mink_candidates(region, n);
    const int64_t nblk = M / kBlock;
    const uint64_t skey = sm_stream_key(seed, d4 ? kStreamMink4 : kStreamMink3);
    if (d4) hipLaunchKernelGGL(k_mink_count<4>, dim3((unsigned)nblk), dim3(kBlock), 0, st, skey,
                               w.blk_count);
    else hipLaunchKernelGGL(k_mink_count<3>, dim3((unsigned)nblk), dim3(kBlock), 0, st, skey,
                            w.blk_count);
    CS_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, st, w.blk_count, 1, nblk, w.blk_offset);
    CS_LAUNCH_CHECK();
    if (d4) hipLaunchKernelGGL(k_mink_scatter<4>, dim3((unsigned)nblk), dim3(kBlock), 0, st, skey,
                               n, w.blk_offset, w.raw, out);
    else hipLaunchKernelGGL(k_mink_scatter<3>, dim3((unsigned)nblk), dim3(kBlock), 0, st, skey,
                            n, w.blk_offset, w.raw, out);
    CS_LAUNCH_CHECK();
    if (d4) hipLaunchKernelGGL(k_mink_tail<4>, dim3(1), dim3(kBlock), 0, st, skey, n, M,
                               w.blk_offset + nblk, w.raw, out);
    else hipLaunchKernelGGL(k_mink_tail<3>, dim3(1), dim3(kBlock), 0, st, skey, n, M,
                            w.blk_offset + nblk, w.raw, out);
    CS_LAUNCH_CHECK();
  } else if (region == CS_DS2_SLAB) {
    hipLaunchKernelGGL(k_sprinkle_ds2, dim3(grid), dim3(kBlock), 0, st,
                       sm_stream_key(seed, kStreamDs2), tan(eta0), n, w.raw, out);
    CS_LAUNCH_CHECK();
  } else {
    hipLaunchKernelGGL(k_sprinkle_ds4, dim3(grid), dim3(kBlock), 0, st,
                       sm_stream_key(seed, kStreamDsTime), sm_stream_key(seed, kStreamDsSphere),
                       tan(eta0), n, w.raw, out);
    CS_LAUNCH_CHECK();
  }
  if (n <= kRankMaxN) {
    hipLaunchKernelGGL(k_rank_place, dim3((unsigned)ceil_div(n, kRankPer)), dim3(kRankThreads), 0,
                       st, w.keys, w.raw, planes, n, coords);
    CS_LAUNCH_CHECK();
    return CS_OK;
  }
  hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, st, w.bkt_count, kBucketPad, B,
                     w.bkt_start);
  CS_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_bucket_scatter, dim3(grid), dim3(kBlock), 0, st, n, w.bkt_of, w.arrive,
                     w.bkt_start, w.slots);
  CS_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_bucket_place, grid_rows(B), dim3(kPlaceThreads), 0, st, w.keys, w.slots,
                     w.bkt_start, B, w.raw, planes, n, coords);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

cs_status launch_sprinkle_batch(bool small, const uint64_t* seeds, const BatchInst* inst,
                                const RankInst* rank, const uint32_t* ids, int64_t count,
                                double* coords, uint32_t* uv, char* rank_base, uint64_t* hist,
                                uint64_t* zero, int nzero, hipStream_t st) {
  if (count <= 0) return CS_OK;
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)count), dim3(threads), 0, st, seeds, inst, rank, ids,
                       coords, uv, rank_base, hist, zero, nzero);
  };
  if (small) go(k_sprinkle_mink2_batch<(int)kSmallN>, kSortThreads<(int)kSmallN>);
  else go(k_sprinkle_mink2_batch<(int)kBatchMaxN>, kSortThreads<(int)kBatchMaxN>);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

}  // namespace cs
