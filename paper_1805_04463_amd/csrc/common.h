// Shared device helpers of the gfx950 causal-set library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/causal.h"

namespace cs {

constexpr int kWave = 64;

// ---------------------------------------------------------------------------
// Counter-based SplitMix64 (Steele, Lea & Flood 2014).  Output c of a generator
// whose state is s is mix(s + (c+1) * golden), i.e. the published next() called
// c+1 times.  A stream key is output `stream` of the generator seeded with
// output 0 of the generator seeded with `seed`.
// ---------------------------------------------------------------------------
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;

__host__ __device__ inline uint64_t sm_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__host__ __device__ inline uint64_t sm_output(uint64_t state, uint64_t c) {
  return sm_mix(state + (c + 1) * kGolden);
}
__host__ __device__ inline uint64_t sm_stream_key(uint64_t seed, uint64_t stream) {
  return sm_output(sm_output(seed, 0), stream);
}
__device__ inline double unit53(uint64_t w) { return (double)(w >> 11) * 0x1.0p-53; }

// Streams of the generator per region.
enum : uint64_t {
  kStreamMink2 = 0,
  kStreamMink4 = 1,
  kStreamDsTime = 2,
  kStreamDsSphere = 3,
  kStreamDs2 = 4,
  kStreamMink3 = 5
};

// Rejection sampling of the S^3 direction gives up after this many tries (probability
// 0.69^4096: never reached in practice, but every loop has a bound).
constexpr int kSphereTries = 4096;

// The time order: (key, generation index), lexicographically.
__device__ inline bool key_less(uint64_t ka, uint32_t ga, uint64_t kb, uint32_t gb) {
  return ka < kb || (ka == kb && ga < gb);
}

// Monotone map double -> uint64 (unsigned order equals numeric order).
__device__ inline uint64_t order_bits(double x) {
  uint64_t b = (uint64_t)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// Bucket in [0, B) (or past it, for the caller to clamp) of point g of n in a slab whose time x
// = tan(eta) lies in [-X, X]: monotone in (order_bits(x), g).  In slabs below 2^-900 the quotient
// B / 2X can overflow, and few different times may be representable: there the times are
// counted in steps of the smallest double, two to spare at each end for the rounding of the
// samplers and one from -0 to 0, and points of equal time are spread by their index, so that
// no bucket holds them all.
__host__ __device__ inline uint64_t bucket_of_time(double x, double X, uint64_t g, uint64_t n,
                                                   uint64_t B) {
  double b;
  if (X >= 0x1p-900) {
    b = (x + X) * ((double)B / (2.0 * X));
  } else {
    const double at = ldexp(x, 1074) + ldexp(X, 1074) + (__builtin_signbit(x) ? 2.0 : 3.0);
    const double steps = 2.0 * ldexp(X, 1074) + 6.0;
    b = (at + (double)g / (double)n) * ((double)B / steps);
  }
  return b > 0.0 ? (uint64_t)b : 0ull;
}

inline int64_t ld_words(int64_t n) { return ((n + 511) / 512) * 8; }
__host__ __device__ inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// A step s coprime to m near the golden section of m: t -> t s mod m goes through 0 .. m-1 with
// consecutive t far apart.
inline int64_t scatter_step(int64_t m) {
  auto coprime = [](int64_t a, int64_t b) {
    while (b) {
      const int64_t r = a % b;
      a = b;
      b = r;
    }
    return a == 1;
  };
  int64_t s = (int64_t)(0.6180339887 * (double)m) | 1;
  while (!coprime(s, m)) s += 2;
  return s;
}

// Grid of `groups` workgroups in rows of at most 2^21: a launch holds less than 2^32 work-items
// along x, a row here at most 2^31.  The kernel's workgroup is group_index(), which in the last
// of several rows can be `groups` or more.
constexpr int64_t kGridRow = (int64_t)1 << 21;
inline dim3 grid_rows(int64_t groups) {
  return groups <= kGridRow ? dim3((unsigned)groups)
                            : dim3((unsigned)kGridRow, (unsigned)ceil_div(groups, kGridRow));
}
__device__ inline int64_t group_index() { return (int64_t)blockIdx.y * kGridRow + blockIdx.x; }

// Coordinate planes per region.
inline int coord_planes(int region) {
  switch (region) {
    case CS_MINK2_DIAMOND: return 2;
    case CS_MINK4_DIAMOND: return 4;
    case CS_DS4_SLAB: return 7;
    case CS_DS2_SLAB: return 3;
    case CS_MINK3_DIAMOND: return 3;
    default: return -1;
  }
}

#define CS_HIP_CHECK(expr)                      \
  do {                                          \
    hipError_t _e = (expr);                     \
    if (_e != hipSuccess) return CS_ERR_HIP;    \
  } while (0)

#define CS_LAUNCH_CHECK()                                   \
  do {                                                      \
    hipError_t _e = hipGetLastError();                      \
    if (_e != hipSuccess) return CS_ERR_HIP;                \
  } while (0)

// One instance of an ensemble: size, row stride (uint64 words) and offsets of its
// coordinates (doubles), matrix (uint64 words) and histogram (uint64 bins) in the
// concatenated buffers.  Its u and v places (uint32) are at coord_off / 2.
struct BatchInst {
  int64_t n, ld, coord_off, bits_off, hist_off;
};

// Tables of an instance counted by ranks (ranks.hip), in the workspace's rank area: n
// points (0: not counted by ranks), in nb blocks of 64 of the u order.
//   sigma  uint16[64 nb]  u place by v place          pi  uint16[64 nb]  v place by u place
//   row    uint32[64 nb]  pi << 16 | 4 D per point, D = its number of predecessors
//   tab    uint32, row J < nb of 64 J entries: pi_i << 16 | 4 F(64 J, pi_i) for i < 64 J
//   seg    uint16, row s (1 <= s <= (nb - 1) / 4) of 64 nb entries: F(256 s, pi_j), j >= 256 s
// where F(a, x) is the number of points with u place below a and v place below x.
constexpr int kRankSegBlocks = 4;  // row blocks per unit of counting work
struct RankInst {
  int64_t base;      // byte offset in the rank area
  int64_t hist_off;  // uint64 bins
  int32_t n, nb;
  __host__ __device__ int64_t sigma_off() const { return base; }
  __host__ __device__ int64_t pi_off() const { return base + 128ll * nb; }
  __host__ __device__ int64_t row_off() const { return base + 256ll * nb; }
  __host__ __device__ int64_t tab_off(int64_t J) const { return base + 512ll * nb + 128 * J * (J - 1); }
  __host__ __device__ int64_t seg_off(int64_t s) const { return tab_off(nb) + 128ll * nb * (s - 1); }
  int64_t end() const { return seg_off((nb - 1) / kRankSegBlocks + 1); }
  // units of counting work: column block J with the segments of its row blocks 0 .. J
  int64_t units() const {
    const int64_t q = nb / kRankSegBlocks, r = nb % kRankSegBlocks;
    return (q + 1) * (kRankSegBlocks / 2 * q + r);
  }
};

// Largest instance of an ensemble (its whole histogram fits the LDS bins, its sort
// fits one workgroup's LDS).
constexpr int64_t kBatchMaxN = 8192;
// Instances of up to kSmallN points can take forms of the ensemble kernels with less LDS and
// fewer wavefronts per instance, in launches of their own: a workgroup sized for 8192 points
// keeps half a CU or a whole one to itself for microseconds whatever its instance holds.  They
// do where there are kSmallMany of them, or where the whole ensemble has at most kTinyN points
// an instance.  Whole runs, us, in the large / the small forms: 60000 of 30 points 3650 / 960,
// 2000 of 512 212 / 138, 600 of 512 87 / 76, 300 of 512 57 / 65, one of 512 34 / 55 (its units on
// four wavefronts), one of 200 28.4 / 26.9, one of 64 23.1 / 19.0.
constexpr int64_t kSmallN = 512, kSmallMany = 512, kTinyN = 192;
// Padding entry of the ensemble builder's per-XCD item lists.
constexpr uint32_t kNoBuildItem = 0xFFFFFFFFu;

// ---------------------------------------------------------------------------
// Internal launchers (each returns CS_OK or CS_ERR_HIP).
// ---------------------------------------------------------------------------
size_t sprinkle_ws_bytes(int region, int64_t n);
cs_status launch_sprinkle(int region, double eta0, uint64_t seed, int64_t n, double* coords,
                          void* ws, hipStream_t st);
cs_status launch_causal_matrix(int region, const double* coords, int64_t n, uint64_t* bits,
                               int64_t ld, hipStream_t st);
size_t histogram_ws_bytes(int64_t n, int counter);
constexpr size_t kFieldWsMin = 256;  // what the d'Alembertian cannot do without
size_t field_ws_bytes(int64_t n, int counter);
long double prefactor_c3();  // (pi / (3 sqrt 2))^(2/3) / Gamma(5/3), the 2+1 constant
cs_status launch_dalembertian(const uint64_t* bits, int64_t n, int64_t ld, int counter, int dim,
                              double ell, const double* phi, double* out, void* ws, size_t ws_bytes, hipStream_t st);
cs_status launch_histogram(const uint64_t* bits, int64_t n, int64_t ld, int counter,
                           uint64_t* hist, void* ws, hipStream_t st);
cs_status launch_action(const uint64_t* hist, int64_t n, int dim, double eps, double* out,
                        hipStream_t st);
cs_status launch_fill_u64(uint64_t* p, int64_t count, uint64_t value, hipStream_t st);
size_t chain_ws_bytes(int64_t n, int64_t count);
// Blocks until the rounds are done (reads a per-round progress count back).
cs_status launch_longest_chain(const uint64_t* bits, int64_t n, int64_t ld, const int64_t* lo,
                               const int64_t* hi, int64_t count, int32_t* length,
                               int32_t* height, void* ws, hipStream_t st);
cs_status launch_degrees(const uint64_t* bits, int64_t n, int64_t ld, int64_t* indeg,
                         int64_t* outdeg, hipStream_t st);
int device_cu_count();

// Allocation-free entry points: bytes of the per-device static scratch array, and its
// device address on the current device (looked up once per device).
constexpr size_t kScratchBytes = 16384;
cs_status scratch_for_current_device(void** out);

// Ensemble pieces (1+1 diamonds).
// small: the forms for instances of at most kSmallN points.  ids: the instances of the launch
// (null: 0 .. count - 1).
cs_status launch_sprinkle_batch(bool small, const uint64_t* seeds, const BatchInst* inst,
                                const RankInst* rank, const uint32_t* ids, int64_t count,
                                double* coords, uint32_t* uv, char* rank_base, uint64_t* hist,
                                uint64_t* zero, int nzero, hipStream_t st);
// Rank tables (items: instance << 16 | group of kTabBlocks column blocks), then the counts from
// them (items: instance << 16 | chunk of `per_item` units; counter: one work counter, zero at
// launch).
cs_status launch_rank_tables(bool small, const RankInst* rank, const uint32_t* items, int64_t nitems,
                             char* rank_base, hipStream_t st);
cs_status launch_count_ranks(bool small, const RankInst* rank, const uint32_t* items, int64_t nitems,
                             int per_item, const char* rank_base, uint64_t* hist,
                             unsigned int* counter, hipStream_t st);
constexpr int kRankWaves = 16;  // wavefronts per workgroup of the rank counter
constexpr int kTabBlocks = 16;  // column blocks per workgroup of the rank tables
constexpr int kSmallWaves = 4;  // both for small instances
cs_status launch_build_batch(bool small, const uint32_t* uv, const BatchInst* inst,
                             const uint32_t* items, int64_t nitems, uint64_t* bits, hipStream_t st);
// Launch configuration of an ensemble counter: mode 0 is the bitset counter (128 tiles;
// tiles with more than pair_max related-pair tasks take the dense product, pair_max < 0:
// every tile), modes 2 / 4 the MFMA counter with 128 / 256 tiles on the int8 or (fp4 =
// true) the fp4 matrix cores; per_cu persistent workgroups per compute unit (1 or 2; the
// 256 tiles fit one).
struct BatchTile {
  int mode;
  int per_cu;
  int pair_max;
};
// An ensemble counter's work list in one queue per XCD: queue x is items[off[x] .. off[x+1]).
constexpr int kBatchQueues = 8;
struct BatchQueues {
  uint32_t off[kBatchQueues + 1];
};
// counter: kBatchQueues work counters, zero at launch.
cs_status launch_count_batch(const BatchTile& cfg, bool fp4, const uint64_t* bits,
                             const BatchInst* inst, const uint32_t* items,
                             const BatchQueues& queues, uint64_t* hist, unsigned int* counter,
                             hipStream_t st);
cs_status launch_action_batch(const uint64_t* hist, const BatchInst* inst, int64_t count,
                              int dim, const double* eps, int n_eps, double* out,
                              hipStream_t st);

}  // namespace cs
