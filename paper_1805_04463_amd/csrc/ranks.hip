// Interval abundances of 1+1 diamonds from ranks (ensembles).
//
// In a 1+1 diamond i ≺ j when both light-cone coordinates grow, so the interval of a
// related pair is the set of points in a rectangle (eq. IOIs), and the pairs need no inner
// product over the matrix.  Number the points by their place in u and let pi_i be the
// place of point i in v: i ≺ j iff i < j and pi_i < pi_j, and the interval size is
//
//   n_ij = #{i < k < j : pi_i < pi_k < pi_j} = A_j(i) - B_i(j),
//   A_j(i) = #{i < k < j : pi_k < pi_j},   B_i(j) = #{i < k < j : pi_k < pi_i}
//
// (for a related pair every k with pi_k < pi_i is in both).  Both terms change by at most
// one from a pair to its neighbour, so a pair costs a handful of integer operations
// instead of the N/64 words, or matrix-core steps, of its two rows: O(N^2) for an
// instance where the counters over the matrix take O(N^3).
//
// A wavefront takes a block J of 64 columns j (one per lane) and walks rows i downwards.
// For each row, which is the same for all lanes, one compare gives the relation mask;
// A_j grows by the mask's bit (a carry-in add); and B_i(j) is B_i at the block's first
// column plus the unrelated lanes below j, i.e. lane - mbcnt(mask).  With F(a, x) the
// number of points with u place < a and v place < x, and D_i = F(i, pi_i):
//   B_i(64 J) = F(64 J, pi_i) - D_i        (scalar, from a table by k_rank_tables)
//   A_j(i)    = D_j - F(i + 1, pi_j)       (from the table at the first row of a unit)
// so rows can be cut anywhere: a unit is one column block by up to 256 rows.
#include "common.h"

namespace cs {
namespace {

// ---------------------------------------------------------------------------
// Tables: a workgroup per (instance of up to CAP points, group of TB column blocks), one
// wavefront per column block J.  F(64 J, x) is a rank query on the set of v places of the points
// with u place below 64 J: a bit per v place, with the running count beside every 32 of them.
// The group's first set comes from sigma (one ballot per 64 places), the others add the
// preceding blocks' points.  A query is one 8-byte LDS gather and a popcount, about nine
// operations per table entry; scattering F through LDS from a scan of sigma by every
// wavefront took 146 us for 256 diamonds of 512 to 8192 points, this takes 70 us (97 MB
// written).  30000 diamonds of 64 points take 36 us with CAP = 512, TB = 4, and 184 with 8192, 16.
// ---------------------------------------------------------------------------
template <int CAP, int TB>
__global__ __launch_bounds__(64 * TB) void k_rank_tables(const RankInst* __restrict__ rank,
                                                         const uint32_t* __restrict__ items,
                                                         char* __restrict__ base) {
  constexpr int kThreads = 64 * TB, kWords = CAP / 32;
  __shared__ uint16_t pis[CAP] __attribute__((aligned(16)));
  __shared__ uint32_t first[kWords] __attribute__((aligned(16)));
  __shared__ uint32_t own[TB][kWords] __attribute__((aligned(16)));
  __shared__ uint2 sets[TB][kWords] __attribute__((aligned(16)));  // bits, count below
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t item = __builtin_amdgcn_readfirstlane(items[blockIdx.x]);
  const RankInst d = rank[item >> 16];
  const int J0 = (int)(item & 0xFFFFu) * TB, J = J0 + wave;
  const int n = d.n, lim = 64 * J;
  const uint16_t* __restrict__ sigma = (const uint16_t*)(base + d.sigma_off());
  const uint16_t* __restrict__ pi = (const uint16_t*)(base + d.pi_off());
  for (int r = 8 * threadIdx.x; r < 64 * d.nb; r += 8 * kThreads)
    *(uint4*)(pis + r) = *(const uint4*)(pi + r);
  for (int w = wave; w < d.nb; w += TB) {  // sigma is 0xFFFF past n
    const uint64_t m = __ballot((int)sigma[64 * w + lane] < 64 * J0);
    if (lane == 0) *(uint2*)(first + 2 * w) = make_uint2((uint32_t)m, (uint32_t)(m >> 32));
  }
  for (int w = 2 * d.nb + threadIdx.x; w < kWords; w += kThreads) first[w] = 0;
  const bool mine = 4 * lane < kWords;  // a lane's four words of a set
  const int at = mine ? 4 * lane : 0;
  if (mine) *(uint4*)(own[wave] + at) = make_uint4(0, 0, 0, 0);
  const int i = lim + lane;  // the block's own points
  const uint32_t p = i < n ? pi[i] : 0u;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (i < n) atomicOr(&own[wave][p >> 5], 1u << (p & 31));
  __syncthreads();
  if (J >= d.nb) return;  // no barrier below
  {
    uint4 v = mine ? *(const uint4*)(first + at) : make_uint4(0, 0, 0, 0);
    for (int w = 0; w < wave && mine; ++w) {
      const uint4 o = *(const uint4*)(own[w] + at);
      v.x |= o.x;
      v.y |= o.y;
      v.z |= o.z;
      v.w |= o.w;
    }
    const uint32_t c0 = __popc(v.x), c1 = c0 + __popc(v.y), c2 = c1 + __popc(v.z);
    const uint32_t sum = c2 + __popc(v.w);
    uint32_t x = sum;
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
      const uint32_t y = __shfl_up(x, k);
      if (lane >= k) x += y;
    }
    x -= sum;
    if (mine) {
      *(uint4*)(sets[wave] + at) = make_uint4(v.x, x, v.y, x + c0);
      *(uint4*)(sets[wave] + at + 2) = make_uint4(v.z, x + c1, v.w, x + c2);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  auto F = [&](uint32_t x) -> uint32_t {
    const uint2 w = sets[wave][x >> 5];
    return w.y + __popc(w.x & ((1u << (x & 31)) - 1u));
  };
  auto entry = [&](uint32_t x) -> uint32_t { return x << 16 | F(x) << 2; };
  uint32_t* __restrict__ tab = (uint32_t*)(base + d.tab_off(J));
#pragma unroll 2
  for (int r = 4 * lane; r < lim; r += 256) {  // 64 J entries, four per lane
    const uint2 q = *(const uint2*)(pis + r);
    *(uint4*)(tab + r) = make_uint4(entry(q.x & 0xFFFFu), entry(q.x >> 16), entry(q.y & 0xFFFFu),
                                    entry(q.y >> 16));
  }
  if (J > 0 && J % kRankSegBlocks == 0) {
    uint16_t* seg = (uint16_t*)(base + d.seg_off(J / kRankSegBlocks));
#pragma unroll 2
    for (int r = lim + 4 * lane; r < n; r += 256) {
      const uint2 q = *(const uint2*)(pis + r);
      *(uint2*)(seg + r) = make_uint2(F(q.x & 0xFFFFu) | F(q.x >> 16) << 16,
                                      F(q.y & 0xFFFFu) | F(q.y >> 16) << 16);
    }
  }
  // D_i = F(64 J, pi_i) + #{64 J <= k < i : pi_k < pi_i}.
  uint32_t D = F(p);
#pragma unroll 8
  for (int k = 0; k < 63; ++k) {
    const uint32_t pk = __builtin_amdgcn_readlane(p, k);
    if (lane > k && pk < p) ++D;
  }
  ((uint32_t*)(base + d.row_off()))[i] = i < n ? (p << 16 | D << 2) : 0u;
}

// ---------------------------------------------------------------------------
// Counts.  Persistent workgroups of WAVES wavefronts, one LDS histogram each; an item
// is `per_item` units of one instance, dealt to the wavefronts in turn.  A row costs five
// VALU and three scalar operations for 64 pairs and one LDS add on the related lanes (about
// half): 256 diamonds of 512 to 8192 points (3.1e9 pairs) take 0.66 ms, 7.3 cycles per
// row and CU, where the fp4 matrix-core tiles took 3.15 ms.  Issue is the bound: the VALU
// is busy 79 % of the time (instructions times 4 cycles), the scalar unit 72 %, and bank
// conflicts of the adds take 39 % of the LDS (without the adds a copy of the kernel took
// 0.60 ms; 16 rows per fetch 0.68 ms).  Thousands of small instances are
// bound by the one work counter, 12 ns an item (30000 of 128 points 374 us; with 16 wavefronts
// and all 8191 bins 504).
// ---------------------------------------------------------------------------
constexpr int kRankRows = 8;   // rows per scalar fetch

// One row against the 64 columns of the lanes.  x: pi_i << 16 with low bits of no weight
// (x < pi_j << 16 is the relation); c = 4 (D_i - F(64 J, pi_i)), the row's share of the bin's
// byte address; H = A_j(i) - lane.  The add runs on the related lanes only: every lane is
// active around it, and written out it leaves the rows one straight block of code instead
// of a branch per row.
__device__ __forceinline__ void rank_row(uint32_t x, int32_t c, bool keep, uint32_t pj, int32_t& H,
                                         uint32_t hist, uint32_t one) {
  const bool rel = (x < pj) & keep;
  const uint64_t m = __builtin_amdgcn_ballot_w64(rel);
  const uint32_t t = __builtin_amdgcn_mbcnt_hi(
      (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)H));
  const uint32_t addr = (t << 2) + (uint32_t)c + hist;
  asm volatile("s_mov_b64 exec, %0\n\tds_add_u32 %1, %2\n\ts_mov_b64 exec, -1"
               :
               : "s"(m), "v"(addr), "v"(one));
  H += rel ? 1 : 0;        // a carry-in add of m, kept apart from the next row's:
  asm("" : "+v"(H));  // combined, the two would take a select more
}

// kRankRows rows of the point and table arrays (wave-uniform: scalar loads).
struct RowChunk {
  uint32_t x[kRankRows], y[kRankRows];
  __device__ __forceinline__ void fetch(const uint32_t* __restrict__ row,
                                        const uint32_t* __restrict__ tab, int i) {
#pragma unroll
    for (int q = 0; q < kRankRows; ++q) {
      x[q] = row[i + q];
      y[q] = tab[i + q];
    }
  }
  // Waits for the fetch here, so that the next one can be issued before these rows are
  // used (scalar loads return out of order: any wait is for all of them).
  __device__ __forceinline__ void arrive() {
    asm volatile("" ::"s"(x[0]), "s"(y[0]) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
};

// hist: LDS byte address of the workgroup's bins.
__device__ inline void rank_unit(const RankInst& d, const char* __restrict__ base, int J, int s,
                                 uint32_t hist) {
  const int lane = threadIdx.x & 63;
  const int n = d.n, j = 64 * J + lane;
  const uint32_t* __restrict__ row = (const uint32_t*)(base + d.row_off());
  const uint32_t* __restrict__ tab = (const uint32_t*)(base + d.tab_off(J));
  const uint32_t own = j < n ? row[j] : 0u;
  const uint32_t pj = own & 0xFFFF0000u;  // 0 past n: above no row
  const uint32_t one = 1u;
  const int lo = 64 * kRankSegBlocks * s;
  int hi = lo + 64 * kRankSegBlocks;
  int32_t H = -lane;
  if (hi <= 64 * J) {
    const uint16_t* seg = (const uint16_t*)(base + d.seg_off(s + 1));
    if (j < n) H += (int32_t)((own & 0xFFFFu) >> 2) - (int32_t)seg[j];
  } else {  // the diagonal block: columns above the row's own, B_i counted from there
    hi = 64 * J;
    const int last = n - hi < 64 ? n - hi : 64;
    for (int r = last - 1; r >= 0; --r)
      rank_row(__builtin_amdgcn_readlane(pj, r), 4 * (r + 1), lane > r, pj, H, hist, one);
  }
  auto rows = [&](const RowChunk& c) {
#pragma unroll
    for (int q = kRankRows - 1; q >= 0; --q)
      rank_row(c.x[q], (int32_t)(c.x[q] - c.y[q]), true, pj, H, hist, one);
  };
  if (hi > lo) {  // a multiple of 64 rows, two chunks in turn
    RowChunk a, b;
    a.fetch(row, tab, hi - kRankRows);
    for (int i = hi - kRankRows; i > lo; i -= 2 * kRankRows) {
      a.arrive();
      b.fetch(row, tab, i - kRankRows);
      rows(a);
      b.arrive();
      a.fetch(row, tab, i - kRankRows > lo ? i - 2 * kRankRows : lo);
      rows(b);
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the adds have reached LDS
}

template <int CAP, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 8) void k_count_ranks(
    const RankInst* __restrict__ rank, const uint32_t* __restrict__ items, int64_t nitems,
    int per_item, const char* __restrict__ base, unsigned long long* __restrict__ ghist,
    unsigned int* __restrict__ counter) {
  constexpr int kThreads = 64 * WAVES, kBins = CAP - 1;
  __shared__ uint32_t hist[kBins];
  __shared__ int slot;
  for (int b = threadIdx.x; b < kBins; b += kThreads) hist[b] = 0;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const bool direct = nitems <= (int64_t)gridDim.x;  // an item per workgroup: no counter
  int cur = -1;
  RankInst d{};
  for (bool first = true;; first = false) {
    int64_t q;
    if (direct) {
      if (!first) break;
      q = blockIdx.x;
      __syncthreads();
    } else {
      __syncthreads();
      if (threadIdx.x == 0) slot = (int)atomicAdd(counter, 1u);
      __syncthreads();
      q = __builtin_amdgcn_readfirstlane(slot);
    }
    if (q >= nitems) break;
    const uint32_t it = items[q];
    const int k = (int)(it >> 16);
    if (k != cur) {
      if (cur >= 0) {
        for (int b = threadIdx.x; b < d.n - 1; b += kThreads)
          if (const uint32_t v = hist[b]) {
            atomicAdd(ghist + d.hist_off + b, (unsigned long long)v);
            hist[b] = 0;
          }
        __syncthreads();
      }
      cur = k;
      d = rank[k];
    }
    const int64_t u0 = (int64_t)(it & 0xFFFFu) * per_item;
    const int64_t total = (int64_t)(d.nb / kRankSegBlocks + 1) *
                          (kRankSegBlocks / 2 * (d.nb / kRankSegBlocks) + d.nb % kRankSegBlocks);
    const int64_t u1 = u0 + per_item < total ? u0 + per_item : total;
    for (int64_t u = u0 + wave; u < u1; u += WAVES) {
      // Unit u: the column blocks 4q .. 4q + 3 have q + 1 segments each, 2q (q + 1) units
      // before them.
      int Q = (int)((sqrtf(2.0f * (float)u + 1.0f) - 1.0f) * 0.5f);
      while (2ll * Q * (Q + 1) > u) --Q;
      while (2ll * (Q + 1) * (Q + 2) <= u) ++Q;
      const int rest = (int)(u - 2ll * Q * (Q + 1));
      const int J = __builtin_amdgcn_readfirstlane(kRankSegBlocks * Q + rest / (Q + 1));
      const int s = __builtin_amdgcn_readfirstlane(rest % (Q + 1));
      rank_unit(d, base, J, s, (uint32_t)(uintptr_t)hist);
    }
  }
  __syncthreads();
  if (cur >= 0)
    for (int b = threadIdx.x; b < d.n - 1; b += kThreads)
      if (const uint32_t v = hist[b]) atomicAdd(ghist + d.hist_off + b, (unsigned long long)v);
}

}  // namespace

cs_status launch_rank_tables(bool small, const RankInst* rank, const uint32_t* items, int64_t nitems,
                             char* rank_base, hipStream_t st) {
  if (nitems <= 0) return CS_OK;
  auto go = [&](auto kernel, int blocks) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)nitems), dim3(64 * blocks), 0, st, rank, items, rank_base);
  };
  if (small) go(k_rank_tables<(int)kSmallN, kSmallWaves>, kSmallWaves);
  else go(k_rank_tables<(int)kBatchMaxN, kTabBlocks>, kTabBlocks);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

cs_status launch_count_ranks(bool small, const RankInst* rank, const uint32_t* items, int64_t nitems,
                             int per_item, const char* rank_base, uint64_t* hist,
                             unsigned int* counter, hipStream_t st) {
  if (nitems <= 0) return CS_OK;
  auto go = [&](auto kernel, int waves) {
    const int64_t resident = 32 / waves * (int64_t)device_cu_count();
    hipLaunchKernelGGL(kernel, dim3((unsigned)(nitems < resident ? nitems : resident)),
                       dim3(64 * waves), 0, st, rank, items, nitems, per_item, rank_base,
                       (unsigned long long*)hist, counter);
  };
  if (small) go(k_count_ranks<(int)kSmallN, kSmallWaves>, kSmallWaves);
  else go(k_count_ranks<(int)kBatchMaxN, kRankWaves>, kRankWaves);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

}  // namespace cs
