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
// Tables: one wavefront per (instance, column block J).  Along the v order the number of
// points seen with u place < 64 J is F(64 J, x); it is scattered to u order in LDS and
// written in whole lines.  Work: n steps per column block, n^2 / 64 per instance; bound by
// latency (0.19 ms for 256 diamonds of 512 to 8192 points, two workgroups per CU).
// ---------------------------------------------------------------------------
constexpr int kTabWaves = 4;
constexpr int kTabUnroll = 4;

__global__ __launch_bounds__(64 * kTabWaves) void k_rank_tables(const RankInst* __restrict__ rank,
                                                                const uint32_t* __restrict__ items,
                                                                int64_t nitems,
                                                                char* __restrict__ base) {
  __shared__ uint16_t lds[kTabWaves][kBatchMaxN];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t it = (int64_t)blockIdx.x * kTabWaves + wave;
  if (it >= nitems) return;  // no workgroup barrier below
  const uint32_t item = items[it];
  const RankInst d = rank[item >> 16];
  const int J = (int)(item & 0xFFFFu), n = d.n, lim = 64 * J;
  const uint16_t* sigma = (const uint16_t*)(base + d.sigma_off());
  const uint16_t* pi = (const uint16_t*)(base + d.pi_off());
  uint16_t* F = lds[wave];  // F[i] = F(64 J, pi_i)
  uint32_t run = 0;
  for (int x0 = 0; x0 < n; x0 += 64 * kTabUnroll) {
    uint32_t s[kTabUnroll];
#pragma unroll
    for (int q = 0; q < kTabUnroll; ++q) {
      const int x = x0 + 64 * q + lane;
      s[q] = x < n ? sigma[x] : 0xFFFFu;
    }
#pragma unroll
    for (int q = 0; q < kTabUnroll; ++q) {
      const uint64_t m = __ballot((int)s[q] < lim);
      const uint32_t f = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, run));
      if (s[q] != 0xFFFFu) F[s[q]] = (uint16_t)f;
      run += (uint32_t)__popcll(m);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  uint32_t* tab = (uint32_t*)(base + d.tab_off(J));
  for (int i = 2 * lane; i < lim; i += 128) {  // 64 J entries, two per lane
    const uint32_t f2 = *(const uint32_t*)(F + i);
    *(uint2*)(tab + i) = make_uint2((f2 & 0xFFFFu) << 2, (f2 >> 16) << 2);
  }
  if (J > 0 && J % kRankSegBlocks == 0) {
    uint16_t* seg = (uint16_t*)(base + d.seg_off(J / kRankSegBlocks));
    for (int i = lim + lane; i < n; i += 64) seg[i] = F[i];
  }
  // The block's own points: D_i = F(64 J, pi_i) + #{64 J <= k < i : pi_k < pi_i}.
  const int i = lim + lane;
  const uint32_t p = i < n ? pi[i] : 0u;
  uint32_t D = i < n ? F[i] : 0u;
#pragma unroll 8
  for (int k = 0; k < 63; ++k) {
    const uint32_t pk = __builtin_amdgcn_readlane(p, k);
    if (lane > k && pk < p) ++D;
  }
  ((uint32_t*)(base + d.row_off()))[i] = i < n ? (p << 16 | D << 2) : 0u;
}

// ---------------------------------------------------------------------------
// Counts.  Persistent workgroups of kRankWaves wavefronts, one LDS histogram each; an item
// is `per_item` units of one instance, dealt to the wavefronts in turn.  A row costs five
// VALU operations for 64 pairs and one LDS add on the related lanes (about half), which
// is the bound: 256 diamonds of 512 to 8192 points (3.1e9 pairs) take 0.73 ms, 8.1 cycles
// per row and CU, where the fp4 matrix-core tiles took 3.15 ms.
// ---------------------------------------------------------------------------
constexpr int kRankThreads = 64 * kRankWaves;
constexpr int kRankBins = (int)kBatchMaxN - 1;
constexpr int kRankRows = 8;  // rows per scalar fetch

// One row against the 64 columns of the lanes.  x: pi_i << 16 plus 4 (D_i - F(64 J, pi_i)),
// a difference in [-4 pi_i, 256], so x < pi_j << 16 is the relation, and its low half,
// sign-extended, the row's share of the bin's byte address.  H = A_j(i) - lane.
__device__ __forceinline__ void rank_row(uint32_t x, uint64_t keep, uint32_t pj, int32_t& H,
                                         uint32_t* hist) {
  const uint64_t m = __builtin_amdgcn_ballot_w64(x < pj) & keep;
  const int32_t t = (int32_t)__builtin_amdgcn_mbcnt_hi(
      (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)H));
  const int32_t addr = (t << 2) + (int32_t)(int16_t)(uint16_t)x;
  if (__builtin_amdgcn_inverse_ballot_w64(m)) atomicAdd((uint32_t*)((char*)hist + addr), 1u);
  uint64_t carry_out;  // H + this lane's bit of m, in one add
  asm("v_addc_co_u32_e64 %0, %1, %2, 0, %3" : "=v"(H), "=s"(carry_out) : "v"(H), "s"(m));
}

__device__ inline void rank_unit(const RankInst& d, const char* __restrict__ base, int J, int s,
                                 uint32_t* hist) {
  const int lane = threadIdx.x & 63;
  const int n = d.n, j = 64 * J + lane;
  const uint32_t* __restrict__ row = (const uint32_t*)(base + d.row_off());
  const uint32_t* __restrict__ tab = (const uint32_t*)(base + d.tab_off(J));
  const uint32_t own = j < n ? row[j] : 0u;
  const uint32_t pj = own & 0xFFFF0000u;  // 0 past n: above no row
  const int lo = 64 * kRankSegBlocks * s;
  int hi = lo + 64 * kRankSegBlocks;
  int32_t H = -lane;
  if (hi <= 64 * J) {
    const uint16_t* seg = (const uint16_t*)(base + d.seg_off(s + 1));
    if (j < n) H += (int32_t)((own & 0xFFFFu) >> 2) - (int32_t)seg[j];
  } else {  // the diagonal block: columns above the row's own, B_i counted from there
    hi = 64 * J;
    const int last = n - hi < 64 ? n - hi : 64;
    for (int r = last - 1; r >= 0; --r) {
      const uint32_t pr = __builtin_amdgcn_readlane(pj, r);
      rank_row(pr + 4u * (uint32_t)(r + 1), r == 63 ? 0ull : ~0ull << (r + 1), pj, H, hist);
    }
  }
  for (int i = hi - kRankRows; i >= lo; i -= kRankRows) {
    uint32_t x[kRankRows];
#pragma unroll
    for (int q = 0; q < kRankRows; ++q) x[q] = row[i + q] - tab[i + q];
#pragma unroll
    for (int q = kRankRows - 1; q >= 0; --q) rank_row(x[q], ~0ull, pj, H, hist);
  }
}

__global__ __launch_bounds__(kRankThreads, 8) void k_count_ranks(
    const RankInst* __restrict__ rank, const uint32_t* __restrict__ items, int64_t nitems,
    int per_item, const char* __restrict__ base, unsigned long long* __restrict__ ghist,
    unsigned int* __restrict__ counter) {
  __shared__ uint32_t hist[kRankBins];
  __shared__ int slot;
  for (int b = threadIdx.x; b < kRankBins; b += kRankThreads) hist[b] = 0;
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
        for (int b = threadIdx.x; b < d.n - 1; b += kRankThreads)
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
    for (int64_t u = u0 + wave; u < u1; u += kRankWaves) {
      // Unit u: the column blocks 4q .. 4q + 3 have q + 1 segments each, 2q (q + 1) units
      // before them.
      int Q = (int)((sqrtf(2.0f * (float)u + 1.0f) - 1.0f) * 0.5f);
      while (2ll * Q * (Q + 1) > u) --Q;
      while (2ll * (Q + 1) * (Q + 2) <= u) ++Q;
      const int rest = (int)(u - 2ll * Q * (Q + 1));
      const int J = __builtin_amdgcn_readfirstlane(kRankSegBlocks * Q + rest / (Q + 1));
      const int s = __builtin_amdgcn_readfirstlane(rest % (Q + 1));
      rank_unit(d, base, J, s, hist);
    }
  }
  __syncthreads();
  if (cur >= 0)
    for (int b = threadIdx.x; b < d.n - 1; b += kRankThreads)
      if (const uint32_t v = hist[b]) atomicAdd(ghist + d.hist_off + b, (unsigned long long)v);
}

}  // namespace

cs_status launch_rank_tables(const RankInst* rank, const uint32_t* items, int64_t nitems,
                             char* rank_base, hipStream_t st) {
  if (nitems <= 0) return CS_OK;
  hipLaunchKernelGGL(k_rank_tables, dim3((unsigned)ceil_div(nitems, kTabWaves)),
                     dim3(64 * kTabWaves), 0, st, rank, items, nitems, rank_base);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

cs_status launch_count_ranks(const RankInst* rank, const uint32_t* items, int64_t nitems,
                             int per_item, const char* rank_base, uint64_t* hist,
                             unsigned int* counter, hipStream_t st) {
  if (nitems <= 0) return CS_OK;
  const unsigned grid = (unsigned)(nitems < 2 * device_cu_count() ? nitems : 2 * device_cu_count());
  hipLaunchKernelGGL(k_count_ranks, dim3(grid), dim3(kRankThreads), 0, st, rank, items, nitems,
                     per_item, rank_base, (unsigned long long*)hist, counter);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

}  // namespace cs
