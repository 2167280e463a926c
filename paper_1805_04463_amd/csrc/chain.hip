// Longest chains inside Alexandroff sets (Sec. 2.5.2 "Set Partitions", algorithm "Maximal
// Chain Length") and the degree vectors of the causal matrix (Sec. 3.2).
//
// The algorithm walks an Alexandroff set A_ij recursively with a memo of distances.  A
// recursion is a poor fit for 64-wide wavefronts, so the same quantity is computed
// through Mirsky's theorem instead: in a finite order, the elements whose longest chain
// (counted from below) has h elements are exactly those removed in round h when minimal
// elements are removed repeatedly.  For the set X = A_ij ∪ {j}, round h removes the
// elements h links above i, and j goes last: the number of rounds is the number of links
// of the longest chain from i to j.
//
// A member k is minimal when no element of its past is left, so each k keeps a witness: the
// latest past element still in X that a scan of its row, from k downward, last found.  A
// round tests one bit per member, whether its witness is still there, and scans on, from
// the witness's word down, only for the members that lost theirs.  Words above it were
// seen empty of remaining elements and stay empty, because X only shrinks; a hit is the
// new witness, and no hit down to the lowest word that holds a member (which rises with
// the rounds) makes k minimal.  Over a whole 3+1 order an element is scanned 2.4 times, the
// last time to be removed, and half of its row is read.
//
// Rounds are a chain of dependent steps, so what counts is the latency of one.  Two forms:
//   - k_chain_round, a launch per round: a workgroup owns the 64 elements of one word of a
//     pair's X, collects those that lost their witness in LDS and deals their scans to its
//     wavefronts.  Removals stay unseen in their round: each word of X is rewritten by its
//     owner into the bitmap that the next round tests.  The host launches rounds in batches
//     over the words that still have members and surveys them after each batch.  Round 0,
//     every element's first search, is bandwidth (75 us for the 3+1 order of 131072
//     elements); the others take 6 to 30 us, of which 5 are launch and bookkeeping.  The
//     order's 41 rounds take 0.93 ms, against 1.67 ms with two launches per round and
//     scans of one wavefront down to word 0.
//   - k_chain_pair, for many rounds on a set that fits the LDS: one workgroup runs the rest
//     of one pair's rounds with X, the witnesses and the work list in LDS, so a round
//     costs two barriers and the latency of its row reads, and no launch (100 pairs of a
//     1+1 diamond of 16384 points, 245 rounds: 4.0 us a round; the call 1.40 ms, against
//     7.5 to 9.1 ms).  After each batch the host takes the form that the costs below say
//     is faster for the rounds left.
#include <math.h>

#include <algorithm>
#include <vector>

#include "common.h"

namespace cs {
namespace {

constexpr int kChainBlock = 256;  // four wavefronts
constexpr int kChainWaves = kChainBlock / kWave;
constexpr int kScanDepth = 4;        // 64-word loads in flight per wave in a long scan step
// Threads for each word of a round over `active` words of pairs of W words.  Few words take many
// wavefronts each, as long as the workgroups are resident together (512 of 1024 threads), or
// four times as many where rows are long and their scans outweigh the test; many short rows
// take two wavefronts, as one does the test.  Calls, us, with 1024 / 512 / 256 / 128 threads: the
// whole 3+1 order of 131072 elements (2048 words) 896 / 991 / 1379 / 2289, eight of 16384 (2048
// words) 429 / 390 / 413 / 513, one of 4096 (64 words) 203 / 217 / 238 / 294, 100 of 500 (800
// words) 164 / 149 / 157 / 172, seven of 60000 (6566 words) 1218 / 1000 / 890 / 1085; 40000
// random pairs of a 1+1 diamond of 500 (8 words a pair) 3545 / 2367 / 1585 / 1353, of 65 (2)
// 993 / 691 / 516 / 473.
int round_threads(int64_t W, unsigned long long active) {
  if (active <= 512 || (active <= 2048 && W >= 512)) return 1024;
  if (active <= 2048) return 512;
  return active > 16384 && W <= 64 ? 128 : 256;
}
// Costs that decide between the two forms after each batch, in us: a round's launch, plus
// so much per word that it visits; a round of k_chain_pair, plus so much per member of
// the largest pair for the scans of its one workgroup.  (Fitted to both forms alone on 1+1,
// 2+1 and 3+1 diamonds of 2000 to 32768 points and 1 to 200 pairs: rounds of the whole 3+1
// order of 32768 points take 0.37 ms, the workgroup alone 2.9 ms; 200 pairs of the 1+1 one
// 12 to 99 ms and 3.2 ms.)
constexpr double kRoundUs = 5.0, kWordUs = 6e-4, kPairRoundUs = 3.5, kPairMemberUs = 0.03;
constexpr uint64_t kNoWord = ~0ull;  // unused entry of the word list
// Up to this many words in all, round 0 is launched over every one before the first look at
// the members (entries past the list's end return at once): the host round trip costs 20 us, e.g.
// 896 -> 921 for the whole 3+1 order of 131072 elements without.  A limit of 16384 words made
// seven random pairs of 131072, few of whose words have members, take 120 us instead of 57.
constexpr int64_t kBlindWords = 4096;
constexpr int64_t kPairMaxN = 32768;  // k_chain_pair: 16-bit indices, 140 KiB of LDS

// Members of pair s in word w, one lane per element: lo ≺ k and (k ≺ hi or k = hi), lo = -1
// / hi = n being the virtual elements below / above everything.
__device__ __forceinline__ bool chain_member(const uint64_t* __restrict__ bits, int64_t n,
                                             int64_t ld, int64_t lo, int64_t hi, int64_t w,
                                             int lane) {
  const int64_t k = w * kWave + lane;
  bool in = k < n && k > lo && k <= hi;
  if (in && lo >= 0) in = (bits[lo * ld + w] >> lane) & 1;              // lo ≺ k
  if (in && hi < n && k < hi) in = (bits[hi * ld + w] >> lane) & 1;     // k ≺ hi
  return in;
}

// X_0, zero heights and an empty word list.
__global__ __launch_bounds__(kChainBlock) void k_chain_init(
    const uint64_t* __restrict__ bits, int64_t n, int64_t ld, int64_t W,
    const int32_t* __restrict__ lohi, uint64_t* __restrict__ X0, int32_t* __restrict__ height,
    uint64_t* __restrict__ list) {
  const int s = blockIdx.y;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t w = (int64_t)blockIdx.x * kChainWaves + (threadIdx.x >> 6);
  if (w >= W) return;
  const uint64_t word =
      __ballot(chain_member(bits, n, ld, lohi[2 * s], lohi[2 * s + 1], w, lane));
  const int64_t k = w * kWave + lane;
  if (k < n) height[(int64_t)s * n + k] = 0;
  if (lane == 0) {
    X0[(int64_t)s * W + w] = word;
    list[(int64_t)s * W + w] = kNoWord;
  }
}

// What a batch of rounds starts from, one workgroup per pair: the members left in all and
// in the largest pair, the list of words with a member (pair << 32 | word << 1 | whether it
// is the pair's lowest) and each pair's lowest.  Words without members leave the other
// bitmap too, as no round visits them again.  (Counting removals in the rounds instead, an
// add per workgroup to one address, cost each round several us.)
struct Survey {
  unsigned long long left, most, active, unused;
};
constexpr int kSurveyThreads = 1024;
__global__ __launch_bounds__(kSurveyThreads) void k_chain_survey(
    const uint64_t* __restrict__ R, uint64_t* __restrict__ other, int64_t W,
    int32_t* __restrict__ low, uint64_t* __restrict__ list, Survey* __restrict__ out) {
  __shared__ uint32_t left, lowest, active;
  __shared__ unsigned long long first;
  const int s = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t* r = R + (int64_t)s * W;
  if (threadIdx.x == 0) {
    left = active = 0;
    lowest = (uint32_t)W;
  }
  __syncthreads();
  uint32_t members = 0, words = 0, mine = (uint32_t)W;
  for (int64_t w = threadIdx.x; w < W; w += kSurveyThreads) {
    const uint64_t x = r[w];
    if (x == 0) {
      other[(int64_t)s * W + w] = 0;
      continue;
    }
    members += (uint32_t)__popcll(x);
    ++words;
    mine = min(mine, (uint32_t)w);
  }
  for (int off = kWave / 2; off > 0; off >>= 1) {
    members += __shfl_xor(members, off);
    words += __shfl_xor(words, off);
    mine = min(mine, (uint32_t)__shfl_xor(mine, off));
  }
  if (lane == 0 && words) {
    atomicAdd(&left, members);
    atomicAdd(&active, words);
    atomicMin(&lowest, mine);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    low[s] = (int32_t)lowest;
    if (left) {
      first = atomicAdd(&out->active, (unsigned long long)active);
      atomicAdd(&out->left, (unsigned long long)left);
      atomicMax(&out->most, (unsigned long long)left);
    }
    active = 0;
  }
  __syncthreads();
  if (left == 0) return;
  for (int64_t w0 = threadIdx.x & ~(kWave - 1); w0 < W; w0 += kSurveyThreads) {
    const int64_t w = w0 + lane;
    const bool some = w < W && r[w] != 0;
    const uint64_t m = __ballot(some);
    if (m == 0) continue;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&active, (uint32_t)__popcll(m));
    at = __shfl(at, 0) + (uint32_t)__popcll(m & ((1ull << lane) - 1));
    if (some) list[first + at] = (uint64_t)s << 32 | (uint64_t)w << 1 | (w == (int64_t)lowest ? 1u : 0u);
  }
}

// The same for more than kSurveyPairs pairs: a wavefront per pair, pairs dealt to the wavefronts
// of few workgroups, as each adds three times to the survey's one line (12 ns) while a
// wavefront spends about 1.2 us on a pair of a few words: about sqrt(2 count) workgroups balance
// the two.  (40000 pairs of 65 elements: 20 us, where a workgroup per pair took 777; 5000: 8.6
// us, 12.1 with 256 workgroups.)
constexpr int kSurveyPairs = 256, kSurveyGroups = 256;
constexpr int kSurveyWaves = kSurveyThreads / kWave;
__global__ __launch_bounds__(kSurveyThreads) void k_chain_survey_many(
    const uint64_t* __restrict__ R, uint64_t* __restrict__ other, int64_t W, int64_t count,
    int32_t* __restrict__ low, uint64_t* __restrict__ list, Survey* __restrict__ out) {
  __shared__ unsigned long long wave_left[kSurveyWaves], wave_most[kSurveyWaves],
      wave_active[kSurveyWaves];  // the last: then where the wavefront's entries go
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t step = (int64_t)gridDim.x * kSurveyWaves;
  unsigned long long left = 0, most = 0, active = 0;
  for (int64_t s = (int64_t)blockIdx.x * kSurveyWaves + wave; s < count; s += step) {
    uint32_t members = 0;
    int64_t lowest = W;
    for (int64_t w0 = 0; w0 < W; w0 += kWave) {
      const int64_t w = w0 + lane;
      const uint64_t x = w < W ? R[s * W + w] : 0ull;
      if (w < W && x == 0) other[s * W + w] = 0;
      const uint64_t m = __ballot(x != 0);
      members += (uint32_t)__popcll(x);
      active += (unsigned long long)__popcll(m);
      if (m && lowest == W) lowest = w0 + __builtin_ctzll(m);
    }
    for (int off = kWave / 2; off > 0; off >>= 1) members += __shfl_xor(members, off);
    if (lane == 0) low[s] = (int32_t)lowest;
    left += members;
    most = max(most, (unsigned long long)members);
  }
  if (lane == 0) {
    wave_left[wave] = left;
    wave_most[wave] = most;
    wave_active[wave] = active;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long words = 0;
    for (int i = 0; i < kSurveyWaves; ++i) words += wave_active[i];
    if (words) {
      unsigned long long at = atomicAdd(&out->active, words);
      left = most = 0;
      for (int i = 0; i < kSurveyWaves; ++i) {
        left += wave_left[i];
        most = max(most, wave_most[i]);
        const unsigned long long own = wave_active[i];
        wave_active[i] = at;
        at += own;
      }
      atomicAdd(&out->left, left);
      atomicMax(&out->most, most);
    }
  }
  __syncthreads();
  if (active == 0) return;
  unsigned long long at = wave_active[wave];
  for (int64_t s = (int64_t)blockIdx.x * kSurveyWaves + wave; s < count; s += step) {
    bool first = true;
    for (int64_t w0 = 0; w0 < W; w0 += kWave) {
      const int64_t w = w0 + lane;
      const bool some = w < W && R[s * W + w] != 0;
      const uint64_t m = __ballot(some);
      if (m == 0) continue;
      const int below = __popcll(m & ((1ull << lane) - 1));
      if (some) list[at + below] = (uint64_t)s << 32 | (uint64_t)w << 1 | (first && below == 0 ? 1u : 0u);
      at += (unsigned long long)__popcll(m);
      first = false;
    }
  }
}

// Highest word q in [wlo, top] of row k holding a member of R, looking at J * 64 words
// (lane l, load j: word top - l - 64 j), and that word's members in *hit; -1 if none of
// them has one.  first: mask of the word `top` (the past part of k's own word).
template <int J>
__device__ __forceinline__ int64_t scan_step(const uint64_t* __restrict__ row,
                                             const uint64_t* __restrict__ R, int64_t top,
                                             int64_t wlo, int lane, uint64_t first, uint64_t* hit) {
  uint64_t v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int64_t q = top - lane - (int64_t)kWave * j;
    v[j] = q >= wlo ? (row[q] & R[q]) : 0ull;
  }
  if (lane == 0) v[0] &= first;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const uint64_t m = __ballot(v[j] != 0);
    if (m) {
      const int src = __builtin_ctzll(m);
      const uint32_t l = __builtin_amdgcn_readlane((uint32_t)v[j], src);
      const uint32_t h = __builtin_amdgcn_readlane((uint32_t)(v[j] >> 32), src);
      *hit = (uint64_t)h << 32 | l;
      return top - (int64_t)src - (int64_t)kWave * j;
    }
  }
  return -1;
}

// One wavefront: k's first witness, the latest member of R in its past, from word w (its own)
// down to word wlo, or -1.  It is usually found about a hundred words down, so the steps
// grow: 64, 128, then 256 words.
__device__ __forceinline__ int64_t first_witness(const uint64_t* __restrict__ row,
                                                 const uint64_t* __restrict__ R, int64_t w,
                                                 int64_t wlo, int lane, uint64_t mask) {
  uint64_t hit = 0;
  int64_t q = scan_step<1>(row, R, w, wlo, lane, mask, &hit), top = w - kWave;
  if (q < 0 && top >= wlo) {
    q = scan_step<2>(row, R, top, wlo, lane, ~0ull, &hit);
    top -= 2 * kWave;
  }
  for (; q < 0 && top >= wlo; top -= (int64_t)kWave * kScanDepth)
    q = scan_step<kScanDepth>(row, R, top, wlo, lane, ~0ull, &hit);
  return q < 0 ? -1 : q * kWave + 63 - __builtin_clzll(hit);
}

// Round t for the 64 elements of each of the `active` listed words, a workgroup per word.  R:
// the members (read only); R_next: the members without this round's minimal elements.  ROWS:
// the grid has several rows (testing the index in every round cost 0.3 us each).
template <int THREADS, bool ROWS = false>
__global__ __launch_bounds__(THREADS, 8) void k_chain_round(
    const uint64_t* __restrict__ bits, int64_t n, int64_t ld, int64_t W,
    const uint64_t* __restrict__ list, int64_t active, const uint64_t* __restrict__ R,
    uint64_t* __restrict__ R_next, int32_t* __restrict__ wit, int32_t* __restrict__ height, const int32_t* __restrict__ low,
    int32_t* __restrict__ low_next, int32_t t) {
  constexpr int kWaves = THREADS / kWave;
  __shared__ int32_t todo[kWave], top_of[kWave];  // element of the word; word to resume at
  __shared__ int32_t best[kWave];                 // its witness found this round, or -1
  __shared__ uint64_t removed;
  __shared__ int ntodo;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t group = ROWS ? group_index() : (int64_t)blockIdx.x;
  if (ROWS && group >= active) return;  // the whole workgroup, here and below
  const uint64_t entry = list[group];
  if (entry == kNoWord) return;
  const int s = (int)(entry >> 32);
  const int64_t w = (int64_t)((uint32_t)entry >> 1);
  const uint64_t* r = R + (int64_t)s * W;
  const int64_t wlo = low[s];
  uint64_t word = 0;
  if (wave == 0) {
    const int64_t k = w * kWave + lane;
    word = r[w];
    // read beside the word, not after it: a stale entry of a former member is not used
    const int32_t m = t > 0 && k < n ? wit[(int64_t)s * n + k] : 0;
    bool need = (word >> lane) & 1;
    int64_t top = w;
    if (need && t > 0) {
      top = m >> 6;
      need = !((r[top] >> (m & 63)) & 1);
    }
    const uint64_t mask = __ballot(need);
    if (need) {
      const int at = __popcll(mask & ((1ull << lane) - 1));
      todo[at] = lane;
      top_of[at] = (int32_t)top;
      best[at] = -1;
    }
    if (lane == 0) {
      ntodo = __popcll(mask);
      removed = 0;
    }
  }
  __syncthreads();
  const int items = ntodo;
  // After round 0 most scans end in removal, all the way down to wlo, so a scan is cut into
  // pieces of 256 words, each a wavefront's single step; the pieces of all items are dealt
  // to the wavefronts and the highest hit counts.
  constexpr int kPiece = kWave * kScanDepth;
  const int pieces = t == 0 ? 1 : (int)((w - wlo) / kPiece) + 1;
  for (int x = wave; x < items * pieces; x += kWaves) {
    const int i = x % items, u = x / items;
    const int64_t k = w * kWave + __builtin_amdgcn_readfirstlane(todo[i]);
    const int64_t top = (int64_t)__builtin_amdgcn_readfirstlane(top_of[i]) - (int64_t)u * kPiece;
    if (top < wlo) continue;
    const uint64_t mask = top == w ? (1ull << (k & 63)) - 1ull : ~0ull;
    const uint64_t* row = bits + k * ld;
    int64_t m = -1;
    if (t == 0) {
      m = first_witness(row, r, top, wlo, lane, mask);
    } else {
      uint64_t hit = 0;
      const int64_t q = scan_step<kScanDepth>(row, r, top, wlo, lane, mask, &hit);
      if (q >= 0) m = q * kWave + 63 - __builtin_clzll(hit);
    }
    if (m >= 0 && lane == 0) atomicMax(&best[i], (int32_t)m);
  }
  if ((entry & 1) && wave == kWaves - 1) {  // the lowest word with a member of R
    int64_t q = wlo;
    for (; q < W; q += kWave) {
      const uint64_t m = __ballot(q + lane < W && r[q + lane] != 0);
      if (m) {
        q += __builtin_ctzll(m);
        break;
      }
    }
    if (lane == 0) low_next[s] = (int32_t)(q < W ? q : W);
  }
  __syncthreads();
  if (wave != 0) return;
  if (lane < items) {
    const int e = todo[lane];
    const int64_t at = (int64_t)s * n + w * kWave + e;
    const int32_t m = best[lane];
    if (m >= 0) {
      wit[at] = m;
    } else {
      height[at] = t + 1;
      atomicOr((unsigned long long*)&removed, 1ull << e);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (lane == 0) R_next[(int64_t)s * W + w] = word & ~removed;
}

// The rounds from t on of pair blockIdx.x (t >= 1: every member has a witness), with the
// members X0 and witnesses left by the rounds before; n <= kPairMaxN.  Dynamic LDS: two bitmaps of the members
// (W words each: a round tests one, and its removals are cleared in the other, which the
// next round tests), the round's removals (W words, cleared in the first bitmap a round
// later), witnesses and work list (n 16-bit entries each).  A round is two phases with a
// barrier each: list the members that lost their witness, scan for each.  A scan takes a
// group of 8 lanes and 64 words per step, so a wavefront serves 8 members at once.
constexpr int kPairGroup = 8;    // lanes per scan
constexpr int kPairUnroll = 4;   // words per wavefront and check step; loads per scan step
constexpr int64_t kNarrowWords = 16;  // more pairs than CUs take 256 threads for up to so many
                                      // words, which four wavefronts check in a step (5000
                                      // pairs of 65 elements 8 us, with 1024 threads 10)

template <int kPairThreads>
__global__ __launch_bounds__(kPairThreads) void k_chain_pair(
    const uint64_t* __restrict__ bits, int64_t n, int64_t ld, int64_t W64,
    const uint64_t* __restrict__ X0, const int32_t* __restrict__ wit0,
    const int32_t* __restrict__ low0, int32_t* __restrict__ height, int t) {
  constexpr int kPairWaves = kPairThreads / kWave;
  extern __shared__ uint64_t chain_lds[];
  const int W = (int)W64;
  uint64_t* X = chain_lds;      // bitmap c at X + c W
  uint64_t* gone = X + 2 * W;
  uint16_t* wit = (uint16_t*)(gone + W);
  uint16_t* todo = wit + W * kWave;
  __shared__ int ntodo[2], left, low[2];
  const int s = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int32_t* h = height + (int64_t)s * n;
  if (threadIdx.x == 0) {
    ntodo[0] = ntodo[1] = left = 0;
    low[t & 1] = low0[s];
  }
  __syncthreads();
  for (int w = wave; w < W; w += kPairWaves) {
    const uint64_t word = X0[(int64_t)s * W + w];
    const int64_t k = (int64_t)w * kWave + lane;
    if (word) wit[k] = (uint16_t)(k < n ? wit0[(int64_t)s * n + k] : 0);
    if (lane == 0) {
      X[w] = X[W + w] = word;
      gone[w] = 0;
      if (word) atomicAdd(&left, __popcll(word));
    }
  }
  __syncthreads();
  const int grp = lane / kPairGroup, sub = lane % kPairGroup;
  // every round removes at least the member of the lowest index: n rounds in all at most
  for (; t <= n && left > 0; ++t) {
    const uint64_t* R = X + (t & 1) * W;
    uint64_t* R_next = X + ((t + 1) & 1) * W;
    const int wlo = low[t & 1];
    int* count = &ntodo[t & 1];
    for (int w0 = wlo + wave; w0 < W; w0 += kPairWaves * kPairUnroll) {
      uint64_t word[kPairUnroll];
      uint32_t m[kPairUnroll];
      uint64_t at_m[kPairUnroll];
#pragma unroll
      for (int u = 0; u < kPairUnroll; ++u) {
        const int w = w0 + u * kPairWaves;
        word[u] = w < W ? R[w] : 0ull;
        // (members' entries count; others may hold anything: kept inside the bitmap)
        m[u] = w < W ? min((uint32_t)wit[w * kWave + lane], (uint32_t)(W * kWave - 1)) : 0u;
      }
#pragma unroll
      for (int u = 0; u < kPairUnroll; ++u) at_m[u] = R[m[u] >> 6];
#pragma unroll
      for (int u = 0; u < kPairUnroll; ++u) {
        const int w = w0 + u * kPairWaves;
        const bool need = ((word[u] >> lane) & 1) && !((at_m[u] >> (m[u] & 63)) & 1);
        const uint64_t mask = __ballot(need);
        if (mask == 0) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(count, __popcll(mask));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(mask & ((1ull << lane) - 1));
        if (need) todo[at] = (uint16_t)(w * kWave + lane);
      }
    }
    for (int w = threadIdx.x; w < W; w += kPairThreads) {  // the last round's removals
      const uint64_t g = gone[w];
      if (g) {
        R_next[w] &= ~g;
        gone[w] = 0;
      }
    }
    if (wave == kPairWaves - 1) {  // the lowest word with a member, for the next round
      int w = wlo;
      for (; w < W; w += kWave) {
        const uint64_t v = __ballot(w + lane < W && R[w + lane < W ? w + lane : 0] != 0);
        if (v) {
          w += __builtin_ctzll(v);
          break;
        }
      }
      if (lane == 0) low[(t + 1) & 1] = w;
    }
    __syncthreads();
    const int items = *count;
    if (threadIdx.x == 0) ntodo[(t + 1) & 1] = 0;
    for (int i = threadIdx.x / kPairGroup; i < items; i += kPairThreads / kPairGroup) {
      const int k = todo[i];
      const uint64_t* row = bits + (int64_t)k * ld;
      int top = wit[k] >> 6;
      uint64_t first = top == k >> 6 ? (1ull << (k & 63)) - 1ull : ~0ull;
      int m = -1;
      for (; top >= wlo && m < 0; top -= 2 * kPairGroup * kPairUnroll) {
        // two words per lane and load, from the pair of words that holds `top` down
        const int p0 = (top >> 1) - sub;
        uint64_t v[kPairUnroll][2];
#pragma unroll
        for (int j = 0; j < kPairUnroll; ++j) {
          const int p = p0 - kPairGroup * j;
          v[j][0] = v[j][1] = 0;
          if (2 * p + 1 >= wlo) {
            const ulonglong2 b = *(const ulonglong2*)(row + 2 * p);  // rows start on 64 bytes
            const int q = 2 * p;
            v[j][0] = b.x & R[q];
            v[j][1] = q + 1 <= top ? b.y & R[q + 1 < W ? q + 1 : q] : 0ull;
            if (q == top) v[j][0] &= first;
            if (q + 1 == top) v[j][1] &= first;
          }
        }
        first = ~0ull;
#pragma unroll
        for (int j = 0; j < kPairUnroll; ++j) {
          const uint32_t b = (uint32_t)(__ballot((v[j][0] | v[j][1]) != 0) >> (kPairGroup * grp)) &
                             ((1u << kPairGroup) - 1u);
          if (m < 0 && b) {
            const int src = __builtin_ctz(b);
            const uint64_t x1 = __shfl((unsigned long long)v[j][1], kPairGroup * grp + src);
            const uint64_t x0 = __shfl((unsigned long long)v[j][0], kPairGroup * grp + src);
            const int q = 2 * ((top >> 1) - src - kPairGroup * j);
            m = x1 ? (q + 1) * kWave + 63 - __builtin_clzll(x1) : q * kWave + 63 - __builtin_clzll(x0);
          }
        }
        top |= 1;  // the next step starts at the pair below the last one read
      }
      if (sub == 0) {
        if (m >= 0) {
          wit[k] = (uint16_t)m;
        } else {
          h[k] = t + 1;
          atomicAnd((unsigned long long*)&R_next[k >> 6], ~(1ull << (k & 63)));
          atomicOr((unsigned long long*)&gone[k >> 6], 1ull << (k & 63));
          atomicSub(&left, 1);
        }
      }
    }
    __syncthreads();
  }
}

// maxh[s] = the largest height of pair s (pairs ending at the virtual top only); blocks of
// blockIdx.x split the n heights, one atomicMax each.
__global__ __launch_bounds__(kChainBlock) void k_chain_maxh(const int32_t* __restrict__ lohi,
                                                           const int32_t* __restrict__ height,
                                                           int64_t n, int32_t* __restrict__ maxh) {
  const int s = blockIdx.y;
  if (lohi[2 * s + 1] != n) return;
  const int32_t* h = height + (int64_t)s * n;
  __shared__ int32_t part[kChainWaves];
  int32_t mx = 0;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * blockDim.x)
    mx = max(mx, h[k]);
  for (int off = kWave / 2; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
  if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kChainWaves; ++i) mx = max(mx, part[i]);
    if (mx) atomicMax(&maxh[s], mx);
  }
}

// length[s]: the height of hi (0 when hi is not in X, i.e. lo does not precede it), or,
// for the virtual top, one link above the highest element.
__global__ void k_chain_length(const int32_t* __restrict__ lohi, const int32_t* __restrict__ height,
                               const int32_t* __restrict__ maxh, int64_t count, int64_t n,
                               int32_t* __restrict__ length) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= count) return;
  const int64_t hi = lohi[2 * s + 1];
  length[s] = hi < n ? height[s * n + hi] : maxh[s] + 1;
}

// Degree vectors: one wavefront per row, 128 words per step (16-byte loads).
__global__ __launch_bounds__(kChainBlock) void k_degrees(const uint64_t* __restrict__ bits,
                                                        int64_t n, int64_t ld, int64_t W,
                                                        int64_t* __restrict__ indeg,
                                                        int64_t* __restrict__ outdeg) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t k = (int64_t)blockIdx.x * kChainWaves + (threadIdx.x >> 6);
  if (k >= n) return;
  const uint64_t* row = bits + k * ld;
  const int64_t kw = k >> 6;
  const uint64_t below = (k & 63) ? (~0ull >> (64 - (k & 63))) : 0ull;
  const uint64_t tail = (n & 63) ? (~0ull >> (64 - (n & 63))) : ~0ull;
  uint32_t cin = 0, cout = 0;
  for (int64_t w0 = 2 * lane; w0 < W; w0 += 2 * kWave) {
    const ulonglong2 v2 = *reinterpret_cast<const ulonglong2*>(row + w0);  // W <= ld, ld even
    uint64_t v[2] = {v2.x, v2.y};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t w = w0 + j;
      if (w >= W) break;
      uint64_t x = v[j];
      if (w == W - 1) x &= tail;
      if (w < kw) {
        cin += __popcll(x);
      } else if (w > kw) {
        cout += __popcll(x);
      } else {
        cin += __popcll(x & below);
        cout += __popcll(x & ~below & ~(1ull << (k & 63)));
      }
    }
  }
  for (int off = kWave / 2; off > 0; off >>= 1) {
    cin += __shfl_xor(cin, off);
    cout += __shfl_xor(cout, off);
  }
  if (lane == 0) {
    if (indeg) indeg[k] = cin;
    if (outdeg) outdeg[k] = cout;
  }
}

struct ChainWs {
  int32_t* lohi;
  uint64_t* books;  // zeroed at the start, book_words in all:
  Survey* survey;  //   before round 0, then after each batch
  int32_t* maxh;   //   largest height of each pair
  int64_t book_words;
  int32_t* low[2];
  uint64_t* X[2];
  uint64_t* list;  // words with members
  int32_t* wit;
  int32_t* height;  // used when the caller passes none
  size_t bytes;
};

int64_t max_batches(int64_t n) { return n / 2 + 2; }  // every batch has at least 2 rounds

ChainWs chain_layout(void* base, int64_t n, int64_t count) {
  const int64_t W = ceil_div(n, kWave);
  ChainWs L{};
  size_t off = 0;
  auto take = [&](size_t b) {
    const size_t o = off;
    off = align_up(off + b, 256);
    return (char*)base + o;
  };
  L.lohi = (int32_t*)take(sizeof(int32_t) * 2 * count);
  const size_t book = off;
  L.books = (uint64_t*)((char*)base + book);
  L.survey = (Survey*)take(sizeof(Survey) * (max_batches(n) + 1));
  L.maxh = (int32_t*)take(sizeof(int32_t) * count);
  L.book_words = (int64_t)((off - book) / sizeof(uint64_t));
  for (int b = 0; b < 2; ++b) L.low[b] = (int32_t*)take(sizeof(int32_t) * count);
  for (int b = 0; b < 2; ++b) L.X[b] = (uint64_t*)take(sizeof(uint64_t) * W * count);
  L.list = (uint64_t*)take(sizeof(uint64_t) * W * count);
  L.wit = (int32_t*)take(sizeof(int32_t) * n * count);
  L.height = (int32_t*)take(sizeof(int32_t) * n * count);
  L.bytes = off;
  return L;
}

}  // namespace

size_t chain_ws_bytes(int64_t n, int64_t count) {
  return chain_layout(nullptr, n, count).bytes;
}

cs_status launch_longest_chain(const uint64_t* bits, int64_t n, int64_t ld, const int64_t* lo,
                               const int64_t* hi, int64_t count, int32_t* length,
                               int32_t* height, void* ws, hipStream_t st) {
  ChainWs L = chain_layout(ws, n, count);
  int32_t* h = height ? height : L.height;
  const int64_t W = ceil_div(n, kWave);
  std::vector<int32_t> lohi(2 * count);
  for (int64_t s = 0; s < count; ++s) {
    lohi[2 * s] = (int32_t)lo[s];
    lohi[2 * s + 1] = (int32_t)hi[s];
  }
  CS_HIP_CHECK(hipMemcpyAsync(L.lohi, lohi.data(), sizeof(int32_t) * 2 * count,
                              hipMemcpyHostToDevice, st));
  cs_status s0 = launch_fill_u64(L.books, L.book_words, 0, st);
  if (s0 != CS_OK) return s0;
  hipLaunchKernelGGL(k_chain_init, dim3((unsigned)ceil_div(W, kChainWaves), (unsigned)count),
                     dim3(kChainBlock), 0, st, bits, n, ld, W, L.lohi, L.X[0], h, L.list);
  CS_LAUNCH_CHECK();
  // Round t removes the minimal elements of what the rounds before left; every X is empty
  // after at most n rounds.  Batches of rounds end with a survey that the host reads; the
  // next batch is sized from the rate of removal so far, so that few rounds run past the
  // end, and its launches cover the words that still have members.
  const int64_t words = W * count;
  Survey seen[2] = {};  // before the last batch and now
  Survey& now = seen[1];
  for (int64_t t = 0, batch = 8, b = 0;; ++b) {
    // the members before round t; low[] is read by round t from the other parity
    if (count <= kSurveyPairs)
      hipLaunchKernelGGL(k_chain_survey, dim3((unsigned)count), dim3(kSurveyThreads), 0, st,
                         L.X[t & 1], L.X[(t + 1) & 1], W, L.low[(t + 1) & 1], L.list, L.survey + b);
    else
      hipLaunchKernelGGL(k_chain_survey_many,
                         dim3((unsigned)std::min<int64_t>(kSurveyGroups, (int64_t)sqrt(2.0 * (double)count))),
                         dim3(kSurveyThreads), 0, st, L.X[t & 1], L.X[(t + 1) & 1], W, count,
                         L.low[(t + 1) & 1], L.list, L.survey + b);
    CS_LAUNCH_CHECK();
    if (t == 0 && words <= kBlindWords) {
      now.active = (unsigned long long)words;
    } else {
      const int64_t from = b > 0 ? b - 1 : 0;
      CS_HIP_CHECK(hipMemcpyAsync(seen + (b > 0 ? 0 : 1), L.survey + from,
                                  sizeof(Survey) * (b > 0 ? 2 : 1), hipMemcpyDeviceToHost, st));
      CS_HIP_CHECK(hipStreamSynchronize(st));
      if (now.left == 0) break;
    }
    if (t > n || b >= max_batches(n)) return CS_ERR_HIP;  // unreachable: a round removes members
    if (t > 0) {
      const double rate = (double)(seen[0].left - now.left) / (double)batch;  // >= 1 per round
      // Layers thin out towards the end, so the rate so far under-estimates the rounds
      // left; half again as many rounds (a round past the end is a near-empty launch) saves
      // host round trips.
      const double rounds = 1.5 * (double)now.left / rate;
      if (n <= kPairMaxN && rounds * (kRoundUs + kWordUs * (double)now.active) >
                                rounds * kPairRoundUs + kPairMemberUs * (double)now.most) {
        const size_t lds = (size_t)W * (3 * sizeof(uint64_t) + 2 * kWave * sizeof(uint16_t));
        const bool narrow = W <= kNarrowWords && count > kSurveyPairs;
        auto pairs = [&](auto kernel, int threads) {
          hipLaunchKernelGGL(kernel, dim3((unsigned)count), dim3(threads), lds, st, bits, n, ld, W,
                             L.X[t & 1], L.wit, L.low[(t + 1) & 1], h, (int)t);
        };
        if (narrow) pairs(k_chain_pair<256>, 256);
        else pairs(k_chain_pair<1024>, 1024);
        CS_LAUNCH_CHECK();
        CS_HIP_CHECK(hipStreamSynchronize(st));  // the call returns after its rounds in either form
        break;
      }
      batch = std::max<int64_t>(2, std::min<int64_t>(64, (int64_t)ceil(rounds)));
    }
    const int64_t end = std::min<int64_t>(t + batch, n + 1);
    batch = end - t;
    const int threads = round_threads(W, now.active);
    for (; t < end; ++t) {
      const int c = (int)(t & 1);
      auto round = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid_rows((int64_t)now.active), dim3(threads), 0, st, bits, n, ld, W,
                           L.list, (int64_t)now.active, L.X[c], L.X[c ^ 1], L.wit, h, L.low[c ^ 1],
                           L.low[c], (int32_t)t);
      };
      const bool rows = (int64_t)now.active > kGridRow;
      if (threads == 1024) round(k_chain_round<1024>);
      else if (threads == 512) round(k_chain_round<512>);
      else if (threads == 256) rows ? round(k_chain_round<256, true>) : round(k_chain_round<256>);
      else rows ? round(k_chain_round<128, true>) : round(k_chain_round<128>);
      CS_LAUNCH_CHECK();
    }
  }
  hipLaunchKernelGGL(k_chain_maxh, dim3((unsigned)std::min<int64_t>(64, ceil_div(n, 4096)),
                                        (unsigned)count),
                     dim3(kChainBlock), 0, st, L.lohi, h, n, L.maxh);
  CS_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_chain_length, dim3((unsigned)ceil_div(count, 256)), dim3(256), 0, st,
                     L.lohi, h, L.maxh, count, n, length);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

cs_status launch_degrees(const uint64_t* bits, int64_t n, int64_t ld, int64_t* indeg,
                         int64_t* outdeg, hipStream_t st) {
  const int64_t W = ceil_div(n, kWave);
  hipLaunchKernelGGL(k_degrees, dim3((unsigned)ceil_div(n, kChainWaves)), dim3(kChainBlock), 0,
                     st, bits, n, ld, W, indeg, outdeg);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

}  // namespace cs
