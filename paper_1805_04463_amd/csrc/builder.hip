// Causal-matrix builder: writes the symmetric packed bitset S = C + C^T of n
// time-ordered points (Sec. 3.2 "Data Structures for Graphs": a topologically
// sorted DAG kept as P + P^T; Ch. 4: i ≺ j iff timelike separated).
//
// Work decomposition: one wave per 64x64 block (bi <= bj) of the upper triangle.
// Lane l owns row i = 64*bi + l (coordinates in registers) and tests it against the
// 64 column points of block bj, the same for every lane: scalar loads in the 2+1 and
// 3+1 diamonds, staged in LDS elsewhere.  Its 64 answers form row i's word for column
// block bj.  A 64x64 bit transpose across the wave (six butterfly stages of lane
// shuffles) turns those row words into the words of rows j for column block bi, so each
// unordered pair is tested once and both halves of the symmetric matrix are written.
// Workgroups walk 1024 x 1024-point patches, one XCD per patch (k_build).  The ensemble
// builder takes its words from the points' places in u and v instead (k_build_batch).
//
// Arithmetic: fp64, in the order written, no contraction (built with
// -ffp-contract=off and explicit round-to-nearest intrinsics); on CDNA4 fp64 VALU
// runs at the rate of non-packed fp32, so no fp32 prefilter is used.
#include "common.h"

namespace cs {
namespace {

template <int R>
struct Pt;
template <>
struct Pt<CS_MINK2_DIAMOND> {
  double u, v;
};
template <>
struct Pt<CS_MINK4_DIAMOND> {
  double t, x, y, z;
};
template <>
struct Pt<CS_DS4_SLAB> {
  double x, c, s, n0, n1, n2, n3;
};
template <>
struct Pt<CS_DS2_SLAB> {
  double eta, th;
};
template <>
struct Pt<CS_MINK3_DIAMOND> {
  double t, x, y;
};

__device__ inline Pt<CS_MINK2_DIAMOND> load_pt(const double* c, int64_t n, int64_t i,
                                               Pt<CS_MINK2_DIAMOND>*) {
  return {c[i], c[n + i]};
}
__device__ inline Pt<CS_MINK4_DIAMOND> load_pt(const double* c, int64_t n, int64_t i,
                                               Pt<CS_MINK4_DIAMOND>*) {
  return {c[i], c[n + i], c[2 * n + i], c[3 * n + i]};
}
__device__ inline Pt<CS_DS4_SLAB> load_pt(const double* c, int64_t n, int64_t i,
                                          Pt<CS_DS4_SLAB>*) {
  return {c[i], c[n + i], c[2 * n + i], c[3 * n + i], c[4 * n + i], c[5 * n + i], c[6 * n + i]};
}

__device__ inline Pt<CS_DS2_SLAB> load_pt(const double* c, int64_t n, int64_t i,
                                          Pt<CS_DS2_SLAB>*) {
  return {c[n + i], c[2 * n + i]};
}
__device__ inline Pt<CS_MINK3_DIAMOND> load_pt(const double* c, int64_t n, int64_t i,
                                               Pt<CS_MINK3_DIAMOND>*) {
  return {c[i], c[n + i], c[2 * n + i]};
}

// a ≺ b for a earlier than b in time order.
__device__ inline bool precedes(const Pt<CS_MINK2_DIAMOND>& a, const Pt<CS_MINK2_DIAMOND>& b) {
  return (a.u < b.u) & (a.v < b.v);
}
__device__ inline bool precedes(const Pt<CS_MINK4_DIAMOND>& a, const Pt<CS_MINK4_DIAMOND>& b) {
  double dt = __dsub_rn(b.t, a.t);
  double dx = __dsub_rn(b.x, a.x);
  double dy = __dsub_rn(b.y, a.y);
  double dz = __dsub_rn(b.z, a.z);
  double s = __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy));
  s = __dadd_rn(s, __dmul_rn(dz, dz));
  return (dt > 0.0) & (__dmul_rn(dt, dt) > s);
}
__device__ inline bool precedes(const Pt<CS_DS4_SLAB>& a, const Pt<CS_DS4_SLAB>& b) {
  // eta_a < eta_b and cos(eta_b - eta_a) < n_a . n_b (both angles in [0, pi]).
  double cd = __dadd_rn(__dmul_rn(a.c, b.c), __dmul_rn(a.s, b.s));
  double dot = __dadd_rn(__dmul_rn(a.n0, b.n0), __dmul_rn(a.n1, b.n1));
  dot = __dadd_rn(dot, __dmul_rn(a.n2, b.n2));
  dot = __dadd_rn(dot, __dmul_rn(a.n3, b.n3));
  return (a.x < b.x) & (cd < dot);
}
__device__ inline bool precedes(const Pt<CS_MINK3_DIAMOND>& a, const Pt<CS_MINK3_DIAMOND>& b) {
  double dt = __dsub_rn(b.t, a.t);
  double dx = __dsub_rn(b.x, a.x);
  double dy = __dsub_rn(b.y, a.y);
  return (dt > 0.0) & (__dmul_rn(dt, dt) > __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)));
}
__device__ inline bool precedes(const Pt<CS_DS2_SLAB>& a, const Pt<CS_DS2_SLAB>& b) {
  // The angular separation the short way round, pi - |pi - |theta_a - theta_b||, below
  // the conformal-time separation (fabs is exact; pi is the double nearest pi).
  const double pi = 3.141592653589793;
  double dth = fabs(__dsub_rn(a.th, b.th));
  dth = __dsub_rn(pi, fabs(__dsub_rn(pi, dth)));
  return (a.eta < b.eta) & (dth < __dsub_rn(b.eta, a.eta));
}

// a ≺ b for points a, b with b no earlier than a in time order (the builder only
// asks this).  In the diamonds dt = t_b - t_a >= 0 exactly, and dt * dt > s >= 0 then
// already excludes dt == 0, so the dt > 0 test of precedes() is dropped: the same answer
// with one compare fewer.  The other regions ask precedes() as it stands.
template <int R>
__device__ inline bool later_precedes(const Pt<R>& a, const Pt<R>& b) {
  return precedes(a, b);
}
template <>
__device__ inline bool later_precedes(const Pt<CS_MINK4_DIAMOND>& a,
                                      const Pt<CS_MINK4_DIAMOND>& b) {
  double dt = __dsub_rn(b.t, a.t);
  double dx = __dsub_rn(b.x, a.x);
  double dy = __dsub_rn(b.y, a.y);
  double dz = __dsub_rn(b.z, a.z);
  double s = __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy));
  s = __dadd_rn(s, __dmul_rn(dz, dz));
  return __dmul_rn(dt, dt) > s;
}
template <>
__device__ inline bool later_precedes(const Pt<CS_MINK3_DIAMOND>& a,
                                      const Pt<CS_MINK3_DIAMOND>& b) {
  double dt = __dsub_rn(b.t, a.t);
  double dx = __dsub_rn(b.x, a.x);
  double dy = __dsub_rn(b.y, a.y);
  return __dmul_rn(dt, dt) > __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy));
}

// The wave's lane mask of later_precedes(a, b).  Where the relation is the AND of two
// compares, each compare writes its lane mask to scalar registers and the masks are
// ANDed there: a ballot of the AND would first turn it into a per-lane value and back
// (two VALU instructions more per pair test).  fcmp predicate 4 is ordered less-than,
// false for NaN like the C operator.
// APART: every a of the wave is strictly earlier than b (see block_apart), so the slabs
// drop their compare of the times.
template <bool APART, int R>
__device__ inline uint64_t precedes_mask(const Pt<R>& a, const Pt<R>& b) {
  return __builtin_amdgcn_ballot_w64(later_precedes(a, b));
}
template <bool APART>
__device__ inline uint64_t precedes_mask(const Pt<CS_MINK2_DIAMOND>& a,
                                         const Pt<CS_MINK2_DIAMOND>& b) {
  return __builtin_amdgcn_fcmp(a.u, b.u, 4) & __builtin_amdgcn_fcmp(a.v, b.v, 4);
}
template <bool APART>
__device__ inline uint64_t precedes_mask(const Pt<CS_DS4_SLAB>& a, const Pt<CS_DS4_SLAB>& b) {
  double cd = __dadd_rn(__dmul_rn(a.c, b.c), __dmul_rn(a.s, b.s));
  double dot = __dadd_rn(__dmul_rn(a.n0, b.n0), __dmul_rn(a.n1, b.n1));
  dot = __dadd_rn(dot, __dmul_rn(a.n2, b.n2));
  dot = __dadd_rn(dot, __dmul_rn(a.n3, b.n3));
  if constexpr (APART) return __builtin_amdgcn_fcmp(cd, dot, 4);
  return __builtin_amdgcn_fcmp(a.x, b.x, 4) & __builtin_amdgcn_fcmp(cd, dot, 4);
}
template <bool APART>
__device__ inline uint64_t precedes_mask(const Pt<CS_DS2_SLAB>& a, const Pt<CS_DS2_SLAB>& b) {
  const double pi = 3.141592653589793;
  double dth = fabs(__dsub_rn(a.th, b.th));
  dth = __dsub_rn(pi, fabs(__dsub_rn(pi, dth)));
  if constexpr (APART) return __builtin_amdgcn_fcmp(dth, __dsub_rn(b.eta, a.eta), 4);
  return __builtin_amdgcn_fcmp(a.eta, b.eta, 4) & __builtin_amdgcn_fcmp(dth, __dsub_rn(b.eta, a.eta), 4);
}

// The slabs' time of a point.
__device__ inline double time_of(const Pt<CS_DS4_SLAB>& p) { return p.x; }
__device__ inline double time_of(const Pt<CS_DS2_SLAB>& p) { return p.eta; }
template <int R>
constexpr bool kSlab = R == CS_DS4_SLAB || R == CS_DS2_SLAB;

// Whether all rows of the wave are strictly earlier than all columns (one per lane): true of
// time-ordered blocks above the diagonal but for ties, and then one compare of the 13 (3+1)
// or 7 (1+1) operations of a pair test is known (fp64 issue bounds these blocks; measured:
// 3+1 builder and degrees at 30001 points 258 -> 247 us, the 1+1 pass at 4001 57.2 -> 56.5).
// False when a time is NaN.
template <int R, int RB>
__device__ inline bool block_apart(const Pt<R> (&rows)[RB], const Pt<R>& col) {
  double first = time_of(col);
  bool ordered = first == first;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(first, off);
    first = o < first ? o : first;
  }
#pragma unroll
  for (int r = 0; r < RB; ++r) ordered = ordered & (time_of(rows[r]) < first);
  return __builtin_amdgcn_ballot_w64(!ordered) == 0;
}

// 2 w + (this lane's bit of the wave mask m): one add with m as the carry-in.
__device__ inline uint32_t shift_in(uint32_t w, uint64_t m) {
  uint32_t r;
  uint64_t carry_out;
  asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(r), "=s"(carry_out) : "v"(w), "s"(m));
  return r;
}

constexpr int kWavesPerBlock = 4;

// 64x64 bit transpose across a wave: lane l holds word x with bit c = element (l, c);
// afterwards lane c holds bit l = element (l, c).  Six butterfly stages; at stage s the
// off-diagonal s x s sub-blocks are swapped with the partner lane l ^ s.
__device__ inline uint64_t wave_transpose64(uint64_t x) {
  const int lane = threadIdx.x & 63;
  const uint64_t lo_masks[6] = {0x00000000FFFFFFFFull, 0x0000FFFF0000FFFFull,
                                0x00FF00FF00FF00FFull, 0x0F0F0F0F0F0F0F0Full,
                                0x3333333333333333ull, 0x5555555555555555ull};
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int s = 32 >> k;
    const uint64_t mlo = lo_masks[k], mhi = ~mlo;
    const uint32_t ylo = (uint32_t)__shfl_xor((int)(uint32_t)x, s);
    const uint32_t yhi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), s);
    const uint64_t y = ((uint64_t)yhi << 32) | ylo;
    x = (lane & s) ? ((x & mhi) | ((y & mhi) >> s)) : ((x & mlo) | ((y & mlo) << s));
  }
  return x;
}

// Row words of lane l for the 64 column points j0 .. j0+63, one per row point pi[r]:
// bit c is column c.  Columns enter from the top, 63 first, each compare's wave mask
// shifted in as a carry.  The columns are wave-uniform, and each is read once for all RB
// rows of the lane.  In the 3+1 and 2+1 diamonds they come through scalar loads into
// SGPRs and feed the fp64 operations directly, instead of broadcast reads from LDS (16
// bytes per lane per instruction: the LDS bound of those blocks).  The other regions
// stage them in LDS: the 7-plane de Sitter slab's columns, loaded ahead, do not fit the
// scalar registers, and the two-plane predicates are too short to hide the scalar load
// latency (both measured slower); with several rows per lane a broadcast read serves RB
// rows.  A block that ends past n repeats point n-1 for the missing columns (masked off
// by the caller).
template <int R>
constexpr bool kScalarColumns = R == CS_MINK4_DIAMOND || R == CS_MINK3_DIAMOND;

template <int R, bool FULL, int RB, bool APART>
__device__ __attribute__((always_inline)) inline void row_words(
    const double* __restrict__ coords, int64_t n, int64_t j0, const Pt<R> (&pi)[RB], Pt<R>* cols,
    uint64_t (&out)[RB]) {
  uint32_t half[RB][2];
#pragma unroll
  for (int h = 1; h >= 0; --h) {
    uint32_t w[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) w[r] = 0;
#pragma unroll
    for (int c = 31; c >= 0; --c) {
      int64_t j = j0 + 32 * h + c;
      if (!FULL) j = j < n ? j : n - 1;
      const Pt<R> q = kScalarColumns<R> ? load_pt(coords, n, j, (Pt<R>*)nullptr) : cols[32 * h + c];
#pragma unroll
      for (int r = 0; r < RB; ++r)
        w[r] = shift_in(w[r], precedes_mask<APART>(pi[r], q));
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) half[r][h] = w[r];
  }
#pragma unroll
  for (int r = 0; r < RB; ++r) out[r] = ((uint64_t)half[r][1] << 32) | half[r][0];
}

// One wave: the 64x64 blocks (bi0 + r, bj), r < RB, of an n-point matrix S with stride ld,
// those with bi0 + r <= bj (bi0 <= bj; both wave-uniform).  Lane l owns rows
// i = 64 (bi0 + r) + l and collects their row words for the 64 column points of block bj.
// The transposed words (rows of block bj, columns of block bi0 + r) come from a 64x64 bit
// transpose of each row word, so each unordered pair is tested once.  Blocks below the
// diagonal are tested but not written.  The wave owning the last column block of a row
// block also zeroes that row block's padding words [nb, ld), so every word of S is written
// exactly once.
template <int R, int RB>
__device__ __attribute__((always_inline)) inline void build_block(
    const double* __restrict__ coords, int64_t n, uint64_t* __restrict__ S, int64_t ld, int64_t nb,
    int64_t bi0, int64_t bj, Pt<R>* cols) {
  const int lane = threadIdx.x & 63;
  Pt<R> pi[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const int64_t i = (bi0 + r) * 64 + lane;
    pi[r] = load_pt(coords, n, i < n ? i : n - 1, (Pt<R>*)nullptr);
  }
  uint64_t rows[RB];
  const int64_t j0 = bj * 64;
  bool apart = false;
  if constexpr (!kScalarColumns<R>) {
    const Pt<R> col = load_pt(coords, n, j0 + lane < n ? j0 + lane : n - 1, (Pt<R>*)nullptr);
    cols[lane] = col;
    if constexpr (kSlab<R>) apart = block_apart<R, RB>(pi, col);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's LDS writes have landed
    __builtin_amdgcn_wave_barrier();
  }
  if (j0 + 64 > n) row_words<R, false, RB, false>(coords, n, j0, pi, cols, rows);
  else if (kSlab<R> && apart) row_words<R, true, RB, kSlab<R>>(coords, n, j0, pi, cols, rows);
  else row_words<R, true, RB, false>(coords, n, j0, pi, cols, rows);
  if constexpr (!kScalarColumns<R>) __builtin_amdgcn_wave_barrier();
  const int64_t j = bj * 64 + lane;
  const bool jv = j < n;
  const int64_t ncols = n - bj * 64;  // valid columns of the block (>= 1)
  if constexpr (RB == 4) {
    if (bi0 + RB - 1 < bj) {
      // Every block lies above the diagonal and every row is valid: a lane's four
      // transposed words of row j (column blocks bi0 .. bi0 + 3) are contiguous and 16-byte
      // aligned (bi0 is a multiple of 4, rows start on 64-byte boundaries), so they go out
      // as 16-byte stores instead of 8-byte ones.
      uint64_t cw[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        if (ncols < 64) rows[r] &= (1ull << ncols) - 1ull;
        const int64_t i = (bi0 + r) * 64 + lane;
        S[i * ld + bj] = rows[r];
        if (bj == nb - 1)
          for (int64_t w = nb; w < ld; ++w) S[i * ld + w] = 0;
        cw[r] = wave_transpose64(rows[r]);
      }
      if (jv) {
        uint4* dst = (uint4*)(S + j * ld + bi0);
        dst[0] = make_uint4((uint32_t)cw[0], (uint32_t)(cw[0] >> 32), (uint32_t)cw[1], (uint32_t)(cw[1] >> 32));
        dst[1] = make_uint4((uint32_t)cw[2], (uint32_t)(cw[2] >> 32), (uint32_t)cw[3], (uint32_t)(cw[3] >> 32));
      }
      return;
    }
  }
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const int64_t bi = bi0 + r;
    if (bi > bj) break;  // this and the later row blocks lie below the diagonal
    const int64_t i = bi * 64 + lane;
    const bool iv = i < n;
    uint64_t row = rows[r];
    if (ncols < 64) row &= (1ull << ncols) - 1ull;
    if (bi == bj) row &= lane == 63 ? 0ull : (~0ull << (lane + 1));  // only j > i
    if (!iv) row = 0;
    const uint64_t col = wave_transpose64(row);  // lane l: row j's bits for columns of bi
    if (bi == bj) {
      if (iv) S[i * ld + bi] = row | col;
    } else {
      if (iv) S[i * ld + bj] = row;
      if (jv) S[j * ld + bi] = col;
    }
    if (bj == nb - 1 && iv)
      for (int64_t w = nb; w < ld; ++w) S[i * ld + w] = 0;
  }
}

// Patches of 16 x 16 blocks (1024 x 1024 points) of the upper triangle, 64 / RB workgroups
// each (16 / RB groups of RB block rows x 4 groups of 4 block columns; a wave takes RB row
// blocks against one column block).  Workgroups are dealt to the 8
// XCDs in turn, so the workgroups of patch p get ids 8 apart: a patch is built
// inside one XCD, whose L2 then holds every 128-byte line of its row segments and of
// its transposed segments until the line is complete, instead of sending partial lines
// from several L2s to HBM.  Below 8 patches (n <= 3072) they are not dealt: the grid is
// the patches' own workgroups.  Patch p counts row-major over the patches (py, px >= py).
#ifndef CS_BUILD_PATCH
#define CS_BUILD_PATCH 16
#endif
constexpr int kPatch = CS_BUILD_PATCH;                       // blocks per patch side
constexpr int kGroups = kPatch / kWavesPerBlock;             // column groups per patch
template <int RB>
constexpr int kPatchWgs = kPatch / RB * kGroups;             // workgroups per patch
// Row blocks per wave, from 8 patches up (n > 3072: below that, the fewer, longer waves
// cost more latency than they save): four, so that each column point read from LDS (or
// loaded into SGPRs) serves four rows of a lane.
template <int R>
constexpr int kRowBlocks = 4;

__device__ inline int64_t patch_row_start(int64_t r, int64_t P) { return r * P - r * (r - 1) / 2; }

template <int R, int RB>
__global__ __launch_bounds__(256) void k_build(const double* __restrict__ coords, int64_t n,
                                               uint64_t* __restrict__ S, int64_t ld, int64_t nb,
                                               int64_t P, int64_t npatch) {
  constexpr int PW = kPatchWgs<RB>;
  __shared__ Pt<R> cols[kScalarColumns<R> ? 1 : kWavesPerBlock][64];
  const int64_t g = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const bool dealt = npatch >= 8;
  const int64_t p = dealt ? (g / (8 * PW)) * 8 + (g & 7) : g / PW;
  if (p >= npatch) return;
  const int l = (int)(dealt ? (g >> 3) % PW : g % PW);
  // smaller root of r^2 - (2P+1) r + 2p = 0, then exact correction
  const double s2 = 2.0 * (double)P + 1.0;
  int64_t py = (int64_t)((s2 - sqrt(s2 * s2 - 8.0 * (double)p)) * 0.5);
  while (py > 0 && patch_row_start(py, P) > p) --py;
  while (patch_row_start(py + 1, P) <= p) ++py;
  const int64_t px = py + (p - patch_row_start(py, P));
  const int64_t bi = py * kPatch + RB * (l / kGroups);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t bj = (px * kGroups + l % kGroups) * kWavesPerBlock + wave;
  if (bi >= nb || bj >= nb || bj < bi) return;  // wave-uniform exit; no block barriers below
  build_block<R, RB>(coords, n, S, ld, nb, bi, bj, cols[kScalarColumns<R> ? 0 : wave]);
}

// Ensemble of 1+1 diamonds, from the points' places in u and v (uv: u place << 16 | v place
// per point, in time order; equal coordinates hold opposite orders in the two, as they are
// unrelated).  Two points are related exactly when their places compare the same way in u
// and v, so the word of a row for a block of 64 columns is the XNOR of two masks: the
// block's points above the row's in u, and in v.  Each mask depends only on how many of
// the block's points lie below the row's place: that count is a rank query (a bit per
// place with running counts, as in the rank tables) and picks one of 65 precomputed
// masks.  Four 8-byte LDS gathers and a dozen operations give 64 pairs of one row, against
// 192 operations for testing the pairs, and rows below the diagonal need no transpose: 256
// diamonds of 512 to 8192 points take 0.19 ms for 0.82 GB of matrices (4.3 TB/s; the VALU
// is busy 58 % of the time, bank conflicts take half of the LDS), against 0.41 ms with the pair
// tests.
//
// A workgroup takes kBuildBlocks column blocks of an instance (512 columns: a lane's words
// of a row are 64 contiguous bytes, padding words included) against all its rows.  The
// items (instance << 16 | column group) form kBatchQueues lists of equal length, one per
// XCD, padded with kNoBuildItem: workgroup b takes entry b div kBatchQueues of list
// b mod kBatchQueues, the XCD that the dispatcher gives it, whose L2 completes the lines.
constexpr int kBuildBlocks = 8;
constexpr int kBuildTables = 2 * kBuildBlocks;  // (block, axis)
// Wavefronts, for instances of up to CAP points: one per table, or four, with eight workgroups per
// CU (30000 diamonds of 64 points 45 us, 298 with sixteen).
template <int CAP>
constexpr int kBuildWaves = CAP == kBatchMaxN ? kBuildTables : 4;

template <int CAP>
__global__ __launch_bounds__(64 * kBuildWaves<CAP>, 8) void k_build_batch(
    const uint32_t* __restrict__ uvs, const BatchInst* __restrict__ inst,
    const uint32_t* __restrict__ items, int64_t nitems, uint64_t* __restrict__ bits) {
  constexpr int kWaves = kBuildWaves<CAP>, kWords = CAP / 32;
  constexpr bool kAll = kWaves == kBuildTables;  // empty blocks have tables too
  __shared__ uint2 sets[kBuildTables][kWords] __attribute__((aligned(16)));  // bits, count below
  __shared__ uint64_t above[kBuildTables][66];  // [c]: columns with at least c of the block below
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t it = items[(int64_t)(blockIdx.x % kBatchQueues) * (nitems / kBatchQueues) +
                            blockIdx.x / kBatchQueues];
  if (it == kNoBuildItem) return;  // the whole workgroup
  const BatchInst d = inst[it >> 16];
  const uint32_t* __restrict__ uv = uvs + d.coord_off / 2;
  const int n = (int)d.n, nb = (n + 63) / 64, b0 = (int)(it & 0xFFFFu) * kBuildBlocks;
  auto query = [&](int a, uint32_t x) -> uint32_t {  // points of table a with place below x
    const uint2 w = sets[a][x >> 5];
    return w.y + __popc(w.x & ((1u << (x & 31)) - 1u));
  };
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const int blocks = nb - b0 < kBuildBlocks ? nb - b0 : kBuildBlocks;
  for (int a = wave; a < (kAll ? kBuildTables : 2 * blocks); a += kWaves) {
    // table 2 b + axis: column block b0 + b
    const int j = 64 * (b0 + (a >> 1)) + lane;
    const bool valid = j < n, mine = 4 * lane < kWords;  // a lane's four words of the set
    const uint32_t t = valid ? uv[j] : 0u;
    const uint32_t place = (a & 1) ? t & 0xFFFFu : t >> 16;
    uint4* s4 = (uint4*)(sets[a] + (mine ? 4 * lane : 0));
    if (mine) s4[0] = s4[1] = make_uint4(0, 0, 0, 0);
    above[a][lane] = 0;
    if (lane < 2) above[a][64 + lane] = 0;
    wave_sync();
    if (valid) atomicOr(&sets[a][place >> 5].x, 1u << (place & 31));
    wave_sync();
    const uint4 none = make_uint4(0, 0, 0, 0), p0 = mine ? s4[0] : none, p1 = mine ? s4[1] : none;
    const uint32_t c0 = __popc(p0.x), c1 = c0 + __popc(p0.z), c2 = c1 + __popc(p1.x);
    const uint32_t sum = c2 + __popc(p1.z);
    uint32_t x = sum;
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
      const uint32_t y = __shfl_up(x, k);
      if (lane >= k) x += y;
    }
    x -= sum;
    if (mine) {
      s4[0] = make_uint4(p0.x, x, p0.z, x + c0);
      s4[1] = make_uint4(p1.x, x + c1, p1.z, x + c2);
    }
    wave_sync();
    if (valid) above[a][query(a, place)] = 1ull << lane;
    wave_sync();
    uint64_t m = above[a][lane];
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {  // suffix OR over the lanes
      const uint32_t lo = __shfl_down((uint32_t)m, k), hi = __shfl_down((uint32_t)(m >> 32), k);
      if (lane + k < 64) m |= (uint64_t)hi << 32 | lo;
    }
    above[a][lane] = m;
  }
  __syncthreads();
  // Four lanes per row, two words each: a store instruction writes 16 whole 64-byte
  // segments.  (With a row per lane, its eight words in four stores, L2 took four partial
  // requests per segment: 0.25 ms.)
  const int quarter = lane & 3, own = 2 * quarter;  // this lane's blocks: b0 + own, + 1
  const bool edge = 64 * (b0 + kBuildBlocks) > n;   // columns past n in this group
  uint64_t* __restrict__ S = bits + d.bits_off + b0 + own;
  for (int rb = wave; rb < nb; rb += kWaves) {
    uint32_t t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = 64 * rb + 16 * k + (lane >> 2);
      t[k] = i < n ? uv[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = 64 * rb + 16 * k + (lane >> 2);
      const uint32_t pu = t[k] >> 16, pv = t[k] & 0xFFFFu;
      uint64_t w[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int a = 2 * (own + e);
        w[e] = kAll || own + e < blocks
                   ? ~(above[a][query(a, pu)] ^ above[a + 1][query(a + 1, pv)]) : 0ull;
        if (rb - b0 == own + e) w[e] &= ~(1ull << (i & 63));  // not related to itself
        if (edge) {
          const int left = n - 64 * (b0 + own + e);
          w[e] &= left >= 64 ? ~0ull : (left <= 0 ? 0ull : (1ull << left) - 1ull);
        }
      }
      if (i < n)
        *(uint4*)(S + (int64_t)i * d.ld) = make_uint4((uint32_t)w[0], (uint32_t)(w[0] >> 32),
                                                      (uint32_t)w[1], (uint32_t)(w[1] >> 32));
    }
  }
}

template <int R, int RB>
cs_status launch_build_rb(const double* coords, int64_t n, uint64_t* S, int64_t ld, int64_t nb,
                          int64_t P, int64_t npatch, hipStream_t st) {
  // Grid rows of at most 64 rounds of 8 patches: a row stays far below 2^32 work-items.
  constexpr int PW = kPatchWgs<RB>;
  const int64_t rounds = ceil_div(npatch, 8);  // nb <= 65535: at most 2^20 rounds
  const dim3 grid = npatch >= 8 ? dim3((unsigned)(8 * PW * std::min<int64_t>(rounds, 64)),
                                       (unsigned)ceil_div(rounds, 64))
                                : dim3((unsigned)(PW * npatch));
  hipLaunchKernelGGL((k_build<R, RB>), grid, dim3(64 * kWavesPerBlock), 0, st, coords, n, S, ld, nb,
                     P, npatch);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

template <int R>
cs_status launch_build(const double* coords, int64_t n, uint64_t* S, int64_t ld, hipStream_t st) {
  const int64_t nb = ceil_div(n, 64);
  const int64_t P = ceil_div(nb, kPatch), npatch = P * (P + 1) / 2;
  if (kRowBlocks<R> > 1 && npatch >= 8)
    return launch_build_rb<R, kRowBlocks<R>>(coords, n, S, ld, nb, P, npatch, st);
  return launch_build_rb<R, 1>(coords, n, S, ld, nb, P, npatch, st);
}

}  // namespace

cs_status launch_causal_matrix(int region, const double* coords, int64_t n, uint64_t* bits,
                               int64_t ld, hipStream_t st) {
  switch (region) {
    case CS_MINK2_DIAMOND: return launch_build<CS_MINK2_DIAMOND>(coords, n, bits, ld, st);
    case CS_MINK4_DIAMOND: return launch_build<CS_MINK4_DIAMOND>(coords, n, bits, ld, st);
    case CS_DS4_SLAB: return launch_build<CS_DS4_SLAB>(coords, n, bits, ld, st);
    case CS_DS2_SLAB: return launch_build<CS_DS2_SLAB>(coords, n, bits, ld, st);
    case CS_MINK3_DIAMOND: return launch_build<CS_MINK3_DIAMOND>(coords, n, bits, ld, st);
    default: return CS_ERR_UNSUPPORTED;
  }
}

cs_status launch_build_batch(bool small, const uint32_t* uv, const BatchInst* inst,
                             const uint32_t* items, int64_t nitems, uint64_t* bits, hipStream_t st) {
  if (nitems <= 0) return CS_OK;
  if (nitems % kBatchQueues != 0) return CS_ERR_INVALID_ARG;
  auto go = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)nitems), dim3(64 * waves), 0, st, uv, inst, items, nitems,
                       bits);
  };
  if (small) go(k_build_batch<(int)kSmallN>, kBuildWaves<(int)kSmallN>);
  else go(k_build_batch<(int)kBatchMaxN>, kBuildWaves<(int)kBatchMaxN>);
  CS_LAUNCH_CHECK();
  return CS_OK;
}

}  // namespace cs
