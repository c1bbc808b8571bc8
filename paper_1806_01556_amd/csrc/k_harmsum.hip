// Harmonic summing with threshold detection and candidate compaction
// (Section 2.2, Algorithm 1), all harmonic planes at once without storing
// them (the MultipleHP organisation of Section 2.2).
//
//   HP_1(i, j) = FOP(i, j)
//   HP_k(i, j) = HP_{k-1}(i, j) + FOP(trunc(i/k), floor(j/k)),  k = 2..NH
//   a cell with HP_k(i, j) > TA(k, i) is appended to list k.
//
// Sums are FP32 in k order (no reassociation, no contraction: there are only
// additions), so every kernel here is bit-identical to a sequential FP32 sum.
// In the stretch-map kernels each thread owns 4 adjacent columns j0..j0+3;
// for k >= 2 those columns read at most two adjacent source columns
// (floor(j/k) spans <= 2 values).  The kernels of the other index maps
// interleave a thread's columns across the wave instead (see there).

#include <algorithm>

#include "fdas_internal.h"

namespace fdas {
namespace {

constexpr int HS_THREADS = 256;

// ---------------------------------------------------------------------------
// Any row count, and the two other index maps (plan option hsum_index).  A
// pulsar whose fundamental sits at (z, r) has its m-th harmonic at (m z, m r).
//
// All three work in two phases, as the 85-row kernel below does.  Phase 1 gives
// a thread four columns and a segment of the rows, and only notes which rows
// hold a cell above threshold: the maximum of a row's four sums is compared once
// per plane, and one bit per row is kept.  Phase 2 (k_emit_map) gives every
// noted (columns, row) to a lane, forms its sums again from memory in the same
// order and appends the candidates.  Appending inside phase 1 made a row cost
// some 20 vector instructions per plane whether it had a hit or not, and left a
// tile near a strong pulsar waiting for 85 rows of atomics one after another:
// 244 us for the fundamental-anchored sum of 20,003 bins, 0.93 ms of 2^22.
//
// The row segments (blockIdx.y) fill the chip where the columns alone do not:
// 256 columns make a wave, so n below about 3072 waves x 256 = 786,432 bins is
// split, up to 8 ways.  The highest-anchored map, whose rows take longest, is split
// four ways from 2^18 to 2^20 bins: 512 to 1024 workgroups of whole columns are two or
// three to a compute unit, and the time is that of the units with one more (2^19 bins
// 272 -> 212 us, 235 before there were segments; 400,000 224 -> 173, 2^20 465 ->
// 388).  A launch covers at most 96 rows (the bits of an entry).

constexpr int XT = 4 * HS_THREADS;
constexpr int kRowsPerPass = 96;
constexpr int kSplitBins = 786432;
constexpr int kMaxSegs = 8;
constexpr int kHighSegs = 4;
constexpr int kHighSplitLo = 1 << 18, kHighSplitHi = 1 << 20;
// entries past those of ceil(n / 4) threads: the last tile's and block's hold fewer than four columns each
constexpr int kHitSlack = kMaxSegs * (kStrideHigh + HS_THREADS);

// Columns of a thread's group: c0 + STRIDE a, a = 0..3.
constexpr int kStrideFund = HS_THREADS;  // a wave's load covers 64 columns at stride m
// 840 = lcm(1..8): rho(p (j + 840 a), q) = rho(p j, q) + 840 a p / q, so the
// four columns' source offsets differ by constants and one offset per fraction
// serves them (kStrideHigh)
static_assert(kStrideHigh == 840 && HS_THREADS == 256, "harmsum_high_tiles counts 256 groups of 840 to a block");

// rows [r0, r1) of this block: segment blockIdx.y of the launch's [rbase, rend)
__device__ __forceinline__ void row_segment(int rbase, int rend, int& r0, int& r1) {
  const int len = rend - rbase;
  r0 = rbase + (int)((int64_t)len * blockIdx.y / gridDim.y);
  r1 = rbase + (int)((int64_t)len * (blockIdx.y + 1) / gridDim.y);
}

struct RowMask {
  unsigned w[3] = {0u, 0u, 0u};
  // bit is uniform: the branches are scalar
  __device__ __forceinline__ void note(bool hit, int bit) {
    const unsigned v = hit ? 1u << (bit & 31) : 0u;
    if (bit < 32)
      w[0] |= v;
    else if (bit < 64)
      w[1] |= v;
    else
      w[2] |= v;
  }
};

// Append {c0, mask} of the threads with hits to the list (at most `cap` entries;
// the launch has checked that every thread's would fit).
__device__ __forceinline__ void flush_mask(const RowMask& mk, int c0, int4* __restrict__ hitrows, int cap,
                                           int32_t* __restrict__ hit_count) {
  const bool any = (mk.w[0] | mk.w[1] | mk.w[2]) != 0u;
  const unsigned long long b = __ballot(any);
  if (b == 0ull) return;  // uniform
  const int lead = (int)__builtin_ctzll(b);
  int base = 0;
  if ((int)(threadIdx.x & 63) == lead) base = atomicAdd(hit_count, __popcll(b));
  base = __shfl(base, lead);
  if (any) {
    const int pos =
        base + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
    if ((unsigned)pos < (unsigned)cap) hitrows[pos] = make_int4(c0, (int)mk.w[0], (int)mk.w[1], (int)mk.w[2]);
  }
}

__device__ __forceinline__ float max4(const float (&v)[4]) { return fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])); }

// Stretch map, any row count: four adjacent columns; a source value of harmonic
// k is fetched once per change of trunc(i/k) and kept across the k rows sharing
// it.
template <int NH>
__global__ __launch_bounds__(HS_THREADS) void k_detect_stretch(const float* __restrict__ fop, int64_t ld, int n,
                                                               int z_max, int rbase, int rend,
                                                               const int* __restrict__,
                                                               const float* __restrict__ ta,
                                                               int4* __restrict__ hitrows, int hit_cap,
                                                               int32_t* __restrict__ hit_count) {
  const int64_t g = (int64_t)blockIdx.x * HS_THREADS + threadIdx.x;
  const int rows = 2 * z_max + 1;
  int r0, r1;
  row_segment(rbase, rend, r0, r1);
  const int j0 = (int)min((int64_t)n - 1, g * 4) / 4 * 4;
  int lo[NH + 1], hi[NH + 1];
  bool selhi[NH + 1][4];
#pragma unroll
  for (int m = 2; m <= NH; ++m) {
    lo[m] = j0 / m;
    hi[m] = min(lo[m] + 1, n - 1);
#pragma unroll
    for (int a = 0; a < 4; ++a) selhi[m][a] = ((j0 + a) / m) != lo[m];
  }
  float cache[NH + 1][4];
  RowMask mk;
  for (int r = r0; r < r1; ++r) {
    const int i = r - z_max;
    // ld >= n and ld % 4 == 0: the last group's read stays inside the row, and
    // phase 2 does not emit columns past n - 1
    const float4 q = *reinterpret_cast<const float4*>(fop + (size_t)r * ld + j0);
    float hp[4] = {q.x, q.y, q.z, q.w};
    bool hit = max4(hp) > ta[r];
#pragma unroll
    for (int m = 2; m <= NH; ++m) {
      const int si = i / m;  // C division: truncation toward zero
      if (r == r0 || si != (i - 1) / m) {
        const float* src = fop + (size_t)(si + z_max) * ld;
        const float vl = src[lo[m]];
        const float vh = src[hi[m]];
#pragma unroll
        for (int a = 0; a < 4; ++a) cache[m][a] = selhi[m][a] ? vh : vl;
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) hp[a] = hp[a] + cache[m][a];
      hit = hit || max4(hp) > ta[(m - 1) * rows + r];
    }
    mk.note(hit, r - rbase);
  }
  if (g * 4 >= n) mk = RowMask();
  flush_mask(mk, j0, hitrows, hit_cap, hit_count);
}

// Raw buffer resource over part of one FOP row: loads at byte offsets >=
// bytes read 0 (the hardware range check), so columns past n - 1 need no
// compare.  The resource starts at the first column a workgroup reads, so
// offsets stay below 64 KB whatever n is.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const float* base, int64_t cols_left) {
  const uint32_t bytes = cols_left <= 0 ? 0u : (cols_left >= 16384 ? 65536u : (uint32_t)cols_left * 4u);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ float row_load(__amdgpu_buffer_rsrc_t rs, int lane_off, int const_off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, lane_off, const_off, 0));
}

// Fundamental-anchored: HP_k(i, j) = HP_{k-1}(i, j) + FOP(k i, k j), a term
// being 0 where (k i, k j) is outside the plane.  Cumulative in k.  Row i has
// the terms m <= z_max / |i|; rows are walked in groups of equal term count MV,
// R rows at a time, so that a wave always has about 28 loads in flight (half of
// the rows have the fundamental only).  Planes past MV hold the same sum: it is
// compared with the smallest of their thresholds.  Bound by the lines it moves from
// beyond L2: 2.75 planes (3.9 GB of 2^22 bins) at 5.4 TB/s without sharing.
//
// Row i0 + r of [a, b], clamped to b (a repeated row sets its bit again).
template <int NH, int MV, int R>
__device__ __forceinline__ void fund_rows(const float* __restrict__ fop, int64_t ld, int n, int z_max, int64_t t0,
                                          int a0, int b0, const float* __restrict__ s_ta, int rbase, RowMask& mk) {
  const int t = (int)threadIdx.x;
  for (int i0 = a0; i0 <= b0; i0 += R) {
    float v[R][MV][4];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int i = min(i0 + q, b0);
#pragma unroll
      for (int m = 1; m <= MV; ++m) {
        // harmonic m of the tile starting at column t0 reads columns m t0 + m (t + 256 a)
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(fop + (size_t)(m * i + z_max) * ld + m * t0, (int64_t)n - m * t0);
#pragma unroll
        for (int a = 0; a < 4; ++a) v[q][m - 1][a] = row_load(rs, 4 * m * t, 4 * m * kStrideFund * a);
      }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = min(i0 + q, b0) + z_max;
      const float* th = s_ta + 8 * r;
      float hp[4];
      bool hit = false;
#pragma unroll
      for (int m = 1; m <= MV; ++m) {
#pragma unroll
        for (int a = 0; a < 4; ++a) hp[a] = m == 1 ? v[q][0][a] : hp[a] + v[q][m - 1][a];
        hit = hit || max4(hp) > th[m - 1];
      }
      mk.note(hit, r - rbase);
    }
  }
}

template <int NH, int MV>
__device__ __forceinline__ void fund_groups(const float* __restrict__ fop, int64_t ld, int n, int z_max, int64_t t0,
                                            int i0, int i1, const float* __restrict__ s_ta, int rbase, RowMask& mk) {
  constexpr int R = MV == 1 ? 7 : MV == 2 ? 4 : MV <= 4 ? 2 : 1;
  // |i| in [lo, hi] has MV terms (row 0 all of them)
  const int hi = z_max / MV, lo = MV == NH ? 0 : z_max / (MV + 1) + 1;
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    int a = side ? lo : -hi, b = side ? hi : -lo;
    if (MV == NH) {
      if (side) break;
      b = hi;
    }
    a = max(a, i0);
    b = min(b, i1);
    if (a <= b) fund_rows<NH, MV, R>(fop, ld, n, z_max, t0, a, b, s_ta, rbase, mk);
  }
  if constexpr (MV < NH) fund_groups<NH, MV + 1>(fop, ld, n, z_max, t0, i0, i1, s_ta, rbase, mk);
}

// All rows of a long spectrum, one row step for the two signs of a node: rows +-i
// with their MV terms, and with CH = 2 rows +-c0, +-c1 (one term each, equal where
// only one is wanted: a repeated row sets its bit again).
template <int MV, int CH>
__device__ __forceinline__ void fund_node(const float* __restrict__ fop, int64_t ld, int n, int z_max, int64_t t0,
                                          int i, int c0, int c1, const float* __restrict__ s_ta, RowMask& mk) {
  const int t = (int)threadIdx.x;
  float v[2][MV][4], w[2][CH + 1][4];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
#pragma unroll
    for (int m = 1; m <= MV; ++m) {
      const int row = z_max + (g ? -m * i : m * i);
      const __amdgpu_buffer_rsrc_t rs = row_rsrc(fop + (size_t)row * ld + m * t0, (int64_t)n - m * t0);
#pragma unroll
      for (int a = 0; a < 4; ++a) v[g][m - 1][a] = row_load(rs, 4 * m * t, 4 * m * kStrideFund * a);
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int row = z_max + (g ? -1 : 1) * (c ? c1 : c0);
      const __amdgpu_buffer_rsrc_t rs = row_rsrc(fop + (size_t)row * ld + t0, (int64_t)n - t0);
#pragma unroll
      for (int a = 0; a < 4; ++a) w[g][c][a] = row_load(rs, 4 * t, 4 * kStrideFund * a);
    }
  }
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int r = z_max + (g ? -i : i);
    float hp[4];
    bool hit = false;
#pragma unroll
    for (int m = 1; m <= MV; ++m) {
#pragma unroll
      for (int a = 0; a < 4; ++a) hp[a] = m == 1 ? v[g][0][a] : hp[a] + v[g][m - 1][a];
      hit = hit || max4(hp) > s_ta[8 * r + m - 1];
    }
    mk.note(hit, r);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int rc = z_max + (g ? -1 : 1) * (c ? c1 : c0);
      mk.note(max4(w[g][c]) > s_ta[8 * rc], rc);
    }
  }
}

template <int NH, int MV>
__device__ __forceinline__ void fund_visit(const float* __restrict__ fop, int64_t ld, int n, int z_max, int64_t t0,
                                           int mv, int i, int c0, int c1, const float* __restrict__ s_ta, RowMask& mk) {
  if (mv == MV) {
    if (c0 == 0) {
      fund_node<MV, 0>(fop, ld, n, z_max, t0, i, 0, 0, s_ta, mk);
      return;
    }
    // c0 > z_max / 2 and i = c0 / 2: more than four terms cannot be here unless z_max < 10
    fund_node<MV, 2>(fop, ld, n, z_max, t0, i, c0, c1, s_ta, mk);
    return;
  }
  if constexpr (MV < NH) fund_visit<NH, MV + 1>(fop, ld, n, z_max, t0, mv, i, c0, c1, s_ta, mk);
}

// The row |i| = 2 i' (or 2 i' + 1) follows its half i' at once: rows 1 .. L = z_max / 2
// (two terms and more) in preorder of the binary tree i -> 2 i, 2 i + 1, each with
// those of its children that have one term.  The lines that a tile reads as term m
// of row i are those that the tile at twice the column reads as term m / 2 of row
// 2 i, and the tile order runs the two together on one XCD, so part of them is
// still in its L2: 3.4 GB from beyond it for 2^22 bins, 3.75 GB with the rows in
// groups of equal term count (2.4 GB, 1.7 planes, if the tiles kept step).
// Measured, whole call: 2^22 bins 720 -> 671 us, 3,000,001 545 -> 514, 1,500,001
// 315 -> 288, 4,000,001 with z_max 17 333 -> 289; 1,000,003 242 -> 251, so up to
// 2^20 bins, where one round of workgroups holds all tiles, the groups stay.
constexpr int kTreeAboveN = 1 << 20;
static_assert(kTreeAboveN >= kSplitBins, "a launch above it has one row segment");
template <int NH>
__device__ __forceinline__ void fund_tree(const float* __restrict__ fop, int64_t ld, int n, int z_max, int64_t t0,
                                          const float* __restrict__ s_ta, RowMask& mk) {
  const int L = z_max / 2;
  fund_node<NH, 0>(fop, ld, n, z_max, t0, 0, 0, 0, s_ta, mk);
  int i = 1;
#pragma unroll 1
  while (i > 0) {
    int c0 = 0, c1 = 0;
    if (2 * i + 1 > L) {
      c0 = 2 * i > L ? 2 * i : 2 * i + 1;
      c1 = min(2 * i + 1, z_max);
    }
    fund_visit<NH, 2>(fop, ld, n, z_max, t0, min(NH, z_max / i), i, c0, c1, s_ta, mk);
    if (2 * i <= L) {
      i = 2 * i;
    } else {  // the next sibling of the node or of the nearest ancestor that has one
      while (i > 0 && ((i & 1) || i + 1 > L)) i >>= 1;
      if (i > 0) i += 1;
    }
  }
}

template <int NH>
__global__ __launch_bounds__(HS_THREADS, 4) void k_detect_fund(const float* __restrict__ fop, int64_t ld, int n,
                                                               int z_max, int rbase, int rend,
                                                               const int* __restrict__ tile_of_block,
                                                               const float* __restrict__ ta,
                                                               int4* __restrict__ hitrows, int hit_cap,
                                                               int32_t* __restrict__ hit_count) {
  __shared__ float s_ta[129 * 8];  // [row][m - 1]; the last term's entry is the smallest of the planes from there on
  const int rows = 2 * z_max + 1;
  for (int r = threadIdx.x; r < rows; r += HS_THREADS) {
    const int i = r < z_max ? z_max - r : r - z_max;
    const int mv = i == 0 ? NH : min(NH, z_max / i);
    float low = ta[(NH - 1) * rows + r];
    for (int m = NH - 1; m >= mv; --m) low = fminf(low, ta[(m - 1) * rows + r]);
    for (int m = 1; m < mv; ++m) s_ta[r * 8 + m - 1] = ta[(m - 1) * rows + r];
    s_ta[r * 8 + mv - 1] = low;
  }
  __syncthreads();
  const int tile = tile_of_block ? tile_of_block[blockIdx.x] : (int)blockIdx.x;
  if (tile < 0 || (int64_t)tile * XT >= n) return;  // uniform
  int r0, r1;
  row_segment(rbase, rend, r0, r1);
  const int64_t t0 = (int64_t)tile * XT;
  RowMask mk;
  // a segment or a pass holds a contiguous part of the rows, where few doubles meet
  bool tree = false;
  if constexpr (NH > 1) tree = n > kTreeAboveN && rend - rbase == rows && z_max >= 2;
  if (tree) {
    if constexpr (NH > 1) fund_tree<NH>(fop, ld, n, z_max, t0, s_ta, mk);
  } else {
    fund_groups<NH, 1>(fop, ld, n, z_max, t0, r0 - z_max, r1 - 1 - z_max, s_ta, rbase, mk);
  }
  const int c0 = (int)t0 + (int)threadIdx.x;
  if (c0 >= n) mk = RowMask();
  flush_mask(mk, c0, hitrows, hit_cap, hit_count);
}

// Highest-harmonic-anchored: HP_k(i, j) = sum_{m=1..k} FOP(rho(m i, k), rho(m j, k)),
// summed in m order, rho = rounding to the nearest integer with halves away
// from zero.  Every index is inside the plane; the planes are not cumulative.
//
// rho(m x, k) depends on m/k only, so the terms of all k <= NH read one value
// per reduced fraction p/q (q <= NH): 22 fractions for NH = 8.  Each
// fraction's four values stay in registers while its source row rho(p i, q)
// is unchanged (it changes on about p/q of the rows).

__host__ __device__ constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }

// reduced fractions p/q, 1 <= p <= q <= nh, ordered by q, then p
__host__ __device__ constexpr int frac_count(int nh) {
  int c = 0;
  for (int q = 1; q <= nh; ++q)
    for (int p = 1; p <= q; ++p) c += gcd_c(p, q) == 1 ? 1 : 0;
  return c;
}
__host__ __device__ constexpr int frac_index(int m, int k) {
  const int g = gcd_c(m, k), p = m / g, q = k / g;
  int idx = frac_count(q - 1);
  for (int pp = 1; pp < p; ++pp) idx += gcd_c(pp, q) == 1 ? 1 : 0;
  return idx;
}
__host__ __device__ constexpr int frac_num(int idx) {
  for (int q = 1;; ++q)
    for (int p = 1; p <= q; ++p)
      if (gcd_c(p, q) == 1 && idx-- == 0) return p;
}
__host__ __device__ constexpr int frac_den(int idx) {
  for (int q = 1;; ++q)
    for (int p = 1; p <= q; ++p)
      if (gcd_c(p, q) == 1 && idx-- == 0) return q;
}
static_assert(frac_count(8) == 22 && frac_index(4, 8) == 1 && frac_num(5) == 3 && frac_den(5) == 4, "fractions");

// rho(p |i|, q) of every fraction for |i| <= 65, and the fractions whose value
// differs between |i| and |i| + 1: looked up with scalar loads, where 22
// divisions a row would outweigh the row's sums.
struct HighTable {
  unsigned row[66][8];   // fraction f in byte f % 4 of word f / 4
  unsigned changes[65];  // bit f: rho at |i| + 1 is not rho at |i|
};
constexpr HighTable make_high_table() {
  HighTable t{};
  for (int f = 0; f < frac_count(8); ++f) {
    const unsigned p = (unsigned)frac_num(f), q = (unsigned)frac_den(f);
    unsigned last = 0;
    for (unsigned x = 0; x < 66; ++x) {
      const unsigned s = (2u * p * x + q) / (2u * q);
      t.row[x][f / 4] |= s << (8 * (f % 4));
      if (x > 0 && s != last) t.changes[x - 1] |= 1u << f;
      last = s;
    }
  }
  return t;
}
constexpr HighTable kHighTableValue = make_high_table();
__constant__ const HighTable kHighTable = kHighTableValue;

template <int NH>
struct HighState {
  float val[frac_count(NH)][4];
  int off[frac_count(NH)];  // byte offset of the lane's first source column from the workgroup's
};

// rho(P x, Q) for 0 <= x < 2^31 (n <= 2^30): with x = Q u + w (w < Q), P x / Q =
// P u + P w / Q, so the rounding only involves P w < P Q.
template <int P, int Q>
__device__ __forceinline__ int rho_pos(int x) {
  const unsigned u = (unsigned)x / Q, w = (unsigned)x - u * Q;
  return (int)(P * u + (2u * P * w + Q) / (2u * Q));
}

// source row of fraction P/Q for output row i
template <int P, int Q>
__device__ __forceinline__ int high_row(int i, int z_max) {
  const int s = rho_pos<P, Q>(i < 0 ? -i : i);
  return (i < 0 ? -s : s) + z_max;
}

template <int NH, int F>
__device__ __forceinline__ void hi_offsets(HighState<NH>& st, int d) {
  if constexpr (F < frac_count(NH)) {
    st.off[F] = 4 * rho_pos<frac_num(F), frac_den(F)>(d);
    hi_offsets<NH, F + 1>(st, d);
  }
}

// Load the fractions of output row i whose bit is set in `mask` (uniform), F and
// the ones after it; c0 = the workgroup's first column, a multiple of 4 x 840.
template <int NH, int F>
__device__ __forceinline__ void hi_refresh(HighState<NH>& st, const float* __restrict__ fop, int64_t ld, int n,
                                           int z_max, int i, unsigned mask, const unsigned (&srows)[8], int c0) {
  if constexpr (F < frac_count(NH)) {
    if ((mask >> F) & 1u) {
      constexpr int P = frac_num(F), Q = frac_den(F);
      const int sr = (int)((srows[F / 4] >> (8 * (F % 4))) & 255u);
      const int64_t s0 = (int64_t)(c0 / Q) * P;
      const __amdgpu_buffer_rsrc_t rs =
          row_rsrc(fop + (size_t)((i < 0 ? -sr : sr) + z_max) * ld + s0, (int64_t)n - s0);
#pragma unroll
      for (int a = 0; a < 4; ++a) st.val[F][a] = row_load(rs, st.off[F], 4 * (kStrideHigh * a / Q * P));
    }
    hi_refresh<NH, F + 1>(st, fop, ld, n, z_max, i, mask, srows, c0);
  }
}

// HP_K = terms m = 1..K in m order
template <int NH, int K, int M>
__device__ __forceinline__ void hi_sum(const float (&val)[frac_count(NH)][4], float (&hp)[4]) {
  if constexpr (M <= K) {
    constexpr int FI = frac_index(M, K);
#pragma unroll
    for (int a = 0; a < 4; ++a) hp[a] = M == 1 ? val[FI][a] : hp[a] + val[FI][a];
    hi_sum<NH, K, M + 1>(val, hp);
  }
}

template <int NH, int K>
__device__ __forceinline__ bool hi_hit(const HighState<NH>& st, int r, int rows, const float* __restrict__ ta) {
  float hp[4];
  hi_sum<NH, K, 1>(st.val, hp);
  const bool hit = max4(hp) > ta[(K - 1) * rows + r];
  if constexpr (K < NH)
    return hit | hi_hit<NH, K + 1>(st, r, rows, ta);
  else
    return hit;
}

// Threads run over groups of four columns 840 apart, 840 groups to a block of
// 3360 columns.  Columns past n - 1 read zeros (or other columns, where
// rho(p j, q) < n) and are never emitted.  Bound by the lines it moves from
// beyond L2: sum over the fractions of (p/q)^2 = 7.5 planes (a column's sources at
// other fractions lie in other tiles, read at other rows).  Measured on 2^22
// bins 2.06 ms (5.2 TB/s of those lines), 1,500,001 bins 0.72 ms (0.06 ms more
// without the chunks, 0.12 ms more in ascending order); 2.17-2.23 and 0.85-0.97 ms
// with candidates appended row by row and offsets formed by division per load.
template <int NH>
__global__ __launch_bounds__(HS_THREADS, 3) void k_detect_high(const float* __restrict__ fop, int64_t ld, int n,
                                                               int z_max, int rbase, int rend,
                                                               const int* __restrict__ tile_of_block,
                                                               const float* __restrict__ ta,
                                                               int4* __restrict__ hitrows, int hit_cap,
                                                               int32_t* __restrict__ hit_count) {
  const int rows = 2 * z_max + 1;
  const int tile = tile_of_block ? tile_of_block[blockIdx.x] : (int)blockIdx.x;
  if (tile < 0 || (int64_t)tile * HS_THREADS / kStrideHigh * (4 * kStrideHigh) >= n) return;  // uniform
  const int g0 = tile * HS_THREADS;
  const int first_blk = g0 / kStrideHigh;
  const int c0 = first_blk * 4 * kStrideHigh;  // <= n: fits
  const int g = g0 + (int)threadIdx.x;
  const int64_t col0 = (int64_t)(g / kStrideHigh) * 4 * kStrideHigh + g % kStrideHigh;
  int r0, r1;
  row_segment(rbase, rend, r0, r1);
  HighState<NH> st;
  hi_offsets<NH, 0>(st, (int)(col0 - c0));
  RowMask mk;
  for (int r = r0; r < r1; ++r) {
    const int i = r - z_max, x = i < 0 ? -i : i;
    unsigned srows[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) srows[q] = kHighTable.row[x][q];
    hi_refresh<NH, 0>(st, fop, ld, n, z_max, i, r == r0 ? ~0u : kHighTable.changes[i > 0 ? i - 1 : x], srows, c0);
    mk.note(hi_hit<NH, 1>(st, r, rows, ta), r - rbase);
  }
  if (col0 >= n) mk = RowMask();
  flush_mask(mk, (int)min(col0, (int64_t)n), hitrows, hit_cap, hit_count);
}

// Sums hk[1..NH] of row i at the four columns c0 + STRIDE a, in phase 1's order.
// Columns past n - 1 are left 0.
template <int NH, int F>
__device__ __forceinline__ void high_values(float (&val)[frac_count(NH)][4], const float* __restrict__ fop, int64_t ld,
                                            int n, int z_max, int i, int c0) {
  if constexpr (F < frac_count(NH)) {
    constexpr int P = frac_num(F), Q = frac_den(F);
    const float* src = fop + (size_t)high_row<P, Q>(i, z_max) * ld;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int c = c0 + kStrideHigh * a;
      val[F][a] = c < n ? src[rho_pos<P, Q>(c)] : 0.0f;
    }
    high_values<NH, F + 1>(val, fop, ld, n, z_max, i, c0);
  }
}

template <int NH, int K>
__device__ __forceinline__ void high_planes(const float (&val)[frac_count(NH)][4], float (&hk)[NH + 1][4]) {
  if constexpr (K <= NH) {
    hi_sum<NH, K, 1>(val, hk[K]);
    high_planes<NH, K + 1>(val, hk);
  }
}

template <int MAP, int NH>
__device__ __forceinline__ void map_sums(float (&hk)[NH + 1][4], const float* __restrict__ fop, int64_t ld, int n,
                                         int z_max, int i, int c0) {
  if constexpr (MAP == FDAS_HSUM_HIGHEST) {
    float val[frac_count(NH)][4];
    high_values<NH, 0>(val, fop, ld, n, z_max, i, c0);
    high_planes<NH, 1>(val, hk);
  } else {
    constexpr int STRIDE = MAP == FDAS_HSUM_FUNDAMENTAL ? kStrideFund : 1;
    float v[NH + 1][4];
#pragma unroll
    for (int m = 1; m <= NH; ++m) {
      const int si = MAP == FDAS_HSUM_FUNDAMENTAL ? m * i : i / m;
      const bool row_in = si >= -z_max && si <= z_max;
      const float* src = fop + (size_t)((row_in ? si : 0) + z_max) * ld;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int c = c0 + STRIDE * a;
        const int64_t sc = MAP == FDAS_HSUM_FUNDAMENTAL ? (int64_t)m * c : (int64_t)(c / m);
        v[m][a] = row_in && c < n && sc < n ? src[sc] : 0.0f;
      }
    }
#pragma unroll
    for (int m = 1; m <= NH; ++m)
#pragma unroll
      for (int a = 0; a < 4; ++a) hk[m][a] = m == 1 ? v[1][a] : hk[m - 1][a] + v[m][a];
  }
}

// ---------------------------------------------------------------------------
// Fast path for a compile-time row count (2*Z+1 rows), in two phases.
//
// Phase 1 (k_harmsum_z): each thread owns 4 adjacent columns and walks all
// rows.  Rows and harmonics are unrolled at compile time (template
// recursion), so every source row and register slot is a constant.  Loads are
// issued DEPTH rows ahead of their use: the unstretched row r+DEPTH, and for
// each k >= 2 the source row trunc((r+DEPTH-Z)/k) when it first appears.  A
// row costs 4*(NH-1) adds plus one max-reduction and compare per harmonic; the
// thread only records which of its rows hold a cell above threshold (a bit
// mask), and a block appends one entry {j0, mask} per thread with hits to a
// global list.
//
// Phase 2 (k_harmsum_emit): a grid-stride kernel gives every (entry, row) with
// its bit set to one thread, which re-forms that row's sums from memory in the
// same k order (bit-identical to phase 1) and appends the candidates.  Hits
// cluster around strong pulsars, so spreading them over the whole GPU keeps a
// few dense tiles from serialising the kernel.
//
// Source columns of the 4 columns j0..j0+3 (j0 = 4g) for harmonic k:
//   k = 2:        (j0/2, j0/2, j0/2+1, j0/2+1)        -- fixed pattern
//   k = 4, 8:     j0/k for all four (j0 mod k + 3 < k)
//   k = 3,5,6,7:  column a reads j0/k + 1 iff (j0 mod k) + a >= k

constexpr int DEPTH = 8;
constexpr int RING = DEPTH / 2 + 3;  // > source rows of one harmonic first used within DEPTH rows

__host__ __device__ constexpr int src_row(int r, int m, int Z) { return (r - Z) / m + Z; }  // C truncation
__host__ __device__ constexpr int slot_of(int r, int m, int Z) { return (src_row(r, m, Z) - src_row(0, m, Z)) % RING; }
// row r of a segment that begins at r0 needs harmonic m's next source row
__host__ __device__ constexpr bool starts(int r, int m, int Z, int r0) {
  return r == r0 || src_row(r, m, Z) != src_row(r - 1, m, Z);
}
__host__ __device__ constexpr bool needs_hi(int m) { return m != 4 && m != 8; }

template <int NH>
struct HsState {
  float4 ring1[DEPTH];
  float lo_ring[NH + 1][RING];
  float hi_ring[NH + 1][RING];
  float val[NH + 1][4];
  unsigned hitmask[3];
};

// loads of the stretched source rows first needed at row R
template <int Z, int NH, int R0, int R, int M>
__device__ __forceinline__ void hs_issue_m(HsState<NH>& st, const float* __restrict__ fop, int64_t ld,
                                           const int (&lo)[NH + 1]) {
  if constexpr (M <= NH) {
    if constexpr (starts(R, M, Z, R0)) {
      constexpr int S = src_row(R, M, Z);
      constexpr int SL = slot_of(R, M, Z);
      const float* src = fop + (size_t)S * ld + lo[M];
      if constexpr (M == 2) {
        const float2 q = *reinterpret_cast<const float2*>(src);  // j0/2 is even
        st.lo_ring[M][SL] = q.x;
        st.hi_ring[M][SL] = q.y;
      } else {
        st.lo_ring[M][SL] = src[0];
        if constexpr (needs_hi(M)) st.hi_ring[M][SL] = src[1];
      }
    }
    hs_issue_m<Z, NH, R0, R, M + 1>(st, fop, ld, lo);
  }
}

template <int Z, int NH, int R0, int R1, int R>
__device__ __forceinline__ void hs_issue(HsState<NH>& st, const float* __restrict__ fop, int64_t ld, int j0,
                                         const int (&lo)[NH + 1]) {
  if constexpr (R < R1) {
    st.ring1[R % DEPTH] = *reinterpret_cast<const float4*>(fop + (size_t)R * ld + j0);
    hs_issue_m<Z, NH, R0, R, 2>(st, fop, ld, lo);
  }
}

template <int Z, int NH, int R0, int R, int M>
__device__ __forceinline__ void hs_harm(HsState<NH>& st, float (&hp)[4], bool& hit, const int (&rmod)[NH + 1],
                                        const float* __restrict__ s_ta) {
  if constexpr (M <= NH) {
    if constexpr (starts(R, M, Z, R0)) {
      constexpr int SL = slot_of(R, M, Z);
      const float vl = st.lo_ring[M][SL];
      if constexpr (M == 2) {
        const float vh = st.hi_ring[M][SL];
        st.val[M][0] = vl;
        st.val[M][1] = vl;
        st.val[M][2] = vh;
        st.val[M][3] = vh;
      } else if constexpr (!needs_hi(M)) {
#pragma unroll
        for (int a = 0; a < 4; ++a) st.val[M][a] = vl;
      } else {
        const float vh = st.hi_ring[M][SL];
        st.val[M][0] = vl;
#pragma unroll
        for (int a = 1; a < 4; ++a) st.val[M][a] = (rmod[M] + a >= M) ? vh : vl;
      }
    }
    const float t = s_ta[R * 8 + (M - 1)];
#pragma unroll
    for (int a = 0; a < 4; ++a) hp[a] = hp[a] + st.val[M][a];
    // one compare per harmonic: any of the 4 columns above threshold (NaN never is)
    hit = hit || fmaxf(fmaxf(hp[0], hp[1]), fmaxf(hp[2], hp[3])) > t;
    hs_harm<Z, NH, R0, R, M + 1>(st, hp, hit, rmod, s_ta);
  }
}

template <int Z, int NH, int R0, int R1, int R>
__device__ __forceinline__ void hs_rows(HsState<NH>& st, const float* __restrict__ fop, int64_t ld, int j0,
                                        const int (&lo)[NH + 1], const int (&rmod)[NH + 1],
                                        const float* __restrict__ s_ta) {
  // take row R out of its ring slot before the slot is refilled with row R + DEPTH
  const float4 v = st.ring1[R % DEPTH];
  hs_issue<Z, NH, R0, R1, R + DEPTH>(st, fop, ld, j0, lo);
  float hp[4] = {v.x, v.y, v.z, v.w};
  bool hit = fmaxf(fmaxf(hp[0], hp[1]), fmaxf(hp[2], hp[3])) > s_ta[R * 8];
  hs_harm<Z, NH, R0, R, 2>(st, hp, hit, rmod, s_ta);
  st.hitmask[R / 32] |= hit ? (1u << (R % 32)) : 0u;
  // Keep the software pipeline as written: the row's sums are consumed here
  // (an empty asm that reads and rewrites the hit word), and no instruction
  // crosses the row boundary.
  __asm__ volatile("" : "+v"(st.hitmask[R / 32]));
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (R + 1 < R1) hs_rows<Z, NH, R0, R1, R + 1>(st, fop, ld, j0, lo, rmod, s_ta);
}

template <int Z, int NH, int R0, int R1, int R>
__device__ __forceinline__ void hs_prologue(HsState<NH>& st, const float* __restrict__ fop, int64_t ld, int j0,
                                            const int (&lo)[NH + 1]) {
  hs_issue<Z, NH, R0, R1, R>(st, fop, ld, j0, lo);
  if constexpr (R + 1 < R0 + DEPTH) hs_prologue<Z, NH, R0, R1, R + 1>(st, fop, ld, j0, lo);
}

// Phase 1 for one thread: rows [R0, R1) of columns j0..j0+3 of a plane with n
// columns.  Returns the bit mask of rows holding a cell above threshold (3 words).
template <int Z, int NH, int R0 = 0, int R1 = 2 * Z + 1>
__device__ __forceinline__ void hs_phase1_thread(const float* __restrict__ fop, int64_t ld, int j0,
                                                 const float* __restrict__ s_ta, unsigned (&mask)[3]) {
  int lo[NH + 1], rmod[NH + 1];
#pragma unroll
  for (int m = 0; m <= NH; ++m) {
    lo[m] = m >= 2 ? j0 / m : 0;
    rmod[m] = m >= 2 ? j0 - lo[m] * m : 0;
  }
  HsState<NH> st;
  st.hitmask[0] = st.hitmask[1] = st.hitmask[2] = 0u;
  hs_prologue<Z, NH, R0, R1, R0>(st, fop, ld, j0, lo);
  hs_rows<Z, NH, R0, R1, R0>(st, fop, ld, j0, lo, rmod, s_ta);
  mask[0] = st.hitmask[0];
  mask[1] = st.hitmask[1];
  mask[2] = st.hitmask[2];
}

template <int Z, int NH>
__device__ __forceinline__ void hs_load_ta(const float* __restrict__ ta, float* __restrict__ s_ta) {
  constexpr int ROWS = 2 * Z + 1;
  for (int e = threadIdx.x; e < ROWS * 8; e += blockDim.x) {
    const int r = e / 8, m = e % 8;
    s_ta[e] = m < NH ? ta[m * ROWS + r] : 0.0f;
  }
}

// Append this block's entries {j0, mask words} to the global hit-row list.
__device__ __forceinline__ void hs_flush_entries(const int4* __restrict__ s_ent, int cnt, int* s_base,
                                                 int4* __restrict__ hitrows, int32_t* __restrict__ hitrow_count) {
  if (cnt == 0) return;  // uniform
  if (threadIdx.x == 0) *s_base = atomicAdd(hitrow_count, cnt);
  __syncthreads();
  if (threadIdx.x < cnt) hitrows[*s_base + threadIdx.x] = s_ent[threadIdx.x];
}

// Phase 1 over all columns [0, n) in groups of 4 (the last group may be
// partial).  The 16-byte read of the last group stays inside the row because
// ld >= n and ld % 4 == 0; a source column j/k + 1 read for k >= 2 is at most
// (n-1)/2 + 1 <= ld - 1.  Values read beyond column n - 1 only reach columns
// >= n, which phase 2 never emits.
// SEGS > 1: blockIdx.y is one of SEGS segments of the rows.  A thread walks its
// rows one memory latency after another (8 rows ahead), so a spectrum too short
// to fill the chip takes the time of 85 rows whatever its length: up to 2^18
// bins (1024 waves) the rows go to four workgroups.  Measured phase 1: 16,384
// bins 18.8 -> 8.0 us, 200,003 bins 20.4 -> 18.8 us; both phases at 2^18 bins 28.7 ->
// 27.9 us.
constexpr int kSegRows = 4;
constexpr int kSegMaxN = 1 << 18;
template <int Z, int NH, int TH = HS_THREADS, int SEGS = 1>
__global__ __launch_bounds__(TH) void k_harmsum_z(const float* __restrict__ fop, int64_t ld, int n,
                                                          const int* __restrict__ tile_of_block,
                                                          const float* __restrict__ ta, int4* __restrict__ hitrows,
                                                          int32_t* __restrict__ hitrow_count) {
  constexpr int ROWS = 2 * Z + 1;
  static_assert(ROWS <= 96, "hit mask holds 96 rows");
  __shared__ float s_ta[ROWS * 8];  // [row][k-1]
  __shared__ int4 s_ent[TH];
  __shared__ int s_nent, s_base;
  hs_load_ta<Z, NH>(ta, s_ta);
  if (threadIdx.x == 0) s_nent = 0;
  __syncthreads();
  const int groups = (n + 3) / 4;
  const int tile = tile_of_block[blockIdx.x];  // -1: no tile for this block
  const int g = tile * TH + threadIdx.x;
  if (tile >= 0 && g < groups) {
    const int j0 = 4 * g;
    unsigned mask[3];
    if constexpr (SEGS == 1) {
      hs_phase1_thread<Z, NH>(fop, ld, j0, s_ta, mask);
    } else {
      static_assert(SEGS == 4, "four row segments");
      constexpr int Q1 = ROWS / 4, Q2 = ROWS / 2, Q3 = 3 * ROWS / 4;
      switch (blockIdx.y) {
        case 0: hs_phase1_thread<Z, NH, 0, Q1>(fop, ld, j0, s_ta, mask); break;
        case 1: hs_phase1_thread<Z, NH, Q1, Q2>(fop, ld, j0, s_ta, mask); break;
        case 2: hs_phase1_thread<Z, NH, Q2, Q3>(fop, ld, j0, s_ta, mask); break;
        default: hs_phase1_thread<Z, NH, Q3, ROWS>(fop, ld, j0, s_ta, mask); break;
      }
    }
    if (mask[0] | mask[1] | mask[2]) {
      const int pos = atomicAdd(&s_nent, 1);
      s_ent[pos] = make_int4(j0, (int)mask[0], (int)mask[1], (int)mask[2]);
    }
  }
  __syncthreads();
  hs_flush_entries(s_ent, s_nent, &s_base, hitrows, hitrow_count);
}

// Batch form: workgroup blk_begin + blockIdx.x belongs to the last trial whose
// block0 is <= it; its tile comes from that trial's tile order.  Entries carry
// the trial in bits 21..31 of the third mask word (rows 64..84 use bits 0..20).
template <int Z, int NH, int TH>
__global__ __launch_bounds__(TH) void k_harmsum_z_batch(const HsTrial* __restrict__ trials, int ntrials,
                                                                int blk_begin, const float* __restrict__ ta,
                                                                int4* __restrict__ hitrows,
                                                                int32_t* __restrict__ hitrow_count) {
  constexpr int ROWS = 2 * Z + 1;
  static_assert(ROWS <= 85, "the trial tag uses bits 21..31 of the third mask word");
  __shared__ float s_ta[ROWS * 8];
  __shared__ int4 s_ent[TH];
  __shared__ int s_nent, s_base;
  hs_load_ta<Z, NH>(ta, s_ta);
  if (threadIdx.x == 0) s_nent = 0;
  __syncthreads();
  const int b = blk_begin + (int)blockIdx.x;
  int lo = 0, hi = ntrials - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (trials[mid].block0 <= b) lo = mid; else hi = mid - 1;
  }
  const HsTrial tr = trials[lo];
  const int groups = (tr.n + 3) / 4;
  const int lb = b - tr.block0;
  const int tile = lb < tr.nblocks ? tr.tile_of_block[lb] : -1;
  const int g = tile * TH + threadIdx.x;
  if (tile >= 0 && g < groups) {
    const int j0 = 4 * g;
    unsigned mask[3];
    hs_phase1_thread<Z, NH>(tr.fop, tr.ld, j0, s_ta, mask);
    if (mask[0] | mask[1] | mask[2]) {
      const int pos = atomicAdd(&s_nent, 1);
      s_ent[pos] = make_int4(j0, (int)mask[0], (int)mask[1], (int)(mask[2] | ((unsigned)lo << 21)));
    }
  }
  __syncthreads();
  hs_flush_entries(s_ent, s_nent, &s_base, hitrows, hitrow_count);
}

// Phase 2 for one (entry, row): re-form the row's sums from memory in the
// same k order as phase 1 (bit-identical) and append its candidates.  Every
// column index read stays < ld (same bound as phase 1).
template <int Z, int NH>
__device__ __forceinline__ void hs_emit_row(const float* __restrict__ fop, int64_t ld, int n, int j0, int r,
                                            const float* __restrict__ ta, fdas_cand* __restrict__ cands, int cap,
                                            int32_t* __restrict__ counts) {
  constexpr int ROWS = 2 * Z + 1;
  const int i = r - Z;
  // all loads first (independent), then the sums in k order
  const float4 v = *reinterpret_cast<const float4*>(fop + (size_t)r * ld + j0);
  float src[NH + 1][4];
#pragma unroll
  for (int m = 2; m <= NH; ++m) {
    const float* rowp = fop + (size_t)(i / m + Z) * ld;
#pragma unroll
    for (int a = 0; a < 4; ++a) src[m][a] = rowp[(j0 + a) / m];
  }
  float hk[NH + 1][4];
  hk[1][0] = v.x;
  hk[1][1] = v.y;
  hk[1][2] = v.z;
  hk[1][3] = v.w;
#pragma unroll
  for (int m = 2; m <= NH; ++m)
#pragma unroll
    for (int a = 0; a < 4; ++a) hk[m][a] = hk[m - 1][a] + src[m][a];
  // reserve per plane, then write
#pragma unroll
  for (int m = 1; m <= NH; ++m) {
    const float t = ta[(m - 1) * ROWS + r];
    int c = 0;
#pragma unroll
    for (int a = 0; a < 4; ++a) c += (j0 + a < n && hk[m][a] > t) ? 1 : 0;
    if (c) {
      int slot = atomicAdd(&counts[m - 1], c);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (j0 + a < n && hk[m][a] > t) {
          if ((unsigned)slot < (unsigned)cap)
            *reinterpret_cast<int4*>(cands + (size_t)(m - 1) * cap + slot) =
                make_int4(m, i, j0 + a, __float_as_int(hk[m][a]));
          ++slot;
        }
      }
    }
  }
}

// Append the candidates of a wave: every active lane holds the sums hk[1..NH] of
// row i (threshold row r) at the columns c0 + STRIDE a.  Each plane's slots are
// reserved for the whole wave in one round of atomics: lane m - 1 reserves plane
// m, lane offsets come from ballots of the 3-bit per-lane counts.  A plan keeps
// (2 z_max + 1) n_max below 2^31, so a count cannot wrap; the unsigned compare
// still keeps any slot that is not in [0, cap) from being written.
template <int NH, int STRIDE>
__device__ __forceinline__ void hs_append_wave(const float (&hk)[NH + 1][4], int n, int rows, int c0, int i, int r,
                                               bool act, const float* __restrict__ ta, fdas_cand* __restrict__ cands,
                                               int cap, int32_t* __restrict__ counts, int lane) {
  unsigned hits = 0u;  // bit 4 * (m - 1) + a: column c0 + STRIDE a is a candidate of plane m
  int below_m[NH + 1], total[NH + 1];
  auto below = [&](unsigned long long b) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
  };
  int mine = 0;
#pragma unroll
  for (int m = 1; m <= NH; ++m) {
    int c = 0;
    const float t = act ? ta[(m - 1) * rows + r] : 0.0f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const bool h = act && c0 + STRIDE * a < n && hk[m][a] > t;
      hits |= h ? 1u << (4 * (m - 1) + a) : 0u;
      c += h ? 1 : 0;
    }
    const unsigned long long b0 = __ballot(c & 1), b1 = __ballot(c & 2), b2 = __ballot(c & 4);
    total[m] = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
    below_m[m] = below(b0) + 2 * below(b1) + 4 * below(b2);
    if (lane == m - 1) mine = total[m];
  }
  int base = 0;
  if (lane < NH && mine > 0) base = atomicAdd(&counts[lane], mine);
#pragma unroll
  for (int m = 1; m <= NH; ++m) {
    if (total[m] == 0) continue;  // uniform
    int slot = __shfl(base, m - 1) + below_m[m];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      if ((hits >> (4 * (m - 1) + a)) & 1u) {
        if ((unsigned)slot < (unsigned)cap)
          *reinterpret_cast<int4*>(cands + (size_t)(m - 1) * cap + slot) =
              make_int4(m, i, c0 + STRIDE * a, __float_as_int(hk[m][a]));
        ++slot;
      }
    }
  }
}

// Phase 2 for one wave: every active lane re-forms the sums of its row r of
// columns j0..j0+3 (same k order as phase 1, so bit-identical) and the wave
// appends the candidates of all lanes to one plane set (fop, cands, counts
// uniform across the wave).
template <int Z, int NH>
__device__ __forceinline__ void hs_emit_wave(const float* __restrict__ fop, int64_t ld, int n, int j0, int r,
                                             bool act, const float* __restrict__ ta,
                                             fdas_cand* __restrict__ cands, int cap,
                                             int32_t* __restrict__ counts, int lane) {
  const int i = r - Z;
  float hk[NH + 1][4];
  if (act) {
    const float4 v = *reinterpret_cast<const float4*>(fop + (size_t)r * ld + j0);
    float src[NH + 1][4];
#pragma unroll
    for (int m = 2; m <= NH; ++m) {
      const float* rowp = fop + (size_t)(i / m + Z) * ld;
#pragma unroll
      for (int a = 0; a < 4; ++a) src[m][a] = rowp[(j0 + a) / m];
    }
    hk[1][0] = v.x;
    hk[1][1] = v.y;
    hk[1][2] = v.z;
    hk[1][3] = v.w;
#pragma unroll
    for (int m = 2; m <= NH; ++m)
#pragma unroll
      for (int a = 0; a < 4; ++a) hk[m][a] = hk[m - 1][a] + src[m][a];
  }
  hs_append_wave<NH, 1>(hk, n, 2 * Z + 1, j0, i, r, act, ta, cands, cap, counts, lane);
}

// Position of the k-th (from 0) of the set bits of the 96-bit mask {y, z, w}, which
// has more than k.
__device__ __forceinline__ int set_bit(int k, int y, int z, int w) {
  const int c0 = __popc(y), c1 = __popc(z);
  int pos = 0;
  unsigned word = (unsigned)y;
  if (k >= c0) {
    k -= c0;
    pos = 32;
    word = (unsigned)z;
    if (k >= c1) {
      k -= c1;
      pos = 64;
      word = (unsigned)w;
    }
  }
#pragma unroll
  for (int s = 16; s > 0; s >>= 1) {
    const int c = __popc(word & ((1u << s) - 1u));
    if (k >= c) {
      k -= c;
      pos += s;
      word >>= s;
    }
  }
  return pos;
}

// The noted rows of a hit-row list (ROWS to an entry) dealt to the lanes of the
// grid's waves: work(c0, bit, act) of every set bit, a whole wave at a time (act:
// this lane has one).  While the grid has a thread for every row of every entry,
// item = entry * ROWS + row: the row is known before the entry is read and nothing
// is passed between lanes, 0.5-1.3 us less for the usual short list.  For longer ones
// a wave takes up to 32 entries at once and its lanes their set bits: as many rounds
// as 64 rows of hits, where a lane for every row, set or not, spent most of a round on
// rows without (and in segments on rows of other segments).
constexpr int kDealEntries = 32;
template <int ROWS, typename Work>
__device__ __forceinline__ void deal_rows(const int4* __restrict__ hitrows, int entries, Work work) {
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * (HS_THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = gridDim.x * (HS_THREADS / 64);
  const bool once = __builtin_expect((int64_t)entries * ROWS <= (int64_t)waves * 64, 1);  // uniform
  int G = 1;
  if (!once) G = min(kDealEntries, (int)((unsigned)(entries + waves - 1) / (unsigned)waves));
  const unsigned w = wave * 64u + lane;  // of a short list
  // one call of work, as its code is long
  // (entries and e0 + waves * G stay far below 2^31)
  for (int e0 = once ? (int)(wave * 64u / ROWS) : wave * G; e0 < entries; e0 += waves * G) {
    int4 ent = make_int4(0, 0, 0, 0);
    int e = (int)(w / ROWS);
    if (!once) e = lane < G ? e0 + lane : entries;
    if (e < entries) ent = hitrows[e];
    int cnt = 0, upto = 0;  // bits of this lane's entry and of those up to it, for lanes under kDealEntries
    int bits = 64, at = lane;
    if (!once) {
      asm volatile("" : "+v"(at));  // what follows from it stays out of the short list's instructions
      cnt = upto = __popc(ent.y) + __popc(ent.z) + __popc(ent.w);
#pragma unroll
      for (int o = 1; o < kDealEntries; o <<= 1) {
        const int u = __builtin_amdgcn_ds_bpermute((at - o) * 4, upto);
        if (at >= o) upto += u;
      }
      bits = __builtin_amdgcn_readlane(upto, kDealEntries - 1);
    }
    for (int t0 = 0; t0 < bits; t0 += 64) {
      int c0 = ent.x, bit = (int)(w % ROWS);
      bool act;
      if (once) {
        const unsigned word = (unsigned)(bit < 32 ? ent.y : (bit < 64 ? ent.z : ent.w));
        act = ((word >> (bit % 32)) & 1u) != 0;
        if (__ballot(act) == 0ull) return;  // uniform
      } else {
        const int t = t0 + at;
        int src = 0;  // the entry that holds bit t
#pragma unroll
        for (int o = kDealEntries / 2; o > 0; o >>= 1) src += t >= __shfl(upto, src + o - 1) ? o : 0;
        const int first = __shfl(upto - cnt, src);
        bit = set_bit(t - first, __shfl(ent.y, src), __shfl(ent.z, src), __shfl(ent.w, src));
        c0 = __shfl(ent.x, src);
        act = t < bits;
      }
      work(c0, bit, act);
    }
    if (once) return;
  }
}

// Phase 2 of the kernels for any row count and of the other index maps.  Measured,
// both phases, 2^22 bins and 85 rows at a false-alarm probability of 1e-4 (some
// 36,000 candidates to a plane): fundamental map 1162 -> 675 us, highest 4556 -> 2122, of
// which phase 1 takes 627 and 1842.
template <int MAP, int NH>
__global__ __launch_bounds__(HS_THREADS) void k_emit_map(const float* __restrict__ fop, int64_t ld, int n, int z_max,
                                                         int rbase, const int4* __restrict__ hitrows, int hit_cap,
                                                         const int32_t* __restrict__ hit_count,
                                                         const float* __restrict__ ta, fdas_cand* __restrict__ cands,
                                                         int cap, int32_t* __restrict__ counts) {
  constexpr int STRIDE =
      MAP == FDAS_HSUM_HIGHEST ? kStrideHigh : MAP == FDAS_HSUM_FUNDAMENTAL ? kStrideFund : 1;
  deal_rows<kRowsPerPass>(hitrows, min(*hit_count, hit_cap), [&](int c0, int bit, bool act) {
    const int r = rbase + bit, i = r - z_max;
    float hk[NH + 1][4];
    if (act) map_sums<MAP, NH>(hk, fop, ld, n, z_max, i, c0);
    hs_append_wave<NH, STRIDE>(hk, n, 2 * z_max + 1, c0, i, r, act, ta, cands, cap, counts, threadIdx.x & 63);
  });
}

// Phase 2 of the 85-row kernel: work item w = entry * ROWS + row, grid-stride over
// all items in wave-uniform steps so the whole wave reaches the compaction together
// (hits crowd into rows near pulsars, and single waves would have dozens of rounds
// if the set rows were dealt); with row segments, which have few rows each, as
// deal_rows does: 2^18 bins with most rows above threshold took 3.77 ms with all
// rows to an entry, take 0.46 this way.
template <int Z, int NH, int SEGS = 1>
__global__ __launch_bounds__(HS_THREADS) void k_harmsum_emit(const float* __restrict__ fop, int64_t ld, int n,
                                                             const int4* __restrict__ hitrows,
                                                             const int32_t* __restrict__ hitrow_count,
                                                             const float* __restrict__ ta,
                                                             fdas_cand* __restrict__ cands, int cap,
                                                             int32_t* __restrict__ counts) {
  const int lane = threadIdx.x & 63;
  if constexpr (SEGS > 1) {
    deal_rows<2 * Z + 1>(hitrows, *hitrow_count, [&](int c0, int bit, bool act) {
      hs_emit_wave<Z, NH>(fop, ld, n, c0, bit, act, ta, cands, cap, counts, lane);
    });
    return;
  }
  constexpr int ROWS = 2 * Z + 1;
  const int64_t items = (int64_t)(*hitrow_count) * ROWS;
  const int64_t stride = (int64_t)gridDim.x * HS_THREADS;
  for (int64_t w0 = (int64_t)blockIdx.x * HS_THREADS + (threadIdx.x & ~63); w0 < items; w0 += stride) {
    const int64_t w = w0 + lane;
    bool act = w < items;
    int4 ent = make_int4(0, 0, 0, 0);
    int r = 0;
    if (act) {
      ent = hitrows[w / ROWS];
      r = (int)(w % ROWS);
      const unsigned word = (unsigned)(r < 32 ? ent.y : (r < 64 ? ent.z : ent.w));
      act = ((word >> (r % 32)) & 1u) != 0;
    }
    if (__ballot(act) == 0ull) continue;  // uniform
    hs_emit_wave<Z, NH>(fop, ld, n, ent.x, r, act, ta, cands, cap, counts, lane);
  }
}

// counts[0 .. nh) = 0 and *extra = 0 in one launch
__global__ void k_fill_counts(int32_t* __restrict__ counts, int nh, int32_t* __restrict__ extra) {
  const int t = threadIdx.x;
  if (t < nh) counts[t] = 0;
  if (extra && t == 63) *extra = 0;
}

// Batch form of phase 2: the entry's trial is in bits 21..31 of its third word.
template <int Z, int NH>
__global__ __launch_bounds__(HS_THREADS) void k_harmsum_emit_batch(const HsTrial* __restrict__ trials,
                                                                   const int4* __restrict__ hitrows,
                                                                   const int32_t* __restrict__ hitrow_count,
                                                                   const float* __restrict__ ta, int cap) {
  constexpr int ROWS = 2 * Z + 1;
  const int64_t items = (int64_t)(*hitrow_count) * ROWS;
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * HS_THREADS;
  // wave-uniform steps; a wave whose active lanes all belong to one trial (the
  // usual case: a phase-1 block appends its entries together) reserves slots
  // per plane for the whole wave, a mixed wave falls back to one atomic per
  // lane and plane
  for (int64_t w0 = (int64_t)blockIdx.x * HS_THREADS + (threadIdx.x & ~63); w0 < items; w0 += stride) {
    const int64_t w = w0 + lane;
    bool act = w < items;
    int4 ent = make_int4(0, 0, 0, 0);
    int r = 0;
    if (act) {
      ent = hitrows[w / ROWS];
      r = (int)(w % ROWS);
      const unsigned w2 = (unsigned)ent.w & 0x1FFFFFu;
      const unsigned word = (unsigned)(r < 32 ? ent.y : (r < 64 ? ent.z : (int)w2));
      act = ((word >> (r % 32)) & 1u) != 0;
    }
    const unsigned long long am = __ballot(act);
    if (am == 0ull) continue;  // uniform
    const int tri = (int)((unsigned)ent.w >> 21);
    const int lead = __builtin_amdgcn_readlane(tri, (int)__builtin_ctzll(am));
    if (__ballot(act && tri != lead) == 0ull) {  // uniform
      const HsTrial& tr = trials[lead];
      hs_emit_wave<Z, NH>(tr.fop, tr.ld, tr.n, ent.x, r, act, ta, tr.cands, cap, tr.counts, lane);
    } else if (act) {
      const HsTrial& tr = trials[tri];
      hs_emit_row<Z, NH>(tr.fop, tr.ld, tr.n, ent.x, r, ta, tr.cands, cap, tr.counts);
    }
  }
}

// counts[0 .. nh) of every trial of a batch set to 0
__global__ void k_zero_counts_batch(const HsTrial* __restrict__ trials, int ntrials, int nh) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ntrials * nh) trials[i / nh].counts[i % nh] = 0;
}

__global__ void k_fill_i32(int32_t* p, int count, int32_t value) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = value;
}

// Tile order of the 85-row kernel computed on the device (the order
// harmsum_tile_order builds on the host): tile t has the key
// (frac << 6) | (octave + 1), frac = (t - 2^octave) << (top - octave), key 0
// for t = 0; tiles are ranked by key and rank q goes to workgroup
// (q mod per) * 8 + q / per, per = ceil(T / 8).  Keys are distinct, so the
// rank of t is the number of smaller keys.
__device__ __forceinline__ uint64_t tile_key(int t, int top) {
  if (t == 0) return 0;
  const int o = 31 - __clz(t);
  const uint64_t frac = (uint64_t)(t - (1 << o)) << (top - o);
  return (frac << 6) | (uint64_t)(o + 1);
}

// With high_tiles > 0, t is a chunk of kHighChunk tiles of the highest-anchored
// kernel and rank q goes where harmsum_high_order puts it.
__global__ void k_tile_order(int* __restrict__ order, int T, int top, int per, int high_tiles) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const uint64_t k = tile_key(t, top);
  int q = 0;
  for (int u = 0; u < T; ++u) q += tile_key(u, top) < k ? 1 : 0;
  if (high_tiles > 0) {
    for (int e = 0; e < kHighChunk; ++e)
      if (t * kHighChunk + e < high_tiles) order[((q / 8) * kHighChunk + e) * 8 + q % 8] = t * kHighChunk + e;
  } else {
    order[(q % per) * 8 + q / per] = t;
  }
}

// Scratch of fdas_harmonic_sum_noalloc in static device memory (one copy per
// GPU, kept until the process ends): hit-row counter, tile order, hit-row list.
constexpr int64_t kNoAllocMaxN = (int64_t)1 << 22;
constexpr size_t kNaOrderOff = 256;
constexpr size_t kNaOrderInts = ((size_t)kNoAllocMaxN / (4 * HS_THREADS) + 128 + 63) / 64 * 64;
constexpr size_t kNaHitOff = kNaOrderOff + kNaOrderInts * sizeof(int);
constexpr int kNaHitCap = (int)(kNoAllocMaxN / 4) + kHitSlack;
constexpr size_t kNaBytes = kNaHitOff + (size_t)kNaHitCap * sizeof(int4);
static __device__ __align__(256) unsigned char scratch[kNaBytes];

}  // namespace

int64_t harmsum_noalloc_max_n() { return kNoAllocMaxN; }
size_t harmsum_noalloc_scratch_bytes() { return kNaBytes; }

hipError_t harmsum_noalloc_scratch(void** ptr) {
  // the caller has made the device current; the address is per device
  return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
}

hipError_t launch_harmsum_noalloc(const float* fop, int64_t n, int64_t ld, int z_max, int n_harm, const float* ta,
                                  fdas_cand* cands, int cap, int32_t* counts, void* scr, int emit_blocks,
                                  int index, hipStream_t s) {
  if (n < 1 || n > kNoAllocMaxN || !scr) return hipErrorInvalidValue;
  unsigned char* base = static_cast<unsigned char*>(scr);
  int* order = reinterpret_cast<int*>(base + kNaOrderOff);
  int4* hitrows = reinterpret_cast<int4*>(base + kNaHitOff);
  int32_t* hit_count = reinterpret_cast<int32_t*>(base);
  const int cols = 4 * HS_THREADS;
  const bool high = index == FDAS_HSUM_HIGHEST;
  const int tiles = (int)(high ? harmsum_high_tiles(n) : (n + cols - 1) / cols);
  const int T = high ? (tiles + kHighChunk - 1) / kHighChunk : tiles;  // tiles or chunks to order
  const int per = high ? (T + 7) / 8 * kHighChunk : (T + 7) / 8;       // workgroups per XCD
  const bool ordered = (z_max == 42 && index == FDAS_HSUM_STRETCH) || index == FDAS_HSUM_FUNDAMENTAL || high;
  if (ordered) {
    int top = 0;
    while ((1LL << (top + 1)) <= (int64_t)(T > 2 ? T - 1 : 1)) ++top;
    hipError_t e = launch_fill_i32(order, per * 8, -1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tile_order, dim3((T + 255) / 256), dim3(256), 0, s, order, T, top, per, high ? tiles : 0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const HsWork wk{order, per * 8, hitrows, hit_count, emit_blocks, kNaHitCap};
  return launch_harmsum(fop, n, ld, z_max, n_harm, ta, cands, cap, counts, wk, index, s);
}

int harmsum_tile_columns() { return 4 * HS_THREADS; }

hipError_t launch_fill_i32(int32_t* p, int count, int32_t value, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((count + 255) / 256), dim3(256), 0, s, p, count, value);
  return hipGetLastError();
}

hipError_t launch_zero_counts_batch(const HsTrial* trials, int ntrials, int nh, hipStream_t s) {
  const int total = ntrials * nh;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_counts_batch, dim3((total + 255) / 256), dim3(256), 0, s, trials, ntrials, nh);
  return hipGetLastError();
}

template <int TH>
hipError_t launch_phase1_batch(const HsTrial* trials, int ntrials, int blk_begin, unsigned blocks, int n_harm,
                               const float* ta, int4* hitrows, int32_t* hitrow_count, hipStream_t s) {
  switch (n_harm) {
#define FDAS_HSP_CASE(NH)                                                                                     \
  case NH:                                                                                                    \
    hipLaunchKernelGGL((k_harmsum_z_batch<42, NH, TH>), dim3(blocks), dim3(TH), 0, s, trials, ntrials,        \
                       blk_begin, ta, hitrows, hitrow_count);                                                 \
    break;
    FDAS_HSP_CASE(1)
    FDAS_HSP_CASE(2)
    FDAS_HSP_CASE(3)
    FDAS_HSP_CASE(4)
    FDAS_HSP_CASE(5)
    FDAS_HSP_CASE(6)
    FDAS_HSP_CASE(7)
    FDAS_HSP_CASE(8)
#undef FDAS_HSP_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

bool harmsum_tile_built(int cols) { return cols == 256 || cols == 512 || cols == 1024; }

hipError_t launch_harmsum_batch85(const HsTrial* trials, int ntrials, int blk_begin, int blk_end, int n_harm,
                                  const float* ta, int cap, int4* hitrows, int32_t* hitrow_count, int eblocks,
                                  int tile_cols, hipStream_t s) {
  if (blk_end <= blk_begin) return hipSuccess;
  hipError_t e = launch_fill_i32(hitrow_count, 1, 0, s);
  if (e != hipSuccess) return e;
  const unsigned blocks = (unsigned)(blk_end - blk_begin);
  switch (tile_cols) {
    case 256: e = launch_phase1_batch<64>(trials, ntrials, blk_begin, blocks, n_harm, ta, hitrows, hitrow_count, s); break;
    case 512: e = launch_phase1_batch<128>(trials, ntrials, blk_begin, blocks, n_harm, ta, hitrows, hitrow_count, s); break;
    case 1024: e = launch_phase1_batch<256>(trials, ntrials, blk_begin, blocks, n_harm, ta, hitrows, hitrow_count, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  switch (n_harm) {
#define FDAS_HSB_CASE(NH)                                                                                     \
  case NH:                                                                                                    \
    hipLaunchKernelGGL((k_harmsum_emit_batch<42, NH>), dim3(eblocks), dim3(HS_THREADS), 0, s, trials, hitrows, \
                       hitrow_count, ta, cap);                                                                \
    break;
    FDAS_HSB_CASE(1)
    FDAS_HSB_CASE(2)
    FDAS_HSB_CASE(3)
    FDAS_HSB_CASE(4)
    FDAS_HSB_CASE(5)
    FDAS_HSB_CASE(6)
    FDAS_HSB_CASE(7)
    FDAS_HSB_CASE(8)
#undef FDAS_HSB_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// one pass (at most 96 rows) of both phases
template <int MAP, int NH, typename Detect>
hipError_t launch_map(Detect detect, const float* fop, int n, int64_t ld, int z_max, int rbase, int rend,
                      const int* order, const float* ta, fdas_cand* cands, int cap, int32_t* counts,
                      const HsWork& wk, unsigned blocks, unsigned segs, unsigned eblocks, hipStream_t s) {
  // The other maps' kernels reserve LDS they do not use, so that fewer waves share
  // a compute unit than registers allow: the waves' source rows evict each
  // other's lines.  Highest: three workgroups (2^22 bins 2.06 ms; four 2.19-2.24,
  // two 2.19).  Fundamental: four beside its 4 KB table (1,500,001 bins 0.301 ms;
  // seven 0.352).
  const size_t reserve = MAP == FDAS_HSUM_HIGHEST ? 50000 : MAP == FDAS_HSUM_FUNDAMENTAL ? 36000 : 0;
  hipLaunchKernelGGL(detect, dim3(blocks, segs), dim3(HS_THREADS), reserve, s, fop, ld, n, z_max, rbase, rend, order, ta,
                     wk.hitrows, wk.hit_cap, wk.hitrow_count);
  hipLaunchKernelGGL((k_emit_map<MAP, NH>), dim3(eblocks), dim3(HS_THREADS), 0, s, fop, ld, n, z_max, rbase,
                     wk.hitrows, wk.hit_cap, wk.hitrow_count, ta, cands, cap, counts);
  return hipGetLastError();
}

int64_t harmsum_hit_entries(int64_t n_max, int index) {
  // segments x groups of the longest spectrum, and of the one with the most of either split
  const int64_t maps = std::min<int64_t>(kMaxSegs * ((n_max + 3) / 4), kSplitBins / 4);
  const int64_t rows85 = kSegRows * ((std::min<int64_t>(n_max, kSegMaxN) + 3) / 4);
  const int64_t high = index == FDAS_HSUM_HIGHEST && n_max > kHighSplitLo
                           ? kHighSegs * ((std::min<int64_t>(n_max, kHighSplitHi) + 3) / 4)
                           : 0;
  return std::max({(n_max + 3) / 4, maps, rows85, high}) + kHitSlack;
}

hipError_t launch_harmsum(const float* fop, int64_t n, int64_t ld, int z_max, int n_harm, const float* ta,
                          fdas_cand* cands, int cap, int32_t* counts, const HsWork& wk, int index, hipStream_t s) {
  // the counts and the hit-row counter start at zero, in one launch
  hipLaunchKernelGGL(k_fill_counts, dim3(1), dim3(64), 0, s, counts, n_harm, wk.hitrow_count);
  {
    hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
  }
  const unsigned eblocks = (unsigned)(wk.emit_blocks > 0 ? wk.emit_blocks : 1024);
  const int nn = (int)n;
  if (z_max == 42 && index == FDAS_HSUM_STRETCH) {
    // two-phase fast path for the 85-template plane
    const unsigned blocks = (unsigned)wk.blocks;
    const bool segs = n <= kSegMaxN && (n + 3) / 4 * kSegRows <= wk.hit_cap;
    switch (n_harm) {
#define FDAS_HSZ_CASE(NH)                                                                                          \
  case NH:                                                                                                         \
    if (segs) {                                                                                                    \
      hipLaunchKernelGGL((k_harmsum_z<42, NH, HS_THREADS, kSegRows>), dim3(blocks, kSegRows), dim3(HS_THREADS), 0, \
                         s, fop, ld, nn, wk.tile_of_block, ta, wk.hitrows, wk.hitrow_count);                       \
      hipLaunchKernelGGL((k_harmsum_emit<42, NH, kSegRows>), dim3(eblocks), dim3(HS_THREADS), 0, s, fop, ld, nn,   \
                         wk.hitrows, wk.hitrow_count, ta, cands, cap, counts);                                     \
    } else {                                                                                                       \
      hipLaunchKernelGGL((k_harmsum_z<42, NH>), dim3(blocks), dim3(HS_THREADS), 0, s, fop, ld, nn,                 \
                         wk.tile_of_block, ta, wk.hitrows, wk.hitrow_count);                                       \
      hipLaunchKernelGGL((k_harmsum_emit<42, NH>), dim3(eblocks), dim3(HS_THREADS), 0, s, fop, ld, nn, wk.hitrows, \
                         wk.hitrow_count, ta, cands, cap, counts);                                                 \
    }                                                                                                              \
    break;
      FDAS_HSZ_CASE(1)
      FDAS_HSZ_CASE(2)
      FDAS_HSZ_CASE(3)
      FDAS_HSZ_CASE(4)
      FDAS_HSZ_CASE(5)
      FDAS_HSZ_CASE(6)
      FDAS_HSZ_CASE(7)
      FDAS_HSZ_CASE(8)
#undef FDAS_HSZ_CASE
      default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  // threads (groups of four columns) and workgroups of phase 1
  int64_t groups;
  unsigned blocks;
  const int* order = nullptr;
  if (index == FDAS_HSUM_FUNDAMENTAL) {
    groups = (n + XT - 1) / XT * HS_THREADS;
    order = wk.tile_of_block;
    blocks = order ? (unsigned)wk.blocks : (unsigned)((n + XT - 1) / XT);
  } else if (index == FDAS_HSUM_HIGHEST) {
    groups = harmsum_high_tiles(n) * HS_THREADS;
    order = wk.tile_of_block;
    blocks = order ? (unsigned)wk.blocks : (unsigned)harmsum_high_tiles(n);
  } else {
    groups = (n + 3) / 4;
    blocks = (unsigned)((groups + HS_THREADS - 1) / HS_THREADS);
  }
  if (groups > wk.hit_cap) return hipErrorInvalidValue;
  // row segments: enough waves to fill the chip, if the list can hold every thread's entry
  int64_t want = std::min<int64_t>(kMaxSegs, kSplitBins / n);
  if (index == FDAS_HSUM_HIGHEST && n > kHighSplitLo && n <= kHighSplitHi) want = kHighSegs;
  const unsigned segs = (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, wk.hit_cap / groups));
  const int rows = 2 * z_max + 1;
  for (int rbase = 0; rbase < rows; rbase += kRowsPerPass) {
    const int rend = std::min(rows, rbase + kRowsPerPass);
    if (rbase > 0) {
      hipError_t e = launch_fill_i32(wk.hitrow_count, 1, 0, s);
      if (e != hipSuccess) return e;
    }
    hipError_t e = hipErrorInvalidValue;
    switch (n_harm) {
#define FDAS_HSX_CASE(NH)                                                                                          \
  case NH:                                                                                                         \
    e = index == FDAS_HSUM_FUNDAMENTAL                                                                             \
            ? launch_map<FDAS_HSUM_FUNDAMENTAL, NH>(k_detect_fund<NH>, fop, nn, ld, z_max, rbase, rend, order, ta, \
                                                    cands, cap, counts, wk, blocks, segs, eblocks, s)              \
        : index == FDAS_HSUM_HIGHEST                                                                               \
            ? launch_map<FDAS_HSUM_HIGHEST, NH>(k_detect_high<NH>, fop, nn, ld, z_max, rbase, rend, order, ta,     \
                                                cands, cap, counts, wk, blocks, segs, eblocks, s)                  \
            : launch_map<FDAS_HSUM_STRETCH, NH>(k_detect_stretch<NH>, fop, nn, ld, z_max, rbase, rend, order, ta,  \
                                                cands, cap, counts, wk, blocks, segs, eblocks, s);                 \
    break;
      FDAS_HSX_CASE(1)
      FDAS_HSX_CASE(2)
      FDAS_HSX_CASE(3)
      FDAS_HSX_CASE(4)
      FDAS_HSX_CASE(5)
      FDAS_HSX_CASE(6)
      FDAS_HSX_CASE(7)
      FDAS_HSX_CASE(8)
#undef FDAS_HSX_CASE
      default:
        break;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace fdas
