// Direct FIR correlation of the spectrum with every acceleration template on
// the matrix cores, fused with the power (Section 2.1.1, eq. (1): the
// time-domain FIR form, here as a Toeplitz-window x template contraction).
//
//   Y[j, z] = sum_d X[j + d] h_z[d],   FOP[z + z_max][j] = |Y[j, z]|^2.
//
// As a matrix product, row j of the window matrix is X[j + d] over the taps d
// and column z of the template matrix is h_z[d]; the window matrix is never
// formed: a workgroup stages its strip of X in LDS once and every MFMA operand
// is read from the strip at offset (row + tap).
//
// Two symmetries of the response cut the sum to a quarter.  A(q, -z) is the
// conjugate of A(-q, z) and, for integer q, A(-q, z) = A(q, z) (substitute
// u -> 1 - u in the integral), so h_-z = conj(h_z) and h_z[-d] = h_z[d] (to
// 1e-14 in the plan's float64 taps; the tap at d = -L/2 has no partner):
//   - with h_z = a + ib, the real-filter correlations A = X * a and B = X * b
//     serve both signs: Y_z = A + iB, Y_-z = A - iB;
//   - each filter runs over distances d >= 0 with X[j + d] + X[j - d] as
//     the operand, d = 0 with half the tap; the unpaired tap is added on the
//     vector units at the end.
//
// MFMA mapping of the FP32 kernel (v_mfma_f32_16x16x4f32, one 16 x 16 FP32
// output block, K = 4 distances; the split kernel below has K = 32):
//   rows    = 16 consecutive output bins;
//   columns = 8 |z| x {Re h, Im h};
//   one instruction for Re X and one for Im X, in accumulators of their own.
// A lane and its neighbour then hold A and B of 4 consecutive bins, swap them
// (DPP quad permutation), form |Y_z|^2 and |Y_-z|^2 and store 16 bytes each.
//
// Templates are grouped by |z| in tiles of 8 from the widest down, and a tile
// only runs over its widest member's support, so short templates do not pay
// for the 394-tap ones.
//
// Work split: a workgroup = 4 waves covers 256 consecutive bins (FP32; split 128), a
// wave 4 sub-tiles of 16 bins (split 2).

#include <algorithm>

#include "fdas_internal.h"

namespace fdas {
namespace {

constexpr int DW = 4;                 // waves per workgroup
constexpr int SUB = 4;                // 16-bin sub-tiles per wave
constexpr int WAVE_BINS = 16 * SUB;   // 64
constexpr int BLK_BINS = DW * WAVE_BINS;  // 256
constexpr int MAX_P = 296;            // L(64)/2, the widest template the plan allows
constexpr int FOLD_PAD = 8;           // strip bins past the widest template (zero-padded steps read them)

typedef float v4f __attribute__((ext_vector_type(4)));

// value of the neighbouring lane (lanes 2q and 2q+1 swap)
__device__ __forceinline__ float swap_pair(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}

// What the epilogue needs of a column, staged in LDS: a global load there would
// wait for the stores of the tile before it.
struct ColumnInfo {
  int row;    // FOP row, -1: none
  int edge;   // L/2
  float tap;  // unpaired tap
  float scale;
};

__device__ __forceinline__ void load_columns(ColumnInfo* col, int columns, const int* __restrict__ rows,
                                             const int* __restrict__ edge, const float* __restrict__ edge_tap,
                                             const float* __restrict__ tscale, int tid) {
  if (tid < columns) col[tid] = {rows[tid], edge[tid / 2], edge_tap[tid], tscale ? tscale[tid / 16] : 1.0f};
}

// The unpaired tap at d = -P of this lane's column: a += X[j - P] h for its 4
// bins of each sub-tile, STEP bins apart.
template <int STEP, int N>
__device__ __forceinline__ void edge_add(const float2* __restrict__ here, int P, float h, v4f (&ar)[N], v4f (&ai)[N]) {
#pragma unroll
  for (int s = 0; s < N; ++s)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float2 f = here[STEP * s + v - P];
      ar[s][v] = fmaf(f.x, h, ar[s][v]);
      ai[s][v] = fmaf(f.y, h, ai[s][v]);
    }
}

// Powers of one +-z pair from its two real-filter correlations, and their
// store.  An even lane holds A = X * Re h (a: its real, b: its imaginary
// part), its odd neighbour B = X * Im h; Y_z = A + iB, Y_-z = A - iB.  The even
// lane forms row z, the odd lane row -z, for 4 consecutive bins each (`left`
// of them inside the spectrum).  With (a, b) a lane's own and (oa, ob) its
// neighbour's values both are (a - ob)^2 + (b + oa)^2: the odd lane's real and
// imaginary part are b + oa and ob - a.
__device__ __forceinline__ void pair_store(const v4f& a, const v4f& b, int row, float* dst, int64_t left) {
  float pw[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const float d = a[v] - swap_pair(b[v]), t = b[v] + swap_pair(a[v]);
    pw[v] = d * d + t * t;
  }
  if (row >= 0) {
    typedef float f4v __attribute__((ext_vector_type(4)));
    if (left >= 4) {
      const f4v v = {pw[0], pw[1], pw[2], pw[3]};
      __builtin_nontemporal_store(v, reinterpret_cast<f4v*>(dst));
    } else {
#pragma unroll
      for (int v = 0; v < 3; ++v)
        if (v < left) __builtin_nontemporal_store(pw[v], dst + v);
    }
  }
}

// Bins that the matrix products must not see: NaN, infinities, and values whose
// folded sum could overflow.  A tile multiplies every bin within its widest
// member's support, by zero past a narrower member's own, and 0 x Inf is NaN.
// Such bins are staged as zero, and the cells whose own support holds one are
// formed again by repair_cells.  Spectra without them are as fast as before (2^20
// bins FP32 381 and 381 us, 2^22 bins FP16 760 and 758); one infinity among 2^22
// bins costs 1.6 ms, NaN throughout 2.6 ms (FP32) and 5.0 ms (split).
constexpr float kBadBin = 1.7e38f;
__device__ __forceinline__ bool bad_bin(const float2& v) {
  return !(fabsf(v.x) < kBadBin && fabsf(v.y) < kBadBin);
}

// The cells of NB bins from j0 on whose own support holds a bad bin, as the sum
// over their taps; tap(t, col, d) is the value of column col of tile t at
// distance d >= 0 (half of it at d = 0).  Called by a whole workgroup of 256
// after its stores; a thread takes one bin.  Only blocks that met a bad bin come here.
template <int NB, int TG, typename Tap>
__device__ __forceinline__ void repair_cells(const float2* __restrict__ x, int64_t n, float* __restrict__ fop,
                                             int64_t ld, int64_t j0, int reach, const ColumnInfo* cols, Tap tap) {
  // the stores of this block's cells come first
  __threadfence();
  __syncthreads();
  constexpr int PER = 256 / NB;  // threads to a bin: each takes every PER-th slot
  // opaque, so that nothing formed from it is kept in registers through the products
  int tid = (int)threadIdx.x;
  __asm__ volatile("" : "+v"(tid));
  const int64_t j = j0 + tid % NB;
  if (j >= n) return;
  auto bin = [&](int64_t i) { return i >= 0 && i < n ? x[i] : make_float2(0.0f, 0.0f); };
  // distance of the nearest bad bin, and of the nearest NaN, before and from j
  int left = reach + 1, right = reach + 1, nan_left = reach + 1, nan_right = reach + 1;
  for (int d = reach; d >= 0; --d) {
    const float2 a = bin(j - d), b = bin(j + d);
    if (bad_bin(a)) left = d;
    if (bad_bin(b)) right = d;
    if (a.x != a.x || a.y != a.y) nan_left = d;
    if (b.x != b.x || b.y != b.y) nan_right = d;
  }
  for (int slot = tid / NB; slot < 8 * TG; slot += PER) {
    const ColumnInfo re = cols[2 * slot], im = cols[2 * slot + 1];
    const int P = re.edge;
    if (re.row < 0 || (left > P && right > P - 1)) continue;
    float yr[2], yi[2];  // +z, -z
    if (nan_left <= P || nan_right < P) {
      // whatever the taps: spectra that are NaN throughout end here
      yr[0] = yi[0] = yr[1] = yi[1] = __builtin_nanf("");
    } else {
      const float2 v = bin(j - P);
      const float a = re.tap * re.scale, b = im.tap * im.scale;
      yr[0] = v.x * a - v.y * b;
      yi[0] = v.x * b + v.y * a;
      yr[1] = v.x * a + v.y * b;
      yi[1] = v.y * a - v.x * b;
      for (int d = 0; d < P; ++d) {
        const float ta = tap(slot >> 3, 2 * (slot & 7), d) * re.scale;
        const float tb = tap(slot >> 3, 2 * (slot & 7) + 1, d) * im.scale;
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          const float2 w = bin(side ? j - d : j + d);
          yr[0] += w.x * ta - w.y * tb;
          yi[0] += w.x * tb + w.y * ta;
          yr[1] += w.x * ta + w.y * tb;
          yi[1] += w.y * ta - w.x * tb;
        }
      }
    }
    fop[(size_t)re.row * ld + j] = yr[0] * yr[0] + yi[0] * yi[0];
    if (im.row >= 0) fop[(size_t)im.row * ld + j] = yr[1] * yr[1] + yi[1] * yi[1];
  }
}

// Operand entry of step p of tile t in a group (entries are step-major, and a step
// holds the tiles that still run).
template <int TG>
__device__ __forceinline__ int group_entry(const int* __restrict__ steps, int t, int p) {
  int e = t;
#pragma unroll
  for (int q = 0; q < TG; ++q) e += min(steps[q], p);
  return e;
}

// A group of TG tiles at once: steps[t] of tile t's folded steps (falling with
// t), rows[t * 16 + col] = FOP row of column col (-1: none),
// edge[t * 8 + slot] = L/2 of the slot's template, edge_tap[t * 16 + col] its
// unpaired tap.  The operand holds 64 floats per (step, tile) in lane order: step p
// (lane group kk: distance d = 4 p + kk) of every tile with more than p steps.  Dynamic LDS: the operand
// (`count` entries, and as much again as one step holds, read ahead) and two
// strips of X (Pm + 8 bins on either side of the workgroup's bins).  The
// unpaired taps are added on the vector units (8 multiply-adds per tile and
// sub-tile against 4 matrix instructions of 32 cycles).
//
// Bound by the FP32 matrix pipe (2 instructions of 32 cycles per 4 distances,
// 16 bins and 8 |z|).  A folded operand is read and added once and used by
// every tile that still runs at its distance: the accumulators of all tiles
// stay in registers (8 per tile and sub-tile), which leaves two waves per
// SIMD, so the next step's LDS reads are issued before this step's products.
// FP32 matrix and vector instructions do not overlap on a SIMD (measured side
// by side: the times add), so every vector instruction counts.
// Measured on 2^20 bins and 85 templates: 0.382 ms, the matrix pipe busy 80 % of
// the time; without the two symmetries 1.265 ms; one tile at a time with
// the folded operand re-read per tile and three or four waves per SIMD
// 0.413-0.456 ms.
template <int TG>
struct FoldState {
  v4f ar[TG][SUB], ai[TG][SUB];
  float2 f[SUB], r[SUB];  // X[j + d], X[j - d] of the next step
  float b[TG];            // its template values
  const float2* up;
  const float2* dn;
  const float* bp;
};

template <int TG, int T>
__device__ __forceinline__ void fold_steps(FoldState<TG>& st, const int* __restrict__ steps, int p) {
  // tiles 0 .. T-1 still run: to the end of tile T-1
  const int end = steps[T - 1];
  for (; p < end; ++p) {
    float fr[SUB], fi[SUB], bv[T];
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      fr[s] = st.f[s].x + st.r[s].x;
      fi[s] = st.f[s].y + st.r[s].y;
    }
#pragma unroll
    for (int t = 0; t < T; ++t) bv[t] = st.b[t];
    // reads past the last step stay inside the strip's padding and the operand's tail
    st.up += 4;
    st.dn -= 4;
    st.bp += 64 * T;
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      st.f[s] = st.up[16 * s];
      st.r[s] = st.dn[16 * s];
    }
#pragma unroll
    for (int t = 0; t < T; ++t) st.b[t] = st.bp[64 * t];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int s = 0; s < SUB; ++s) {
        st.ar[t][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(fr[s], bv[t], st.ar[t][s], 0, 0, 0);
        st.ai[t][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(fi[s], bv[t], st.ai[t][s], 0, 0, 0);
      }
  }
  if constexpr (T > 1) fold_steps<TG, T - 1>(st, steps, p);
}

template <int TG>
__global__ __launch_bounds__(DW * 64, 2) void k_direct_conv(
    const float2* __restrict__ x, int64_t n, float* __restrict__ fop, int64_t ld, const float4* __restrict__ Bpk,
    const int* __restrict__ steps, const int* __restrict__ rows, const int* __restrict__ edge,
    const float* __restrict__ edge_tap, int count, int Pm, int blocks) {
  extern __shared__ float4 lds4[];
  __shared__ ColumnInfo cols[16 * TG];
  __shared__ int s_bad[2];  // 1 + the last block staged in this strip that met a bad bin
  const int tid = threadIdx.x;
  load_columns(cols, 16 * TG, rows, edge, edge_tap, nullptr, tid);
  if (tid < 2) s_bad[tid] = 0;
  __syncthreads();
  const int halo = Pm + FOLD_PAD;
  const int strip = BLK_BINS + 2 * halo;  // bins jb - halo + u
  const float* bs = reinterpret_cast<const float*>(lds4);
  float2* xs = reinterpret_cast<float2*>(lds4 + 16 * (count + TG));
  for (int i = tid; i < count * 16; i += DW * 64) lds4[i] = Bpk[i];
  const int lane = tid & 63;
  const int w = tid >> 6;
  const int m = lane & 15;   // A row (bin) / output column
  const int kk = lane >> 4;  // A/B k index; output row group
  const int blk0 = (int)((int64_t)blocks * blockIdx.x / gridDim.x);
  const int blk1 = (int)((int64_t)blocks * (blockIdx.x + 1) / gridDim.x);
  for (int blk = blk0; blk < blk1; ++blk) {
    // the other strip may still be read: one barrier per block
    float2* cur = xs + ((blk - blk0) & 1) * strip;
    for (int u = tid; u < strip; u += DW * 64) {
      const int64_t idx = (int64_t)blk * BLK_BINS - halo + u;
      float2 v = (idx >= 0 && idx < n) ? x[idx] : make_float2(0.0f, 0.0f);
      if (bad_bin(v)) {
        v = make_float2(0.0f, 0.0f);
        s_bad[(blk - blk0) & 1] = blk + 1;
      }
      cur[u] = v;
    }
    __syncthreads();
    const int64_t jb = (int64_t)blk * BLK_BINS + w * WAVE_BINS;
    const float2* __restrict__ centre = cur + w * WAVE_BINS + m + halo;
    FoldState<TG> st;
#pragma unroll
    for (int t = 0; t < TG; ++t)
#pragma unroll
      for (int s = 0; s < SUB; ++s) st.ar[t][s] = st.ai[t][s] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    st.up = centre + kk;
    st.dn = centre - kk;
    st.bp = bs + lane;
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      st.f[s] = st.up[16 * s];
      st.r[s] = st.dn[16 * s];
    }
#pragma unroll
    for (int t = 0; t < TG; ++t) st.b[t] = st.bp[64 * t];
    fold_steps<TG, TG>(st, steps, 0);
    const int64_t left = n - (jb + 4 * kk);  // bins from this lane's first to the end
    const bool whole = jb + WAVE_BINS <= n;  // uniform
    const float2* __restrict__ here = cur + w * WAVE_BINS + 4 * kk + halo;  // this lane's first output bin
#pragma unroll
    for (int t = 0; t < TG; ++t) {
      const ColumnInfo ci = cols[t * 16 + m];
      edge_add<16>(here, ci.edge, ci.tap, st.ar[t], st.ai[t]);
      const int row = ci.row;
      float* dst = fop + (size_t)(row < 0 ? 0 : row) * ld + jb + 4 * kk;
      if (whole) {
#pragma unroll
        for (int s = 0; s < SUB; ++s) pair_store(st.ar[t][s], st.ai[t][s], row, dst + 16 * s, 4);
      } else {
#pragma unroll
        for (int s = 0; s < SUB; ++s) pair_store(st.ar[t][s], st.ai[t][s], row, dst + 16 * s, left - 16 * s);
      }
    }
    if (__builtin_amdgcn_readfirstlane(s_bad[(blk - blk0) & 1]) == blk + 1)
      repair_cells<BLK_BINS, TG>(x, n, fop, ld, (int64_t)blk * BLK_BINS, Pm, cols, [&](int t, int col, int d) {
        return bs[64 * group_entry<TG>(steps, t, d / 4) + 16 * (d & 3) + col];
      });
  }
}

// ---------------------------------------------------------------------------
// Split precision on the 16-bit matrix cores (v_mfma_f32_16x16x32_{f16,bf16}):
// every operand value v is carried as hi = round16(v), lo = round16(v - hi),
// and a product as hi*hi + hi*lo + lo*hi with FP32 accumulation.  The lo*lo
// term is ~2^-22 of a product for FP16 and dropped; for BF16 it is as large as
// the rounding of the halves and kept (2-norm error 5.1e-6 without it, 4.0e-6
// with, 2^22 bins 0.77 and 0.85 ms).  One instruction takes 16 bins x 32
// distances x 16 real filters (8 |z|).  FP16 has a narrow exponent range, so the
// block's strip of X is scaled by 2^ex (largest |Re|, |Im| brought to 2^14 .. 32752,
// so that a folded value stays within 65504) and each template tile by a
// plan-chosen 2^eh; both scalings are exact and undone on the accumulator.  What is
// left of a bin 2^18 and more under the strip's largest is a multiple of 2^-24
// scaled: with the strip at 2^13 the error of such bins beside a line was twice this.

constexpr int SSUB = 2;                      // 16-bin sub-tiles per wave, 32 bins apart
constexpr int SBLK_BINS = 128;               // 4 waves: wave w takes bins 64 (w / 2) + 16 (w % 2) + 32 s
constexpr int SPER = (SBLK_BINS + 2 * 32 * ((MAX_P + 31) / 32 + 3) + 255) / 256;  // strip bins per thread

template <typename T>
struct Split16;

// pack: two values rounded to nearest even, the first in the low half;
// low: v minus half `i` of a packed pair
template <>
struct Split16<_Float16> {
  static constexpr bool kLowLow = false;  // 2^-22 of a product
  typedef _Float16 v8 __attribute__((ext_vector_type(8)));
  static __device__ __forceinline__ unsigned pack(float a, float b) {
    typedef _Float16 v2 __attribute__((ext_vector_type(2)));
    const v2 h = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(unsigned, h);
  }
  static __device__ __forceinline__ float low(float v, unsigned p, int i) {
    // v - half in one instruction (a conversion and a subtraction otherwise)
    float r;
    if (i == 0)
      __asm__("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(v));
    else
      __asm__("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(v));
    return r;
  }
  static __device__ __forceinline__ v4f mfma(const v8& a, const v8& b, const v4f& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

template <>
struct Split16<__bf16> {
  static constexpr bool kLowLow = true;  // up to 2^-16 of a product: as large as the halves' own rounding
  typedef __bf16 v8 __attribute__((ext_vector_type(8)));
  static __device__ __forceinline__ unsigned pack(float a, float b) {
    typedef __bf16 v2 __attribute__((ext_vector_type(2)));
    const v2 h = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(unsigned, h);
  }
  static __device__ __forceinline__ float low(float v, unsigned p, int i) {
    return v - __uint_as_float(i ? p & 0xffff0000u : p << 16);
  }
  static __device__ __forceinline__ v4f mfma(const v8& a, const v8& b, const v4f& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// The 16 folded values of one sub-tile and step (Re, Im of 8 distances) as hi
// and lo halves.
template <typename T>
struct Folded {
  typename Split16<T>::v8 rh, rl, ih, il;
};

// hi and lo halves of 8 values; the packed hi pairs are opaque to the compiler,
// which would otherwise round every value a second time to form its lo half
template <typename T>
__device__ __forceinline__ void split8(const float (&v)[8], typename Split16<T>::v8& hi, typename Split16<T>::v8& lo) {
  typedef Split16<T> S;
  unsigned h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    h[e] = S::pack(v[2 * e], v[2 * e + 1]);
    __asm__("" : "+v"(h[e]));
    l[e] = S::pack(S::low(v[2 * e], h[e], 0), S::low(v[2 * e + 1], h[e], 1));
  }
  hi = __builtin_bit_cast(typename S::v8, make_uint4(h[0], h[1], h[2], h[3]));
  lo = __builtin_bit_cast(typename S::v8, make_uint4(l[0], l[1], l[2], l[3]));
}

template <typename T>
__device__ __forceinline__ Folded<T> fold_split(const float2 (&u)[8], const float2 (&d)[8]) {
  Folded<T> o;
  float re[8], im[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    re[e] = u[e].x + d[e].x;
    im[e] = u[e].y + d[e].y;
  }
  split8<T>(re, o.rh, o.rl);
  split8<T>(im, o.ih, o.il);
  return o;
}

// 8 consecutive strip values, upwards from p or downwards to it
__device__ __forceinline__ void strip_up(const float2* __restrict__ p, float2 (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = p[e];
}
__device__ __forceinline__ void strip_down(const float2* __restrict__ p, float2 (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = p[-e];
}

// A group of TG tiles at once, as in the FP32 kernel, with steps of 32
// distances: lane group kg holds distances 32 q + 8 kg + e.  Bsp holds 2 KiB
// per (step, tile): 64 lanes x 8 hi values, then 64 x 8 lo values; tscale[t] =
// 2^-eh.  The strip of X stays FP32 (scaled so that a folded value is at most
// 65504) and every folded value is split when it is used: the sum of two 16-bit
// halves is no 16-bit value.  A wave's two sub-tiles lie 32 bins, one step,
// apart, so sub-tile 0 of the next step reads upwards what sub-tile 1 reads
// now, and sub-tile 1 downwards what sub-tile 0 reads now: one upward and one
// downward read per step instead of two each (`PAR` says which registers hold
// which).  Dynamic LDS: the operand, one entry read ahead, and one strip.
// Measured on 2^22 bins: 0.766 ms (FP16); 1.53 ms with every template and tap
// multiplied on its own.  The fold and split cost 48 vector instructions per
// sub-tile and step against 12 matrix instructions per tile, which 16-bit
// matrix instructions overlap in part; both pipes together bound it.
template <typename T, int TG, int PAR>
__device__ __forceinline__ void split_step(v4f (&ar)[TG][SSUB], v4f (&ai)[TG][SSUB], float2 (&u)[2][8],
                                           float2 (&d)[2][8], const float2* __restrict__ up,
                                           const float2* __restrict__ dn, const uint4* __restrict__ b, int active) {
  typedef Split16<T> S;
  typedef typename S::v8 v8;
  v8 bh = __builtin_bit_cast(v8, b[0]), bl = __builtin_bit_cast(v8, b[64]);
  // u[PAR], d[PAR]: sub-tile 0; u[1 - PAR], d[1 - PAR]: sub-tile 1
  Folded<T> f[SSUB];
  f[0] = fold_split<T>(u[PAR], d[PAR]);
  f[1] = fold_split<T>(u[1 - PAR], d[1 - PAR]);
  strip_up(up, u[PAR]);        // the next step's sub-tile 1
  strip_down(dn, d[1 - PAR]);  // the next step's sub-tile 0
#pragma unroll
  for (int t = 0; t < TG; ++t) {
    if (t < active) {  // uniform
      // the next tile's values (past the last one: unused) while this one multiplies
      const v8 nh = __builtin_bit_cast(v8, b[128 * (t + 1)]);
      const v8 nl = __builtin_bit_cast(v8, b[128 * (t + 1) + 64]);
#pragma unroll
      for (int s = 0; s < SSUB; ++s) {
        ar[t][s] = S::mfma(f[s].rh, bh, ar[t][s]);
        ai[t][s] = S::mfma(f[s].ih, bh, ai[t][s]);
      }
#pragma unroll
      for (int s = 0; s < SSUB; ++s) {
        ar[t][s] = S::mfma(f[s].rl, bh, ar[t][s]);
        ai[t][s] = S::mfma(f[s].il, bh, ai[t][s]);
      }
#pragma unroll
      for (int s = 0; s < SSUB; ++s) {
        ar[t][s] = S::mfma(f[s].rh, bl, ar[t][s]);
        ai[t][s] = S::mfma(f[s].ih, bl, ai[t][s]);
      }
      if constexpr (S::kLowLow) {
#pragma unroll
        for (int s = 0; s < SSUB; ++s) {
          ar[t][s] = S::mfma(f[s].rl, bl, ar[t][s]);
          ai[t][s] = S::mfma(f[s].il, bl, ai[t][s]);
        }
      }
      bh = nh;
      bl = nl;
    }
  }
}

// NB parts of 128 bins to a block, one after another on one staged strip: narrow
// banks have so few steps that staging, with its halo of three steps and the wait
// for its loads, is most of the time.
template <typename T, int TG, int NB>
__global__ __launch_bounds__(256, 2) void k_direct_conv_split(
    const float2* __restrict__ x, int64_t n, float* __restrict__ fop, int64_t ld, const uint4* __restrict__ Bsp,
    const int* __restrict__ steps, const float* __restrict__ tscale, const int* __restrict__ rows,
    const int* __restrict__ edge, const float* __restrict__ edge_tap, int count, int halo, int Pm, int blocks) {
  extern __shared__ uint4 lds_u4[];
  __shared__ ColumnInfo cols[16 * TG];
  __shared__ float s_max[4];
  const int tid = threadIdx.x;
  load_columns(cols, 16 * TG, rows, edge, edge_tap, tscale, tid);
  const int strip = NB * SBLK_BINS + 2 * halo;  // bins jb - halo + u
  float2* xs = reinterpret_cast<float2*>(lds_u4 + 128 * (count + 1));
  for (int i = tid; i < count * 128; i += 256) lds_u4[i] = Bsp[i];
  const int lane = tid & 63;
  const int w = tid >> 6;
  const int m = lane & 15;
  const int kg = lane >> 4;
  const int w0 = 64 * (w >> 1) + 16 * (w & 1);  // first bin of this wave's sub-tile 0
  int run[TG];
#pragma unroll
  for (int t = 0; t < TG; ++t) run[t] = steps[t];
  const int blk0 = (int)((int64_t)blocks * blockIdx.x / gridDim.x);
  const int blk1 = (int)((int64_t)blocks * (blockIdx.x + 1) / gridDim.x);
  float2 nx[SPER];  // the next block's strip, loaded while this one is worked on
  auto fetch = [&](int blk) {
#pragma unroll
    for (int i = 0; i < SPER; ++i) {
      const int u = tid + 256 * i;
      const int64_t idx = (int64_t)blk * (NB * SBLK_BINS) - halo + u;
      nx[i] = (u < strip && idx >= 0 && idx < n) ? x[idx] : make_float2(0.0f, 0.0f);
    }
  };
  // largest |Re|, |Im| of this wave's share of the fetched strip, negated when
  // the share held a bad bin (which becomes zero).  Taken before
  // the block's stores are issued: a wait for the loads then waits for no store.
  auto note_max = [&]() {
    auto share_max = [&]() {  // NaN if one is met
      float m = 0.0f;
#pragma unroll
      for (int i = 0; i < SPER; ++i)
        m = __builtin_elementwise_maximum(m, __builtin_elementwise_maximum(fabsf(nx[i].x), fabsf(nx[i].y)));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m = __builtin_elementwise_maximum(m, __shfl_xor(m, o));
      return m;
    };
    float mx = share_max();
    if (!(mx < kBadBin)) {  // uniform
#pragma unroll
      for (int i = 0; i < SPER; ++i)
        if (bad_bin(nx[i])) nx[i] = make_float2(0.0f, 0.0f);
      mx = -share_max();
    }
    if (lane == 0) s_max[w] = mx;
  };
  fetch(blk0);
  note_max();
  for (int blk = blk0; blk < blk1; ++blk) {
    const int64_t j0 = (int64_t)blk * (NB * SBLK_BINS);
    __syncthreads();  // every wave is done with the previous strip
    const float mx = fmaxf(fmaxf(fabsf(s_max[0]), fabsf(s_max[1])), fmaxf(fabsf(s_max[2]), fabsf(s_max[3])));
    const int bad = __builtin_amdgcn_readfirstlane(__float_as_int(s_max[0]) | __float_as_int(s_max[1]) |
                                                   __float_as_int(s_max[2]) | __float_as_int(s_max[3]));  // sign
    int ex = 0;
    if (mx > 0.0f) {
      // 2^14 <= max * 2^ex, and the sum of two bins at most 65504, FP16's largest
      ex = 14 - ilogbf(mx);
      if (ldexpf(mx, ex) > 32752.0f) --ex;
    }
#pragma unroll
    for (int i = 0; i < SPER; ++i) {
      const int u = tid + 256 * i;
      if (u < strip) xs[u] = make_float2(ldexpf(nx[i].x, ex), ldexpf(nx[i].y, ex));
    }
    __syncthreads();
    if (blk + 1 < blk1) fetch(blk + 1);
    for (int nb = 0; nb < NB; ++nb) {
      if (NB > 1 && nb > 0 && j0 + nb * SBLK_BINS >= n) break;  // uniform
      const float2* part = xs + halo + nb * SBLK_BINS;
      v4f ar[TG][SSUB], ai[TG][SSUB];
#pragma unroll
      for (int t = 0; t < TG; ++t)
#pragma unroll
        for (int s = 0; s < SSUB; ++s) ar[t][s] = ai[t][s] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
      const float2* up = part + w0 + m + 8 * kg;
      const float2* dn = part + w0 + m - 8 * kg;
      const uint4* b = lds_u4 + lane;
      float2 u[2][8], d[2][8];
      strip_up(up, u[0]);
      strip_up(up + 32, u[1]);
      strip_down(dn, d[0]);
      strip_down(dn + 32, d[1]);
      up += 64;
      dn -= 32;
      for (int q = 0; q < run[0]; q += 2) {
        int active = 0, next = 0;
#pragma unroll
        for (int t = 0; t < TG; ++t) {
          active += q < run[t] ? 1 : 0;
          next += q + 1 < run[t] ? 1 : 0;
        }
        split_step<T, TG, 0>(ar, ai, u, d, up, dn, b, active);
        b += 128 * active;
        if (next == 0) break;  // uniform: an odd number of steps
        split_step<T, TG, 1>(ar, ai, u, d, up + 32, dn - 32, b, next);
        b += 128 * next;
        up += 64;
        dn -= 64;
      }
      if (nb == 0 && blk + 1 < blk1) note_max();
      const int64_t jb = j0 + nb * SBLK_BINS + w0;
      const int64_t left = n - (jb + 4 * kg);
      const bool whole = j0 + (nb + 1) * SBLK_BINS <= n;  // uniform
      const float2* __restrict__ here = part + w0 + 4 * kg;
#pragma unroll
      for (int t = 0; t < TG; ++t) {
        const ColumnInfo ci = cols[t * 16 + m];
        edge_add<32>(here, ci.edge, ci.tap, ar[t], ai[t]);
        const float unscale = ldexpf(ci.scale, -ex);
        const int row = ci.row;
        float* dst = fop + (size_t)(row < 0 ? 0 : row) * ld + jb + 4 * kg;
#pragma unroll
        for (int s = 0; s < SSUB; ++s) {
          const v4f a = ar[t][s] * unscale, c = ai[t][s] * unscale;
          if (whole)
            pair_store(a, c, row, dst + 32 * s, 4);
          else
            pair_store(a, c, row, dst + 32 * s, left - 32 * s);
        }
      }
    }
    if (bad < 0) {
      auto tap = [&](int t, int col, int d) {
        // lane 16 ((d / 8) % 4) + col, value d % 8: hi, and lo 64 lanes on
        const T* e = reinterpret_cast<const T*>(lds_u4 + 128 * group_entry<TG>(steps, t, d / 32));
        const int at = (16 * ((d >> 3) & 3) + col) * 8 + (d & 7);
        return (float)e[at] + (float)e[at + 512];
      };
      constexpr int RB = NB * SBLK_BINS < 256 ? NB * SBLK_BINS : 256;
      for (int q = 0; q < NB * SBLK_BINS; q += RB) repair_cells<RB, TG>(x, n, fop, ld, j0 + q, Pm, cols, tap);
    }
  }
}

}  // namespace

template <typename T, int TG, int NB>
hipError_t launch_split_group(const float2* x, int64_t n, float* fop, int64_t ld, const DirectTables& t,
                              const DirectGroup& gr, int halo, int blocks, unsigned grid, hipStream_t s) {
  const size_t lds = (size_t)2048 * (gr.count + 1) + sizeof(float2) * (size_t)(NB * SBLK_BINS + 2 * halo);
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_direct_conv_split<T, TG, NB>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_direct_conv_split<T, TG, NB>), dim3(grid), dim3(256), lds, s, x, n, fop, ld,
                     t.Bsp + (size_t)128 * gr.offset, t.steps + gr.first, t.tscale + gr.first, t.rows + 16 * gr.first,
                     t.edge + 8 * gr.first, t.edge_tap + 16 * gr.first, gr.count, halo, t.P_max, blocks);
  return hipGetLastError();
}

hipError_t launch_direct_conv_split(const float2* x, int64_t n, float* fop, int64_t ld, const DirectTables& t,
                                    int cus, bool bf16, hipStream_t s) {
  if (t.P_max > MAX_P || t.ngroups < 1 || n < 1 || !t.Bsp || !t.tscale || !t.groups) return hipErrorInvalidValue;
  // steps of 32 distances, run in pairs and read one step ahead
  const int halo = 32 * ((t.P_max + 31) / 32 + 3);
  // Banks of two tiles (z_max 8 .. 15; narrower ones run in FP32): four parts to a
  // strip where every workgroup has that many.  2^22 bins in FP16, z_max 8 and 15:
  // 196 and 263 us in blocks of 128 bins, 170 and 250 in 512.
  const bool narrow = t.ngroups == 1 && t.groups[0].tiles == 2 && n >= (int64_t)4 * SBLK_BINS * 2 * cus;
  const int bins = (narrow ? 4 : 1) * SBLK_BINS;
  if (bins + 2 * halo > 256 * SPER) return hipErrorInvalidValue;
  const int64_t blocks = (n + bins - 1) / bins;
  const unsigned grid = (unsigned)std::min<int64_t>(blocks, 2 * cus);
  for (int g = 0; g < t.ngroups; ++g) {
    const DirectGroup& gr = t.groups[g];
    hipError_t e = hipErrorInvalidValue;
    switch (gr.tiles) {
#define FDAS_SPLIT_CASE(TG, NB)                                                                            \
  e = bf16 ? launch_split_group<__bf16, TG, NB>(x, n, fop, ld, t, gr, halo, (int)blocks, grid, s)          \
           : launch_split_group<_Float16, TG, NB>(x, n, fop, ld, t, gr, halo, (int)blocks, grid, s);       \
  break;
      case 2:
        if (narrow) {
          FDAS_SPLIT_CASE(2, 4)
        }
        FDAS_SPLIT_CASE(2, 1)
      case 3: FDAS_SPLIT_CASE(3, 1)
      case 4: FDAS_SPLIT_CASE(4, 1)
      case 5: FDAS_SPLIT_CASE(5, 1)
      case 6: FDAS_SPLIT_CASE(6, 1)
#undef FDAS_SPLIT_CASE
      default:
        break;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_direct_conv(const float2* x, int64_t n, float* fop, int64_t ld, const DirectTables& t, int cus,
                              hipStream_t s) {
  if (t.P_max > MAX_P || t.ngroups < 1 || n < 1 || !t.Bpk || !t.groups) return hipErrorInvalidValue;
  const int64_t blocks = (n + BLK_BINS - 1) / BLK_BINS;
  // A workgroup stages its operand once for a contiguous range of blocks.  Two to a
  // compute unit are all that the registers of large groups allow; one tile takes 80,
  // and six hide each other's staging (z_max 0, 2^22 bins: 63 -> 43 us, z_max 7: 142 ->
  // 123).
  const bool one = t.ngroups == 1 && t.groups[0].tiles == 1;
  const unsigned grid = (unsigned)std::min<int64_t>(blocks, (one ? 6 : 2) * cus);
  for (int g = 0; g < t.ngroups; ++g) {
    const DirectGroup& gr = t.groups[g];
    const size_t lds = sizeof(float) * 64 * (size_t)(gr.count + gr.tiles) +
                       sizeof(float2) * 2 * (size_t)(BLK_BINS + 2 * (t.P_max + FOLD_PAD));
    switch (gr.tiles) {
#define FDAS_DIRECT_CASE(TG)                                                                                        \
  case TG: {                                                                                                        \
    if (lds > 65536) {                                                                                              \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_direct_conv<TG>),                          \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                     \
      if (e != hipSuccess) return e;                                                                                \
    }                                                                                                               \
    hipLaunchKernelGGL(k_direct_conv<TG>, dim3(grid), dim3(DW * 64), lds, s, x, n, fop, ld,                         \
                       reinterpret_cast<const float4*>(t.Bpk) + (size_t)16 * gr.offset, t.steps + gr.first,         \
                       t.rows + 16 * gr.first, t.edge + 8 * gr.first, t.edge_tap + 16 * gr.first, gr.count, t.P_max, \
                       (int)blocks);                                                                                \
    break;                                                                                                          \
  }
      FDAS_DIRECT_CASE(1)
      FDAS_DIRECT_CASE(2)
      FDAS_DIRECT_CASE(3)
      FDAS_DIRECT_CASE(4)
      FDAS_DIRECT_CASE(5)
      FDAS_DIRECT_CASE(6)
#undef FDAS_DIRECT_CASE
      default:
        return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace fdas
