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
//     the operand (FP32 kernel), d = 0 with half the tap, and the unpaired tap
//     in a step of its own.
//
// MFMA mapping of the FP32 kernel (v_mfma_f32_16x16x4f32, one 16 x 16 FP32
// output block, K = 4 distances):
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
// Work split: a workgroup = 4 waves covers 256 consecutive bins (FP32), a wave 4
// sub-tiles of 16 bins.

#include <algorithm>

#include "fdas_internal.h"

namespace fdas {
namespace {

// Two adjacent FOP values stored non-temporally: the plane is written once and
// read back only after the whole convolution, so it should not stay in the
// caches (the same policy as the overlap-save kernel's stores).
__device__ __forceinline__ void store2_nt(float* dst, float a, float b) {
  typedef float f2v __attribute__((ext_vector_type(2)));
  const f2v v = {a, b};
  __builtin_nontemporal_store(v, reinterpret_cast<f2v*>(dst));
}

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

// A group of TG tiles at once: tiles[t] = {folded steps, 0, 0, 0} (steps fall
// with t), rows[t * 16 + col] = FOP row of column col (-1: none),
// edge[t * 8 + slot] = L/2 of the slot's template.  The operand holds 64
// floats per (step, tile) in lane order: step p (lane group kk: distance
// d = 4 p + kk) of every tile with more than p steps, then two edge steps per
// tile (step e: the taps at -edge[4 e + kk]).  Dynamic LDS: the operand
// (`count` entries) and two strips of X (Pm + 8 bins on either side of the
// workgroup's bins).
//
// Bound by the FP32 matrix pipe (2 instructions of 32 cycles per 4 distances,
// 16 bins and 8 |z|).  A folded operand is read and added once and used by
// every tile that still runs at its distance: the accumulators of all tiles
// stay in registers (8 per tile and sub-tile), which leaves two waves per
// SIMD, so the next step's LDS reads are issued before this step's products.
// Measured on 2^20 bins and 85 templates: 0.393 ms, 127 TFLOP/s issued, matrix
// pipe busy 80 %; without the two symmetries 1.265 ms; one tile at a time with
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
__device__ __forceinline__ void fold_steps(FoldState<TG>& st, const int4* __restrict__ tiles, int p) {
  // tiles 0 .. T-1 still run: to the end of tile T-1
  const int end = tiles[T - 1].x;
  for (; p < end; ++p) {
    float fr[SUB], fi[SUB], bv[T];
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      fr[s] = st.f[s].x + st.r[s].x;
      fi[s] = st.f[s].y + st.r[s].y;
    }
#pragma unroll
    for (int t = 0; t < T; ++t) bv[t] = st.b[t];
    // reads past the last step stay inside the strip's padding and the edge steps
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
  if constexpr (T > 1) fold_steps<TG, T - 1>(st, tiles, p);
}

template <int TG>
__global__ __launch_bounds__(DW * 64, 2) void k_direct_conv(
    const float2* __restrict__ x, int64_t n, float* __restrict__ fop, int64_t ld, const float4* __restrict__ Bpk,
    const int4* __restrict__ tiles, const int* __restrict__ rows, const int* __restrict__ edge, int count, int Pm,
    int blocks) {
  extern __shared__ float4 lds4[];
  const int tid = threadIdx.x;
  const int halo = Pm + FOLD_PAD;
  const int strip = BLK_BINS + 2 * halo;  // bins jb - halo + u
  const float* bs = reinterpret_cast<const float*>(lds4);
  float2* xs = reinterpret_cast<float2*>(lds4 + 16 * count);
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
      cur[u] = (idx >= 0 && idx < n) ? x[idx] : make_float2(0.0f, 0.0f);
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
    fold_steps<TG, TG>(st, tiles, 0);
    const int64_t left = n - (jb + 4 * kk);  // bins from this lane's first to the end
    const bool whole = jb + WAVE_BINS <= n;  // uniform
    const float* eb = bs + 64 * (count - 2 * TG) + lane;
#pragma unroll
    for (int t = 0; t < TG; ++t) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float2* __restrict__ ed = centre - edge[t * 8 + 4 * e + kk];
        const float bv = eb[64 * (2 * t + e)];
#pragma unroll
        for (int s = 0; s < SUB; ++s) {
          const float2 f = ed[16 * s];
          st.ar[t][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.x, bv, st.ar[t][s], 0, 0, 0);
          st.ai[t][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.y, bv, st.ai[t][s], 0, 0, 0);
        }
      }
      const int row = rows[t * 16 + m];
      float* dst = fop + (size_t)(row < 0 ? 0 : row) * ld + jb + 4 * kk;
      if (whole) {
#pragma unroll
        for (int s = 0; s < SUB; ++s) pair_store(st.ar[t][s], st.ai[t][s], row, dst + 16 * s, 4);
      } else {
#pragma unroll
        for (int s = 0; s < SUB; ++s) pair_store(st.ar[t][s], st.ai[t][s], row, dst + 16 * s, left - 16 * s);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Split precision on the 16-bit matrix cores (v_mfma_f32_16x16x32_{f16,bf16}):
// every operand value v is carried as hi = round16(v), lo = round16(v - hi),
// and a product as hi*hi + hi*lo + lo*hi with FP32 accumulation (the lo*lo
// term, ~2^-22 of the product for FP16, is dropped).  One instruction takes
// 16 bins x 16 complex taps x 8 templates: K = 32 real values, lane group
// g = lane/16 holding taps 4g..4g+3 of the 16 as (Re, Im) pairs.  FP16 has a
// narrow exponent range, so the block's strip of X is scaled by 2^ex
// (largest |Re|, |Im| brought to about 2^14) and each template tile by a
// plan-chosen 2^eh; both scalings are exact and undone on the accumulator.

constexpr int SDW = 4;                       // waves per workgroup
constexpr int SSUB = 8;                      // 16-bin sub-tiles per wave
constexpr int SWAVE_BINS = 16 * SSUB;        // 128
constexpr int SBLK_BINS = SDW * SWAVE_BINS;   // 512

template <typename T>
struct Split16;

template <>
struct Split16<_Float16> {
  typedef _Float16 v8 __attribute__((ext_vector_type(8)));
  static __device__ __forceinline__ unsigned short bits(float v) {
    const _Float16 h = (_Float16)v;
    return __builtin_bit_cast(unsigned short, h);
  }
  static __device__ __forceinline__ float value(unsigned short b) {
    return (float)__builtin_bit_cast(_Float16, b);
  }
  static __device__ __forceinline__ v4f mfma(const v8& a, const v8& b, const v4f& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

template <>
struct Split16<__bf16> {
  typedef __bf16 v8 __attribute__((ext_vector_type(8)));
  static __device__ __forceinline__ unsigned short bits(float v) {
    const __bf16 h = (__bf16)v;  // round to nearest even
    return __builtin_bit_cast(unsigned short, h);
  }
  static __device__ __forceinline__ float value(unsigned short b) {
    return __uint_as_float((unsigned)b << 16);
  }
  static __device__ __forceinline__ v4f mfma(const v8& a, const v8& b, const v4f& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// 8 16-bit values from 4 (possibly only 4-byte aligned) 32-bit LDS words
template <typename V8>
__device__ __forceinline__ V8 lds_v8(const unsigned* __restrict__ p) {
  uint4 u;
  u.x = p[0];
  u.y = p[1];
  u.z = p[2];
  u.w = p[3];
  return __builtin_bit_cast(V8, u);
}

// tiles[g] = {P, first 16-tap group in Bsp, member count, P rounded up to 8};
// Bsp holds per tile and 16-tap group 64 lanes x 8 hi values, then 64 x 8 lo
// values (2 KiB); tscale[g] = 2^-eh of the tile.  Dynamic LDS: hi and lo
// strips of X (2 x (SBLK_BINS + 2 Pm + 16) words) and one tile's operand.
// Four waves per SIMD (at most 128 registers: the accumulators stay in VGPRs)
// keep the 16-bit matrix pipe busier than the compiler's default of three
// with AGPR accumulators (measured 1.67 against 1.85 ms on 2^22 bins).
template <typename T>
__global__ __launch_bounds__(SDW * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_direct_conv_split(const float2* __restrict__ x, int64_t n,
                                                               float* __restrict__ fop, int64_t ld,
                                                               const uint4* __restrict__ Bsp,
                                                               const int4* __restrict__ tiles,
                                                               const float* __restrict__ tscale,
                                                               const int* __restrict__ rows, int ntiles, int Pm) {
  typedef Split16<T> S;
  typedef typename S::v8 v8;
  extern __shared__ uint4 lds_u4[];
  __shared__ unsigned s_max;
  unsigned* xhi = reinterpret_cast<unsigned*>(lds_u4);
  const int tid = threadIdx.x;
  const int64_t jb = (int64_t)blockIdx.x * SBLK_BINS;
  const int strip = SBLK_BINS + 2 * Pm + 16;  // even
  unsigned* xlo = xhi + strip;
  uint4* bs = reinterpret_cast<uint4*>(xlo + strip);
  if (tid == 0) s_max = 0u;
  __syncthreads();
  // largest |Re|, |Im| of the strip (bit patterns of non-negative floats order like integers)
  {
    float mx = 0.0f;
    for (int u = tid; u < strip; u += SDW * 64) {
      const int64_t idx = jb - Pm + u;
      if (idx >= 0 && idx < n) {
        const float2 v = x[idx];
        mx = fmaxf(mx, fmaxf(fabsf(v.x), fabsf(v.y)));
      }
    }
    atomicMax(&s_max, __float_as_uint(mx));
  }
  __syncthreads();
  int ex = 0;
  {
    const float mx = __uint_as_float(s_max);
    if (mx > 0.0f && mx < 3.0e38f) ex = 14 - ilogbf(mx);  // 2^14 <= max * 2^ex < 2^15
  }
  for (int u = tid; u < strip; u += SDW * 64) {
    const int64_t idx = jb - Pm + u;
    const float2 v = (idx >= 0 && idx < n) ? x[idx] : make_float2(0.0f, 0.0f);
    const float re = ldexpf(v.x, ex), im = ldexpf(v.y, ex);
    const unsigned short hr = S::bits(re), hi_ = S::bits(im);
    const unsigned short lr = S::bits(re - S::value(hr)), li = S::bits(im - S::value(hi_));
    xhi[u] = (unsigned)hr | ((unsigned)hi_ << 16);
    xlo[u] = (unsigned)lr | ((unsigned)li << 16);
  }

  const int lane = tid & 63;
  const int w = tid >> 6;
  const int m = lane & 15;
  const int kg = lane >> 4;  // lane group: taps 4kg..4kg+3 of each 16
  const int col = lane & 15;
  const int slot = col >> 1;
  const int c = col & 1;

  for (int g = 0; g < ntiles; ++g) {
    const int4 tg = tiles[g];
    const int P = tg.x;
    const int groups16 = tg.w / 8;  // P8 pairs = 2 P8 taps = P8/8 groups of 16 taps
    {
      const uint4* __restrict__ src = Bsp + (size_t)tg.y * 128;  // 2 KiB = 128 uint4 per group, hi then lo
      __syncthreads();
      for (int i = tid; i < groups16 * 128; i += SDW * 64) bs[i] = src[i];
      __syncthreads();
    }
    // strip word of this lane's first tap for group 0, sub-tile 0.  The A
    // operand of sub-tile s and tap group q starts at a0 + 16 (s + q): it
    // depends on s + q only, so a window of SSUB operands slides along q, one
    // new (hi, lo) pair loaded per group (ring slot (s + q) % SSUB, a
    // compile-time index inside the unrolled block of SSUB groups).  Loading
    // the next group's operands one group ahead was slower (more registers,
    // two waves per SIMD instead of three).
    const int a0 = w * SWAVE_BINS + m + Pm - P + 4 * kg;
    v4f acc[SSUB];
#pragma unroll
    for (int s = 0; s < SSUB; ++s) acc[s] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    v8 ah[SSUB], al[SSUB];
#pragma unroll
    for (int i = 0; i < SSUB - 1; ++i) {
      ah[i] = lds_v8<v8>(xhi + a0 + 16 * i);
      al[i] = lds_v8<v8>(xlo + a0 + 16 * i);
    }
    for (int q0 = 0; q0 < groups16; q0 += SSUB) {
#pragma unroll
      for (int dq = 0; dq < SSUB; ++dq) {
        const int q = q0 + dq;
        if (q < groups16) {  // uniform
          ah[(dq + SSUB - 1) % SSUB] = lds_v8<v8>(xhi + a0 + 16 * (q + SSUB - 1));
          al[(dq + SSUB - 1) % SSUB] = lds_v8<v8>(xlo + a0 + 16 * (q + SSUB - 1));
          const v8 b_hi = __builtin_bit_cast(v8, bs[q * 128 + lane]);
          const v8 b_lo = __builtin_bit_cast(v8, bs[q * 128 + 64 + lane]);
#pragma unroll
          for (int s = 0; s < SSUB; ++s) {
            const v8 a_hi = ah[(dq + s) % SSUB];
            const v8 a_lo = al[(dq + s) % SSUB];
            acc[s] = S::mfma(a_hi, b_hi, acc[s]);
            acc[s] = S::mfma(a_hi, b_lo, acc[s]);
            acc[s] = S::mfma(a_lo, b_hi, acc[s]);
          }
        }
      }
    }
    const float unscale = ldexpf(tscale[g], -ex);
    const int row = slot < tg.z ? rows[g * 8 + slot] : -1;
#pragma unroll
    for (int s = 0; s < SSUB; ++s) {
      float pw[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float y = acc[s][v] * unscale;
        const float o = swap_pair(y);
        pw[v] = y * y + o * o;
      }
      if (row >= 0) {
        const int64_t j = jb + w * SWAVE_BINS + 16 * s + 4 * kg + 2 * c;
        float* dst = fop + (size_t)row * ld + j;
        const float p0 = c ? pw[2] : pw[0];
        const float p1 = c ? pw[3] : pw[1];
        if (j + 2 <= n) {
          store2_nt(dst, p0, p1);
        } else if (j < n) {
          __builtin_nontemporal_store(p0, dst);
        }
      }
    }
  }
}

}  // namespace

int direct_block_bins() { return SBLK_BINS; }
int direct_max_half_taps() { return MAX_P; }
size_t direct_lds_bytes(int P_max, int P8_max) {
  return sizeof(float) * (2 * (size_t)(SBLK_BINS + 2 * P_max + 16) + 64 * (size_t)P8_max);
}

hipError_t launch_direct_conv_split(const float2* x, int64_t n, float* fop, int64_t ld, const DirectTables& t,
                                    bool bf16, hipStream_t s) {
  if (t.P_max > MAX_P || t.ntiles < 1 || n < 1 || !t.Bsp || !t.tscale) return hipErrorInvalidValue;
  const int64_t blocks = (n + SBLK_BINS - 1) / SBLK_BINS;
  const size_t lds = direct_lds_bytes(t.P_max, t.P8_max);
  const void* fn = bf16 ? reinterpret_cast<const void*>(k_direct_conv_split<__bf16>)
                        : reinterpret_cast<const void*>(k_direct_conv_split<_Float16>);
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (bf16)
    hipLaunchKernelGGL(k_direct_conv_split<__bf16>, dim3((unsigned)blocks), dim3(SDW * 64), lds, s, x, n, fop, ld,
                       t.Bsp, t.tiles, t.tscale, t.rows, t.ntiles, t.P_max);
  else
    hipLaunchKernelGGL(k_direct_conv_split<_Float16>, dim3((unsigned)blocks), dim3(SDW * 64), lds, s, x, n, fop, ld,
                       t.Bsp, t.tiles, t.tscale, t.rows, t.ntiles, t.P_max);
  return hipGetLastError();
}

hipError_t launch_direct_conv(const float2* x, int64_t n, float* fop, int64_t ld, const DirectTables& t, int cus,
                              hipStream_t s) {
  if (t.P_max > MAX_P || t.ngroups < 1 || n < 1 || !t.Bpk || !t.edge || !t.groups) return hipErrorInvalidValue;
  const int64_t blocks = (n + BLK_BINS - 1) / BLK_BINS;
  // a workgroup stages its operand once for a contiguous range of blocks
  const unsigned grid = (unsigned)std::min<int64_t>(blocks, 2 * cus);
  for (int g = 0; g < t.ngroups; ++g) {
    const DirectGroup& gr = t.groups[g];
    const size_t lds = sizeof(float) * 64 * (size_t)gr.count +
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
                       reinterpret_cast<const float4*>(t.Bpk) + (size_t)16 * gr.offset, t.tiles + gr.first,         \
                       t.rows + 16 * gr.first, t.edge + 8 * gr.first, gr.count, t.P_max, (int)blocks);              \
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
