// Training kernels of the learned block pre-screen (the network is described in
// k_prescreen.hip): forward pass recording activations and max-pool positions,
// data gradients, weight gradients, and the sums of their partials.
//
// The 32-channel layers run on the FP32 matrix cores (v_mfma_f32_16x16x4f32).
// The instruction accumulates its four products one after another with a
// rounding each, in k order, starting from the C operand (checked bit for bit
// against a chain of fmaf), so a convolution whose K index runs over (input
// channel, tap) in order gives the bits of the scalar chain
// acc = fmaf(w, x, acc) that starts at the bias: max-pool positions and ReLU
// signs do not depend on the unit that computed them.
//
// Gradients of pooled layers stay compact: g[b][c][p] is the gradient of pooled
// output p, at position F p + arg[b][c][p] of the layer below its max-pool; a
// workgroup expands its tile when it stages it in LDS, so the three zeros of
// every window are never in memory (the dense form moved 134 MB per 256 blocks
// for the first layer alone).  The last layer is the same with F = 64.

#include <algorithm>

#include "fdas_internal.h"

namespace fdas {
namespace {

constexpr int PC = 32;      // channels
constexpr int PK = 9;       // kernel taps
constexpr int PBLK = 4096;  // bins per block

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f(unsigned short b) { return __uint_as_float((unsigned)b << 16); }
__device__ __forceinline__ float softplus(float x) { return log1pf(expf(-fabsf(x))) + fmaxf(x, 0.0f); }

// Layer 1 forward: one input channel, bias, ReLU, max-pool.  Workgroup = 256
// positions of one sample; a thread owns 32 consecutive outputs of a channel.
constexpr int PT = 256, PQ = 32;
__global__ __launch_bounds__(256) void k_ps_conv1(const float* __restrict__ x, const unsigned short* __restrict__ w,
                                                  const unsigned short* __restrict__ bias, float* __restrict__ out,
                                                  unsigned char* __restrict__ arg) {
  // word u of the tile at u + u / 32: the 8 threads of a channel read windows
  // 32 positions apart, which then fall in different banks
  __shared__ float xs[PT + 8 + (PT + 8) / 32 + 1];
  const int b = blockIdx.y;
  const int t0 = blockIdx.x * PT;
  const int tid = threadIdx.x;
  const float* xb = x + (size_t)b * PBLK;
  for (int u = tid; u < PT + 8; u += 256) {
    const int t = t0 + u - 4;
    xs[u + u / 32] = (t >= 0 && t < PBLK) ? xb[t] : 0.0f;
  }
  const int o = tid / 8, q0 = (tid % 8) * PQ;
  float wk[PK];
#pragma unroll
  for (int k = 0; k < PK; ++k) wk[k] = bf16_to_f(w[o * PK + k]);
  const float bo = bf16_to_f(bias[o]);
  __syncthreads();
  float acc[PQ], xw[PQ + 8];
#pragma unroll
  for (int u = 0; u < PQ + 8; ++u) xw[u] = xs[q0 + u + (q0 + u) / 32];
#pragma unroll
  for (int q = 0; q < PQ; ++q) {
    acc[q] = bo;
#pragma unroll
    for (int k = 0; k < PK; ++k) acc[q] = fmaf(wk[k], xw[q + k], acc[q]);
  }
  // the thread's 8 pooled values are consecutive and 32-byte aligned
  float best[PQ / 4];
  unsigned char ba[PQ / 4];
#pragma unroll
  for (int p = 0; p < PQ / 4; ++p) {
    best[p] = fmaxf(acc[4 * p], 0.0f);
    ba[p] = 0;
#pragma unroll
    for (int qq = 1; qq < 4; ++qq) {
      const float v = fmaxf(acc[4 * p + qq], 0.0f);
      if (v > best[p]) {
        best[p] = v;
        ba[p] = (unsigned char)qq;
      }
    }
  }
  const size_t o0 = ((size_t)b * PC + o) * (PBLK / 4) + (t0 + q0) / 4;
  float4* dst = reinterpret_cast<float4*>(out + o0);
  dst[0] = make_float4(best[0], best[1], best[2], best[3]);
  dst[1] = make_float4(best[4], best[5], best[6], best[7]);
  *reinterpret_cast<uint2*>(arg + o0) = *reinterpret_cast<const uint2*>(ba);
}

// Four consecutive positions t .. t + 3 (t a multiple of 4) of row `row` (sample
// x channel) of an expanded gradient: g has one value per F = 2^fs positions.
__device__ __forceinline__ float4 expand4(const float* __restrict__ g, const unsigned char* __restrict__ arg, size_t row,
                                          int L, int fs, int t) {
  const size_t at = row * (size_t)(L >> fs) + (t >> fs);
  const float v = g[at];
  const int a = (int)arg[at] - (t & ((1 << fs) - 1));
  return make_float4(a == 0 ? v : 0.0f, a == 1 ? v : 0.0f, a == 2 ? v : 0.0f, a == 3 ? v : 0.0f);
}

// Weight operands of k_ps_conv32 in lane order, one per layer 2..4 and direction
// (0: forward, 1: data gradient) and half of the output channels: word
// (((l * 2 + dir) * 2 + half) * 72 + p) * 64 + lane.  Written whenever the BF16
// weights change: a wave then loads its 72 operands as 72 coalesced words
// instead of gathering them from 16 rows each.
constexpr int kOperandWords = 3 * 2 * 2 * 72 * 64;
__global__ __launch_bounds__(256) void k_ps_operands(const unsigned short* __restrict__ w0,
                                                     const unsigned short* __restrict__ w1,
                                                     const unsigned short* __restrict__ w2, float* __restrict__ wt) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= kOperandWords) return;
  const int lane = i & 63, p = (i / 64) % 72, half = (i / (64 * 72)) & 1, dir = (i / (64 * 72 * 2)) & 1,
            l = i / (64 * 72 * 4);
  const unsigned short* w = l == 0 ? w0 : (l == 1 ? w1 : w2);
  const int c = 16 * half + (lane & 15), kappa = 4 * p + (lane >> 4), i2 = kappa / PK, k = kappa % PK;
  // forward: output channel c, input i2, tap k; data gradient: output channel (of
  // the layer below) c, input i2, flipped tap
  wt[i] = bf16_to_f(dir == 0 ? w[(c * PC + i2) * PK + k] : w[(i2 * PC + c) * PK + (PK - 1 - k)]);
}

// Per-sample results of the last layer and the head.
struct HeadOut {
  const float* labels;
  float pos_weight;
  const unsigned short *wf, *bf;
  float* logits;
  float* loss;        // [nb] loss / nb
  float* dlogit;      // [nb]
  float* h;           // [nb][32] channel maxima
  float* g;           // [nb][32] their gradients
  unsigned char* at;  // [nb][32] their positions
};

// 32 -> 32 channel convolution, kernel 9: tiles of TP = 64 SUBT positions of one
// sample; 8 waves = 2 halves of the output channels x 4 groups of 16 SUBT
// positions.  K step p holds kappa = 4 p + kk, kappa = 9 i + tap; a wave keeps
// its 72 weight operands in registers over all its tiles, and an activation
// operand is one LDS word at an address whose lane part repeats every 9 steps
// (4 channels), so the loop is LDS reads and matrix instructions only.
// Row stride = 32 (mod 64) words: the lane groups that cross from tap 8 to the
// next channel read other banks than those before it.
// MODE 0: forward, bias, ReLU, max-pool by 4 -> out, out_arg [nb][32][L / 4].
// MODE 1: data gradient (weights transposed and flipped, input expanded from
//         in / in_arg with F = 2^fs), masked by act > 0 -> out [nb][32][L].
// MODE 2: forward of the last layer (TP = L = 64) and the head.
// Measured on 256 blocks, the three layers together: 71 us forward (with the
// head; 177 us on the vector units) and 69 us for the data gradients (206 us);
// the matrix pipe's floor is 40 us each.
template <int SUBT, int MODE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_ps_conv32(
    const float* __restrict__ in, const unsigned char* __restrict__ in_arg, int L, int fs, int nb,
    const float* __restrict__ wt, const unsigned short* __restrict__ bias, float* __restrict__ out,
    unsigned char* __restrict__ out_arg, const float* __restrict__ act, HeadOut ho) {
  constexpr int TP = 64 * SUBT;
  constexpr int XW = TP + 32;
  constexpr int QUADS = (TP + 8) / 4;
  static_assert(XW % 64 == 32, "bank layout");
  __shared__ float xs[PC * XW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m = lane & 15, kk = lane >> 4;
  const int half = wv & 1, pos0 = (wv >> 1) * 16 * SUBT;
  const int c = 16 * half + m;  // this lane's output channel
  float B[72];
#pragma unroll
  for (int p = 0; p < 72; ++p) B[p] = wt[(half * 72 + p) * 64 + lane];
  const float bo = MODE == 1 ? 0.0f : bf16_to_f(bias[c]);
  int off[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int kappa = 4 * q + kk;
    off[q] = (kappa / PK) * XW + kappa % PK + pos0 + m;
  }
  __shared__ float s_wf[PC + 1];
  if (MODE == 2 && tid <= PC) s_wf[tid] = bf16_to_f(tid < PC ? ho.wf[tid] : ho.bf[0]);
  const int per = L / TP;
  for (int tile = blockIdx.x; tile < nb * per; tile += gridDim.x) {
    const int b = tile / per, t0 = (tile - b * per) * TP;
    const float label = MODE == 2 && tid == 0 ? ho.labels[b] : 0.0f;
    __syncthreads();  // the previous tile is no longer read
    for (int e = tid; e < PC * QUADS; e += 512) {
      const int i = e / QUADS, q = e - i * QUADS;
      const int t = t0 - 4 + 4 * q;
      float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (t >= 0 && t < L) {
        const size_t row = (size_t)b * PC + i;
        if (MODE == 1)
          v = expand4(in, in_arg, row, L, fs, t);
        else
          v = *reinterpret_cast<const float4*>(in + row * L + t);
      }
      *reinterpret_cast<float4*>(xs + i * XW + 4 * q) = v;
    }
    __syncthreads();
    v4f acc[SUBT];
#pragma unroll
    for (int s = 0; s < SUBT; ++s) acc[s] = v4f{bo, bo, bo, bo};
#pragma unroll
    for (int p = 0; p < 72; ++p)
#pragma unroll
      for (int s = 0; s < SUBT; ++s)
        acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[off[p % 9] + (p / 9) * 4 * XW + 16 * s], B[p], acc[s], 0, 0, 0);
    // lane: channel c, positions t0 + pos0 + 16 s + 4 kk + v
    if (MODE == 0) {
      float best[4];
      unsigned ba = 0;  // position of the maximum of sub-tile s in byte s
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        best[s] = fmaxf(acc[s % SUBT][0], 0.0f);
        unsigned a = 0;
#pragma unroll
        for (int v = 1; v < 4; ++v) {
          const float r = fmaxf(acc[s % SUBT][v], 0.0f);
          if (r > best[s]) {
            best[s] = r;
            a = v;
          }
        }
        ba |= a << (8 * s);
      }
      // pooled output 4 s + kk sits in lane group kk: a 4 x 4 transposition over
      // (s, kk) gives lane group kk the outputs 4 kk .. 4 kk + 3, stored as 16 bytes
#pragma unroll
      for (int z = 1; z < 4; z <<= 1) {
        const bool hi = (kk & z) != 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if (s & z) continue;
          const float got = __shfl_xor(hi ? best[s] : best[s | z], 16 * z);
          if (hi)
            best[s] = got;
          else
            best[s | z] = got;
        }
        const unsigned lo_mask = z == 1 ? 0x00ff00ffu : 0x0000ffffu;  // bytes s with bit z clear
        const unsigned got = __shfl_xor(hi ? ba & lo_mask : (ba & ~lo_mask) >> (8 * z), 16 * z);
        ba = hi ? (ba & ~lo_mask) | got : (ba & lo_mask) | (got << (8 * z));
      }
      const size_t at = ((size_t)b * PC + c) * (L / 4) + (t0 + pos0) / 4 + 4 * kk;
      *reinterpret_cast<float4*>(out + at) = make_float4(best[0], best[1], best[2], best[3]);
      *reinterpret_cast<unsigned*>(out_arg + at) = ba;
    } else if (MODE == 1) {
#pragma unroll
      for (int s = 0; s < SUBT; ++s) {
        const size_t at = ((size_t)b * PC + c) * L + t0 + pos0 + 16 * s + 4 * kk;
        const float4 a = *reinterpret_cast<const float4*>(act + at);
        *reinterpret_cast<float4*>(out + at) =
            make_float4(a.x > 0.0f ? acc[s][0] : 0.0f, a.y > 0.0f ? acc[s][1] : 0.0f, a.z > 0.0f ? acc[s][2] : 0.0f,
                        a.w > 0.0f ? acc[s][3] : 0.0f);
      }
    } else {
      __shared__ float s_best[4][PC];
      __shared__ int s_at[4][PC];
      __shared__ float s_h[PC];
      __shared__ float s_dl;
      // first maximum over this wave's 16 positions of a channel
      float best = fmaxf(acc[0][0], 0.0f);
      int at = pos0 + 4 * kk;
#pragma unroll
      for (int v = 1; v < 4; ++v) {
        const float r = fmaxf(acc[0][v], 0.0f);
        if (r > best) {
          best = r;
          at = pos0 + 4 * kk + v;
        }
      }
#pragma unroll
      for (int o = 16; o < 64; o <<= 1) {
        const float ob = __shfl_xor(best, o);
        const int oa = __shfl_xor(at, o);
        if (ob > best || (ob == best && oa < at)) {
          best = ob;
          at = oa;
        }
      }
      if (kk == 0) {
        s_best[wv >> 1][c] = best;
        s_at[wv >> 1][c] = at;
      }
      __syncthreads();
      if (tid < PC) {
        best = s_best[0][tid];
        at = s_at[0][tid];
#pragma unroll
        for (int q = 1; q < 4; ++q)
          if (s_best[q][tid] > best) {
            best = s_best[q][tid];
            at = s_at[q][tid];
          }
        s_h[tid] = best;
      }
      __syncthreads();
      if (tid == 0) {
        float lg = s_wf[PC];
#pragma unroll
        for (int k = 0; k < PC; ++k) lg = fmaf(s_wf[k], s_h[k], lg);
        ho.logits[b] = lg;
        const float y = label;
        const float sg = 1.0f / (1.0f + expf(-lg));
        ho.loss[b] = (ho.pos_weight * y * softplus(-lg) + (1.0f - y) * softplus(lg)) / nb;
        const float dl = (ho.pos_weight * y * (sg - 1.0f) + (1.0f - y) * sg) / nb;
        ho.dlogit[b] = dl;
        s_dl = dl;
      }
      __syncthreads();
      if (tid < PC) {
        const size_t o = (size_t)b * PC + tid;
        ho.h[o] = best;
        ho.at[o] = (unsigned char)at;
        ho.g[o] = best > 0.0f ? s_dl * s_wf[tid] : 0.0f;
      }
    }
  }
}

// Weight and bias gradients of the three 32-channel layers in one launch:
// dW[o][i][k] = sum over samples and positions of dz[b][o][t] x[b][i][t + k - 4],
// a product with K = positions.  A workgroup walks units of min(128, L)
// positions of one sample; each of its 12 waves (three per SIMD) owns three taps
// of 16 x 16 channel pairs, so nothing is summed across waves; the workgroup's partial
// sums go to `part` (no atomics: the sums do not depend on the run) and
// k_ps_reduce adds them up.  Row strides of 4 (mod 8) x odd words put the 16
// rows x 4 positions of an operand on 64 banks.
// Measured (256 blocks, all three layers): 70 us against 655 us with scalar
// windows and atomics; the matrix pipe's floor is 41 us.  Nine waves of one tap
// each (three on one SIMD, two on the others) took 81 us.
struct WgJob {
  const float* g;  // compact gradient, F = 2^fs
  const unsigned char* arg;
  const float* x;
  int L, fs;
  int wg0, nwg;  // its workgroups
};
struct WgJobs {
  WgJob j[3];
};

constexpr int WT = 128;      // positions per unit
constexpr int WDS = WT + 4;  // 132
constexpr int WXS = WT + 12; // 140

constexpr int WTH = 768;
__global__ __launch_bounds__(WTH) void k_ps_wgrad32(WgJobs jobs, int nb, float* __restrict__ part,
                                                    float* __restrict__ partb) {
  __shared__ float ds[PC * WDS];
  __shared__ float xs[PC * WXS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m = lane & 15, kk = lane >> 4;
  const int a = wv & 1, h = (wv >> 1) & 1, k0 = 3 * (wv >> 2);  // output, input half; first tap
  const int q = (int)blockIdx.x >= jobs.j[2].wg0 ? 2 : (int)blockIdx.x >= jobs.j[1].wg0 ? 1 : 0;
  const WgJob jb = jobs.j[q];
  const int T = min(WT, jb.L), per = jb.L / T;
  const int dq = T / 4, xq = T / 4 + 2;  // quads of a row
  v4f acc[3];
  float accb = 0.0f;
#pragma unroll
  for (int j = 0; j < 3; ++j) acc[j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  for (int u = (int)blockIdx.x - jb.wg0; u < nb * per; u += jb.nwg) {
    const int b = u / per, t0 = (u - b * per) * T;
    __syncthreads();
    for (int e = tid; e < PC * xq; e += WTH) {
      const int i = e / xq, c = e - i * xq;
      const int t = t0 - 4 + 4 * c;
      float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (t >= 0 && t < jb.L) v = *reinterpret_cast<const float4*>(jb.x + ((size_t)b * PC + i) * jb.L + t);
      *reinterpret_cast<float4*>(xs + i * WXS + 4 * c) = v;
    }
    for (int e = tid; e < PC * dq; e += WTH) {
      const int o = e / dq, c = e - o * dq;
      *reinterpret_cast<float4*>(ds + o * WDS + 4 * c) =
          expand4(jb.g, jb.arg, (size_t)b * PC + o, jb.L, jb.fs, t0 + 4 * c);
    }
    __syncthreads();
    const float* dp = ds + (16 * a + m) * WDS + kk;
    const float* xp = xs + (16 * h + m) * WXS + kk + k0;
#pragma unroll 4
    for (int p = 0; p < T; p += 4) {
      const float d = dp[p];
#pragma unroll
      for (int j = 0; j < 3; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(d, xp[p + j], acc[j], 0, 0, 0);
      if (wv < 2) accb += d;  // uniform; h = 0, k0 = 0
    }
  }
  // lane: o = 16 a + 4 kk + v, i = 16 h + m
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    float* dst = part + (((size_t)blockIdx.x * PK + k0 + j) * 16 + a * 8 + h * 4) * 64 + lane;
#pragma unroll
    for (int v = 0; v < 4; ++v) dst[v * 64] = acc[j][v];
  }
  if (wv < 2) {
    accb += __shfl_xor(accb, 16);
    accb += __shfl_xor(accb, 32);
    if (kk == 0) partb[blockIdx.x * PC + 16 * a + m] = accb;
  }
}

// Weight and bias gradients of the one-channel layer: columns 0..8 are the taps
// f[t + k - 4], column 9 is one (the bias).  A workgroup walks units of 128
// positions, its 4 waves 32 each; their sums meet in LDS.  Bound by the compact
// gradient's read (46 MB for 256 blocks) and the latency of a unit's loads: 21 us
// with 2048 workgroups; 26 us with units of 256 positions and 1024, 42 us with 512;
// 188 us with the dense gradient and atomics.
constexpr int W1T = 128;
constexpr int W1DS = W1T + 4;
__global__ __launch_bounds__(256) void k_ps_wgrad1(const float* __restrict__ g, const unsigned char* __restrict__ arg,
                                                   const float* __restrict__ x, int nb, float* __restrict__ part) {
  __shared__ float ds[PC * W1DS];
  __shared__ float fs[W1T + 24];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m = lane & 15, kk = lane >> 4;
  constexpr int per = PBLK / W1T;
  v4f acc[2] = {v4f{0.0f, 0.0f, 0.0f, 0.0f}, v4f{0.0f, 0.0f, 0.0f, 0.0f}};
  for (int u = blockIdx.x; u < nb * per; u += gridDim.x) {
    const int b = u / per, t0 = (u - b * per) * W1T;
    __syncthreads();
    for (int e = tid; e < W1T + 24; e += 256) {
      const int t = t0 - 4 + e;
      fs[e] = (t >= 0 && t < PBLK) ? x[(size_t)b * PBLK + t] : 0.0f;
    }
    for (int e = tid; e < PC * (W1T / 4); e += 256) {
      const int o = e / (W1T / 4), c = e % (W1T / 4);
      *reinterpret_cast<float4*>(ds + o * W1DS + 4 * c) = expand4(g, arg, (size_t)b * PC + o, PBLK, 2, t0 + 4 * c);
    }
    __syncthreads();
    const float* dp = ds + m * W1DS + kk + W1T / 4 * wv;
    const float* xp = fs + kk + m + W1T / 4 * wv;
#pragma unroll 4
    for (int p = 0; p < W1T / 4; p += 4) {
      const float xv = m == PK ? 1.0f : xp[p];
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[p], xv, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[p + 16 * W1DS], xv, acc[1], 0, 0, 0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v) ds[(wv * 8 + a * 4 + v) * 64 + lane] = acc[a][v];
  __syncthreads();
  for (int e = tid; e < 512; e += 256)
    part[(size_t)blockIdx.x * 512 + e] = (ds[e] + ds[512 + e]) + (ds[1024 + e] + ds[1536 + e]);
}

// Sums of the partials, written to grad (and grad2 when given) and loss.
// Workgroup = 64 elements x 16 segments of the partials.
//   blocks 0 .. 431: 144 per 32-channel layer, weights in lane order
//   432 .. 434: their biases; 435: head and loss
//   436 .. 467: the one-channel layer, 16 elements x 64 segments each (its 2048
//   partials in 16 segments took longer than all the rest)
struct ReduceIn {
  const float *part, *partb, *part1;
  int wg0[3], nwg[3], n1;
  const float *dlogit, *h, *loss;
  int nb;
  int off_w[4], off_b[4], off_fc;
};
constexpr int kReduceBlocks = 3 * 144 + 3 + 1 + 32;

__global__ __launch_bounds__(1024) void k_ps_reduce(ReduceIn in, float* __restrict__ grad, float* __restrict__ grad2,
                                                    float* __restrict__ loss) {
  __shared__ float s_sum[16][64];
  const int lane = threadIdx.x & 63, seg = threadIdx.x >> 6;
  const int blk = blockIdx.x;
  float s = 0.0f;
  int dst = -1;
  bool to_loss = false;
  if (blk < 432) {
    const int q = blk / 144, r = blk - 144 * q;  // r = 16 k + register
    const float* p = in.part + ((size_t)in.wg0[q] * 144 + r) * 64 + lane;
#pragma unroll 8
    for (int i = seg; i < in.nwg[q]; i += 16) s += p[(size_t)i * 144 * 64];
    const int k = r >> 4, reg = r & 15;
    const int o = 16 * (reg >> 3) + 4 * (lane >> 4) + (reg & 3), i = 16 * ((reg >> 2) & 1) + (lane & 15);
    dst = in.off_w[3 - q] + (o * PC + i) * PK + k;
  } else if (blk < 435) {
    const int q = blk - 432;
    if (lane < PC) {
      const float* p = in.partb + (size_t)in.wg0[q] * PC + lane;
#pragma unroll 8
      for (int i = seg; i < in.nwg[q]; i += 16) s += p[(size_t)i * PC];
      dst = in.off_b[3 - q] + lane;
    }
  } else if (blk > 435) {
    // element e = 16 (blk - 436) + lane % 16: register e / 64, lane e % 64
    const int e = 16 * (blk - 436) + (lane & 15);
    const float* p = in.part1 + e;
#pragma unroll 8
    for (int i = 4 * seg + (lane >> 4); i < in.n1; i += 64) s += p[(size_t)i * 512];
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    const int reg = e >> 6, o = 16 * (reg >> 2) + 4 * ((e & 63) >> 4) + (reg & 3), col = e & 15;
    if (lane < 16) dst = col < PK ? in.off_w[0] + o * PK + col : col == PK ? in.off_b[0] + o : -1;
  } else {
    if (lane < PC) {
#pragma unroll 8
      for (int b = seg; b < in.nb; b += 16) s = fmaf(in.dlogit[b], in.h[(size_t)b * PC + lane], s);
      dst = in.off_fc + lane;
    } else if (lane == PC) {
#pragma unroll 8
      for (int b = seg; b < in.nb; b += 16) s += in.dlogit[b];
      dst = in.off_fc + PC;
    } else if (lane == PC + 1) {
#pragma unroll 8
      for (int b = seg; b < in.nb; b += 16) s += in.loss[b];
      to_loss = true;
    }
  }
  s_sum[seg][lane] = s;
  __syncthreads();
  if (seg == 0) {
    s = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) s += s_sum[q][lane];
    if (dst >= 0) {
      grad[dst] = s;
      if (grad2) grad2[dst] = s;
    }
    if (to_loss) loss[0] = s;
  }
}

constexpr int kWg32 = 512;  // workgroups of k_ps_wgrad32, two per compute unit
constexpr int kWg1 = 2048;

}  // namespace

size_t ps_operand_floats() { return kOperandWords; }

hipError_t ps_operands(const PsBuffers& pb, hipStream_t s) {
  const unsigned short* w = pb.wbf;
  hipLaunchKernelGGL(k_ps_operands, dim3((kOperandWords + 255) / 256), dim3(256), 0, s, w + ps_off_w(1),
                     w + ps_off_w(2), w + ps_off_w(3), pb.wtrain);
  return hipGetLastError();
}

size_t ps_partial_floats() { return (size_t)kWg32 * (PK * 16 * 64 + PC) + (size_t)kWg1 * 512; }

hipError_t ps_gradient(const PsBuffers& pb, const float* feats, int nb, const float* labels, float pos_weight,
                       float* logits, float* loss, float* grad2, hipStream_t s) {
  const unsigned short* w = pb.wbf;
  int off_w[4], off_b[4];
  for (int l = 0; l < 4; ++l) {
    off_w[l] = ps_off_w(l);
    off_b[l] = ps_off_b(l);
  }
  const int off_fc = ps_off_fc();
  const HeadOut none{};
  const HeadOut head{labels, pos_weight, w + off_fc, w + off_fc + PC, logits, pb.lossb, pb.dlogit, pb.h, pb.g4, pb.arg4};
  const dim3 blk(512);
  auto wt = [&](int l, int dir) { return pb.wtrain + (size_t)(l * 2 + dir) * 2 * 72 * 64; };
  auto grid = [&](int tiles) { return dim3((unsigned)std::min(tiles, 512)); };
  // forward, recording the activations and the max-pool positions
  hipLaunchKernelGGL(k_ps_conv1, dim3(PBLK / PT, nb), dim3(256), 0, s, feats, w + off_w[0], w + off_b[0], pb.a1, pb.arg1);
  hipLaunchKernelGGL((k_ps_conv32<4, 0>), grid(4 * nb), blk, 0, s, pb.a1, nullptr, 1024, 0, nb, wt(0, 0),
                     w + off_b[1], pb.a2, pb.arg2, nullptr, none);
  hipLaunchKernelGGL((k_ps_conv32<4, 0>), grid(nb), blk, 0, s, pb.a2, nullptr, 256, 0, nb, wt(1, 0), w + off_b[2],
                     pb.a3, pb.arg3, nullptr, none);
  hipLaunchKernelGGL((k_ps_conv32<1, 2>), grid(nb), blk, 0, s, pb.a3, nullptr, 64, 0, nb, wt(2, 0), w + off_b[3],
                     nullptr, nullptr, nullptr, head);
  // data gradients down to layer 1's pooled outputs
  hipLaunchKernelGGL((k_ps_conv32<1, 1>), grid(nb), blk, 0, s, pb.g4, pb.arg4, 64, 6, nb, wt(2, 1), nullptr, pb.g3,
                     nullptr, pb.a3, none);
  hipLaunchKernelGGL((k_ps_conv32<4, 1>), grid(nb), blk, 0, s, pb.g3, pb.arg3, 256, 2, nb, wt(1, 1), nullptr, pb.g2,
                     nullptr, pb.a2, none);
  hipLaunchKernelGGL((k_ps_conv32<4, 1>), grid(4 * nb), blk, 0, s, pb.g2, pb.arg2, 1024, 2, nb, wt(0, 1), nullptr,
                     pb.g1, nullptr, pb.a1, none);
  // weight gradients: workgroups in proportion to the units (8, 2 and a half per sample)
  WgJobs jobs;
  ReduceIn in{};
  const int n0 = std::min(8 * nb, 390), n1 = std::min(2 * nb, 98), n2 = std::min(nb, 24);
  static_assert(390 + 98 + 24 == kWg32, "every workgroup has a partial");
  jobs.j[2] = {pb.g2, pb.arg2, pb.a1, 1024, 2, n2 + n1, n0};
  jobs.j[1] = {pb.g3, pb.arg3, pb.a2, 256, 2, n2, n1};
  jobs.j[0] = {pb.g4, pb.arg4, pb.a3, 64, 6, 0, n2};
  float* partb = pb.part + (size_t)kWg32 * PK * 16 * 64;
  float* part1 = partb + (size_t)kWg32 * PC;
  const int w1 = std::min(nb * (PBLK / W1T), kWg1);
  hipLaunchKernelGGL(k_ps_wgrad32, dim3((unsigned)(n0 + n1 + n2)), dim3(WTH), 0, s, jobs, nb, pb.part, partb);
  hipLaunchKernelGGL(k_ps_wgrad1, dim3((unsigned)w1), dim3(256), 0, s, pb.g1, pb.arg1, feats, nb, part1);
  in.part = pb.part;
  in.partb = partb;
  in.part1 = part1;
  for (int q = 0; q < 3; ++q) {
    in.wg0[q] = jobs.j[q].wg0;
    in.nwg[q] = jobs.j[q].nwg;
  }
  in.n1 = w1;
  in.dlogit = pb.dlogit;
  in.h = pb.h;
  in.loss = pb.lossb;
  in.nb = nb;
  for (int l = 0; l < 4; ++l) {
    in.off_w[l] = off_w[l];
    in.off_b[l] = off_b[l];
  }
  in.off_fc = off_fc;
  hipLaunchKernelGGL(k_ps_reduce, dim3(kReduceBlocks), dim3(1024), 0, s, in, pb.grad, grad2, loss);
  return hipGetLastError();
}

}  // namespace fdas
