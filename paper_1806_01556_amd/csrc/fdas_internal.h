// Internal declarations shared by the host library and the kernel launchers.
#pragma once

#include <complex>
#include <cstdint>
#include <vector>

#include <hip/hip_runtime.h>

#include "../../include/fdas.h"

namespace fdas {

// ---- FP64 plan arithmetic (fdas_math.cpp) ---------------------------------
int tap_count(int z);
void gauss_legendre(int n, std::vector<double>& x, std::vector<double>& w);
void template_taps(int z, std::vector<std::complex<double>>& h);
void template_bank(int z_max, std::vector<std::vector<std::complex<double>>>& bank);
void ols_spectra(const std::vector<std::vector<std::complex<double>>>& bank, int C, int P,
                 std::vector<float>& out);
double erlang_threshold(int k, double p_fa);

// Packed template operand of the direct (matrix-core) correlations: slots of
// |z| = z_max, ..., 0 in tiles of 8, column 2 t the real and 2 t + 1 the
// imaginary part of slot t's taps at distances d >= 0 (the taps are symmetric
// in d and conjugate in z).  Consecutive tiles form groups that one launch
// works on together (at most 6 tiles and 64 KiB of operand).  A group's
// entries are step-major: step p of every tile with more than p steps.
//   FP32 (Bpk): a step is 4 distances, an entry 64 lane-ordered floats
//   (column lane % 16, distance 4 p + lane / 16).
//   Split (Bsp): a step is 32 distances, an entry 64 lanes x 8 hi then 64 x 8
//   lo 16-bit patterns (distances 32 p + 8 (lane / 16) + e), the tile's values
//   scaled by 2^eh (largest magnitude brought to about 2^14).
struct DirectGroup {
  int first, tiles;   // tile range
  int offset, count;  // operand entries
};
struct DirectPack {
  std::vector<float> Bpk;
  std::vector<uint16_t> Bsp;
  std::vector<float> tscale;    // [tiles] 2^-eh (split)
  std::vector<int> steps;       // [tiles], falling
  std::vector<int> rows;        // [tiles][16] FOP row of a column (even: +z, odd: -z, -1: none)
  std::vector<int> edge;        // [tiles][8] L/2 of a slot
  std::vector<float> edge_tap;  // [tiles][16] the unpaired tap at d = -L/2 of a column (x 2^eh)
  std::vector<DirectGroup> groups;
  int P_max = 0;                // widest template, L/2
};
// Templates up to |z| = kSplitAboveZ run in FP32 whatever precision a plan asks for:
// a bank of one tile has too few products for the 16-bit matrix cores to make up for
// the split of its operands (2^22 bins, z_max 0, 3, 7: FP32 43, 79, 120 us; split
// FP16 124, 124, 159).
constexpr int kSplitAboveZ = 7;
void direct_pack(const std::vector<std::vector<std::complex<double>>>& bank, int z_max, DirectPack& pk);
void direct_pack_split(const std::vector<std::vector<std::complex<double>>>& bank, int z_max, bool bf16,
                       DirectPack& pk);

// ---- overlap-save geometry -------------------------------------------------
constexpr int kOlsC = 4096;      // default FFT length of one chunk

struct OlsGeom {
  int C;   // chunk FFT length
  int P;   // left context = max L/2
  int V;   // valid outputs per chunk = C - (L_max - 1)
};

// Device tables of one chunk length: template spectra [rows][C] and twiddles
// (tw1 [16][C/16] = w_C^(k t); tw2 [17][TW2] = w_M^(k c), M = C/16, TW2 = M/16,
// and in row 16 w32^p for the 8192-point transform).
struct OlsTables {
  OlsGeom geom{};
  float2* H = nullptr;
  float2* tw1 = nullptr;
  float2* tw2 = nullptr;
};

bool ols_chunk_built(int C);  // 2048, 4096, 8192
int ols_threads(int C);       // threads of a convolution workgroup (C / 16)
int ols_slots_per_cu(int C);  // resident convolution workgroups per compute unit
void fft_twiddles(int C, std::vector<float>& tw1, std::vector<float>& tw2);

// ---- kernel launchers (k_*.hip) -------------------------------------------
// slots: workgroups of the persistent grid (all resident at once).
hipError_t launch_ols_conv(const float2* x, int64_t n, float* fop, int64_t ld, const OlsTables& t, int rows,
                           int slots, hipStream_t s);

// Only the listed overlap-save chunks, with templates (FOP rows) z0 .. z0 + nr - 1
// for each: two lists in one launch (either may be empty); zrow is the row of the
// zero-drift template (written as |X|^2).  With d_n the kernel reads a list's
// length from device memory and n is only its upper bound (the grid is sized
// for it).
struct ChunkList {
  const int* list = nullptr;  // device array
  int n = 0;
  const int* d_n = nullptr;
  int z0 = 0, nr = 0;
};
hipError_t launch_ols_conv_list(const float2* x, int64_t n, float* fop, int64_t ld, const OlsTables& t, ChunkList a,
                                ChunkList b, int zrow, int slots, hipStream_t s);

// FOP rows the stretched harmonic sums read as sources (k = 2 .. nh) of an
// 2*Z+1-row plane: [*lo, *hi]; empty (lo > hi) when nh < 2.
void stretch_source_rows(int Z, int nh, int* lo, int* hi);

// One spectrum of a batch for the convolution queue (device table entry).
struct ConvTrial {
  const float2* x;
  float* fop;
  int64_t n;
  int64_t ld;
  int64_t item0;  // first (chunk, template) pair of this trial: pairs before it = sum of chunks * rows
};

// (chunk, template) pairs [item_begin, item_end) of a batch, split into equal
// contiguous ranges over the resident workgroups; at most tmax templates share
// one forward FFT (0: a whole chunk's templates).
hipError_t launch_ols_conv_batch(const ConvTrial* trials, int ntrials, int64_t item_begin, int64_t item_end,
                                 const OlsTables& t, int rows, int tmax, int slots, hipStream_t s);

// Device tables of the direct correlations, as DirectPack describes them.
struct DirectTables {
  const float* Bpk;
  const uint4* Bsp;
  const float* tscale;
  const int* steps;
  const int* rows;
  const int* edge;
  const float* edge_tap;
  const DirectGroup* groups;  // host memory
  int ngroups;
  int P_max;
};
hipError_t launch_direct_conv(const float2* x, int64_t n, float* fop, int64_t ld, const DirectTables& t, int cus,
                              hipStream_t s);
hipError_t launch_direct_conv_split(const float2* x, int64_t n, float* fop, int64_t ld, const DirectTables& t,
                                    int cus, bool bf16, hipStream_t s);

// Columns handled by one workgroup of the 85-row harmonic-sum kernel.
int harmsum_tile_columns();

// Order in which the 85-row harmonic-sum kernel visits its column tiles of
// `cols` columns: tile_of_block[b] is the tile of workgroup b (-1: none).
void harmsum_tile_order(int64_t n, std::vector<int>& tile_of_block, int cols);
// Tiles of the highest-anchored kernel (256 groups of four columns 840 apart, 840
// groups to 3360 columns) and their order: chunks of 8 consecutive tiles in the
// octave order, a chunk's tiles one after another on one XCD (neighbours share
// the cache lines at their edges), eight chunks at a time over the XCDs.
constexpr int kStrideHigh = 840;
constexpr int kHighChunk = 8;
inline int64_t harmsum_high_tiles(int64_t n) {
  return ((n + 4 * kStrideHigh - 1) / (4 * kStrideHigh) * kStrideHigh + 255) / 256;
}
void harmsum_high_order(int64_t n, std::vector<int>& tile_of_block);
// Tile widths (columns) the 85-row batch harmonic sum is built for: 256, 512, 1024.
bool harmsum_tile_built(int cols);

// Workspace of the two-phase 85-row harmonic sum.
struct HsWork {
  const int* tile_of_block;  // workgroup -> column tile (-1: none)
  int blocks;                // workgroups of phase 1
  int4* hitrows;             // {first column, row mask words}
  int32_t* hitrow_count;     // entries appended by phase 1
  int emit_blocks;           // workgroups of phase 2 (0: default)
  int hit_cap;               // entries the list holds, at least harmsum_hit_entries of the plan's n_max
};
// Hit-row entries a plan for spectra of up to n_max bins and an index map needs: one
// per thread of phase 1, row segments of short spectra included.
int64_t harmsum_hit_entries(int64_t n_max, int index);

// One spectrum of a batch for the harmonic sum (device table entry).
struct HsTrial {
  const float* fop;
  int64_t ld;
  fdas_cand* cands;
  int32_t* counts;
  const int* tile_of_block;  // this length's tile order
  int n;
  int block0;                // first phase-1 workgroup of this trial
  int nblocks;               // phase-1 workgroups of this trial
  int pad;
};

hipError_t launch_zero_counts_batch(const HsTrial* trials, int ntrials, int nh, hipStream_t s);

// Two-phase 85-row stretch sum over phase-1 workgroups [blk_begin, blk_end)
// of a batch (default thresholds ta, capacity cap per plane), column tiles of
// tile_cols columns (each trial's tile order built for that width).
hipError_t launch_harmsum_batch85(const HsTrial* trials, int ntrials, int blk_begin, int blk_end, int n_harm,
                                  const float* ta, int cap, int4* hitrows, int32_t* hitrow_count, int eblocks,
                                  int tile_cols, hipStream_t s);

// index: FDAS_HSUM_* (the stretch map uses the two-phase kernels for 85 rows).
// counts[0 .. n_harm) are reset by the launch.
hipError_t launch_harmsum(const float* fop, int64_t n, int64_t ld, int z_max, int n_harm,
                          const float* ta, fdas_cand* cands, int cap, int32_t* counts,
                          const HsWork& wk, int index, hipStream_t s);

hipError_t launch_fill_i32(int32_t* p, int count, int32_t value, hipStream_t s);

// Allocation-free harmonic sum: the same kernels with their scratch (hit-row
// counter, tile order, hit-row list) in the library's static device array.
// harmsum_noalloc_scratch returns that array's address on the current device.
int64_t harmsum_noalloc_max_n();
size_t harmsum_noalloc_scratch_bytes();
hipError_t harmsum_noalloc_scratch(void** ptr);
hipError_t launch_harmsum_noalloc(const float* fop, int64_t n, int64_t ld, int z_max, int n_harm, const float* ta,
                                  fdas_cand* cands, int cap, int32_t* counts, void* scratch, int emit_blocks,
                                  int index, hipStream_t s);

int sort_tile_count(int m);
int sort_passes(int rows, int bits_r);

// Ordered records [0, min(total, out_cap)) and the nh counts copied into
// device-visible page-locked host memory by a kernel.
hipError_t launch_copy_out(const fdas_cand* sorted, int cap, int nh, const int32_t* counts, int out_cap,
                           fdas_cand* out, int32_t* counts_out, hipStream_t s);

// Table 1's N_cand per plane on the device: from the ordered array (planes
// packed, min(count, cap) records each) keep each plane's top_k highest
// powers (ties: lower z, then lower r), in (z, r) order, packed into out
// (plane k after sum_{k' < k} min(top_k, its records)).  out and counts_out (the
// device counts; NULL skips them) may be page-locked host memory.
hipError_t launch_topk(const fdas_cand* sorted, int cap, int nh, const int32_t* counts, int top_k, fdas_cand* out,
                       int32_t* counts_out, hipStream_t s);

// out[t * nh + k] = ptrs[t][k] for t < count, k < nh
hipError_t launch_gather_counts(int32_t* const* ptrs, int count, int nh, int32_t* out, hipStream_t s);

// Pack the per-plane lists (planes + k*cap, min(counts[k], cap) records each,
// counts read on the device) into `a` and order them by (harm, z, r).  `b` is
// scratch of the same size (nh * cap records), `hist` holds
// 256 * sort_tile_count(nh * cap) ints, `totals` 256 * sort_passes ints.
// *sorted receives a or b.  Nothing waits for the host.
hipError_t launch_sort_candidates(const fdas_cand* planes, int cap, int nh, const int32_t* counts, int rows,
                                  int z_max, int bits_r, fdas_cand* a, fdas_cand* b, int* hist, int* totals,
                                  fdas_cand** sorted, hipStream_t s);

// One trial of a batch readback: its per-plane lists and device counts, and
// the index of its first record in the packed array (host prefix of the
// clamped counts).
struct RbTrial {
  const int4* cands;
  const int32_t* counts;
  int64_t off;
  int64_t pad;
};

// Ordering by buckets, for lists of up to 65,536 records per plane (sort_buckets):
// one list (planes, counts; trials = 1, tab NULL) or the trials of a batch (tab).
// out, early, counts_out and shares_out may be page-locked host memory.
struct BucketSort {
  const fdas_cand* planes;
  const int32_t* counts;
  const RbTrial* tab;
  int trials, cap, nh, rows, z_max, bits_r;
  int64_t most;        // records of the longest list, at most
  int* work;           // bucket_work_ints(trials) ints, zero before the first call
  fdas_cand* scratch;  // as many records as the lists hold
  fdas_cand* out;      // the ordered records, up to out_cap
  int64_t out_cap;
  fdas_cand* early;    // where they go when they are at most early_cap (NULL: never)
  int early_cap;
  int32_t* counts_out;  // one list's counts (NULL skips them)
  int32_t* shares_out;  // set to 0 if none of one list's buckets is left to launch_bucket_shares
};
bool sort_buckets(int cap);
size_t bucket_work_ints(int trials);
hipError_t launch_bucket_sort(const BucketSort& q, hipStream_t s);
// The buckets that launch_bucket_sort left, with the same arguments and nothing
// changed in work and scratch between; of a batch, none is left unless
// batch_shares_possible for a plane.
bool batch_shares_possible(int32_t plane_records);
hipError_t launch_bucket_shares(const BucketSort& q, hipStream_t s);

int sort_passes_batch(int count, int rows, int bits_r);

// Order the lists of `count` trials (m records in all) as one trial-major
// array in (trial, harm, z, r) order.  a, b hold m records, hist
// 256 * sort_tile_count(m) ints, totals 256 * sort_passes_batch ints.
hipError_t launch_sort_batch(const RbTrial* tab, int count, int cap, int nh, int m, int rows, int z_max, int bits_r,
                             fdas_cand* a, fdas_cand* b, int* hist, int* totals, fdas_cand** sorted, hipStream_t s);

// ---- learned block pre-screen (k_prescreen.hip) ----------------------------
struct PsBuffers {
  float* theta;          // FP32 master parameters
  float* grad;           // gradient accumulator (mean over the batch)
  float* m;              // Adam moments
  float* v;
  unsigned short* wbf;   // BF16 copy used by the kernels
  unsigned short* wpack; // layers 1..3 as matrix-core A operands (kPsPackShorts)
  float* wtrain;         // the same layers as the training kernels' operands (ps_operand_floats)
  float *a1, *a2, *a3;                        // pooled activations [B][32][1024 / 256 / 64]
  unsigned char *arg1, *arg2, *arg3, *arg4;   // max-pool positions, as a1..a3; [B][32] for the last maximum
  float *g1, *g2, *g3, *g4;                   // gradients of the pooled values, as arg1..arg4
  float *h, *dlogit, *lossb;                  // [B][32] channel maxima, [B] logit gradients, [B] losses
  float* part;                                // partial weight gradients (ps_partial_floats)
};
int ps_param_count();
constexpr int kPsPackShorts = 3 * 2 * 9 * 64 * 8;
// features of listed 4096-bin blocks: log(1 + |X|^2)
hipError_t ps_features(const float2* x, int64_t n, const int* blocks, int nb, float* out, hipStream_t s);
// parameter offsets: weights and biases of layer l = 0..3, the head
int ps_off_w(int l);
int ps_off_b(int l);
int ps_off_fc();
size_t ps_operand_floats();
size_t ps_partial_floats();
hipError_t ps_operands(const PsBuffers& pb, hipStream_t s);  // wbf -> wtrain
// logits of nb feature blocks
hipError_t ps_forward(const PsBuffers& pb, const float* feats, int nb, float* logits, hipStream_t s);
// logits, mean loss, and the mean gradient into pb.grad (and grad2 unless NULL)
hipError_t ps_gradient(const PsBuffers& pb, const float* feats, int nb, const float* labels, float pos_weight,
                       float* logits, float* loss, float* grad2, hipStream_t s);
// logits of blocks 0..nb-1 of an n-bin spectrum, the features computed in the inference kernel
hipError_t ps_infer_spectrum(const PsBuffers& pb, const float2* x, int64_t n, int nb, float* logits, hipStream_t s);
hipError_t ps_adam(const PsBuffers& pb, float lr, float b1, float b2, float c1, float c2, float eps, hipStream_t s);
hipError_t ps_round(const PsBuffers& pb, hipStream_t s);
hipError_t ps_zero(float* p, int n, hipStream_t s);

// Device-side block selection of the pre-screened search (one workgroup):
// from the logits of blocks 0..nblk-1 and a threshold, writes into `lists` the
// searched-chunk list (cap_c entries), the tile list (cap_t entries, unused
// tail -1), the source-only chunk list (cap_c entries) and the three counts.
// nblk <= kMaxSelBlocks.
constexpr int kMaxSelBlocks = 16384;
hipError_t ps_search_lists(const float* logits, float thr, int64_t n, int nblk, int nh, int V, int tcols, int* lists,
                           int cap_c, int cap_t, hipStream_t s);

}  // namespace fdas
