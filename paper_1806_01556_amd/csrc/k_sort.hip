// Canonical ordering of the candidate lists on the device.
//
// The harmonic-sum kernel appends candidates to per-plane lists in arrival
// order.  Algorithm 1 visits cells in (k, i, j) order, so the list is ordered
// by the key ((k-1)*rows + row) * 2^bits_r + r, which is unique per cell.
//
// Lists of up to 65,536 records per plane (kBucketCap) are ordered in three
// launches, one bucket per (plane, row):
//   k_bucket_count    records per bucket
//   k_bucket_scatter  (r, power) pairs to their bucket's range, in any order
//   k_bucket_sort     a workgroup orders one bucket by r and writes the records
//   k_bucket_shares   only for lists with a bucket of more than 4096 records
// The list sizes are read from the device counts, so nothing waits for the host.
// A readback is bound by launches and their dependent latencies, not by its
// few megabytes: 229 k records took 73 us in the 13 launches of the radix sort
// below and take 32 us here, 7 k records 35 and 17 us.  A bucket holds the cells of
// one row, mostly some hundreds; a workgroup orders up to 4096 in LDS, and a larger
// bucket is divided among workgroups by rank, each of which reads all of it.  That
// does not scale to a row of millions of candidates, so longer lists are packed
// into one array and sorted by the whole key with an LSD radix sort (8-bit digits,
// stable passes):
//   k_sort_pack    packs the per-plane lists (sizes read from the device
//                  counts, so nothing waits for the host) and clears the
//                  per-pass digit totals
//   k_sort_hist    per-tile digit histograms (tile = 1024 records), and the
//                  digit totals of the pass by atomics
//   k_sort_offsets one workgroup per digit turns its row of tile counts into
//                  output offsets (records of smaller digits + the digit's
//                  records in earlier tiles), in place
//   k_sort_scatter stable scatter: ranks within a tile come from wave
//                  ballots (lanes with equal digits) plus per-wave counts
// Every kernel is launched for the largest possible list (n_harm * capacity
// records); tiles past the actual count return at once.
//
// A batch of trials is ordered into one trial-major array: every trial has its
// own buckets, which k_bucket_sort_small (a wave to a bucket) and k_bucket_shares
// order, launched for as many records as the longest trial holds; or, in the radix sort (k_sort_pack_batch), records carry their
// trial number in bits 8 and up of the harmonic field and the key puts the trial
// above the plane slot; the last scatter pass clears the tag.  The batch record
// count is known to the host, so those launches are sized exactly.

#include <algorithm>

#include "fdas_internal.h"

namespace fdas {
namespace {

constexpr int ST = 256;            // threads per block
constexpr int SPT = 4;             // records per thread per tile
constexpr int TILE = ST * SPT;     // 1024 records per tile

struct CandKey {
  int rows, z_max, bits_r;
  int batch;  // records carry their trial in bits 8.. of the harmonic field
};

__device__ __forceinline__ unsigned long long cand_key(const int4 c, const CandKey kp) {
  const int harm = kp.batch ? (c.x & 255) : c.x;
  unsigned long long slot = (unsigned long long)((harm - 1) * kp.rows + (c.y + kp.z_max));
  if (kp.batch) slot += (unsigned long long)((unsigned)c.x >> 8) * 8ull * (unsigned long long)kp.rows;
  return (slot << kp.bits_r) | (unsigned long long)(unsigned)c.z;
}

// plane offsets of the packed array from the device counts (each plane keeps
// at most cap records, and at most keep of them when keep > 0); returns the total
__device__ __forceinline__ int pack_offsets(const int32_t* __restrict__ counts, int nh, int cap, int (&off)[9],
                                            int keep = 0) {
  off[0] = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    int c = k < nh ? min(max(counts[k], 0), cap) : 0;
    if (keep > 0) c = min(c, keep);
    off[k + 1] = off[k] + c;
  }
  return off[8];
}

// records of the list: m_fixed when the host knows it (batch), else from the counts
__device__ __forceinline__ int record_count(const int32_t* __restrict__ counts, int nh, int cap, int m_fixed) {
  if (m_fixed >= 0) return m_fixed;
  int off[9];
  return pack_offsets(counts, nh, cap, off);
}

__global__ __launch_bounds__(ST) void k_sort_pack(const int4* __restrict__ planes, int cap, int nh,
                                                  const int32_t* __restrict__ counts, int4* __restrict__ out,
                                                  int* __restrict__ totals, int ntotals) {
  if (blockIdx.x == 0)
    for (int t = threadIdx.x; t < ntotals; t += ST) totals[t] = 0;
  int off[9];
  const int m = pack_offsets(counts, nh, cap, off);
  const int i = blockIdx.x * ST + threadIdx.x;
  if (i >= m) return;
  int k = 0;
  while (k + 1 < nh && i >= off[k + 1]) ++k;
  out[i] = planes[(size_t)k * cap + (i - off[k])];
}

__global__ __launch_bounds__(ST) void k_sort_hist(const int4* __restrict__ in, int cap, int nh,
                                                  const int32_t* __restrict__ counts, int m_fixed, int shift,
                                                  CandKey kp, int* __restrict__ hist, int maxblk,
                                                  int* __restrict__ totals) {
  const int m = record_count(counts, nh, cap, m_fixed);
  if ((int)blockIdx.x * TILE >= m) return;  // uniform
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * TILE;
  // one LDS atomic per distinct digit of a wave (lanes with equal digits found
  // by ballots, as in the scatter): skewed digits -- the trial and plane bits
  // of the top passes -- would otherwise serialise 64 atomics on one address
#pragma unroll
  for (int j = 0; j < SPT; ++j) {
    const int i = base + j * ST + threadIdx.x;
    const bool valid = i < m;
    const int d = valid ? (int)((cand_key(in[i], kp) >> shift) & 255ull) : 0;
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const unsigned long long m1 = __ballot((d >> b) & 1);
      peers &= ((d >> b) & 1) ? m1 : ~m1;
    }
    const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(peers >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)peers, 0u));
    if (valid && rank == 0) atomicAdd(&h[d], __popcll(peers));
  }
  __syncthreads();
  const int v = h[threadIdx.x];
  hist[threadIdx.x * maxblk + blockIdx.x] = v;
  if (v) atomicAdd(&totals[threadIdx.x], v);
}

// Output offsets of the pass: for digit d (workgroup d) and tile b,
// hist[d * maxblk + b] <- (records with a smaller digit) + (records of digit d
// in tiles before b), computed in place by a workgroup-wide scan of the row.
__global__ __launch_bounds__(ST) void k_sort_offsets(int* __restrict__ hist, int maxblk,
                                                     const int* __restrict__ totals, int cap, int nh,
                                                     const int32_t* __restrict__ counts, int m_fixed) {
  const int m = record_count(counts, nh, cap, m_fixed);
  const int nblk = (m + TILE - 1) / TILE;
  if (nblk == 0) return;
  __shared__ int sc[ST];
  __shared__ int s_carry;
  const int d = blockIdx.x, t = threadIdx.x;
  // records whose digit is below d
  sc[t] = t < d ? totals[t] : 0;
  __syncthreads();
  for (int o = ST / 2; o > 0; o >>= 1) {
    if (t < o) sc[t] += sc[t + o];
    __syncthreads();
  }
  if (t == 0) s_carry = sc[0];
  __syncthreads();
  int* row = hist + (size_t)d * maxblk;
  for (int b0 = 0; b0 < nblk; b0 += ST) {
    const int b = b0 + t;
    const int v = b < nblk ? row[b] : 0;
    sc[t] = v;
    __syncthreads();
    for (int o = 1; o < ST; o <<= 1) {
      const int u = t >= o ? sc[t - o] : 0;
      __syncthreads();
      sc[t] += u;
      __syncthreads();
    }
    const int carry = s_carry;
    if (b < nblk) row[b] = carry + sc[t] - v;
    __syncthreads();
    if (t == ST - 1) s_carry = carry + sc[t];
    __syncthreads();
  }
}

__global__ __launch_bounds__(ST) void k_sort_scatter(const int4* __restrict__ in, int4* __restrict__ out, int cap,
                                                     int nh, const int32_t* __restrict__ counts, int m_fixed,
                                                     int shift, CandKey kp, const int* __restrict__ offs, int maxblk,
                                                     int untag) {
  const int m = record_count(counts, nh, cap, m_fixed);
  if ((int)blockIdx.x * TILE >= m) return;  // uniform
  __shared__ int base[256];      // running position per digit inside this tile's output range
  __shared__ int wcnt[ST / 64][256];
  const int t = threadIdx.x;
  const int w = t >> 6;
  base[t] = offs[(size_t)t * maxblk + blockIdx.x];
#pragma unroll
  for (int q = 0; q < ST / 64; ++q) wcnt[q][t] = 0;
  __syncthreads();
  const int tile0 = blockIdx.x * TILE;
  for (int j = 0; j < SPT; ++j) {
    const int i = tile0 + j * ST + t;
    const bool valid = i < m;
    int4 rec = make_int4(0, 0, 0, 0);
    int d = 0;
    if (valid) {
      rec = in[i];
      d = (int)((cand_key(rec, kp) >> shift) & 255ull);
    }
    // lanes of this wave holding the same digit
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const unsigned long long m1 = __ballot((d >> b) & 1);
      peers &= ((d >> b) & 1) ? m1 : ~m1;
    }
    const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(peers >> 32),
                                               __builtin_amdgcn_mbcnt_lo((unsigned)peers, 0u));
    if (valid && rank == 0) wcnt[w][d] = __popcll(peers);
    __syncthreads();
    if (valid) {
      int pos = base[d] + rank;
      for (int q = 0; q < w; ++q) pos += wcnt[q][d];
      if (untag) rec.x &= 255;
      out[pos] = rec;
    }
    __syncthreads();
    // advance the running bases and clear the per-wave counts
    {
      int add = 0;
#pragma unroll
      for (int q = 0; q < ST / 64; ++q) {
        add += wcnt[q][t];
        wcnt[q][t] = 0;
      }
      base[t] += add;
    }
    __syncthreads();
  }
}

// out[t * nh + k] = ptrs[t][k]: the counts of every trial of a batch in one array
__global__ void k_gather_counts(int32_t* const* __restrict__ ptrs, int count, int nh, int32_t* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count * nh) out[i] = ptrs[i / nh][i % nh];
}

// Batch pack: record i of the packed array belongs to the last trial whose
// first record is <= i (empty trials share their successor's offset), then to
// that trial's plane by its clamped counts.  The trial is tagged into the
// harmonic field.  Block 0 also clears the per-pass digit totals.
__global__ __launch_bounds__(ST) void k_sort_pack_batch(const RbTrial* __restrict__ tr, int count, int cap, int nh,
                                                        int m, int4* __restrict__ out, int* __restrict__ totals,
                                                        int ntotals) {
  if (blockIdx.x == 0)
    for (int t = threadIdx.x; t < ntotals; t += ST) totals[t] = 0;
  const int i = blockIdx.x * ST + threadIdx.x;
  if (i >= m) return;
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tr[mid].off <= (int64_t)i) lo = mid; else hi = mid - 1;
  }
  int off[9];
  pack_offsets(tr[lo].counts, nh, cap, off);
  const int j = i - (int)tr[lo].off;
  int k = 0;
  while (k + 1 < nh && j >= off[k + 1]) ++k;
  int4 rec = tr[lo].cands[(size_t)k * cap + (j - off[k])];
  rec.x |= lo << 8;
  out[i] = rec;
}

// Top-k selection of Table 1's N_cand per plane, on the ordered array: block
// k keeps the top_k highest powers of plane k (ties: lower z, then lower r --
// the earlier record of the (z, r)-ordered plane) and writes them, still in
// (z, r) order, after the kept records of the planes before it.  The k-th
// largest of the distinct keys (power bits << 32 | ~position) is found by an
// 8-bit radix select from the top digit; the records with a key at least as
// large are compacted in order by a workgroup scan.
constexpr int TK = 1024;  // threads of the selection

__device__ __forceinline__ unsigned long long topk_key(const int4* __restrict__ plane, int p) {
  // powers of candidates are above a positive threshold: their bits order them
  return ((unsigned long long)(unsigned)plane[p].w << 32) | (unsigned long long)(~(unsigned)p);
}

__global__ __launch_bounds__(TK) void k_topk(const int4* __restrict__ sorted, int cap, int nh,
                                             const int32_t* __restrict__ counts, int top_k,
                                             int4* __restrict__ out, int32_t* __restrict__ counts_out) {
  __shared__ int s_hist[256];
  __shared__ int s_wave[TK / 64];
  __shared__ unsigned long long s_prefix;
  __shared__ int s_need, s_done;
  const int k = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
  if (k >= nh) return;
  if (counts_out && t == 0) counts_out[k] = counts[k];
  int off[9], okeep[9];
  pack_offsets(counts, nh, cap, off);
  pack_offsets(counts, nh, cap, okeep, top_k);
  const int m = off[k + 1] - off[k];
  const int4* plane = sorted + off[k];
  int4* dst = out + okeep[k];
  if (m <= top_k) {
    for (int i = t; i < m; i += TK) dst[i] = plane[i];
    return;
  }
  // radix select of the top_k-th largest key, until a digit's records are all
  // kept (usually within the four digits of the power)
  if (t == 0) {
    s_prefix = 0ull;
    s_need = top_k;
    s_done = 0;
  }
  for (int shift = 56; shift >= 0; shift -= 8) {
    if (t < 256) s_hist[t] = 0;
    __syncthreads();
    const unsigned long long prefix = s_prefix;
    const unsigned long long hmask = shift == 56 ? 0ull : (~0ull << (shift + 8));
    for (int i0 = 0; i0 < m; i0 += TK) {
      const int i = i0 + t;
      const unsigned long long key = i < m ? topk_key(plane, i) : 0ull;
      const bool in = i < m && (key & hmask) == prefix;
      const int d = in ? (int)((key >> shift) & 255ull) : 0;
      // one LDS atomic per distinct digit of a wave: the powers' top digits are alike
      unsigned long long peers = __ballot(in);
      if (peers == 0ull) continue;  // uniform
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const unsigned long long m1 = __ballot((d >> b) & 1);
        peers &= ((d >> b) & 1) ? m1 : ~m1;
      }
      const int rank =
          __builtin_amdgcn_mbcnt_hi((unsigned)(peers >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)peers, 0u));
      if (in && rank == 0) atomicAdd(&s_hist[d], __popcll(peers));
    }
    __syncthreads();
    // thread t < 256 looks at digit 255 - t: the records with a larger digit stay
    // below the need, those with it or a larger one reach it
    const int need = s_need;
    int own = 0, incl = 0;
    if (t < 256) {
      own = incl = s_hist[255 - t];
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
      }
      if (lane == 63) s_wave[wv] = incl;
    }
    __syncthreads();
    if (t < 256) {
      for (int q = 0; q < wv; ++q) incl += s_wave[q];
      if (incl >= need && incl - own < need) {
        const int left = need - (incl - own);
        s_need = left;
        s_prefix = prefix | ((unsigned long long)(255 - t) << shift);
        s_done = left == own ? 1 : 0;
      }
    }
    __syncthreads();
    if (s_done) break;  // uniform: every record of this digit is kept
  }
  const unsigned long long kth = s_prefix;  // keys are distinct: exactly top_k are >= kth
  // stable compaction of the keys >= kth
  int base = 0;
  for (int i0 = 0; i0 < m; i0 += TK) {
    const int i = i0 + t;
    const bool f = i < m && topk_key(plane, i) >= kth;
    const unsigned long long b = __ballot(f);
    if (lane == 0) s_wave[wv] = __popcll(b);
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < TK / 64; ++q) {
      const int c = s_wave[q];
      before += q < wv ? c : 0;
      all += c;
    }
    if (f)
      dst[base + before +
          __builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u))] = plane[i];
    base += all;
    __syncthreads();
  }
}

constexpr int kBucketCap = 65536;

// --- bucket sort ----------------------------------------------------------------
// Bucket (k - 1) * rows + row; blockIdx.y is the trial.  Work arrays per trial:
// totals[kMaxBuckets] and cursor[kMaxBuckets], zero between calls (the plan
// clears them once, k_bucket_sort or k_bucket_sort_small after use),
// starts[kMaxBuckets + 1], and the shares of the buckets that those kernels leave
// (more than 4096 and 512 records): their number, then {bucket, share << 16} each.

constexpr int kMaxBuckets = 8 * 129;
constexpr int kBucketLds = 4096;                  // records a workgroup orders in LDS
constexpr int kBucketSmall = 512;                 // ... and a wave
constexpr int SHARE_T = 1024;                     // threads of k_bucket_shares
constexpr int kShareCount = 3 * kMaxBuckets + 1;  // index of the number of shares
constexpr int kMaxShares = 8 * kBucketCap / kBucketSmall;  // no share has fewer than 512 records
constexpr int kBucketInts = kShareCount + 1 + kMaxShares;      // per trial
static_assert(kMaxBuckets < (1 << 16) && kBucketCap <= (1 << 16), "share and position fields");

// Shares of a bucket of c records in a list of m, one up to kBucketLds.  Small ones take
// a workgroup the least time, but each reads the whole bucket.  Whole readback of one
// row and of eight rows of 65,536 records: 107 and 275 us in shares of 960, 112 and
// 271 of 1920, 128 and 286 of 3584; eight rows without their way to the host (copying
// readback) 356, 331 and 296 us.
__device__ __forceinline__ int bucket_shares(int c, int m) {
  const int share = c <= kBucketLds ? kBucketLds : m <= 2 * kBucketCap ? 960 : 3584;
  return (c + share - 1) / share;
}

struct BucketList {
  const int4* planes;     // one list
  const int32_t* counts;
  const RbTrial* tab;     // or a batch's
  int cap, nh, rows, z_max;
  int* work;              // [trials][kBucketInts]
};

__device__ __forceinline__ BucketList trial_list(const BucketList& bl, int64_t& base) {
  BucketList one = bl;
  base = 0;
  if (bl.tab) {
    one.planes = bl.tab[blockIdx.y].cands;
    one.counts = bl.tab[blockIdx.y].counts;
    base = bl.tab[blockIdx.y].off;
  }
  one.work = bl.work + (size_t)blockIdx.y * kBucketInts;
  return one;
}

// this workgroup's share [lo, hi) of a list's m records, at least one to a thread
__device__ __forceinline__ void bucket_share(int m, int& lo, int& hi) {
  const int active = min((int)gridDim.x, (m + ST - 1) / ST);
  lo = hi = 0;
  if ((int)blockIdx.x < active) {
    lo = (int)((int64_t)m * blockIdx.x / active);
    hi = (int)((int64_t)m * (blockIdx.x + 1) / active);
  }
}

// record i of the packed list and its bucket (a row outside the plane, which no
// harmonic sum writes, is clamped)
__device__ __forceinline__ int4 bucket_record(const BucketList& bl, const int (&off)[9], int i, int& bucket) {
  int k = 0;
  while (k + 1 < bl.nh && i >= off[k + 1]) ++k;
  const int4 rec = bl.planes[(size_t)k * bl.cap + (i - off[k])];
  bucket = k * bl.rows + min(max(rec.y + bl.z_max, 0), bl.rows - 1);
  return rec;
}

__global__ __launch_bounds__(ST) void k_bucket_count(BucketList all) {
  __shared__ int h[kMaxBuckets];
  int64_t base;
  const BucketList bl = trial_list(all, base);
  int off[9], lo, hi;
  bucket_share(pack_offsets(bl.counts, bl.nh, bl.cap, off), lo, hi);
  if (lo == hi) return;  // uniform
  const int nb = bl.nh * bl.rows;
  for (int b = threadIdx.x; b < nb; b += ST) h[b] = 0;
  __syncthreads();
  for (int i = lo + threadIdx.x; i < hi; i += ST) {
    int b;
    bucket_record(bl, off, i, b);
    atomicAdd(&h[b], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += ST)
    if (h[b]) atomicAdd(&bl.work[b], h[b]);
}

// Buckets of more than `above` records become shares.
__global__ __launch_bounds__(ST) void k_bucket_scatter(BucketList all, int above, int2* __restrict__ pairs) {
  __shared__ int start[kMaxBuckets + 1];
  __shared__ int h[kMaxBuckets];
  __shared__ int s_wave[ST / 64];
  __shared__ int s_shares;
  int64_t base;
  const BucketList bl = trial_list(all, base);
  int off[9], lo, hi;
  const int m = pack_offsets(bl.counts, bl.nh, bl.cap, off);
  bucket_share(m, lo, hi);
  if (lo == hi && blockIdx.x > 0) return;  // uniform; workgroup 0 writes the starts of an empty list too
  const int nb = bl.nh * bl.rows, t = threadIdx.x;
  const int* totals = bl.work;
  int* cursor = bl.work + kMaxBuckets;
  int* starts = bl.work + 2 * kMaxBuckets;
  // exclusive sums of the totals: PER consecutive buckets to a thread
  constexpr int PER = (kMaxBuckets + ST - 1) / ST;
  int own[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = t * PER + q;
    own[q] = b < nb ? totals[b] : 0;
    sum += own[q];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(incl, o);
    if ((t & 63) >= o) incl += u;
  }
  if ((t & 63) == 63) s_wave[t >> 6] = incl;
  if (t == 0) s_shares = 0;
  __syncthreads();
  int at = incl - sum;
  for (int q = 0; q < (t >> 6); ++q) at += s_wave[q];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = t * PER + q;
    if (b < nb) {
      start[b] = at;
      h[b] = 0;
      if (blockIdx.x == 0) {
        starts[b] = at;
        if (own[q] > above) {
          const int W = bucket_shares(own[q], m);
          const int first = atomicAdd(&s_shares, W);
          for (int w = 0; w < W; ++w)
            if (first + w < kMaxShares) bl.work[kShareCount + 1 + first + w] = b | (w << 16);
        }
      }
      at += own[q];
    }
  }
  if (blockIdx.x == 0 && t == 0) starts[nb] = m;
  __syncthreads();
  if (blockIdx.x == 0 && t == 0) bl.work[kShareCount] = min(s_shares, kMaxShares);
  for (int i = lo + t; i < hi; i += ST) {
    int b;
    bucket_record(bl, off, i, b);
    atomicAdd(&h[b], 1);
  }
  __syncthreads();
  for (int b = t; b < nb; b += ST) {
    if (h[b]) start[b] += atomicAdd(&cursor[b], h[b]);
    h[b] = 0;
  }
  __syncthreads();
  for (int i = lo + t; i < hi; i += ST) {
    int b;
    const int4 rec = bucket_record(bl, off, i, b);
    pairs[base + start[b] + atomicAdd(&h[b], 1)] = make_int2(rec.z, rec.w);
  }
}

// Ascending bitonic sort of N keys (a power of two, at least 64) by TH threads, t
// this thread's index among them.  Pairs at a distance of up to 64 stay within a
// wave's 128 keys; with one wave (TH = 64) all of them do.
template <int TH>
__device__ __forceinline__ void bitonic(unsigned long long* keys, int N, int t) {
  for (int size = 2; size <= N; size <<= 1) {
    for (int d = size >> 1; d > 0; d >>= 1) {
      for (int q = t; q < N / 2; q += TH) {
        const int i = 2 * q - (q & (d - 1)), j = i + d;
        const unsigned long long x = keys[i], y = keys[j];
        if ((x > y) == ((i & size) == 0)) {
          keys[i] = y;
          keys[j] = x;
        }
      }
      if (TH > 64 && (d > 64 || (d == 1 && size >= 128))) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}

__device__ __forceinline__ unsigned long long bucket_key(const int2* mine, int i, int c) {
  const int2 v = i < c ? mine[i] : make_int2(-1, -1);  // padding orders last: r >= 0
  return ((unsigned long long)(unsigned)v.x << 32) | (unsigned)v.y;
}

// Orders the buckets of up to kBucketSmall records, a wave to `span` (at most 64)
// of them; larger ones are left to k_bucket_shares.  The trials of a batch have
// thousands of buckets, most with a few records or none: 16 trials of 7 k records
// 46 us with a workgroup and 32 KB of LDS for every bucket, 35 with 4 KB for the
// small ones, 21 with a wave each.
__global__ __launch_bounds__(ST) void k_bucket_sort_small(BucketList all, const int2* __restrict__ pairs, int span,
                                                          int64_t out_cap, int4* __restrict__ out) {
  __shared__ unsigned long long s_keys[ST / 64][kBucketSmall];
  int64_t base;
  const BucketList bl = trial_list(all, base);
  const int nb = bl.nh * bl.rows, lane = threadIdx.x & 63;
  const int b0 = ((int)blockIdx.x * (ST / 64) + (threadIdx.x >> 6)) * span;  // no barrier follows
  const int* starts = bl.work + 2 * kMaxBuckets;
  // lane l looks at bucket b0 + l
  const bool in = lane < span && b0 + lane < nb;
  const int at = in ? starts[b0 + lane] : 0;
  const int held = in ? starts[b0 + lane + 1] - at : 0;
  if (held > 0) {
    bl.work[b0 + lane] = 0;
    bl.work[kMaxBuckets + b0 + lane] = 0;
  }
  unsigned long long* keys = s_keys[threadIdx.x >> 6];
  for (unsigned long long todo = __ballot(held > 0 && held <= kBucketSmall); todo != 0ull; todo &= todo - 1ull) {
    const int l = (int)__builtin_ctzll(todo), b = b0 + l;
    const int s0 = __builtin_amdgcn_readlane(at, l), c = __builtin_amdgcn_readlane(held, l);
    int N = 64;
    while (N < c) N <<= 1;
    for (int i = lane; i < N; i += 64) keys[i] = bucket_key(pairs + base + s0, i, c);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    bitonic<64>(keys, N, lane);
    const int harm = b / bl.rows + 1, z = b % bl.rows - bl.z_max;
    const int64_t room = out_cap - (base + s0);
    for (int i = lane; i < c; i += 64)
      if (i < room) out[base + s0 + i] = make_int4(harm, z, (int)(keys[i] >> 32), (int)(unsigned)keys[i]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Gathers records of a bucket of c, those with ranks [p0, p1) among them, as
// keys (r << 32 | position) in any order: at most kBucketLds, all those of ranks
// [p0 - *skip, p0 - *skip + the count returned) in the order of these keys.  A
// radix select of 12 bits a round over (r, position), distinct whatever the records
// hold, narrows the two ends until what lies between them fits: one round unless a
// digit at an end holds more records than there is room for.  A
// whole workgroup reads the bucket once per round, and once more for the keys;
// `keys` is the histograms' memory until then.  What bounds it is latency: U loads at a
// time without a branch between them, the next ones under way, one LDS reservation
// for all that a wave finds in them.
__device__ __forceinline__ int bucket_share_keys(const int2* __restrict__ mine, int c, int p0, int p1, int bits_r,
                                                 unsigned long long* keys, int* skip) {
  constexpr int DIG = 12, U = 8;
  __shared__ int s_wave[2][SHARE_T / 64];
  __shared__ int s_bin[2], s_need[2], s_size[2], s_n;
  static_assert(2 * sizeof(int) << DIG <= sizeof(unsigned long long) * kBucketLds, "two histograms");
  int(*hist)[1 << DIG] = reinterpret_cast<int(*)[1 << DIG]>(keys);
  const int t = threadIdx.x, lane = t & 63;
  const unsigned top = bits_r < 32 ? (1u << bits_r) - 1u : ~0u;
  // batch(r, i0): r of the records i0 + u SHARE_T, u < U (past the end: the last one's)
  auto each = [&](auto batch) {
    unsigned next[U];
    auto load = [&](int i0) {
#pragma unroll
      for (int u = 0; u < U; ++u) next[u] = (unsigned)mine[min(i0 + u * SHARE_T, c - 1)].x;
    };
    load(t);
    for (int i0 = t; i0 - t < c; i0 += U * SHARE_T) {
      unsigned r[U];
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = min(next[u], top);
      load(i0 + U * SHARE_T);  // in flight while this batch is worked on
      batch(r, i0);
    }
  };
  // the ends: keys below prefix[0] << left rank before p0 - need[0]; those up to
  // prefix[1] << left and its digit's rest rank before p1 - 1 - need[1] + size[1]
  unsigned long long prefix[2] = {0ull, 0ull};
  int need[2] = {p0, p1 - 1}, size[2] = {c, c};
  int left = bits_r + 16;
  auto between = [&]() { return p1 - 1 - need[1] + size[1] - (p0 - need[0]); };
  while (between() > kBucketLds) {  // uniform
    // a digit lies within r or within the position; at no bits left every digit is one record
    const int width = min(DIG, left > 16 ? left - 16 : left), shift = left - width;
    const unsigned mask = (1u << width) - 1u;
    const bool one = prefix[0] == prefix[1];  // the same records count for both ends
    for (int e = t; e < 2 << DIG; e += SHARE_T) (&hist[0][0])[e] = 0;
    __syncthreads();
    if (left == bits_r + 16) {
      const int sh = shift - 16;  // bits_r > 0
      each([&](const unsigned (&r)[U], int i0) {
        const bool whole = i0 - t + U * SHARE_T <= c;  // uniform
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const unsigned d = r[u] >> sh;
          // neighbours in the list are often neighbours in r: one addition for a wave of one digit
          const unsigned first = (unsigned)__builtin_amdgcn_readfirstlane((int)d);
          if (whole && __ballot(d != first) == 0ull) {
            if (lane == 0) atomicAdd(&hist[0][first], 64);
          } else if (i0 + u * SHARE_T < c) {
            atomicAdd(&hist[0][d], 1);
          }
        }
      });
    } else {
      each([&](const unsigned (&r)[U], int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * SHARE_T;
          const unsigned long long v = (((unsigned long long)r[u] << 16) | (unsigned)i) >> shift, up = v >> width;
          if (i < c && up == prefix[0]) atomicAdd(&hist[0][(unsigned)v & mask], 1);
          if (i < c && !one && up == prefix[1]) atomicAdd(&hist[1][(unsigned)v & mask], 1);
        }
      });
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int* h = hist[one ? 0 : j];
      constexpr int PER = (1 << DIG) / SHARE_T;
      int sum = 0;
#pragma unroll
      for (int q = 0; q < PER; ++q) sum += h[t * PER + q];
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
      }
      if (lane == 63) s_wave[j][t >> 6] = incl;
      __syncthreads();
      for (int q = 0; q < (t >> 6); ++q) incl += s_wave[j][q];
      int below = incl - sum;
      if (need[j] >= below && need[j] < incl) {  // one thread
        for (int q = 0; q < PER; ++q) {
          const int v = h[t * PER + q];
          if (need[j] >= below && need[j] < below + v) {
            s_bin[j] = t * PER + q;
            s_need[j] = need[j] - below;
            s_size[j] = v;
          }
          below += v;
        }
      }
      __syncthreads();
      prefix[j] = (prefix[j] << width) | (unsigned)s_bin[j];
      need[j] = s_need[j];
      size[j] = s_size[j];
    }
    left = shift;
  }
  *skip = need[0];
  if (t == 0) s_n = 0;
  __syncthreads();
  each([&](const unsigned (&r)[U], int i0) {
    unsigned found = 0u;  // bit u
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * SHARE_T;
      const unsigned long long k = (((unsigned long long)r[u] << 16) | (unsigned)i) >> left;
      found |= i < c && k >= prefix[0] && k <= prefix[1] ? 1u << u : 0u;
    }
    if (__ballot(found != 0u) == 0ull) return;  // uniform
    const int cnt = __popc(found);
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    int at = 0;
    if (lane == 63) at = atomicAdd(&s_n, incl);
    at = __builtin_amdgcn_readlane(at, 63) + incl - cnt;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((found >> u) & 1u) {
        if (at < kBucketLds) keys[at] = ((unsigned long long)r[u] << 32) | (unsigned)(i0 + u * SHARE_T);
        ++at;
      }
  });
  return between();
}

// Keys [0, got) put in order by TH threads, and cnt of them from `skip` on written
// from out[first] on as records of bucket b: (r, power), or (r, position) of the
// bucket's records in `from`.  Records past out_cap are dropped.
template <int TH>
__device__ __forceinline__ void order_and_write(const BucketList& bl, unsigned long long* keys, int got, int b, int skip,
                                                int cnt, const int2* __restrict__ from, int4* __restrict__ out,
                                                int64_t first, int64_t out_cap) {
  const int t = threadIdx.x;
  int N = 64;
  while (N < got) N <<= 1;
  for (int i = got + t; i < N; i += TH) keys[i] = ~0ull;  // orders last: r >= 0
  __syncthreads();
  bitonic<TH>(keys, N, t);
  __syncthreads();
  const int harm = b / bl.rows + 1, z = b % bl.rows - bl.z_max;
  const int64_t room = out_cap - first;
  for (int i = t; i < cnt; i += TH)
    if (i < room) {
      const unsigned long long k = keys[skip + i];
      const int2 v = from ? from[(unsigned)k] : make_int2((int)(k >> 32), (int)(unsigned)k);
      out[first + i] = make_int4(harm, z, v.x, v.y);
    }
}

// Orders bucket blockIdx.x of a list, if it holds at most kBucketLds records, and
// writes them.  When all the list's records fit in early_cap, they
// go to `early` (page-locked memory) instead of out; with counts_out the counts go
// out too, with shares_out the number of shares left to k_bucket_shares.
__global__ __launch_bounds__(ST) void k_bucket_sort(BucketList all, const int2* __restrict__ pairs, int64_t out_cap, int4* __restrict__ out, int4* __restrict__ early,
                                                    int early_cap, int32_t* __restrict__ counts_out,
                                                    int32_t* __restrict__ shares_out) {
  __shared__ unsigned long long keys[kBucketLds];
  int64_t base;
  const BucketList bl = trial_list(all, base);
  const int b = blockIdx.x, t = threadIdx.x;
  const int* starts = bl.work + 2 * kMaxBuckets;
  const int s0 = starts[b], c = starts[b + 1] - s0;
  if (counts_out && b == 0 && t < bl.nh) counts_out[t] = bl.counts[t];
  if (shares_out && b == 0 && t == 0) *shares_out = bl.work[kShareCount];
  // an empty bucket's total and cursor are zero already
  if (c <= 0) return;  // uniform
  if (t == 0) {
    bl.work[b] = 0;
    bl.work[kMaxBuckets + b] = 0;
  }
  if (c > kBucketLds) return;  // uniform
  if (early && starts[bl.nh * bl.rows] <= early_cap) out = early;
  for (int i = t; i < c; i += ST) keys[i] = bucket_key(pairs + base + s0, i, c);
  order_and_write<ST>(bl, keys, c, b, 0, c, nullptr, out, base + s0, out_cap);
}

// The buckets that the other kernels leave, in shares dealt to the workgroups.
// Interference that fills a row, or a plan of few rows, brings up to 65,536 records
// to a bucket.  For a single list the host launches this only if there is a share,
// which it learns with the counts that it waits for, so the usual readback pays
// nothing for it; for a batch, if a plane holds enough records.  Whole readback
// of 65,536 records of one row: 106 us; 100 us in the radix sort of the whole
// key, 686 us with one workgroup that passed over them in memory.
__global__ __launch_bounds__(SHARE_T) void k_bucket_shares(BucketList all, const int2* __restrict__ pairs, int bits_r,
                                                           int64_t out_cap, int4* __restrict__ out,
                                                           int4* __restrict__ early, int early_cap) {
  __shared__ unsigned long long keys[kBucketLds];
  int64_t base;
  const BucketList bl = trial_list(all, base);
  const int* starts = bl.work + 2 * kMaxBuckets;
  const int shares = bl.work[kShareCount];
  if (early && starts[bl.nh * bl.rows] <= early_cap) out = early;
  for (int e = blockIdx.x; e < shares; e += gridDim.x) {  // uniform
    const int v = bl.work[kShareCount + 1 + e], b = v & 0xffff, w = v >> 16;
    const int s0 = starts[b], c = starts[b + 1] - s0, W = bucket_shares(c, starts[bl.nh * bl.rows]);
    const int2* mine = pairs + base + s0;
    const int p0 = (int)((int64_t)c * w / W), cnt = (int)((int64_t)c * (w + 1) / W) - p0;
    int skip;
    const int got = bucket_share_keys(mine, c, p0, p0 + cnt, bits_r, keys, &skip);  // all of them if c <= kBucketLds
    order_and_write<SHARE_T>(bl, keys, got, b, skip, cnt, mine, out, base + s0 + p0, out_cap);
    __syncthreads();  // the keys are read
  }
}

// The ordered records and the counts written straight into page-locked host
// memory (device-visible pointers), so the host waits once: records
// [0, min(total, out_cap)) of `sorted`, counts[0 .. nh).
__global__ __launch_bounds__(ST) void k_copy_out(const int4* __restrict__ sorted, int cap, int nh,
                                                 const int32_t* __restrict__ counts, int out_cap,
                                                 int4* __restrict__ out, int32_t* __restrict__ counts_out) {
  int off[9];
  const int m = min(pack_offsets(counts, nh, cap, off), out_cap);
  if (blockIdx.x == 0 && (int)threadIdx.x < nh) counts_out[threadIdx.x] = counts[threadIdx.x];
  for (int i = blockIdx.x * ST + threadIdx.x; i < m; i += gridDim.x * ST) out[i] = sorted[i];
}

}  // namespace

hipError_t launch_copy_out(const fdas_cand* sorted, int cap, int nh, const int32_t* counts, int out_cap,
                           fdas_cand* out, int32_t* counts_out, hipStream_t s) {
  const int blocks = std::max(1, std::min(1024, (nh * cap + ST - 1) / ST));
  hipLaunchKernelGGL(k_copy_out, dim3(blocks), dim3(ST), 0, s, reinterpret_cast<const int4*>(sorted), cap, nh,
                     counts, out_cap, reinterpret_cast<int4*>(out), counts_out);
  return hipGetLastError();
}

hipError_t launch_topk(const fdas_cand* sorted, int cap, int nh, const int32_t* counts, int top_k, fdas_cand* out,
                       int32_t* counts_out, hipStream_t s) {
  if (top_k <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_topk, dim3(nh), dim3(TK), 0, s, reinterpret_cast<const int4*>(sorted), cap, nh, counts, top_k,
                     reinterpret_cast<int4*>(out), counts_out);
  return hipGetLastError();
}

hipError_t launch_gather_counts(int32_t* const* ptrs, int count, int nh, int32_t* out, hipStream_t s) {
  const int total = count * nh;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_counts, dim3((total + 255) / 256), dim3(256), 0, s, ptrs, count, nh, out);
  return hipGetLastError();
}

int sort_tile_count(int m) { return (m + TILE - 1) / TILE; }

int sort_passes(int rows, int bits_r) {
  const int slot_bits = 32 - __builtin_clz((unsigned)(8 * rows));  // covers (k-1)*rows + row < 8*rows
  return (slot_bits + bits_r + 7) / 8;
}

bool sort_buckets(int cap) { return cap <= kBucketCap; }

size_t bucket_work_ints(int trials) { return (size_t)trials * kBucketInts; }

namespace {
bool bucket_list(const BucketSort& q, BucketList& bl) {
  if (q.nh < 1 || q.rows < 1 || q.nh * q.rows > kMaxBuckets || !sort_buckets(q.cap) || q.trials < 1 || !q.work)
    return false;
  bl = BucketList{reinterpret_cast<const int4*>(q.planes), q.counts, q.tab, q.cap, q.nh, q.rows, q.z_max, q.work};
  return true;
}
}  // namespace

hipError_t launch_bucket_sort(const BucketSort& q, hipStream_t s) {
  BucketList bl;
  if (!bucket_list(q, bl)) return hipErrorInvalidValue;
  int2* pairs = reinterpret_cast<int2*>(q.scratch);
  int4 *out = reinterpret_cast<int4*>(q.out), *early = reinterpret_cast<int4*>(q.early);
  // Workgroups for the records that a list can hold.  Sized for the capacity, 1024
  // trials of 10 records took 847 us, the readback with the radix sort 372; sized
  // for their records 250.
  const unsigned wgs = (unsigned)std::max<int64_t>(1, std::min<int64_t>(256, (q.most + ST - 1) / ST));
  const unsigned buckets = (unsigned)(q.nh * q.rows), trials = (unsigned)q.trials;
  hipLaunchKernelGGL(k_bucket_count, dim3(wgs, trials), dim3(ST), 0, s, bl);
  hipLaunchKernelGGL(k_bucket_scatter, dim3(wgs, trials), dim3(ST), 0, s, bl, q.tab ? kBucketSmall : kBucketLds, pairs);
  if (q.tab) {
    // a wave to some two buckets with records, or to more where 16,384 waves, two
    // rounds of the chip, have them all
    const int64_t want = std::max<int64_t>(2 * (int64_t)buckets / std::max<int64_t>(1, q.most),
                                           (int64_t)buckets * trials / 16384);
    const int span = (int)std::max<int64_t>(1, std::min<int64_t>(64, want));
    const unsigned waves = (buckets + span - 1) / span;
    hipLaunchKernelGGL(k_bucket_sort_small, dim3((waves + ST / 64 - 1) / (ST / 64), trials), dim3(ST), 0, s, bl, pairs,
                       span, q.out_cap, out);
  } else {
    hipLaunchKernelGGL(k_bucket_sort, dim3(buckets), dim3(ST), 0, s, bl, pairs, q.out_cap, out, early, q.early_cap,
                       q.counts_out, q.shares_out);
  }
  return hipGetLastError();
}

bool batch_shares_possible(int32_t plane_records) { return plane_records > kBucketSmall; }

hipError_t launch_bucket_shares(const BucketSort& q, hipStream_t s) {
  BucketList bl;
  if (!bucket_list(q, bl)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_bucket_shares, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(q.tab ? 96 : 512, q.most / kBucketSmall)), (unsigned)q.trials), dim3(SHARE_T), 0, s, bl,
                     reinterpret_cast<const int2*>(q.scratch), q.bits_r, q.out_cap, reinterpret_cast<int4*>(q.out),
                     reinterpret_cast<int4*>(q.early), q.early_cap);
  return hipGetLastError();
}

hipError_t launch_sort_candidates(const fdas_cand* planes, int cap, int nh, const int32_t* counts, int rows,
                                  int z_max, int bits_r, fdas_cand* a, fdas_cand* b, int* hist, int* totals,
                                  fdas_cand** sorted, hipStream_t s) {
  const int maxm = nh * cap;
  const int maxblk = sort_tile_count(maxm);
  const int passes = sort_passes(rows, bits_r);
  hipLaunchKernelGGL(k_sort_pack, dim3((maxm + ST - 1) / ST), dim3(ST), 0, s, reinterpret_cast<const int4*>(planes),
                     cap, nh, counts, reinterpret_cast<int4*>(a), totals, 256 * passes);
  CandKey kp{rows, z_max, bits_r, 0};
  int4* src = reinterpret_cast<int4*>(a);
  int4* dst = reinterpret_cast<int4*>(b);
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    int* tot = totals + 256 * p;
    hipLaunchKernelGGL(k_sort_hist, dim3(maxblk), dim3(ST), 0, s, src, cap, nh, counts, -1, shift, kp, hist, maxblk,
                       tot);
    hipLaunchKernelGGL(k_sort_offsets, dim3(256), dim3(ST), 0, s, hist, maxblk, tot, cap, nh, counts, -1);
    hipLaunchKernelGGL(k_sort_scatter, dim3(maxblk), dim3(ST), 0, s, src, dst, cap, nh, counts, -1, shift, kp, hist,
                       maxblk, 0);
    int4* tmp = src;
    src = dst;
    dst = tmp;
  }
  *sorted = reinterpret_cast<fdas_cand*>(src);
  return hipGetLastError();
}

int sort_passes_batch(int count, int rows, int bits_r) {
  const int slot_bits = 32 - __builtin_clz((unsigned)(8 * rows * count));  // trial * 8 * rows + plane slot
  return (slot_bits + bits_r + 7) / 8;
}

hipError_t launch_sort_batch(const RbTrial* tab, int count, int cap, int nh, int m, int rows, int z_max, int bits_r,
                             fdas_cand* a, fdas_cand* b, int* hist, int* totals, fdas_cand** sorted, hipStream_t s) {
  *sorted = a;
  if (m <= 0) return hipSuccess;
  const int nblk = sort_tile_count(m);
  const int passes = sort_passes_batch(count, rows, bits_r);
  hipLaunchKernelGGL(k_sort_pack_batch, dim3((m + ST - 1) / ST), dim3(ST), 0, s, tab, count, cap, nh, m,
                     reinterpret_cast<int4*>(a), totals, 256 * passes);
  CandKey kp{rows, z_max, bits_r, 1};
  int4* src = reinterpret_cast<int4*>(a);
  int4* dst = reinterpret_cast<int4*>(b);
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    int* tot = totals + 256 * p;
    hipLaunchKernelGGL(k_sort_hist, dim3(nblk), dim3(ST), 0, s, src, cap, nh, nullptr, m, shift, kp, hist, nblk, tot);
    hipLaunchKernelGGL(k_sort_offsets, dim3(256), dim3(ST), 0, s, hist, nblk, tot, cap, nh, nullptr, m);
    hipLaunchKernelGGL(k_sort_scatter, dim3(nblk), dim3(ST), 0, s, src, dst, cap, nh, nullptr, m, shift, kp, hist,
                       nblk, p == passes - 1 ? 1 : 0);
    int4* tmp = src;
    src = dst;
    dst = tmp;
  }
  *sorted = reinterpret_cast<fdas_cand*>(src);
  return hipGetLastError();
}

}  // namespace fdas
