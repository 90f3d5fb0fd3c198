// Per-sentence minibatch formation on one wavefront (gfx950), shared by the
// epoch kernels and the minibatch export so that all of them draw the same
// minibatches.
//
//  * keep_and_compact: reads a sentence's raw ids, decides subsampling per
//    position (Philox word 0 against the keep threshold) and compacts the
//    kept words into LDS with a ballot prefix count.
//  * form_targets: forms up to 64 targets lane-parallel: window half-width
//    (word 1), the K shared negatives (words 2.., one table read each), the
//    decayed learning rate, and whether a negative id is out of range;
//    form_target_batch leaves them in LDS, export_targets writes them out.
#pragma once

#include "device_common.h"
#include "kernel_args.h"

namespace w2v {

constexpr int kMaxSentence = 1024;
constexpr int kMaxWindow = 16;

struct SentenceLds {
  int32_t ret_id[kMaxSentence];   // kept word ids, in order
  int16_t ret_off[kMaxSentence];  // their offsets in the sentence
};

// Targets q0 .. q0+63 of a sentence.
struct TargetBatch {
  int32_t lo[kWave];              // first retained index of the window
  int32_t n[kWave];               // number of input words
  float alpha[kWave];
  int32_t bad[kWave];             // a negative id outside [0, V)
};

__device__ __forceinline__ uint32_t word_of(const U64x4& b, int j) {
  const int m = j >> 1;
  const uint64_t v = m == 0 ? b.v[0] : m == 1 ? b.v[1] : m == 2 ? b.v[2] : b.v[3];
  return (j & 1) ? (uint32_t)(v >> 32) : (uint32_t)v;
}

// Subsampling and compaction of the sentence [sb, sb + len). Returns the
// number of kept words; counts out-of-range ids in `rejected`. The export
// variant marks every position that forms no minibatch with -1.
template <bool kExport>
__device__ __forceinline__ int keep_and_compact(const EpochArgs& a, int64_t sb,
                                                int len, int lane,
                                                SentenceLds& sl,
                                                int64_t& rejected) {
  const uint64_t e = (uint64_t)a.epoch;
  int n_ret = 0;
  for (int base = 0; base < len; base += kWave) {
    const int off = base + lane;
    const bool in = off < len;
    const int x = in ? a.corpus[sb + off] : 0;
    // -1 marks a word dropped from the vocabulary (w2v_build_vocab): it is
    // removed from the sentence before windows form, as any out-of-range id,
    // but it is no error.
    const bool bad = in && (x < -1 || x >= a.V);
    bool keep = in && x >= 0 && x < a.V;
    if (keep && a.thr != nullptr) {
      const U64x4 blk = stream_block(a.seed, (uint64_t)(sb + off), e, 0);
      keep = (uint32_t)blk.v[0] <= a.thr[x];
    }
    const uint64_t m = __ballot(keep);
    if (keep) {
      const int dst = n_ret + __popcll(m & lanes_below(lane));
      sl.ret_id[dst] = x;
      sl.ret_off[dst] = (int16_t)off;
    }
    n_ret += __popcll(m);
    rejected += __popcll(__ballot(bad));
    if (kExport && in && !keep) a.out_targets[sb + off - a.pos_begin] = -1;
  }
  __syncthreads();
  return n_ret;
}

// One target as formed, in one lane.
struct FormedTarget {
  int id = -1;        // the target word
  int lo = 0;         // first retained index of the window
  int n = 0;          // number of input words (0: no minibatch)
  float alpha = 0.f;
  int bucket = 0;     // loss bucket (formed only with a loss)
};

// Forms targets q0 + j, j < TB (TB a power of two up to 64, q0 + j < n_ret):
// lane j returns target j, its negatives go to negs[j K + k], and `bad` gets
// bit j where one of them is outside [0, V). The 64 / TB lanes l = j mod TB
// share target j: lane l takes every (64 / TB)-th Philox block from block
// l / TB on. The table reads of a block (each a random access to a table of
// up to 400 MB) come before any use of one. With kTogether they are issued
// without a branch, a word that is no negative reading entry 0, and are all
// in flight at once; else each stands behind its test, so nothing is read in
// vain, but the compiler waits for some of them before it issues the next.
// That wait shows where a SIMD holds one wavefront with little else to do
// (grouped epoch, D = 384, G = 4, K = 5, 4e6 tokens: 24.6 ms behind the tests,
// 22.6 together); elsewhere reading together changes the times by 2% either
// way (planted shape, K = 25: 81.4 / 80.2 ms; D = 485, K = 25: 107.7 / 109.5).
template <bool kTogether>
__device__ __forceinline__ FormedTarget form_targets(const EpochArgs& a, int64_t sb,
                                                     int q0, int n_ret, int lane,
                                                     const SentenceLds& sl,
                                                     int32_t* negs, int TB,
                                                     uint64_t& bad) {
  const uint64_t e = (uint64_t)a.epoch;
  const int K = a.K;
  const int w = a.w;
  const int j = lane & (TB - 1);
  const int q = q0 + j;
  const int share = kWave / TB;
  FormedTarget t;
  bool bad_id = false;
  if (q < n_ret) {
    const int64_t p = sb + sl.ret_off[q];
    t.id = sl.ret_id[q];
    const int n_blocks = (K + 9) >> 3;  // words 0 .. K + 1
    for (int b = (int)((unsigned)lane / (unsigned)TB); b < n_blocks; b += share) {
      const U64x4 blk = stream_block(a.seed, (uint64_t)p, e, (uint64_t)b);
      if (b == 0) {
        const int h = w - (int)scale_draw(word_of(blk, 1), (uint64_t)w);
        t.lo = max(q - h, 0);
        t.n = min(q + h, n_ret - 1) - t.lo;
      }
      const int k0 = 8 * b - 2;  // negative of the block's word 0
      int neg[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = k0 + i;
        if constexpr (kTogether) {
          const uint64_t at = scale_draw(word_of(blk, i), (uint64_t)a.table_size);
          neg[i] = a.table[k >= 0 && k < K ? at : 0];
          if (k < 0 || k >= K) neg[i] = 0;
        } else {
          neg[i] = 0;
          if (k >= 0 && k < K)
            neg[i] = a.table[scale_draw(word_of(blk, i), (uint64_t)a.table_size)];
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = k0 + i;
        bad_id |= neg[i] < 0 || neg[i] >= a.V;
        if (k >= 0 && k < K) negs[j * K + k] = neg[i];
      }
    }
    t.alpha = decayed_alpha(a.alpha0, a.min_frac, a.epoch, a.n_epochs, a.T, p);
    if (a.loss != nullptr) t.bucket = (int)(p * (int64_t)a.n_buckets / a.T);
  }
  bad = __ballot(bad_id);
  for (int s = kWave / 2; s >= TB; s /= 2) bad |= bad >> s;
  if (TB < kWave) {
    bad &= (1ull << TB) - 1ull;
    if (lane >= TB) t.n = 0;
  }
  __syncthreads();
  return t;
}

// The same for the 64 targets q0 .. q0 + 63, into LDS.
template <bool kTogether>
__device__ __forceinline__ void form_target_batch(const EpochArgs& a, int64_t sb,
                                                  int q0, int n_ret, int lane,
                                                  const SentenceLds& sl,
                                                  TargetBatch& tb, int32_t* negs) {
  uint64_t bad;
  const FormedTarget t =
      form_targets<kTogether>(a, sb, q0, n_ret, lane, sl, negs, kWave, bad);
  tb.lo[lane] = t.lo;
  tb.n[lane] = t.n;
  tb.alpha[lane] = t.alpha;
  tb.bad[lane] = (int)((bad >> lane) & 1ull);
  __syncthreads();
}

// Writes the formed targets q0 .. q0 + 63 out (minibatch export).
__device__ __forceinline__ void export_targets(const EpochArgs& a, int64_t sb, int q0,
                                               int n_ret, int lane,
                                               const SentenceLds& sl,
                                               const FormedTarget& t,
                                               const int32_t* negs) {
  const int K = a.K;
  const int w = a.w;
  const int q = q0 + lane;
  if (q >= n_ret) return;
  const int64_t r = sb + sl.ret_off[q] - a.pos_begin;
  if (t.n == 0) {
    a.out_targets[r] = -1;
    return;
  }
  a.out_targets[r] = t.id;
  for (int i = 0; i < 2 * w; ++i) {
    int id = -1;
    if (i < t.n) id = sl.ret_id[t.lo + i + (t.lo + i >= q ? 1 : 0)];
    a.out_ctx[r * 2 * w + i] = id;
  }
  for (int k = 0; k < K; ++k) {
    const int neg = negs[lane * K + k];
    a.out_negs[r * K + k] = neg;
    a.out_mask[r * K + k] = (uint8_t)(neg == t.id);
  }
  a.out_alpha[r] = t.alpha;
}

// Adds a wave's loss sums for one bucket (lane 0 holds the input count).
__device__ __forceinline__ void flush_loss(double* loss, int bucket,
                                           double& lsum, double& lcnt,
                                           int lane) {
  double s = lsum;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m);
  if (lane == 0) {
    unsafeAtomicAdd(loss + 2 * bucket, s);
    unsafeAtomicAdd(loss + 2 * bucket + 1, lcnt);
  }
  lsum = 0.0;
  lcnt = 0.0;
}

// Adds a wave's counters into stats[0..4] (lane 0) and raises the device's
// error word if the wave skipped anything for an id outside [0, V).
__device__ __forceinline__ void flush_stats(const EpochArgs& a, int lane,
                                            int64_t n_mb, int64_t sum_n,
                                            int64_t raw, int64_t rejected,
                                            int64_t rows) {
  int64_t* const stats = a.stats;
  if (lane == 0) report_bad_ids(a.status, rejected);
  if (stats != nullptr && lane == 0) {
    atomicAdd((unsigned long long*)&stats[0], (unsigned long long)n_mb);
    atomicAdd((unsigned long long*)&stats[1], (unsigned long long)sum_n);
    atomicAdd((unsigned long long*)&stats[2], (unsigned long long)raw);
    atomicAdd((unsigned long long*)&stats[3], (unsigned long long)rejected);
    atomicAdd((unsigned long long*)&stats[4], (unsigned long long)rows);
  }
}

}  // namespace w2v
