// Sentence-parallel HogBatch epoch on gfx950: the general kernel.
//
// One wavefront owns one sentence at a time (a persistent grid strides over
// the sentences of the range). For its sentence it
//   1. decides subsampling and compacts the kept words (sentence.h);
//   2. forms up to 64 targets at a time lane-parallel (sentence.h; fewer
//      where their negatives would cost LDS residency);
//   3. runs those targets' minibatches in sentence order through the fused
//      minibatch (sgns_core.h), so every minibatch of a sentence sees the
//      updates of the ones before it, while minibatches of different
//      sentences interleave without locks (Hogwild, Sec. 1.1). While a
//      minibatch's rows are on their way the next one's ids are staged.
// Pending input-row updates (PendingSlots, EpochIo): consecutive targets of
// a sentence share most of their input words, so a wavefront adds the
// updates of a cold input row to an LDS slot instead of the matrix, reads
// the row as (matrix row + its pending updates) while the word stays in the
// window, and adds the slot to the matrix once, atomically, when it lets the
// word go. The row traffic of the minibatch path is dominated by its writes;
// this turns about 2 window writes of an input row into one.
// k_export stops after step 2 and writes the minibatches out.
#include <algorithm>
#include <climits>
#include <map>
#include <mutex>
#include <tuple>

#include "group_core.h"
#include "kernel_args.h"
#include "sentence.h"
#include "sgns_core.h"

namespace w2v {

// slots[]: rows of 64 C floats in LDS, the updates a wavefront has made to an
// input row and not yet added to the matrix (lane l's columns l + 64c at
// offset 64c + l). Slot code of distinct input i of a minibatch (lane i):
// -1: no slot, its update goes to the matrix at once; s < kSlotHeld: slot s,
// empty, which takes this minibatch's update; kSlotHeld + s: slot s holds
// pending updates of this word, which the read adds and to which this
// minibatch's update is added. A lane reads and writes its own columns only.
constexpr int kSlotHeld = 64;
constexpr int kMaxPendingSlots = 16;

// Smallest value of lanes 0..15 (x of the other lanes is not used).
__device__ __forceinline__ int row0_min(int x) {
  x = min(x, i_dpp<kDppXor1>(x));
  x = min(x, i_dpp<kDppXor2>(x));
  x = min(x, i_dpp<kDppRowHalfMirror>(x));
  x = min(x, i_dpp<kDppRowMirror>(x));
  return uniform_int(x);
}

// Pending-update slots of a wavefront: lane s < count (at most 16) holds the
// word of slot s (id, -1 if free) and the retained index of the last target
// that used it (used). For the minibatch of target q with the distinct
// inputs mb.in_id[0..n):
//   * a word held in a slot is a hit (find);
//   * any other word with id >= from takes a free slot, else the least
//     recently used slot no input of this minibatch holds (whose pending
//     updates flush(s, id) first adds to the matrix), else none (its update
//     goes to the matrix at once) (assign).
// Slots that this target does not use and that were not used for more than
// `expire` targets before it are flushed and freed, so no update stays
// pending after its word has left the window for good; the caller flushes
// every slot at the end of a sentence. The rows of a minibatch are read
// before its slots are flushed: none of the flushed slots holds one of them.
struct PendingSlots {
  int count, from, expire;
  int id, used;
  uint64_t miss;  // inputs of the current minibatch that may take a slot

  // Finds the slots of target q's words; returns lane i's slot code.
  template <int NMAX>
  __device__ __forceinline__ int find(const Minibatch& mb, int q, int lane) {
    int code = -1;
    miss = __ballot(lane < mb.n && mb.in_id >= from);
    if (miss == 0ull) return code;
    uint64_t hit = 0ull;
    find_from<0, NMAX>(mb, code, hit);
    miss &= ~__ballot(code >= 0);
    if (((hit >> lane) & 1ull) != 0ull) used = q;
    return code;
  }
  // Inputs I, I + 1, ... (free slots and the lanes past the slots hold -1,
  // which no word is).
  template <int I, int NMAX>
  __device__ __forceinline__ void find_from(const Minibatch& mb, int& code,
                                            uint64_t& hit) const {
    if constexpr (I < NMAX) {
      if (I < mb.n) {
        const uint64_t held = __ballot(id == __builtin_amdgcn_readlane(mb.in_id, I));
        const int c = held != 0ull ? kSlotHeld + __builtin_ctzll(held) : -1;
        code = (int)threadIdx.x == I ? c : code;
        hit |= held;
        find_from<I + 1, NMAX>(mb, code, hit);
      }
    }
  }

  // Expires slots and gives slots to the words that have none.
  template <class Flush>
  __device__ __forceinline__ void assign(const Minibatch& mb, int q, int lane, int& code,
                                         const Flush& flush) {
    const bool mine = lane < count;
    for (uint64_t old = __ballot(mine && id >= 0 && used < q - expire); old != 0ull;
         old &= old - 1ull) {
      const int s = __builtin_ctzll(old);
      flush(s, __builtin_amdgcn_readlane(id, s));
      if (lane == s) id = -1;
    }
    for (; miss != 0ull; miss &= miss - 1ull) {
      const int i = __builtin_ctzll(miss);
      // (last use + 1, slot): free slots first, then the least recently used.
      const int key = !mine ? INT_MAX : id < 0 ? lane : (used + 1) * 16 + lane;
      const int least = row0_min(key);
      if (least >= (q + 1) * 16) break;  // every slot holds an input of this minibatch
      const int s = least & 15;
      if (least >= 16) flush(s, __builtin_amdgcn_readlane(id, s));
      if (lane == i) code = s;
      const int word = __builtin_amdgcn_readlane(mb.in_id, i);
      if (lane == s) {
        id = word;
        used = q;
      }
    }
  }

  // Flushes every slot.
  template <class Flush>
  __device__ __forceinline__ void drain(int lane, const Flush& flush) {
    for (uint64_t held = __ballot(lane < count && id >= 0); held != 0ull;
         held &= held - 1ull) {
      const int s = __builtin_ctzll(held);
      flush(s, __builtin_amdgcn_readlane(id, s));
    }
    id = -1;
  }
};

// Rows of the live matrices (Core's Io): read coherently, updated by tier,
// input rows with a slot code in the wavefront's pending slots.
template <int C>
struct EpochIo {
  RowTiers<C> tiers;
  float* M_in;
  float* M_out;
  float* slots;
  PendingSlots pend;
  int q;     // retained index of the current target
  int code;  // lane i: slot code of input i

  // Adds the pending updates of slot s to the M_in row of word id.
  __device__ __forceinline__ void flush(int s, int id) const {
    const float* p = slot_row(s);
    float d[C];
#pragma unroll
    for (int c = 0; c < C; ++c) d[c] = p[kWave * c];
    tiers.add(0, M_in, id, d);
  }
  __device__ __forceinline__ void before_inputs(const Minibatch& mb) {
    if (pend.count > 0)
      pend.assign(mb, q, tiers.lane, code, [&](int s, int id) { flush(s, id); });
  }

  __device__ __forceinline__ void load_in(int id, bool ok, float (&r)[C]) const {
    load_row<C, true>(M_in, id, tiers.ld, ok ? tiers.D : 0, tiers.lane, r);
  }
  __device__ __forceinline__ void load_out(int id, bool ok, float (&r)[C]) const {
    load_row<C, true>(M_out, id, tiers.ld, ok ? tiers.D : 0, tiers.lane, r);
  }
  template <int N>
  __device__ __forceinline__ void settle_in(const Minibatch& mb, float (&a)[N][C]) const {
    const uint64_t split =
        __ballot(tiers.lane < mb.n && mb.in_id < tiers.split_rows);
    add_splits(0, split, [&](int i) { return __builtin_amdgcn_readlane(mb.in_id, i); }, a);
    const uint64_t held = __ballot(code >= kSlotHeld);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (((held >> i) & 1ull) != 0ull) {
        const float* p = slot_row(__builtin_amdgcn_readlane(code, i) - kSlotHeld);
#pragma unroll
        for (int c = 0; c < C; ++c) a[i][c] += p[kWave * c];
      }
    }
  }
  template <int N>
  __device__ __forceinline__ void settle_out(const Minibatch& mb, int k0,
                                             float (&o)[N][C]) const {
    // bit k: column k0 + k is a split row
    const uint64_t neg =
        __ballot(tiers.lane < mb.n_out - 1 && mb.neg_id < tiers.split_rows);
    uint64_t split = k0 == 0 ? neg << 1 : neg >> (k0 - 1);
    if (k0 == 0 && mb.target < tiers.split_rows) split |= 1ull;
    add_splits(1, split & ((1ull << N) - 1ull),
               [&](int k) {
                 return k0 + k == 0 ? mb.target
                                    : __builtin_amdgcn_readlane(mb.neg_id, (k0 + k - 1) & 63);
               },
               o);
  }
  // Adds the partial rows of the rows whose bits are set, one row after the
  // other: split rows are few, and the code for a row is there once.
  template <int N, class Id>
  __device__ __forceinline__ void add_splits(int m, uint64_t rows, const Id& id,
                                             float (&r)[N][C]) const {
#pragma unroll 1
    for (; rows != 0ull; rows &= rows - 1ull) {
      const int i = __builtin_ctzll(rows);
      float t[C];
      tiers.split_sum(m, id(i), t);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        if (j == i) {
#pragma unroll
          for (int c = 0; c < C; ++c) r[j][c] += t[c];
        }
      }
    }
  }
  template <int N>
  __device__ __forceinline__ void put_out(int, int id, const float (&o)[N],
                                          const float (&g)[N], int c0) const {
    tiers.update(1, M_out, id, o, g, c0);
  }
  // A slot's row is read, added to and written back rather than added to by
  // LDS atomics: a ds_add_f32 of a wavefront costs the CU's LDS unit so much
  // that 8 wavefronts per CU waited for it (5e6 uniform tokens at D = 300:
  // 47 ms).
  template <int N>
  __device__ __forceinline__ void fetch_kept(int i, float (&kept)[N], int c0) const {
    const int s = __builtin_amdgcn_readlane(code, i);
    if (s >= kSlotHeld) {
      const float* p = slot_row(s - kSlotHeld) + kWave * c0;
#pragma unroll
      for (int c = 0; c < N; ++c) kept[c] = p[kWave * c];
    } else {
#pragma unroll
      for (int c = 0; c < N; ++c) kept[c] = 0.f;
    }
  }
  template <int N>
  __device__ __forceinline__ void put_in(int i, int id, const float (&row)[N],
                                         const float (&g)[N], const float (&kept)[N],
                                         int c0) const {
    const int s = __builtin_amdgcn_readlane(code, i);
    if (s < 0) {
      tiers.update(0, M_in, id, row, g, c0);
    } else {
      float* p = slot_row(s & (kSlotHeld - 1)) + kWave * c0;
#pragma unroll
      for (int c = 0; c < N; ++c) p[kWave * c] = kept[c] + g[c];
    }
  }
  __device__ __forceinline__ float* slot_row(int s) const {
    return slots + s * (kWave * C) + tiers.lane;
  }
};

// Sentences that run at once per CU in a default launch: the waves per SIMD
// that the row registers of a shape leave, times the four SIMDs. How far
// concurrent sentences drift from the sequential epoch depends on how many
// there are, so this is part of what a launch computes, not only of how fast
// it does: it follows from C, the capacity of input rows and whether the N x
// (K + 1) logits fit one reduction of 64 (several_blocks), and it stays as it
// is when the kernels change. The kernels' own output blocks are another
// matter: Core takes up to 6 columns in one block whatever nmax is, so a
// one-block kernel of nmax 16 or 32 serves K on both sides of this rule, and
// its registers allow the larger of the two values.
constexpr bool several_blocks_of(int nmax, int K) { return K + 1 > kWave / nmax; }

constexpr int sentences_per_simd(int C, int nmax, bool several_blocks) {
  if (nmax == 32) return !several_blocks && C == 1 ? 3 : 2;
  if (nmax == 16) return several_blocks ? (C == 1 ? 3 : C <= 3 ? 2 : 1) : C <= 2 ? 3 : 2;
  return several_blocks ? (C <= 2 ? 3 : C <= 5 ? 2 : 1) : C <= 4 ? 3 : 2;
}

// Waves per SIMD the register allocation must allow: the most sentences per
// SIMD that a launch of the kernel runs.
template <int C, int NMAX, bool kMulti>
constexpr int epoch_waves_per_eu() {
  return sentences_per_simd(C, NMAX, kMulti);
}

// The kernel's arguments, read again from the kernel argument segment: what
// only the start of a sentence or of a batch of targets needs does not hold
// scalar registers (or vector registers, spilled) in between.
__device__ __forceinline__ EpochArgs reread_args() {
  typedef const __attribute__((address_space(4))) EpochArgs* Segment;
  Segment p = (Segment)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const EpochArgs*)p;
}

template <int C, int NMAX, bool kMulti>
__global__ __launch_bounds__(kWave) __attribute__((
    amdgpu_waves_per_eu(epoch_waves_per_eu<C, NMAX, kMulti>()))) void k_epoch(EpochArgs a) {
  __shared__ SentenceLds sl;
  extern __shared__ int32_t negs_lds[];  // [TB][K], then the pending slots
  const int lane = threadIdx.x;
  const int K = a.K;
  const bool want_loss = a.loss != nullptr;
  const int TB = a.target_batch;  // targets formed at once
  EpochIo<C> io{{a.part, a.split_rows, a.hot_rows, a.ld, a.D, lane},
                a.M_in,
                a.M_out,
                reinterpret_cast<float*>(negs_lds + TB * (K > 0 ? K : 1)),
                {a.pend_slots, a.pend_from, 2 * a.w, -1, 0, 0ull},
                0,
                -1};

  int64_t n_mb = 0, sum_n = 0, raw = 0, rejected = 0, rows = 0;
  double lsum = 0.0, lcnt = 0.0;
  int bucket = -1;

  for (int64_t s = blockIdx.x; s < a.n_sent; s += gridDim.x) {
    const EpochArgs ka = reread_args();
    const int64_t sb = ka.pos_begin + s * ka.L;
    const int64_t se = min(sb + (int64_t)ka.L, ka.pos_end);
    const int len = (int)(se - sb);
    raw += len;
    const int n_ret = keep_and_compact<false>(ka, sb, len, lane, sl, rejected);

    for (int q0 = 0; q0 < n_ret; q0 += TB) {
      uint64_t bad;
      const FormedTarget t = form_targets<false>(reread_args(), sb, q0, n_ret, lane, sl,
                                                 negs_lds, TB, bad);
      uint64_t todo = __ballot(t.n > 0);
      rejected += __popcll(todo & bad);
      todo &= ~bad;
      n_mb += __popcll(todo);
      // One minibatch behind the ids: the turn that stages target q0 + j runs
      // the minibatch staged in the turn before, whose rows are on their way.
      Minibatch staged{};
      int j = -1;
      while (j >= 0 || todo != 0ull) {
        const Minibatch mb = staged;
        const int cur = j;
        Core<C, NMAX, kMulti> core;
        if (cur >= 0) core.load(io, mb);
        j = -1;
        if (todo != 0ull) {
          j = __builtin_ctzll(todo);
          todo &= todo - 1ull;
          const int n = __builtin_amdgcn_readlane(t.n, j);
          int jj = __builtin_amdgcn_readlane(t.lo, j) + lane;
          if (jj >= q0 + j) ++jj;
          const int ctx = lane < n ? sl.ret_id[jj] : 0;
          const int neg = lane < K ? negs_lds[j * K + lane] : 0;
          sum_n += n;
          staged = stage_minibatch<(NMAX > 16)>(lane, ctx, (1ull << n) - 1ull,
                                                __builtin_amdgcn_readlane(t.id, j), neg, K);
          rows += staged.n + staged.n_out;
        }
        if (cur < 0) continue;
        io.q = q0 + cur;
        if (io.pend.count > 0) io.code = io.pend.template find<NMAX>(mb, io.q, lane);
        float loss_part = 0.f;
        core.run(io, lane, mb,
                 __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t.alpha), cur)),
                 want_loss, loss_part);
        if (want_loss) {
          const int b = __builtin_amdgcn_readlane(t.bucket, cur);
          if (b != bucket) {
            if (bucket >= 0) flush_loss(a.loss, bucket, lsum, lcnt, lane);
            bucket = b;
          }
          lsum += (double)loss_part;
          lcnt += (double)__builtin_amdgcn_readlane(t.n, cur);
        }
      }
      __syncthreads();
    }
    io.pend.drain(lane, [&](int slot, int id) { io.flush(slot, id); });
  }
  if (want_loss && bucket >= 0) flush_loss(a.loss, bucket, lsum, lcnt, lane);
  flush_stats(a, lane, n_mb, sum_n, raw, rejected, rows);
}

// The minibatches of the epoch written out instead of run.
__global__ __launch_bounds__(kWave) void k_export(EpochArgs a) {
  __shared__ SentenceLds sl;
  extern __shared__ int32_t negs_lds[];  // [kWave][K]
  const int lane = threadIdx.x;
  int64_t n_mb = 0, sum_n = 0, raw = 0, rejected = 0;
  for (int64_t s = blockIdx.x; s < a.n_sent; s += gridDim.x) {
    const int64_t sb = a.pos_begin + s * a.L;
    const int64_t se = min(sb + (int64_t)a.L, a.pos_end);
    const int len = (int)(se - sb);
    raw += len;
    const int n_ret = keep_and_compact<true>(a, sb, len, lane, sl, rejected);
    for (int q0 = 0; q0 < n_ret; q0 += kWave) {
      uint64_t bad;
      const FormedTarget t =
          form_targets<false>(a, sb, q0, n_ret, lane, sl, negs_lds, kWave, bad);
      export_targets(a, sb, q0, n_ret, lane, sl, t, negs_lds);
      const uint64_t formed = __ballot(t.n > 0);
      rejected += __popcll(formed & bad);
      n_mb += __popcll(formed & ~bad);
      sum_n += wave_sum_int(((formed & ~bad) >> lane) & 1ull ? t.n : 0);
      __syncthreads();
    }
  }
  flush_stats(a, lane, n_mb, sum_n, raw, rejected, 0);
}

// Partial rows of the split rows: cleared before an epoch, summed (in the
// order g = 0, 1, ...) and added into the matrices with one rounding, then
// cleared, after it; a row with nothing pending keeps its bits. One thread
// per (matrix, row, column).
__global__ __launch_bounds__(256) void k_part_clear(EpochArgs a) {
  const int64_t n = (int64_t)2 * a.split_rows * kSplitParts * a.ld;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    a.part[i] = 0.f;
}

__global__ __launch_bounds__(256) void k_part_fold(EpochArgs a) {
  const int64_t n = (int64_t)2 * a.split_rows * a.D;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int col = (int)(i % a.D);
    const int64_t mr = i / a.D;  // m * split_rows + row
    const int m = (int)(mr / a.split_rows);
    const int64_t row = mr % a.split_rows;
    float* pb = a.part + mr * kSplitParts * a.ld + col;
    float* dst = (m == 0 ? a.M_in : a.M_out) + row * a.ld + col;
    float sum = 0.f;
    for (int g = 0; g < kSplitParts; ++g) {
      sum += pb[g * a.ld];
      pb[g * a.ld] = 0.f;
    }
    if (sum != 0.f) *dst += sum;
  }
}

// The same epoch with the K negatives shared by groups of G consecutive
// targets (group_core.h): per group, the members' input occurrences and the
// output candidates (member targets, then the group's negatives) are staged
// deduplicated with their group tables, then one snapshot step runs over the
// group (group_core.h) with up to OMAX output columns. Groups start at
// retained indices that are multiples of G (G divides the 64-target
// batches).

// Sentences per SIMD of a default launch, as sentences_per_simd is for
// k_epoch: part of what a launch computes, so it follows from C and OMAX (a
// wavefront's rows: OMAX output rows, their updates and a block of input
// rows) and not from what a build's registers leave. Builds use at most the
// registers that allow it; k_epoch_grouped<4, 16> just fits two waves per
// SIMD and runs one.
constexpr int grouped_sentences_per_simd(int C, int omax) {
  if (omax == 32) return 2;
  if (omax == 16) return C == 1 ? 3 : C <= 3 ? 2 : 1;
  return C <= 2 ? 3 : C <= 5 ? 2 : 1;
}

template <int C, int OMAX>
__global__ __launch_bounds__(kWave) void k_epoch_grouped(EpochArgs a) {
  __shared__ SentenceLds sl;
  __shared__ TargetBatch tb;
  __shared__ GroupRows mb;
  __shared__ GroupLds gl;
  extern __shared__ int32_t negs_lds[];  // [kWave][K]
  const int lane = threadIdx.x;
  const int K = a.K;
  const int G = a.group;
  const bool want_loss = a.loss != nullptr;

  int64_t n_mb = 0, sum_n = 0, raw = 0, rejected = 0, rows = 0;
  double lsum = 0.0, lcnt = 0.0;
  int bucket = -1;

  for (int64_t s = blockIdx.x; s < a.n_sent; s += gridDim.x) {
    const int64_t sb = a.pos_begin + s * a.L;
    const int64_t se = min(sb + (int64_t)a.L, a.pos_end);
    const int len = (int)(se - sb);
    raw += len;
    const int n_ret = keep_and_compact<false>(a, sb, len, lane, sl, rejected);

    for (int q0 = 0; q0 < n_ret; q0 += kWave) {
      form_target_batch<(C >= 6)>(a, sb, q0, n_ret, lane, sl, tb, negs_lds);
      const int cnt = min(kWave, n_ret - q0);
      for (int j0 = 0; j0 < cnt; j0 += G) {
        // Members: lane g < G holds the input count of target j0 + g.
        const int n_g = (lane < G && j0 + lane < cnt) ? tb.n[j0 + lane] : 0;
        const uint64_t members = __ballot(n_g > 0);
        if (members == 0ull) continue;
        if (uniform_int(tb.bad[j0]) != 0) {
          rejected += __popcll(members);
          continue;
        }
        // Input occurrences, member by member, one per lane.
        int off = 0, my_g = -1, my_i = 0;
#pragma unroll
        for (int g = 0; g < kMaxGroup; ++g) {
          if (g < G) {
            const int ng = __builtin_amdgcn_readlane(n_g, g);
            if (lane >= off && lane < off + ng) {
              my_g = g;
              my_i = lane - off;
            }
            off += ng;
          }
        }
        const int total = off;
        if (my_g >= 0) {
          const int q = q0 + j0 + my_g;
          int jj = tb.lo[j0 + my_g] + my_i;
          if (jj >= q) ++jj;
          gl.occ_id[lane] = sl.ret_id[jj];
          gl.occ_g[lane] = my_g;
        }
        if (lane < G)
          gl.alpha[lane] = n_g > 0 ? tb.alpha[j0 + lane] : 0.f;
        // Output candidates: member targets, then the group's negatives
        // (drawn at its first retained position).
        int cid = -1;
        if (lane < G) {
          if (n_g > 0) cid = sl.ret_id[q0 + j0 + lane];
        } else if (lane < G + K) {
          cid = negs_lds[j0 * K + (lane - G)];
        }
        gl.cand_id[lane] = cid;
        __syncthreads();

        // Distinct input rows and their multiplicity per member.
        const int my_id = my_g >= 0 ? gl.occ_id[lane] : -1;
        bool first = my_g >= 0;
        float mult[kMaxGroup];
#pragma unroll
        for (int g = 0; g < kMaxGroup; ++g) mult[g] = 0.f;
        if (my_g >= 0) {
          for (int l2 = 0; l2 < total; ++l2) {
            if (gl.occ_id[l2] != my_id) continue;
            if (l2 < lane) first = false;
            const int g2 = gl.occ_g[l2];
#pragma unroll
            for (int g = 0; g < kMaxGroup; ++g) mult[g] += (g2 == g) ? 1.f : 0.f;
          }
        }
        const uint64_t fin = __ballot(first);
        if (first) {
          const int dst = __popcll(fin & lanes_below(lane));
          mb.ctx[dst] = my_id;
#pragma unroll
          for (int g = 0; g < kMaxGroup; ++g) gl.m[dst][g] = mult[g];
        }
        const int n_in = __popcll(fin);

        // Distinct output columns: member-target bits and negative weight.
        bool cfirst = cid >= 0;
        uint32_t bits = 0u;
        float nw = 0.f;
        if (cid >= 0) {
          for (int c2 = 0; c2 < G + K; ++c2) {
            if (gl.cand_id[c2] != cid) continue;
            if (c2 < lane) cfirst = false;
            if (c2 < G) bits |= 1u << c2;
            else nw += 1.f;
          }
        }
        const uint64_t fout = __ballot(cfirst);
        if (cfirst) {
          const int dst = __popcll(fout & lanes_below(lane));
          mb.out[dst] = cid;
          gl.tbits[dst] = bits;
          gl.negw[dst] = nw;
        }
        const int n_out = __popcll(fout);
        __syncthreads();

        n_mb += __popcll(members);
        sum_n += total;
        rows += n_in + n_out;
        float loss_part = 0.f;
        run_group<C, OMAX>(a, lane, n_in, n_out, mb, gl, G, want_loss, loss_part);
        if (want_loss) {
          const int qf = q0 + j0 + (int)__builtin_ctzll(members);
          const int64_t p = sb + sl.ret_off[qf];
          const int b = (int)(p * (int64_t)a.n_buckets / a.T);
          if (b != bucket) {
            if (bucket >= 0) flush_loss(a.loss, bucket, lsum, lcnt, lane);
            bucket = b;
          }
          lsum += (double)loss_part;
          if (lane == 0) lcnt += (double)total;
        }
        __syncthreads();
      }
      __syncthreads();
    }
  }
  if (want_loss && bucket >= 0) flush_loss(a.loss, bucket, lsum, lcnt, lane);
  flush_stats(a, lane, n_mb, sum_n, raw, rejected, rows);
}

// ------------------------------------------------------------ launchers --

static int part_grid(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return (int)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

hipError_t launch_part_clear(const EpochArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_part_clear,
                     dim3(part_grid((int64_t)2 * a.split_rows * kSplitParts * a.ld)),
                     dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_part_fold(const EpochArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_part_fold, dim3(part_grid((int64_t)2 * a.split_rows * a.D)),
                     dim3(256), 0, s, a);
  return hipGetLastError();
}

#define W2V_TRAIN_SHAPES(X) \
  X(1, 10) X(2, 10) X(3, 10) X(4, 10) X(5, 10) X(6, 10) X(8, 10) X(10, 10) \
  X(1, 16) X(2, 16) X(3, 16) X(4, 16) X(5, 16) X(1, 32) X(2, 32)

using EpochKernel = void (*)(EpochArgs);

// Kernel for C columns per lane, up to nmax input words, and K negatives:
// the single-block variant when the K+1 output columns fit one reduction.
static EpochKernel train_kernel_for(int C, int nmax, int K) {
  const bool multi = K + 1 > Core<1, 10, false>::KB;
#define W2V_PICK(c, n) \
  if (C == c && nmax == n) \
    return multi ? k_epoch<c, n, true> : k_epoch<c, n, false>;
  W2V_TRAIN_SHAPES(W2V_PICK)
#undef W2V_PICK
  return nullptr;
}

bool train_shape_supported(int C, int nmax) {
  return train_kernel_for(C, nmax, 0) != nullptr;
}

int columns_for(int D) {
  static const int kCols[] = {1, 2, 3, 4, 5, 6, 8, 10};
  for (int c : kCols)
    if (D <= kWave * c) return c;
  return 0;
}

int inputs_cap_for(int n) {
  if (n <= 10) return 10;
  if (n <= 16) return 16;
  if (n <= 32) return 32;
  return 0;
}

// gfx950 gives each CU 160 KB of LDS and allocates it to a workgroup in
// granules of 1280 bytes. The runtime's occupancy query admits requests that
// the granules do not: at D = 100, K = 5 it allowed 12 workgroups per CU
// with 12,808 bytes each, 12 x 10 granules would need 168,960 bytes, and a
// twelfth of the persistent grid then waited for a free CU (-34%
// throughput). Both limits apply.
constexpr size_t kLdsPerCu = 160 * 1024;
constexpr size_t kLdsGranule = 1280;

int resident_blocks_per_cu(const void* kernel, size_t dyn_lds) {
  int blocks = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kernel, kWave,
                                                   dyn_lds) != hipSuccess)
    return 0;
  hipFuncAttributes attr{};
  if (hipFuncGetAttributes(&attr, kernel) != hipSuccess) return 0;
  const size_t per = (attr.sharedSizeBytes + dyn_lds + kLdsGranule - 1) /
                     kLdsGranule * kLdsGranule;
  const int by_lds = (int)(kLdsPerCu / per);
  return blocks < by_lds ? blocks : by_lds;
}

static size_t negatives_lds(int K, int batch = kWave) {
  return sizeof(int32_t) * (size_t)batch * (size_t)(K > 0 ? K : 1);
}

static size_t epoch_dyn_lds(const EpochArgs& a) {
  return negatives_lds(a.K);
}

static size_t slot_bytes(int C) { return sizeof(float) * (size_t)kWave * C; }

// Shape of the training launch for (C, nmax, K) on the current device:
// targets formed at once, pending slots and resident workgroups per CU.
// Computed from occupancy queries once per device and shape.
struct TrainShape {
  int target_batch, pending_slots, blocks_per_cu;
};

static TrainShape compute_train_shape(int C, int nmax, int K) {
  TrainShape t{kWave, 0, 0};
  EpochKernel k = train_kernel_for(C, nmax, K);
  if (k == nullptr) return t;
  const void* f = reinterpret_cast<const void*>(k);
  const int by_rule = 4 * sentences_per_simd(C, nmax, several_blocks_of(nmax, K));
  const int best = std::min(resident_blocks_per_cu(f, negatives_lds(K, 8)), by_rule);
  while (t.target_batch > 8 &&
         resident_blocks_per_cu(f, negatives_lds(K, t.target_batch)) < best)
    t.target_batch /= 2;
  const size_t negs = negatives_lds(K, t.target_batch);
  t.blocks_per_cu = std::min(resident_blocks_per_cu(f, negs), by_rule);
  if (t.blocks_per_cu <= 0) return t;
  for (int n = kMaxPendingSlots; n >= 2; --n)
    if (resident_blocks_per_cu(f, negs + n * slot_bytes(C)) >= t.blocks_per_cu) {
      t.pending_slots = n;
      break;
    }
  return t;
}

static TrainShape train_shape(int C, int nmax, int K) {
  static std::mutex mu;
  static std::map<std::tuple<int, int, int, int>, TrainShape> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return compute_train_shape(C, nmax, K);
  const auto key = std::make_tuple(dev, C, nmax, K);
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  const TrainShape t = compute_train_shape(C, nmax, K);
  if (t.blocks_per_cu > 0) cache[key] = t;  // failed queries are retried
  return t;
}

int train_target_batch(int C, int nmax, int K) { return train_shape(C, nmax, K).target_batch; }

int train_pending_slots(int C, int nmax, int K) { return train_shape(C, nmax, K).pending_slots; }

int train_blocks_per_cu(int C, int nmax, int K) { return train_shape(C, nmax, K).blocks_per_cu; }

hipError_t launch_train(int C, int nmax, const EpochArgs& a, int grid,
                        hipStream_t s) {
  EpochKernel k = train_kernel_for(C, nmax, a.K);
  if (k == nullptr) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(grid), dim3(kWave),
                     negatives_lds(a.K, a.target_batch) + a.pend_slots * slot_bytes(C),
                     s, a);
  return hipGetLastError();
}

#define W2V_GROUP_SHAPES(X) \
  X(1, 10) X(2, 10) X(3, 10) X(4, 10) X(5, 10) X(6, 10) X(8, 10) X(10, 10) \
  X(1, 16) X(2, 16) X(3, 16) X(4, 16) X(5, 16) X(6, 16) X(1, 32) X(2, 32)

static EpochKernel grouped_kernel_for(int C, int omax) {
#define W2V_PICK(c, n) \
  if (C == c && omax == n) return k_epoch_grouped<c, n>;
  W2V_GROUP_SHAPES(W2V_PICK)
#undef W2V_PICK
  return nullptr;
}

int group_outputs_cap_for(int n) {
  if (n <= 10) return 10;
  if (n <= 16) return 16;
  if (n <= 32) return 32;
  return 0;
}

bool grouped_shape_supported(int C, int omax) {
  return grouped_kernel_for(C, omax) != nullptr;
}

int grouped_blocks_per_cu(int C, int omax, int K) {
  EpochKernel k = grouped_kernel_for(C, omax);
  if (k == nullptr) return 0;
  // The other part of the rule: no more sentences at once than 160 KB of LDS
  // hold at 11320 bytes and the negatives each.
  const size_t per = (11320 + negatives_lds(K) + kLdsGranule - 1) / kLdsGranule * kLdsGranule;
  const int by_rule = std::min(4 * grouped_sentences_per_simd(C, omax), (int)(kLdsPerCu / per));
  return std::min(resident_blocks_per_cu(reinterpret_cast<const void*>(k), negatives_lds(K)),
                  by_rule);
}

hipError_t launch_grouped(int C, int omax, const EpochArgs& a, int grid,
                          hipStream_t s) {
  EpochKernel k = grouped_kernel_for(C, omax);
  if (k == nullptr) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(grid), dim3(kWave), epoch_dyn_lds(a), s, a);
  return hipGetLastError();
}

hipError_t launch_export(const EpochArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_export, dim3(grid), dim3(kWave),
                     epoch_dyn_lds(a), s, a);
  return hipGetLastError();
}

}  // namespace w2v
