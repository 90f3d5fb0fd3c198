// The fused HogBatch minibatch on one wavefront (gfx950, wave64).
//
// One minibatch = N input words (rows of M_in) and the target plus K shared
// negatives (rows of M_out) (Sec. 1.1, negative sample sharing; Fig. 1
// right). The N x (K+1) logit block, the sigmoid error of Alg. 1 and both
// gradient products are formed here from rows gathered once:
//
//   X = A O^T   E = alpha (l - sigma(X))   dA = E O   dO = E^T A
//
// Rows are staged deduplicated. A negative equal to the target is masked;
// repeated negatives collapse into one column of weight m, and repeated input
// words into one row of weight m (m identical rows or columns have identical
// logits and errors, so one copy with its error scaled by m yields the same
// dA and dO). Every row is then read once and written once per minibatch:
// all reads precede the minibatch's own writes even when the output columns
// take several blocks, and a plain read-modify-write of a row cannot lose a
// sibling update from the same minibatch.
//
// Layout: lane l holds columns l, l+64, ..., l+64(C-1) of every gathered row
// in VGPRs (C = ceil(D/64) rounded up to a compiled size), loaded through
// range-checked buffer descriptors. Ids, multiplicities and slot codes stay
// in registers, one per lane (Minibatch), and are read back with v_readlane:
// a wavefront that handles one minibatch after the other spends its time on
// the chain of LDS round trips and branches between the row accesses (at
// D = 64 and one sentence in flight, 9 of 22 thousand cycles per minibatch
// went into staging and slot bookkeeping through LDS), so the core holds
// neither LDS staging nor per-element loops.
//
// The logits of 8 input rows x 8 output columns (a tile) come from one
// transposing reduction over per-lane partial products (reduce_tile, which
// leaves out the rows and columns a tile lacks). It puts slot (i, k) in lane
// 8 i + k, where the error is evaluated. Four consecutive lanes are then
// four columns of one input row, which is what v_mfma_f32_4x4x1 (16 blocks)
// broadcasts to all its blocks with CBSZ = 4, so both gradient products run
// on the matrix cores straight from the rows in registers: dO takes the
// errors as they lie, dA takes them transposed by one ds_bpermute. One
// instruction does 4 x 64 multiply-adds in 8 cycles without a v_readlane;
// the VALU form took 16 cycles for the multiply-adds and 16 for the four
// v_readlane (each rounds like v_fma_f32).
//
// Update path (live matrices, RowTiers): rows with id < hot_rows receive
// fp32 atomic adds (frequent words, whose concurrent updates would otherwise
// overwrite each other), all other rows a store of (value read + update)
// written through to device scope, the Hogwild write the paper's threads
// perform (Sec. 1.1). Rows below
// split_rows (the head of the Zipf law, written by nearly every concurrent
// wavefront) are spread over kSplitParts partial rows: a wavefront adds its
// update atomically to the partial row of its group (blockIdx mod
// kSplitParts, i.e. its XCD under round-robin dispatch), and reads return
// the matrix row plus every partial row, so atomics to one address come from
// one XCD only and nothing is hidden from a reader. Snapshot batches add
// their updates with fp64 atomics into a delta buffer instead, or write them
// to staging rows for a sorted reduction.
//
// Where rows are read and where updates go is the business of the caller's Io
// (EpochIo, with the pending input-row updates, in the epoch kernel; StepIo
// and StageIo in the snapshot batches).
//
// Output columns go in blocks of KB: 6 where the K + 1 columns fit (the
// paper's K = 5), all of them in one block, else 8 (4 for rows of more than
// 384 columns) with the update of the input rows accumulated over the blocks.
#pragma once

#include "device_common.h"
#include "w2v.h"

namespace w2v {

constexpr int kMaxInputs = 32;   // input words per minibatch (2 * max window)
constexpr int kMaxOutputs = 65;  // target + up to 64 negatives
constexpr int kSplitParts = W2V_SPLIT_PARTS;

// One minibatch's distinct ids and multiplicities, one per lane.
struct Minibatch {
  int n;         // distinct input rows: lanes i < n hold them
  int n_out;     // output columns: 0 is the target, k >= 1 in lane k - 1
  int target;
  int in_id;
  int neg_id;
  float in_w;    // multiplicity of the lane's input row / negative; read
  float neg_w;   // only if `weighted`
  bool weighted; // some multiplicity may be above 1
};

// Whether two of the 64 lanes (kWide) or two lanes of any 16-lane row hold
// the same id: every pair of a row meets in one of eight rotations, and the
// pairs of two rows in the sixteen rotations of one of them.
template <bool kWide>
__device__ __forceinline__ bool has_repeat(int id) {
  uint32_t low = ~0u;
  auto meet = [&](int other) { low = min(low, (uint32_t)(id ^ other)); };
  meet(i_dpp<0x121>(id));
  meet(i_dpp<0x122>(id));
  meet(i_dpp<0x123>(id));
  meet(i_dpp<0x124>(id));
  meet(i_dpp<0x125>(id));
  meet(i_dpp<0x126>(id));
  meet(i_dpp<0x127>(id));
  meet(i_dpp<0x128>(id));
  if constexpr (kWide) {
    const int lane = threadIdx.x;
#pragma unroll
    for (int rows = 1; rows <= 2; ++rows) {
      const int x = __builtin_amdgcn_ds_bpermute(((lane + 16 * rows) & 63) * 4, id);
      meet(x);
      meet(i_dpp<0x121>(x));
      meet(i_dpp<0x122>(x));
      meet(i_dpp<0x123>(x));
      meet(i_dpp<0x124>(x));
      meet(i_dpp<0x125>(x));
      meet(i_dpp<0x126>(x));
      meet(i_dpp<0x127>(x));
      meet(i_dpp<0x128>(x));
      meet(i_dpp<0x129>(x));
      meet(i_dpp<0x12A>(x));
      meet(i_dpp<0x12B>(x));
      meet(i_dpp<0x12C>(x));
      meet(i_dpp<0x12D>(x));
      meet(i_dpp<0x12E>(x));
      meet(i_dpp<0x12F>(x));
    }
  }
  return __ballot(low == 0u) != 0ull;
}

// Moves the distinct ids of the lanes in `present` to lanes 0, 1, ... in
// order of first appearance, with their multiplicities; returns how many.
// The general path: repeated ids and gaps.
__device__ __forceinline__ int compact_distinct(uint64_t present, int lane, int& id,
                                                float& weight) {
  uint64_t firsts = 0ull;
  int mult = 0;
  for (uint64_t m = present; m != 0ull;) {
    const int l = __builtin_ctzll(m);
    const uint64_t eq =
        __ballot(id == __builtin_amdgcn_readlane(id, l)) & present;
    if (lane == l) mult = __popcll(eq);
    firsts |= 1ull << l;
    m &= ~eq;
  }
  // A lane that is no first goes to lane 63, which is then no destination.
  const int dst = ((firsts >> lane) & 1ull) != 0ull ? __popcll(firsts & lanes_below(lane))
                                                    : kWave - 1;
  id = __builtin_amdgcn_ds_permute(dst * 4, id);
  weight = (float)__builtin_amdgcn_ds_permute(dst * 4, mult);
  return __popcll(firsts);
}

// Stages a minibatch from the ids as formed: lane i of `in_present` holds
// input word `in_id`, lane k < K negative `neg_id`. Lanes without a word
// hold any id.
template <bool kWideIn>
__device__ __forceinline__ Minibatch stage_minibatch(int lane, int in_id,
                                                     uint64_t in_present, int target,
                                                     int neg_id, int K) {
  Minibatch mb;
  mb.target = target;
  mb.in_w = mb.neg_w = 1.f;
  mb.weighted = false;
  // Ids that no word has, all different, where there is no word.
  mb.in_id = ((in_present >> lane) & 1ull) != 0ull ? in_id : -1 - lane;
  mb.n = __popcll(in_present);
  const bool gaps = (in_present & (in_present + 1ull)) != 0ull;
  if (gaps || has_repeat<kWideIn>(mb.in_id)) {
    mb.n = compact_distinct(in_present, lane, mb.in_id, mb.in_w);
    mb.weighted = true;
  }
  const uint64_t drawn = K < kWave ? (1ull << K) - 1ull : ~0ull;
  mb.neg_id = lane < K ? neg_id : -1 - lane;
  const uint64_t masked = __ballot(mb.neg_id == target);
  mb.n_out = K + 1;
  bool rep;
  if (K <= 16)
    rep = has_repeat<false>(mb.neg_id);
  else
    rep = has_repeat<true>(mb.neg_id);
  if (masked != 0ull || rep) {
    mb.n_out = 1 + compact_distinct(drawn & ~masked, lane, mb.neg_id, mb.neg_w);
    mb.weighted = true;
  }
  return mb;
}

// Raw buffer descriptor of one matrix row of n_bytes: loads past the end
// return 0 and stores/atomics past it are dropped by the hardware range
// check, so a row of D floats needs no per-lane bounds test.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* row,
                                                          int n_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), (short)0,
                                           n_bytes, kBufferWord3);
}

// Row id of a matrix: ids and strides are below 2^31, so one 32 x 32 -> 64
// bit product.
template <class T>
__device__ __forceinline__ T* row_at(T* base, int id, int64_t ld) {
  return base + (uint64_t)(uint32_t)id * (uint32_t)ld;
}

// Loads columns lane + 64c, c < C, of one row (0 past D). D = 0 gives zeros
// without touching memory, whatever the id.
template <int C, bool kLive>
__device__ __forceinline__ void load_row(const float* base, int id, int64_t ld, int D,
                                         int lane, float (&r)[C]) {
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(row_at(base, id, ld), D * 4);
#pragma unroll
  for (int c = 0; c < C; ++c)
    r[c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
        rs, (lane + kWave * c) * 4, 0, kLive ? kCoherentLoad : 0));
}

// Applies update g to the column sets c0, c0 + 1, ... of one row whose
// values as read are `old`: fp32 atomic adds, or a plain store of old + g.
template <int N>
__device__ __forceinline__ void update_row(float* row, int D, int lane, bool atomic,
                                           const float (&old)[N], const float (&g)[N],
                                           int c0 = 0) {
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(row, D * 4);
  if (atomic) {
#pragma unroll
    for (int c = 0; c < N; ++c)
      __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(
          g[c], rs, (lane + kWave * (c0 + c)) * 4, 0, 0);
  } else {
#pragma unroll
    for (int c = 0; c < N; ++c)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(old[c] + g[c]), rs,
                                            (lane + kWave * (c0 + c)) * 4, 0,
                                            kCoherentStore);
  }
}

// Row access of a minibatch's live rows by tier: rows id < split_rows of
// matrix m (0: input, 1: output) have partial rows part[((m split_rows + id)
// kSplitParts + g) ld], g < kSplitParts, that every read adds and that take
// the updates (atomically, in the partial row of this wavefront's group);
// rows id < hot_rows take fp32 atomic adds; other rows a store of old + g.
template <int C>
struct RowTiers {
  float* part;
  int split_rows;
  int hot_rows;
  int64_t ld;
  int D;
  int lane;

  __device__ __forceinline__ float* part_base(int m, int id) const {
    return part + (int64_t)(m * split_rows + id) * kSplitParts * ld;
  }
  // Partial rows in flight at a time (each is a memory round trip; more take
  // the registers of the rows).
  static constexpr int kSplitLoad = C > 6 ? 1 : 4;
  static_assert(kSplitParts % kSplitLoad == 0, "whole batches of partial rows");
  // Sum of the partial rows of a split row.
  __device__ __forceinline__ void split_sum(int m, int id, float (&r)[C]) const {
    float* pb = part_base(m, id);
#pragma unroll
    for (int c = 0; c < C; ++c) r[c] = 0.f;
#pragma unroll 1
    for (int g = 0; g < kSplitParts; g += kSplitLoad) {
      float t[kSplitLoad][C];
#pragma unroll
      for (int u = 0; u < kSplitLoad; ++u) load_row<C, true>(pb, g + u, ld, D, lane, t[u]);
#pragma unroll
      for (int u = 0; u < kSplitLoad; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) r[c] += t[u][c];
    }
  }
  // Adds the partial rows of a split row to its value as read. Rows of more
  // than 384 columns take them one by one without a sum of their own: C more
  // registers cost them 10% (grouped epoch, D = 640, G = 2, 4e6 tokens: 44.0
  // ms with the sum, 39.1 without; D = 300, G = 4: 23.4 ms with, 24.0 without).
  __device__ __forceinline__ void add_split(int m, int id, float (&r)[C]) const {
    if (id >= split_rows) return;
    if constexpr (C > 6) {
      float* pb = part_base(m, id);
#pragma unroll 1
      for (int g = 0; g < kSplitParts; ++g) {
        float t[C];
        load_row<C, true>(pb, g, ld, D, lane, t);
#pragma unroll
        for (int c = 0; c < C; ++c) r[c] += t[c];
      }
    } else {
      float t[C];
      split_sum(m, id, t);
#pragma unroll
      for (int c = 0; c < C; ++c) r[c] += t[c];
    }
  }
  // Where the updates of row id go.
  __device__ __forceinline__ float* target(int m, float* W, int id) const {
    return id < split_rows ? row_at(part_base(m, id), (int)(blockIdx.x % kSplitParts), ld)
                           : row_at(W, id, ld);
  }
  // Adds g to row id atomically whatever its tier (pending updates).
  __device__ __forceinline__ void add(int m, float* W, int id,
                                      const float (&g)[C]) const {
    update_row(target(m, W, id), D, lane, true, g, g);
  }
  template <int N>
  __device__ __forceinline__ void update(int m, float* W, int id, const float (&old)[N],
                                         const float (&g)[N], int c0) const {
    update_row(target(m, W, id), D, lane, id < hot_rows || id < split_rows, old, g, c0);
  }
};

using v4f = __attribute__((ext_vector_type(4))) float;

// d + e (x) r: adds to four rows (d[m], this lane's column) the products of
// row value r and the errors that lanes 4 kBlock + m hold.
template <int kBlock>
__device__ __forceinline__ v4f outer4(float e, float r, v4f d) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(e, r, d, 4, kBlock, 0);
}

// Logits of a tile of NI x KB partial products (value(i, k), one per lane
// and column set): on return lane 8 i + k holds the sum of value(i, k) over
// the wavefront. The reduction halves the values at each step (rows i, then
// columns k); a missing partner is left out, and tiles of up to 4 and 2 rows
// reduce fewer values and move to their lanes at the end.
template <int NI, int KB, class F>
__device__ __forceinline__ float reduce_tile(const F& value, int lane) {
  static_assert(NI >= 1 && NI <= 8 && KB >= 1 && KB <= 8, "at most 8 x 8 slots");
  constexpr int kRows = NI > 4 ? 8 : NI > 2 ? 4 : NI > 1 ? 2 : 1;
  float w[KB];
  // Rows, one column after the other (few values live at once).
  const bool b3 = (lane & 8) != 0;
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    float r[kRows > 1 ? kRows / 2 : 1];
#pragma unroll
    for (int i = 0; i < (kRows > 1 ? kRows / 2 : 1); ++i)
      r[i] = i + kRows / 2 < NI && kRows > 1
                 ? f_swap_sum32(value(i, k), value(i + kRows / 2, k))
                 : f_sum32(value(i, k));
    if constexpr (kRows == 8) {
      w[k] = f_pair_dpp<kDppRowMirror>(f_swap_sum16(r[0], r[2]), f_swap_sum16(r[1], r[3]), b3);
    } else if constexpr (kRows == 4) {
      w[k] = f_swap_sum16(r[0], r[1]);
    } else {
      w[k] = r[0];
    }
  }
  // Columns: three halvings, by the lane bits that the rows left.
  auto halve = [&](auto step, int bit) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j >= bit || j >= KB) continue;
      w[j] = step(w[j], j + bit < KB ? w[j + bit < KB ? j + bit : 0] : 0.f, j + bit < KB);
    }
  };
  auto by_mirror = [&](float a, float b, bool two) {
    return two ? f_pair_dpp<kDppRowMirror>(a, b, (lane & 8) != 0)
               : a + f_dpp<kDppRowMirror>(a);
  };
  auto by_half = [&](float a, float b, bool two) {
    return two ? f_pair_dpp<kDppRowHalfMirror>(a, b, (lane & 4) != 0)
               : a + f_dpp<kDppRowHalfMirror>(a);
  };
  auto by_2 = [&](float a, float b, bool two) {
    return two ? f_pair_dpp<kDppXor2>(a, b, (lane & 2) != 0) : a + f_dpp<kDppXor2>(a);
  };
  auto by_1 = [&](float a, float b, bool two) {
    return two ? f_pair_dpp<kDppXor1>(a, b, (lane & 1) != 0) : a + f_dpp<kDppXor1>(a);
  };
  auto by_16 = [&](float a, float b, bool two) {
    return two ? f_swap_sum16(a, b) : f_sum16(a);
  };
  if constexpr (kRows == 8) {
    halve(by_half, 4);
    halve(by_2, 2);
    halve(by_1, 1);
    return w[0];
  } else if constexpr (kRows == 4) {
    halve(by_mirror, 4);
    halve(by_half, 2);
    halve(by_2, 1);
    w[0] += f_dpp<kDppXor1>(w[0]);
    return __int_as_float(
        __builtin_amdgcn_ds_bpermute(((2 * lane) & 63) * 4, __float_as_int(w[0])));
  } else {
    halve(by_16, 4);
    halve(by_mirror, 2);
    halve(by_half, 1);
    w[0] += f_dpp<kDppXor2>(w[0]);
    w[0] += f_dpp<kDppXor1>(w[0]);
    return __int_as_float(
        __builtin_amdgcn_ds_bpermute(((4 * lane) & 63) * 4, __float_as_int(w[0])));
  }
}

// a / d for a in [0, 1] and d in [1, 4]: the hardware's reciprocal, and the
// quotient corrected by its residual (sigma of logits in [-1, 1]: 0.36 ulp off
// in the mean; 0.39 as an IEEE divide 1 / (1 + e^-x), 0.41 as a corrected
// reciprocal times a).
__device__ __forceinline__ float quotient_near1(float a, float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  const float q = a * r;
  return fmaf(fmaf(-d, q, a), r, q);
}

// log(1 + t) for t in [0, 1], within about an ulp: 2 atanh(s), s = t / (2 +
// t) <= 1/3, by its series up to s^15 (the next term is below 2e-9 of the
// sum). What the quotient and the sum 2 + t round away is added beside the
// series, so that the last addition is the one that rounds (losses of logits
// in [-1, 1]: 0.33 ulp off in the mean, as with the library's logarithm; 0.48
// with a reciprocal times t).
__device__ __forceinline__ float log1p_unit(float t) {
#pragma clang fp contract(off)  // `rest` belongs to s as rounded
  const float d = 2.f + t;
  const float r = __builtin_amdgcn_rcpf(d);
  const float s = t * r;
  const float rest = fmaf(-(t - (d - 2.f)), s, fmaf(-d, s, t)) * r;  // of t / (2 + t)
  const float q = s * s;
  float p = 1.f / 15.f;
  p = fmaf(p, q, 1.f / 13.f);
  p = fmaf(p, q, 1.f / 11.f);
  p = fmaf(p, q, 1.f / 9.f);
  p = fmaf(p, q, 1.f / 7.f);
  p = fmaf(p, q, 1.f / 5.f);
  p = fmaf(p, q, 1.f / 3.f);
  return 2.f * (s + fmaf(s * q, p, rest));
}

// Error and loss of one slot of a minibatch of one target: column 0 is the
// target (label 1), the others negatives (label 0); both scaled by the row
// and column multiplicities (wgt).
__device__ __forceinline__ float target_error(bool is_target, float x, float wgt,
                                              float alpha, bool want_loss,
                                              float& loss_part) {
  // label - sigma(x) is sigma(-x) for the target and -sigma(x) for a
  // negative; evaluating sigma(z) directly avoids cancelling against 1. With
  // t = e^-|z| it is 1 / (1 + t), or t / (1 + t) where z < 0, and the loss
  // is max(z, 0) + log(1 + t): one exponential, no divide and no library
  // logarithm (a wavefront on its own spent a quarter of a minibatch here).
  const float z = is_target ? -x : x;
  const float t = __expf(-fabsf(z));
  const float sz = quotient_near1(z < 0.f ? t : 1.f, 1.f + t);
  if (want_loss) loss_part += wgt * (fmaxf(z, 0.f) + log1p_unit(t));
  return wgt * alpha * (is_target ? sz : -sz);
}

// The fused minibatch. C: columns per lane; NMAX: input rows (10, 16 or 32);
// kMulti: several output blocks of KB columns, else one of 6 (K <= 5). Io
// says where rows are read and where updates go:
//   load_in(id, ok, row), load_out(id, ok, row): issue the loads of a row
//     (zeros where !ok, without touching memory);
//   settle_in(mb, a), settle_out(mb, k0, o): add to rows as read what is
//     kept elsewhere (partial rows, pending updates);
//   put_out(k, id, row, g, c0): apply update g to output column k, whose
//     values were read as `row`; the arrays hold the columns lane + 64 c of
//     the column sets from c0 on;
//   before_inputs(mb): called once before the input rows are written, for
//     what has to be done first (pending slots that change hands);
//   fetch_kept(i, kept, c0): issue the reads of what put_in needs for row i;
//   put_in(i, id, row, g, kept, c0): apply update g to input row i.
// load() issues every load; run() does the rest, so that the caller can
// work on the next minibatch's ids in between.
template <int C, int NMAX, bool kMulti>
struct Core {
  static constexpr int KB = !kMulti ? 6 : C >= 8 ? 4 : 8;
  static constexpr int kTiles = (NMAX + 7) / 8;
  static constexpr int kGroups = (NMAX + 3) / 4;
  // With several blocks the next one's rows are loaded while this one is
  // computed and written; they are other rows (columns are distinct), so
  // every row is still read before the minibatch writes it.
  static constexpr bool kPrefetch = kMulti && (C <= 4 || C >= 6);
  // Column sets whose updates are formed at once: rows of more than 384
  // columns go in two halves, which keeps the 4 x C accumulators of four
  // rows from taking the registers of the rows.
  static constexpr int CH = C > 6 ? C / 2 : C;
  static_assert(C % CH == 0, "whole halves");

  float a[NMAX][C];
  float o[KB][C];

  template <class Io>
  __device__ __forceinline__ void load_block(Io& io, const Minibatch& mb, int k0,
                                             float (&r)[KB][C]) {
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int id = k0 + k == 0 ? mb.target
                                 : __builtin_amdgcn_readlane(mb.neg_id, (k0 + k - 1) & 63);
      io.load_out(id, k0 + k < mb.n_out, r[k]);
    }
  }

  // Rows are loaded in pairs: tiles go by an even number of rows.
  template <class Io>
  __device__ __forceinline__ void load(Io& io, const Minibatch& mb) {
#pragma unroll
    for (int i = 0; i < NMAX; ++i) {
      if ((i & ~1) < mb.n)
        io.load_in(__builtin_amdgcn_readlane(mb.in_id, i), i < mb.n, a[i]);
    }
    load_block(io, mb, 0, o);
  }

  // Logits of tile T from its first NI rows.
  template <int T, int NI>
  __device__ __forceinline__ float tile(int lane) const {
    return reduce_tile<NI, KB>(
        [&](int i, int k) {
          float acc = a[8 * T + i][0] * o[k][0];
#pragma unroll
          for (int c = 1; c < C; ++c) acc = fmaf(a[8 * T + i][c], o[k][c], acc);
          return acc;
        },
        lane);
  }

  // Logits of tile T with ni rows: as few rows as hold them.
  template <int T>
  __device__ __forceinline__ float logits(int ni, int lane) const {
    constexpr int kRows = NMAX - 8 * T < 8 ? NMAX - 8 * T : 8;
    if constexpr (kRows <= 2) {
      return tile<T, 2>(lane);
    } else {
      if (ni <= 2) return tile<T, 2>(lane);
      if (ni <= 4) return tile<T, 4>(lane);
      if (ni <= 6) return tile<T, 6>(lane);
      return tile<T, 8>(lane);
    }
  }

  // Errors of the block at column k0: e[t] in lane 8 i + k, et[t] in lane
  // 8 k + i (0 for slots that the minibatch has not).
  template <int T>
  __device__ __forceinline__ void errors_of(const Minibatch& mb, int lane, int k0,
                                            float alpha, bool want_loss,
                                            float& loss_part, float (&e)[kTiles],
                                            float (&et)[kTiles]) const {
    if constexpr (T < kTiles) {
      const int li = lane >> 3, lk = lane & 7;
      const int ni = mb.n - 8 * T;
      e[T] = 0.f;
      et[T] = 0.f;
      if (ni > 0) {
        const float x = logits<T>(ni, lane);
        const bool first = k0 + lk == 0;
        const bool valid = li < ni && lk < KB && k0 + lk < mb.n_out;
        float wgt = 1.f;
        if (mb.weighted) {
          wgt = lane_of(mb.in_w, 8 * T + li);
          const float wk = lane_of(mb.neg_w, k0 + lk - 1);
          if (!first) wgt *= wk;
        }
        if (valid) e[T] = target_error(first, x, wgt, alpha, want_loss, loss_part);
        et[T] = lane_of(e[T], lk * 8 + li);
        errors_of<T + 1>(mb, lane, k0, alpha, want_loss, loss_part, e, et);
      }
    }
  }

  template <class Io>
  __device__ __forceinline__ void run(Io& io, int lane, const Minibatch& mb,
                                      float alpha, bool want_loss, float& loss_part) {
    const int n = mb.n;
    io.settle_in(mb, a);
    v4f ga[kMulti ? kGroups : 1][C];
    if constexpr (kMulti) {
#pragma unroll
      for (int g = 0; g < kGroups; ++g)
#pragma unroll
        for (int c = 0; c < C; ++c) ga[g][c] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    float next[kPrefetch ? KB : 1][C];
#pragma unroll 1
    for (int k0 = 0; k0 < (kMulti ? mb.n_out : 1); k0 += KB) {
      if constexpr (kPrefetch) {
        if (k0 + KB < mb.n_out) load_block(io, mb, k0 + KB, next);
      }
      io.settle_out(mb, k0, o);
      // Logits and errors, eight input rows at a time: lane 8 i + k.
      float e[kTiles], et[kTiles];
      errors_of<0>(mb, lane, k0, alpha, want_loss, loss_part, e, et);
      // dO = E^T A, four columns at a time.
#pragma unroll
      for (int g = 0; g < (KB + 3) / 4; ++g) {
        if (k0 + 4 * g < mb.n_out) {
#pragma unroll
          for (int c0 = 0; c0 < C; c0 += CH) {
            v4f d[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) d[c] = v4f{0.f, 0.f, 0.f, 0.f};
            outputs_of<0>(g, n, e, c0, d);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              const int k = 4 * g + m;
              if (k < KB && k0 + k < mb.n_out) {
                float old[CH], gk[CH];
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                  old[c] = o[k < KB ? k : 0][c0 + c];
                  gk[c] = d[c][m];
                }
                const int id = k0 + k == 0
                                   ? mb.target
                                   : __builtin_amdgcn_readlane(mb.neg_id, (k0 + k - 1) & 63);
                io.put_out(k0 + k, id, old, gk, c0);
              }
            }
          }
        }
      }
      if constexpr (!kMulti) io.before_inputs(mb);
      // dA = E O, four rows at a time (summed over the blocks).
#pragma unroll
      for (int g = 0; g < kGroups; ++g) {
        if (4 * g < n) {
          if constexpr (kMulti) {
            inputs_of(g, et, 0, ga[g]);
          } else {
#pragma unroll
            for (int c0 = 0; c0 < C; c0 += CH) {
              v4f d[CH];
#pragma unroll
              for (int c = 0; c < CH; ++c) d[c] = v4f{0.f, 0.f, 0.f, 0.f};
              inputs_of(g, et, c0, d);
              put_inputs(io, mb, g, c0, d);
            }
          }
        }
      }
      if constexpr (kPrefetch) {
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
          for (int c = 0; c < C; ++c) o[k][c] = next[k][c];
      } else if constexpr (kMulti) {
        if (k0 + KB < mb.n_out) load_block(io, mb, k0 + KB, o);
      }
    }
    if constexpr (kMulti) {
      io.before_inputs(mb);
#pragma unroll
      for (int g = 0; g < kGroups; ++g)
        if (4 * g < n) {
#pragma unroll
          for (int c0 = 0; c0 < C; c0 += CH) {
            v4f d[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) d[c] = ga[g][c0 + c];
            put_inputs(io, mb, g, c0, d);
          }
        }
    }
  }

  // The errors alone: io.put_errors(k0, T, e) gets those of the block at
  // column k0 and input rows 8 T .. 8 T + 7, lane 8 i + k holding slot (i, k).
  template <class Io>
  __device__ __forceinline__ void run_errors(Io& io, int lane, const Minibatch& mb,
                                             float alpha) {
#pragma unroll 1
    for (int k0 = 0; k0 < (kMulti ? mb.n_out : 1); k0 += KB) {
      float e[kTiles], et[kTiles], no_loss = 0.f;
      errors_of<0>(mb, lane, k0, alpha, false, no_loss, e, et);
#pragma unroll
      for (int t = 0; t < kTiles; ++t)
        if (8 * t < mb.n) io.put_errors(mb, k0, t, k0 + KB < mb.n_out ? KB : mb.n_out - k0,
                                        e[t]);
      if constexpr (kMulti) {
        if (k0 + KB < mb.n_out) load_block(io, mb, k0 + KB, o);
      }
    }
  }

  static __device__ __forceinline__ float lane_of(float x, int l) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute((l & 63) * 4, __float_as_int(x)));
  }

  // d += the share of input rows I, I + 1, ... in output columns 4 g .. 4 g + 3.
  template <int I>
  __device__ __forceinline__ void outputs_of(int g, int n, const float (&e)[kTiles],
                                             int c0, v4f (&d)[CH]) const {
    if constexpr (I < NMAX) {
      if (I < n) {
#pragma unroll
        for (int i = I; i < I + 2; ++i) {
#pragma unroll
          for (int c = 0; c < CH; ++c)
            d[c] = outer4_at((i % 8) * 2 + g, e[i / 8], a[i][c0 + c], d[c]);
        }
        outputs_of<I + 2>(g, n, e, c0, d);
      }
    }
  }

  // d += the share of the block's output columns in input rows 4 g .. 4 g + 3.
  template <int N>
  __device__ __forceinline__ void inputs_of(int g, const float (&et)[kTiles], int c0,
                                            v4f (&d)[N]) const {
#pragma unroll
    for (int k = 0; k < KB; ++k)
#pragma unroll
      for (int c = 0; c < N; ++c)
        d[c] = outer4_at(2 * k + (g & 1), et[g / 2], o[k][c0 + c], d[c]);
  }

  template <class Io>
  __device__ __forceinline__ void put_inputs(Io& io, const Minibatch& mb, int g, int c0,
                                             const v4f (&d)[CH]) const {
    float kept[4][CH];
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if (4 * g + m < NMAX && 4 * g + m < mb.n) io.fetch_kept(4 * g + m, kept[m], c0);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int i = 4 * g + m;
      if (i < NMAX && i < mb.n) {
        float old[CH], gi[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          old[c] = a[i < NMAX ? i : 0][c0 + c];
          gi[c] = d[c][m];
        }
        io.put_in(i, __builtin_amdgcn_readlane(mb.in_id, i), old, gi, kept[m], c0);
      }
    }
  }

  // outer4 of a block number that is constant once the loops are unrolled.
  static __device__ __forceinline__ v4f outer4_at(int block, float e, float r, v4f d) {
    switch (block) {
      case 0: return outer4<0>(e, r, d);
      case 1: return outer4<1>(e, r, d);
      case 2: return outer4<2>(e, r, d);
      case 3: return outer4<3>(e, r, d);
      case 4: return outer4<4>(e, r, d);
      case 5: return outer4<5>(e, r, d);
      case 6: return outer4<6>(e, r, d);
      case 7: return outer4<7>(e, r, d);
      case 8: return outer4<8>(e, r, d);
      case 9: return outer4<9>(e, r, d);
      case 10: return outer4<10>(e, r, d);
      case 11: return outer4<11>(e, r, d);
      case 12: return outer4<12>(e, r, d);
      case 13: return outer4<13>(e, r, d);
      case 14: return outer4<14>(e, r, d);
      default: return outer4<15>(e, r, d);
    }
  }
};

}  // namespace w2v
