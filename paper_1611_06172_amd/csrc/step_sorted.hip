// Sorted snapshot batch on gfx950: the step of the atomic snapshot batch
// (step_kernels.hip) with every row's updates summed in one fixed order, so
// that a batch gives the same bits on every run and no atomics are needed.
//
//   1. k_stage: one wavefront per minibatch computes its updates from the
//      unchanged matrices (sgns_core.h) and writes them to staging rows
//      (StageIo) instead of applying them. Each staging row gets a sort
//      key naming the matrix row it updates: id for M_in, V + id for M_out,
//      2V for an unused staging row;
//   2. one stable radix sort of (key, staging index) pairs (radix_sort.hip),
//      so each matrix row's updates form one run, in minibatch order;
//   3. k_reduce: one wavefront per chunk of 64 sorted entries sums each run
//      it holds in fp64, in sorted order, loading kBatch staging rows (and
//      the matrix rows of the runs that open among them) at once. A run
//      inside the chunk is applied (M = fp32(M + sum) where the sum is not
//      0); the part of a run that crosses the chunk's first or last border
//      goes to the chunk's head or tail piece;
//   4. k_reduce_spans: a run's head pieces within one span of kSpan chunks
//      are added, in chunk order, into the first of them;
//   5. k_reduce_cross: the chunk in which a crossing run starts finds the
//      run's last chunk (galloping search over chunk borders), adds its
//      tail piece and the run's summed piece of every span it goes through,
//      in span order, and applies the total.
// Traffic per batch: the gathered rows, one staging row written and read
// per update, the keys, and one read and write per touched row.
//
// Pulled batches (w2v_step_batch, whose workspace does not hold the staging
// rows of a large batch): k_stage keeps only the errors E (4 N (K + 1) bytes
// a minibatch), and k_reduce forms an entry's update again from them, E O
// from the K + 1 output rows or E^T A from the N input rows of its
// minibatch, in the same order of fused multiply-adds, so to the same bits.
// The input rows are reduced first, from the unchanged M_out, into rows kept
// aside (next_in); then the output columns, from the unchanged M_in, into
// M_out; then k_reduce_copy moves the new input rows into M_in. The partner
// rows (2 N (K + 1) a minibatch) come from L2 and the memory-side cache:
// 7.9e6 rows of 1.2 KB take 0.74 ms at the kernel-test configuration, where
// the 3.8e7 fp64 atomic requests of the delta buffers took 2.34 ms. (Under
// uniform ids most of the rows come from memory: the whole batch takes 1.80
// ms, 2.10 with atomics.)
#include <hip/hip_runtime.h>

#include "batch_ids.h"
#include "kernel_args.h"
#include "sgns_core.h"

namespace w2v {

constexpr int kChunk = 64;   // sorted entries per wavefront (one per lane)
constexpr int kBatch = 8;    // rows loaded before they are added

// Rows of the unchanged matrices (Core's Io); the update of distinct input i
// goes to row i of `in`, that of output column k to row k of `out`.
template <int C>
struct StageIo {
  const SortedStepArgs& a;
  float* in;
  float* out;
  float* errors;  // [N][K + 1] of this minibatch (pulled batches)
  int lane;

  // Errors of output columns k0 .. k0 + cols - 1 and input rows from 8 t on.
  __device__ __forceinline__ void put_errors(const Minibatch& mb, int k0, int t, int cols,
                                             float e) const {
    const int i = 8 * t + (lane >> 3), k = lane & 7;
    if (i < mb.n && k < cols) errors[i * (a.K + 1) + k0 + k] = e;
  }

  __device__ __forceinline__ void load_in(int id, bool ok, float (&r)[C]) const {
    load_row<C, false>(a.M_in, id, a.ld, ok ? a.D : 0, lane, r);
  }
  __device__ __forceinline__ void load_out(int id, bool ok, float (&r)[C]) const {
    load_row<C, false>(a.M_out, id, a.ld, ok ? a.D : 0, lane, r);
  }
  template <int N>
  __device__ __forceinline__ void settle_in(const Minibatch&, float (&)[N][C]) const {}
  template <int N>
  __device__ __forceinline__ void settle_out(const Minibatch&, int, float (&)[N][C]) const {}
  __device__ __forceinline__ void before_inputs(const Minibatch&) const {}
  template <int N>
  __device__ __forceinline__ void fetch_kept(int, float (&)[N], int) const {}
  template <int N>
  __device__ __forceinline__ void put(float* row, const float (&g)[N], int c0) const {
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int col = lane + kWave * (c0 + c);
      if (col < a.D) row[col] = g[c];
    }
  }
  template <int N>
  __device__ __forceinline__ void put_out(int k, int, const float (&)[N],
                                          const float (&g)[N], int c0) const {
    put(out + k * a.ld, g, c0);
  }
  template <int N>
  __device__ __forceinline__ void put_in(int i, int, const float (&)[N],
                                         const float (&g)[N], const float (&)[N],
                                         int c0) const {
    put(in + i * a.ld, g, c0);
  }
};

// Waves per SIMD the registers of k_stage must allow (1: no bound). It is
// bound by the rows in flight, and without a bound the compiler puts the
// accumulators of the matrix instructions into registers of their own (AGPRs)
// beside those of the rows, which costs the shapes below a wave or more
// (k_stage<5, 10, true, false>: 217 + 88 registers and one wave, with the
// bound 219 and two). Sorted batches of V = 100,000, Zipf(1.0) ids, us
// without / with the bound: (65536, N 10, K 15, D 300) 1797 / 1547, (65536,
// 10, 25, 200) 1990 / 1612, (65536, 32, 15, 128) 1932 / 1433, (65536, 10, 5,
// 384) 1124 / 1104. Where no wave is lost the bound costs 1 to 2% ((65536,
// 10, 5, 300) 982 / 996), and pulled batches have no such accumulators.
// k_step, which the memory side's atomics bound, gained nothing from it.
constexpr int stage_waves_per_eu(int C, int nmax, bool multi, bool pull) {
  if (pull) return 1;
  if (nmax == 10 && multi) return C == 1 ? 4 : C == 2 ? 3 : C <= 5 ? 2 : 1;
  if (nmax == 10) return C == 2 ? 5 : C == 4 ? 4 : C == 6 ? 3 : 1;
  if (nmax == 16 && multi) return C == 1 ? 4 : C == 2 ? 3 : C <= 4 ? 2 : 1;
  if (nmax == 16) return C == 3 ? 4 : C == 4 ? 3 : 1;
  return multi ? (C == 1 ? 3 : 2) : (C == 1 ? 5 : 1);
}

template <int C, int NMAX, bool kMulti, bool kPull>
__global__ __launch_bounds__(kWave) __attribute__((
    amdgpu_waves_per_eu(stage_waves_per_eu(C, NMAX, kMulti, kPull)))) void k_stage(
    SortedStepArgs a) {
  const int lane = threadIdx.x;
  const int n_slots_out = a.K + 1;
  int64_t applied = 0, sum_n = 0, rejected = 0, rows = 0;
  for (int64_t b = blockIdx.x; b < a.B; b += gridDim.x) {
    BatchIds ids;
    const bool bad = read_batch_ids(a, b, lane, ids);
    const int n = __popcll(ids.present);
    const bool use = !bad && n > 0;
    const Minibatch mb = stage_minibatch<(NMAX > 16)>(lane, ids.ctx, ids.present,
                                                      ids.target, ids.neg, a.K);
    const int64_t in0 = b * a.N, out0 = b * n_slots_out;
    StageIo<C> io{a, a.stage_in + in0 * a.ld, a.stage_out + out0 * a.ld,
                  a.errors + in0 * n_slots_out, lane};
    Core<C, NMAX, kMulti> core;
    if (use) core.load(io, mb);
    // Keys of this minibatch's staging rows (2V where nothing is staged).
    const uint32_t unused = 2u * (uint32_t)a.V;
    if (lane < a.N) {
      a.key_in[in0 + lane] = (use && lane < mb.n) ? (uint32_t)mb.in_id : unused;
      a.val_in[in0 + lane] = (int32_t)(in0 + lane);
    }
    if (lane == 0) {
      a.key_out[out0] = use ? (uint32_t)a.V + (uint32_t)mb.target : unused;
      a.val_out[out0] = (int32_t)(a.out_base + out0);
    }
    if (lane < a.K) {
      a.key_out[out0 + 1 + lane] = (use && lane + 1 < mb.n_out)
                                       ? (uint32_t)a.V + (uint32_t)mb.neg_id
                                       : unused;
      a.val_out[out0 + 1 + lane] = (int32_t)(a.out_base + out0 + 1 + lane);
    }
    if (bad) {
      ++rejected;
    } else if (use) {
      ++applied;
      sum_n += n;
      rows += mb.n + mb.n_out;
      const float alpha = a.alpha != nullptr ? a.alpha[b] : a.alpha_scalar;
      float no_loss = 0.f;
      if constexpr (kPull)
        core.run_errors(io, lane, mb, alpha);
      else
        core.run(io, lane, mb, alpha, false, no_loss);
    }
  }
  if (lane == 0) report_bad_ids(a.status, rejected);
  if (a.stats != nullptr && lane == 0) {
    atomicAdd((unsigned long long*)&a.stats[0], (unsigned long long)applied);
    atomicAdd((unsigned long long*)&a.stats[1], (unsigned long long)sum_n);
    atomicAdd((unsigned long long*)&a.stats[3], (unsigned long long)rejected);
    atomicAdd((unsigned long long*)&a.stats[4], (unsigned long long)rows);
  }
}

// The sorted updates of both matrices: n entries (key, staging index),
// staging rows of stride ld, pieces[(2 chunk + h) ld] (h = 0 head, 1 tail).
struct ReduceArgs {
  const uint32_t* key;
  const int32_t* val;
  int64_t n;
  const float* stage;
  float* M_in;
  float* M_out;
  double* pieces;          // [2 n_chunks][pstride], pstride >= 64 C
  int32_t V, D;
  int64_t ld, pstride;
  uint32_t key_lo, key_hi; // pulled batches: k_reduce handles [key_lo, key_hi)
  float* W_in;             // where new M_in rows go: M_in, or (pulled) next_in
  // pulled batches: the errors and ids of the minibatches
  const float* errors;     // [B][N][K + 1]
  const uint32_t* ids_in;  // [B][N], [B][K + 1]: the sort keys as staged
  const uint32_t* ids_out;
  int32_t N, K;
  int32_t out_base;        // entries from here on are output columns
};

// Where the new values of a sort key's row go (keys < 2V).
__device__ __forceinline__ float* key_row_out(const ReduceArgs& r, uint32_t key) {
  return key < (uint32_t)r.V ? r.W_in + (int64_t)key * r.ld
                             : r.M_out + (int64_t)(key - (uint32_t)r.V) * r.ld;
}

// Matrix row a sort key names (keys < 2V).
__device__ __forceinline__ float* key_row(const ReduceArgs& r, uint32_t key) {
  return key < (uint32_t)r.V ? r.M_in + (int64_t)key * r.ld
                             : r.M_out + (int64_t)(key - (uint32_t)r.V) * r.ld;
}

// The row of `key`, whose values were m, becomes fp32(m + sum) where the sum
// is not 0. A pulled batch writes the rows of M_in elsewhere, and whole.
template <int C, bool kPull>
__device__ __forceinline__ void store_sum(const ReduceArgs& r, uint32_t key, int lane,
                                          const float (&m)[C], const double (&sum)[C]) {
  float* row = kPull ? key_row_out(r, key) : key_row(r, key);
  const bool in_place = !kPull || r.W_in == r.M_in;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int col = lane + kWave * c;
    if (col < r.D && (sum[c] != 0.0 || !in_place))
      row[col] = sum[c] != 0.0 ? (float)((double)m[c] + sum[c]) : m[c];
  }
}

template <int C>
__device__ __forceinline__ void apply_sum(const ReduceArgs& r, uint32_t key,
                                          int lane, const double (&sum)[C]) {
  float m[C];
  load_row<C, false>(key_row(r, key), 0, r.ld, r.D, lane, m);
  store_sum<C, true>(r, key, lane, m, sum);
}

// Piece rows hold all 64 C columns (zero past D), so they are written and
// read without per-column tests.
template <int C>
__device__ __forceinline__ void put_piece(const ReduceArgs& r, int64_t chunk,
                                          int h, int lane,
                                          const double (&sum)[C]) {
  double* p = r.pieces + (2 * chunk + h) * r.pstride + lane;
#pragma unroll
  for (int c = 0; c < C; ++c) p[kWave * c] = sum[c];
}

// Lane's columns of the n_bytes-long row at p (range-checked loads: 0 past
// the end, all 0 for n_bytes = 0), issued without a branch so that a batch
// of them stays in flight together.
template <int C>
__device__ __forceinline__ void load_masked(const float* p, int n_bytes, int lane,
                                            float (&x)[C]) {
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(p, n_bytes);
#pragma unroll
  for (int c = 0; c < C; ++c)
    x[c] = __uint_as_float(
        __builtin_amdgcn_raw_buffer_load_b32(rs, (lane + kWave * c) * 4, 0, 0));
}

// Where k_reduce finds the update of a sorted entry. kPull: no staging rows;
// the update of an input row is formed again from its minibatch's errors and
// output rows, that of an output column from the errors and input rows, in
// the staged kernel's order of fused multiply-adds, so to the same bits.
//
// Ids (sort keys) and errors of the partners of slot `slot` of minibatch b,
// one per lane; 2V where there is none.
__device__ __forceinline__ void load_partners(const ReduceArgs& r, int b, int slot,
                                              bool is_in, bool valid, int lane,
                                              uint32_t& key, float& error) {
  const int n_out = r.K + 1;
  const int most = !valid ? 0 : is_in ? n_out : r.N;
  key = 2u * (uint32_t)r.V;
  error = 0.f;
  if (lane < most) {
    const int64_t in0 = (int64_t)b * r.N;
    key = is_in ? r.ids_out[(int64_t)b * n_out + lane] : r.ids_in[in0 + lane];
    const int i = is_in ? slot : lane, k = is_in ? lane : slot;
    error = r.errors[(in0 + i) * n_out + k];
  }
}

template <int C, bool kPull>
__global__ __launch_bounds__(kWave) void k_reduce(ReduceArgs r) {
  constexpr int kBatch = kPull ? 4 : w2v::kBatch;
  constexpr int kRows = 4;  // partner rows in flight
  const int lane = threadIdx.x;
  const int64_t n_chunks = (r.n + kChunk - 1) / kChunk;
  static_assert(kChunk == kWave, "one sorted entry per lane");
  for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
    const int64_t lo = ch * kChunk;
    const int cnt = (int)(lo + kChunk < r.n ? kChunk : r.n - lo);
    // The chunk's keys and staging indices, one per lane.
    const uint32_t kl = lane < cnt ? r.key[lo + lane] : 0xffffffffu;
    const int32_t vl = lane < cnt ? r.val[lo + lane] : 0;
    // The minibatch and the slot within it of this lane's entry.
    int eb = 0, es = 0;
    const bool e_in = vl < r.out_base;
    if constexpr (kPull) {
      const uint32_t idx = (uint32_t)(e_in ? vl : vl - r.out_base);
      const uint32_t per = (uint32_t)(e_in ? r.N : r.K + 1);
      eb = (int)(idx / per);
      es = (int)(idx - (uint32_t)eb * per);
    }
    const uint64_t inputs = kPull ? __ballot(e_in) : 0ull;
    // A pulled batch reduces the keys in [key_lo, key_hi) (sorted: those below
    // come first), a staged one all that name a row: constants, which keep the
    // chain of a small batch short (B = 256, D = 384: 34.2 us, 37.4 with the
    // range read from the arguments).
    const uint32_t key_hi = kPull ? r.key_hi : 2u * (uint32_t)r.V;
    int j_lo = 0;
    if constexpr (kPull) {
      j_lo = __popcll(__ballot(lane < cnt && kl < r.key_lo));
      if (j_lo == cnt || (uint32_t)__builtin_amdgcn_readlane((int)kl, j_lo & 63) >= key_hi)
        continue;
    }
    const uint32_t prev = lo > 0 ? r.key[lo - 1] : 0xffffffffu;
    const uint32_t next = lo + cnt < r.n ? r.key[lo + cnt] : 0xffffffffu;
    uint32_t cur = 0xffffffffu;  // key of the open run (none yet)
    int start = 0, end = cnt;
    double sum[C];
    float mrow[C];               // matrix row of the open run, as read
#pragma unroll
    for (int c = 0; c < C; ++c) {
      sum[c] = 0.0;
      mrow[c] = 0.f;
    }
    // Closes the run [s, e) of key k: applied, or left as the chunk's head
    // piece (it began in an earlier chunk) or tail piece (it goes on).
    auto close = [&](uint32_t k, int s, int e) {
      if (s == 0 && prev == k) {
        put_piece<C>(r, ch, 0, lane, sum);
      } else if (e == cnt && next == k) {
        put_piece<C>(r, ch, 1, lane, sum);
      } else {
        store_sum<C, kPull>(r, k, lane, mrow, sum);
      }
    };
    bool done = false;
    for (int j0 = j_lo; j0 < cnt && !done; j0 += kBatch) {
      // Issue a batch of staging-row loads, and the matrix row of every run
      // that opens in the batch, then add them in order. A run's matrix row
      // is written by no one else before this wavefront applies it.
      float x[kBatch][C], m[kBatch][C];
      uint32_t pk[kPull ? kBatch : 1];
      float pe[kPull ? kBatch : 1];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = j0 + u;
        const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)kl, j & 63);
        const uint32_t kp = j == 0 ? prev : (uint32_t)__builtin_amdgcn_readlane((int)kl, j - 1);
        const bool valid = j < cnt && k < key_hi;
        const int32_t v = __builtin_amdgcn_readlane(vl, j & 63);
        if constexpr (kPull) {
          load_partners(r, __builtin_amdgcn_readlane(eb, j & 63), __builtin_amdgcn_readlane(es, j & 63),
                        ((inputs >> (j & 63)) & 1ull) != 0ull, valid, lane, pk[u], pe[u]);
        } else {
          load_masked<C>(r.stage + (int64_t)(valid ? v : 0) * r.ld, valid ? r.D * 4 : 0,
                         lane, x[u]);
        }
        const bool opens = valid && k != kp;
        load_masked<C>(key_row(r, opens ? k : 0u), opens ? r.D * 4 : 0, lane, m[u]);
      }
      if constexpr (kPull) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const int j = j0 + u;
          const bool is_in = ((inputs >> (j & 63)) & 1ull) != 0ull;
          const float* M = is_in ? r.M_out : r.M_in;
          // Partners are distinct rows first, unused slots after them.
          const int count = __popcll(__ballot(pk[u] < 2u * (uint32_t)r.V));
          const int row = (int)(pk[u] - (is_in ? (uint32_t)r.V : 0u));
#pragma unroll
          for (int c = 0; c < C; ++c) x[u][c] = 0.f;
#pragma unroll 1
          for (int p0 = 0; p0 < count; p0 += kRows) {
            float y[kRows][C];
#pragma unroll
            for (int p = 0; p < kRows; ++p)
              load_masked<C>(row_at(M, __builtin_amdgcn_readlane(row, p0 + p), r.ld),
                             p0 + p < count ? r.D * 4 : 0, lane, y[p]);
#pragma unroll
            for (int p = 0; p < kRows; ++p) {
              if (p0 + p < count) {
                const float e = lane_value(pe[u], p0 + p);
#pragma unroll
                for (int c = 0; c < C; ++c) x[u][c] = fmaf(e, y[p][c], x[u][c]);
              }
            }
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = j0 + u;
        const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)kl, j & 63);
        if (done || j >= cnt || k >= key_hi) {
          if (!done) end = j;
          done = true;
        } else {
          if (k != cur) {
            if (cur != 0xffffffffu) close(cur, start, j);
            cur = k;
            start = j;
#pragma unroll
            for (int c = 0; c < C; ++c) {
              sum[c] = 0.0;
              mrow[c] = m[u][c];
            }
          }
#pragma unroll
          for (int c = 0; c < C; ++c) sum[c] += (double)x[u][c];
        }
      }
    }
    if (cur != 0xffffffffu) close(cur, start, end);
  }
}

// Chunks per span: the head pieces of one run inside one span of kSpan
// chunks are first added into the span's first such piece, so that a run
// over many chunks costs its start chunk one read per span.
constexpr int kSpan = 32;

// Key of the first entry of chunk c, and whether its run began earlier.
__device__ __forceinline__ bool has_head(const ReduceArgs& r, int64_t c,
                                         uint32_t& key) {
  const int64_t lo = c * kChunk;
  if (lo <= 0 || lo >= r.n) return false;
  key = r.key[lo];
  return key < 2u * (uint32_t)r.V && r.key[lo - 1] == key;
}

// Adds `count` piece rows at pieces[2 (c0 + i)] (i < count), a batch at a
// time, in order.
template <int C>
__device__ __forceinline__ void add_heads(const ReduceArgs& r, int64_t c0,
                                          int64_t count, int lane,
                                          double (&sum)[C]) {
  for (int64_t i0 = 0; i0 < count; i0 += kBatch) {
    double x[kBatch][C];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      // past the end: re-read the last piece, not added below
      const int64_t cu = c0 + (i0 + u < count ? i0 + u : count - 1);
      const double* head = r.pieces + 2 * cu * r.pstride + lane;
#pragma unroll
      for (int c = 0; c < C; ++c) x[u][c] = head[kWave * c];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (i0 + u < count)
#pragma unroll
        for (int c = 0; c < C; ++c) sum[c] += x[u][c];
  }
}

// For every (run, span) with head pieces, the wavefront of the first such
// chunk adds the run's head pieces in the span, in chunk order, into that
// chunk's head piece.
template <int C>
__global__ __launch_bounds__(kWave) void k_reduce_spans(ReduceArgs r) {
  const int lane = threadIdx.x;
  const int64_t n_chunks = (r.n + kChunk - 1) / kChunk;
  for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
    uint32_t key;
    if (!has_head(r, ch, key)) continue;
    uint32_t kp;
    if (ch % kSpan != 0 && has_head(r, ch - 1, kp) && kp == key) continue;
    // The run's head pieces in this span: chunks ch, ch+1, ... (lane j
    // tests chunk ch + 1 + j; the run's chunks are consecutive).
    const int64_t span_end = (ch / kSpan + 1) * kSpan;
    const int64_t cj = ch + 1 + lane;
    uint32_t kj = 0u;
    const bool same = cj < span_end && has_head(r, cj, kj) && kj == key;
    const int64_t end = ch + 1 + __builtin_ctzll(~__ballot(same));
    if (end == ch + 1) continue;  // a single head piece is its own sum
    double sum[C];
#pragma unroll
    for (int c = 0; c < C; ++c) sum[c] = 0.0;
    add_heads<C>(r, ch, end - ch, lane, sum);
    put_piece<C>(r, ch, 0, lane, sum);
  }
}

template <int C>
__global__ __launch_bounds__(kWave) void k_reduce_cross(ReduceArgs r) {
  const int lane = threadIdx.x;
  const int64_t n_chunks = (r.n + kChunk - 1) / kChunk;
  for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
    const int64_t lo = ch * kChunk;
    const int64_t hi = lo + kChunk;
    if (hi >= r.n) continue;
    const uint32_t key = r.key[hi - 1];
    if (key >= 2u * (uint32_t)r.V || r.key[hi] != key) continue;
    // The run continues into the next chunk; it starts in this one unless
    // the whole chunk belongs to a run that began earlier.
    if (lo > 0 && r.key[lo] == key && r.key[lo - 1] == key) continue;
    // Last chunk of the run: the chunk ch + d is inside the run when the
    // entry opening it still has the key; gallop over d = 1, 2, 4, ... and
    // bisect, so a run over P chunks costs about 2 log2 P key reads.
    auto inside = [&](int64_t d) {
      const int64_t e = (ch + d) * kChunk;
      return e < r.n && r.key[e] == key;
    };
    int64_t good = 1, step = 1;      // chunk ch + 1 holds part of the run
    while (inside(good + step)) {
      good += step;
      step *= 2;
    }
    int64_t bad = good + step;       // first d known outside
    while (bad - good > 1) {
      const int64_t mid = good + (bad - good) / 2;
      if (inside(mid)) good = mid; else bad = mid;
    }
    const int64_t last_chunk = ch + good;
    double sum[C];
    const double* tail = r.pieces + (2 * ch + 1) * r.pstride + lane;
#pragma unroll
    for (int c = 0; c < C; ++c) sum[c] = tail[kWave * c];
    // One summed piece per span the run goes through (k_reduce_spans), in
    // span order: the first at ch + 1, the others at span starts.
    const int64_t first_span = (ch + 1) / kSpan, last_span = last_chunk / kSpan;
    for (int64_t sp0 = first_span; sp0 <= last_span; sp0 += kBatch) {
      double x[kBatch][C];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int64_t sp = sp0 + u <= last_span ? sp0 + u : last_span;
        const int64_t c1 = sp == first_span ? ch + 1 : sp * kSpan;
        const double* head = r.pieces + 2 * c1 * r.pstride + lane;
#pragma unroll
        for (int c = 0; c < C; ++c) x[u][c] = head[kWave * c];
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (sp0 + u <= last_span)
#pragma unroll
          for (int c = 0; c < C; ++c) sum[c] += x[u][c];
    }
    apply_sum<C>(r, key, lane, sum);
  }
}

// Pulled batches: the new M_in rows, kept aside while M_in was still read,
// go into the matrix (one wavefront per 64 sorted entries; the entries that
// open a run copy its row).
template <int C>
__global__ __launch_bounds__(kWave) void k_reduce_copy(ReduceArgs r) {
  constexpr int kRows = 4;  // rows in flight
  const int lane = threadIdx.x;
  const int64_t n_chunks = (r.n + kChunk - 1) / kChunk;
  for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
    const int64_t e = ch * kChunk + lane;
    const uint32_t k = e < r.n ? r.key[e] : 0xffffffffu;
    const uint32_t before = e > 0 && e < r.n ? r.key[e - 1] : 0xffffffffu;
    uint64_t open = __ballot(k < (uint32_t)r.V && k != before);
    while (open != 0ull) {
      int row[kRows], bytes[kRows];
      float x[kRows][C];
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        const int l = open != 0ull ? __builtin_ctzll(open) : 0;
        row[u] = __builtin_amdgcn_readlane((int)k, l);
        bytes[u] = open != 0ull ? r.D * 4 : 0;
        open &= open - 1ull;
        load_masked<C>(row_at(r.W_in, row[u], r.ld), bytes[u], lane, x[u]);
      }
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(row_at(r.M_in, row[u], r.ld), bytes[u]);
#pragma unroll
        for (int c = 0; c < C; ++c)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[u][c]), rs,
                                                (lane + kWave * c) * 4, 0, 0);
      }
    }
  }
}

#define W2V_SORTED_SHAPES(X) \
  X(1, 10) X(2, 10) X(3, 10) X(4, 10) X(5, 10) X(6, 10) X(8, 10) X(10, 10) \
  X(1, 16) X(2, 16) X(3, 16) X(4, 16) X(5, 16) X(1, 32) X(2, 32)

using StageKernel = void (*)(SortedStepArgs);
using ReduceKernel = void (*)(ReduceArgs);

static StageKernel stage_kernel_for(int C, int nmax, int K, bool pull) {
  const bool multi = K + 1 > Core<1, 10, false>::KB;
#define W2V_PICK(c, n) \
  if (C == c && nmax == n)                                                     \
    return pull ? (multi ? k_stage<c, n, true, true> : k_stage<c, n, false, true>) \
                : (multi ? k_stage<c, n, true, false> : k_stage<c, n, false, false>);
  W2V_SORTED_SHAPES(W2V_PICK)
#undef W2V_PICK
  return nullptr;
}

static bool reduce_kernels_for(int C, bool pull, ReduceKernel& red, ReduceKernel& spans,
                               ReduceKernel& cross, ReduceKernel& copy) {
  switch (C) {
#define W2V_CASE(c) \
  case c:           \
    red = pull ? k_reduce<c, true> : k_reduce<c, false>; spans = k_reduce_spans<c>; cross = k_reduce_cross<c>; copy = k_reduce_copy<c>; return true;
    W2V_CASE(1) W2V_CASE(2) W2V_CASE(3) W2V_CASE(4) W2V_CASE(5) W2V_CASE(6)
    W2V_CASE(8) W2V_CASE(10)
#undef W2V_CASE
    default:
      return false;
  }
}

static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

static int key_bits(int32_t V) {
  return 32 - __builtin_clz(2u * (unsigned)V);  // keys are 0..2V
}

// Doubles per piece row: at least 64 C for the C a row stride of ld can
// need (D <= ld; C = ceil(D/64) rounded up to a compiled size, at most one
// more).
static int64_t piece_stride(int32_t ld) { return (int64_t)kWave * ((ld + kWave - 1) / kWave + 1); }

// Workspace: staging rows (inputs, then outputs) or, for a pulled batch, the
// errors; then keys, sorted keys, values, sorted values, pieces, sort
// temporaries and, for a pulled batch, the new M_in rows (row r of V).
struct SortedLayout {
  int64_t n_in, n;
  size_t stage, ints, pieces, temp, next_in, total;
};

static SortedLayout sorted_layout(int32_t B, int32_t N, int32_t K, int32_t V,
                                  int32_t ld, bool pull) {
  SortedLayout L{};
  L.n_in = (int64_t)B * N;
  L.n = L.n_in + (int64_t)B * (K + 1);
  L.stage = align256(sizeof(float) * (pull ? (size_t)L.n_in * (size_t)(K + 1)
                                           : (size_t)L.n * (size_t)ld));
  L.ints = align256(sizeof(uint32_t) * (size_t)L.n);
  L.pieces = align256(sizeof(double) * 2 * (size_t)((L.n + kChunk - 1) / kChunk) *
                     (size_t)piece_stride(ld));
  L.temp = align256(radix_sort_temp_bytes(L.n, sizeof(uint32_t)));
  L.next_in = pull ? align256(sizeof(float) * (size_t)V * (size_t)ld) : 0;
  L.total = L.stage + 4 * L.ints + L.pieces + L.temp + L.next_in;
  if (L.total == 0) L.total = 256;
  return L;
}

size_t sorted_step_workspace_bytes(int32_t B, int32_t N, int32_t K, int32_t V,
                                   int32_t ld, bool pull) {
  return sorted_layout(B, N, K, V, ld, pull).total;
}

bool sorted_step_supported(int C, int nmax) {
  ReduceKernel r, sp, x, cp;
  return stage_kernel_for(C, nmax, 0, false) != nullptr &&
         reduce_kernels_for(C, false, r, sp, x, cp);
}

hipError_t launch_step_sorted(int C, int nmax, SortedStepArgs a, void* workspace,
                              bool pull, hipStream_t s) {
  StageKernel k = stage_kernel_for(C, nmax, a.K, pull);
  ReduceKernel red, spans, cross, copy;
  if (k == nullptr || !reduce_kernels_for(C, pull, red, spans, cross, copy))
    return hipErrorInvalidValue;
  const SortedLayout L = sorted_layout(a.B, a.N, a.K, a.V, (int32_t)a.ld, pull);
  char* w = (char*)workspace;
  float* stage = (float*)w;
  uint32_t* keys = (uint32_t*)(w + L.stage);
  uint32_t* keys_sorted = (uint32_t*)(w + L.stage + L.ints);
  int32_t* vals = (int32_t*)(w + L.stage + 2 * L.ints);
  int32_t* vals_sorted = (int32_t*)(w + L.stage + 3 * L.ints);
  double* pieces = (double*)(w + L.stage + 4 * L.ints);
  void* temp = (void*)(w + L.stage + 4 * L.ints + L.pieces);
  a.stage_in = stage;
  a.stage_out = pull ? stage : stage + L.n_in * a.ld;
  a.errors = stage;
  a.key_in = keys;
  a.val_in = vals;
  a.key_out = keys + L.n_in;
  a.val_out = vals + L.n_in;
  a.out_base = L.n_in;
  const int grid = a.B < (1 << 20) ? a.B : (1 << 20);
  hipLaunchKernelGGL(k, dim3(grid), dim3(kWave), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = radix_sort_pairs((const uint32_t*)keys, (const int32_t*)vals, keys_sorted,
                       vals_sorted, L.n, key_bits(a.V), temp, s);
  if (e != hipSuccess) return e;
  float* next_in = (float*)((char*)temp + L.temp);
  ReduceArgs r{keys_sorted, vals_sorted, L.n, stage, a.M_in, a.M_out, pieces,
               a.V, a.D, a.ld, piece_stride((int32_t)a.ld),
               0u, 2u * (uint32_t)a.V, pull ? next_in : a.M_in,
               stage, keys, keys + L.n_in, a.N, a.K, (int32_t)L.n_in};
  if (r.pstride < (int64_t)kWave * C) return hipErrorInvalidValue;
  const int64_t n_chunks = (L.n + kChunk - 1) / kChunk;
  const int rgrid = (int)(n_chunks < 65536 ? n_chunks : 65536);
  if (pull) {
    // Input rows first, into next_in: they read M_out as it was. Then the
    // output columns, which read M_in as it was and move M_out.
    r.key_hi = (uint32_t)a.V;
    hipLaunchKernelGGL(red, dim3(rgrid), dim3(kWave), 0, s, r);
    r.key_lo = (uint32_t)a.V;
    r.key_hi = 2u * (uint32_t)a.V;
  }
  hipLaunchKernelGGL(red, dim3(rgrid), dim3(kWave), 0, s, r);
  hipLaunchKernelGGL(spans, dim3(rgrid), dim3(kWave), 0, s, r);
  hipLaunchKernelGGL(cross, dim3(rgrid), dim3(kWave), 0, s, r);
  if (pull) hipLaunchKernelGGL(copy, dim3(rgrid), dim3(kWave), 0, s, r);
  return hipGetLastError();
}

}  // namespace w2v
