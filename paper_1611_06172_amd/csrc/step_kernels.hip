// Snapshot batch of independent HogBatch minibatches on gfx950: the route
// with atomics (w2v_step_batch takes it where its sizes make it the fastest
// and where the matrices share elements; the others are in step_sorted.hip).
//
// Three launches on the caller's stream:
//   1. zero the fp64 delta buffers (workspace);
//   2. one wavefront per minibatch (persistent grid-stride over the batch):
//      rows are read from the matrices, which stay unchanged during this
//      launch, so every minibatch sees the input matrices; the fp32 updates
//      are added with fp64 atomics into the delta buffers;
//   3. every element with a non-zero delta becomes fp32(M + delta), one
//      rounding per element, so the result does not depend on the order in
//      which the atomics landed beyond fp64 rounding.
#include "kernel_args.h"
#include "batch_ids.h"
#include "sgns_core.h"

namespace w2v {

__global__ __launch_bounds__(256) void k_zero(double* p, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    p[i] = 0.0;
}

// Rows of the unchanged matrices (Core's Io); updates are added to the
// delta buffers.
template <int C>
struct StepIo {
  const StepArgs& a;
  int lane;

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
  __device__ __forceinline__ void add(double* d, int id, const float (&g)[N], int c0) const {
    double* row = row_at(d, id, a.ld);
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int col = lane + kWave * (c0 + c);
      if (col < a.D) unsafeAtomicAdd(row + col, (double)g[c]);
    }
  }
  template <int N>
  __device__ __forceinline__ void put_out(int, int id, const float (&)[N],
                                          const float (&g)[N], int c0) const {
    add(a.dM_out, id, g, c0);
  }
  template <int N>
  __device__ __forceinline__ void put_in(int, int id, const float (&)[N],
                                         const float (&g)[N], const float (&)[N],
                                         int c0) const {
    add(a.dM_in, id, g, c0);
  }
};

template <int C, int NMAX, bool kMulti>
__global__ __launch_bounds__(kWave) void k_step(StepArgs a) {
  const int lane = threadIdx.x;
  int64_t applied = 0, sum_n = 0, rejected = 0, rows = 0;
  for (int64_t b = blockIdx.x; b < a.B; b += gridDim.x) {
    BatchIds ids;
    const bool bad = read_batch_ids(a, b, lane, ids);
    if (bad) {
      ++rejected;
      continue;
    }
    const int n = __popcll(ids.present);
    if (n == 0) continue;
    const Minibatch mb = stage_minibatch<(NMAX > 16)>(lane, ids.ctx, ids.present,
                                                      ids.target, ids.neg, a.K);
    StepIo<C> io{a, lane};
    Core<C, NMAX, kMulti> core;
    core.load(io, mb);
    ++applied;
    sum_n += n;
    rows += mb.n + mb.n_out;
    float unused = 0.f;
    core.run(io, lane, mb, a.alpha != nullptr ? a.alpha[b] : a.alpha_scalar, false, unused);
  }
  if (lane == 0) report_bad_ids(a.status, rejected);
  if (a.stats != nullptr && lane == 0) {
    atomicAdd((unsigned long long*)&a.stats[0], (unsigned long long)applied);
    atomicAdd((unsigned long long*)&a.stats[1], (unsigned long long)sum_n);
    atomicAdd((unsigned long long*)&a.stats[3], (unsigned long long)rejected);
    atomicAdd((unsigned long long*)&a.stats[4], (unsigned long long)rows);
  }
}

// M = fp32(M + delta) where delta != 0; one wavefront per row.
__global__ __launch_bounds__(256) void k_finalize(float* M, const double* dM,
                                                  int32_t V, int32_t D,
                                                  int64_t ld) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  for (int64_t r = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
       r < V; r += waves) {
    for (int col = lane; col < D; col += kWave) {
      const double d = dM[r * ld + col];
      if (d != 0.0) M[r * ld + col] = (float)((double)M[r * ld + col] + d);
    }
  }
}

#define W2V_STEP_SHAPES(X) \
  X(1, 10) X(2, 10) X(3, 10) X(4, 10) X(5, 10) X(6, 10) X(8, 10) X(10, 10) \
  X(1, 16) X(2, 16) X(3, 16) X(4, 16) X(5, 16) X(1, 32) X(2, 32)

using StepKernel = void (*)(StepArgs);

static StepKernel step_kernel_for(int C, int nmax, int K) {
  const bool multi = K + 1 > Core<1, 10, false>::KB;
#define W2V_PICK(c, n) \
  if (C == c && nmax == n) return multi ? k_step<c, n, true> : k_step<c, n, false>;
  W2V_STEP_SHAPES(W2V_PICK)
#undef W2V_PICK
  return nullptr;
}

hipError_t launch_step(int C, int nmax, const StepArgs& a, int grid,
                       hipStream_t s) {
  StepKernel k = step_kernel_for(C, nmax, a.K);
  if (k == nullptr) return hipErrorInvalidValue;
  const int64_t n_delta = (int64_t)a.V * a.ld;
  hipLaunchKernelGGL(k_zero, dim3(4096), dim3(256), 0, s, a.dM_in, n_delta);
  hipLaunchKernelGGL(k_zero, dim3(4096), dim3(256), 0, s, a.dM_out, n_delta);
  hipLaunchKernelGGL(k, dim3(grid), dim3(kWave), 0, s, a);
  const int64_t blocks = ((int64_t)a.V + 3) / 4;
  const int fgrid = (int)(blocks < 65536 ? blocks : 65536);
  hipLaunchKernelGGL(k_finalize, dim3(fgrid), dim3(256), 0, s, a.M_in,
                     (const double*)a.dM_in, a.V, a.D, a.ld);
  hipLaunchKernelGGL(k_finalize, dim3(fgrid), dim3(256), 0, s, a.M_out,
                     (const double*)a.dM_out, a.V, a.D, a.ld);
  return hipGetLastError();
}

}  // namespace w2v
