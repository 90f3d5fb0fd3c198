// Ids of one minibatch of a snapshot batch, as the caller gave them.
#pragma once

#include "device_common.h"

namespace w2v {

struct BatchIds {
  int target;        // uniform
  int ctx;           // lane i < N: input word, -1 if absent
  int neg;           // lane k < K: negative
  uint64_t present;  // lanes that hold an input word
};

// Reads minibatch b; returns whether one of its ids is outside [0, V).
template <class Args>
__device__ __forceinline__ bool read_batch_ids(const Args& a, int64_t b, int lane,
                                               BatchIds& ids) {
  ids.target = uniform_int(a.targets[b]);
  ids.ctx = lane < a.N ? a.contexts[b * a.N + lane] : -1;
  ids.neg = lane < a.K ? a.negatives[b * a.K + lane] : 0;
  ids.present = __ballot(ids.ctx >= 0);
  return __ballot(ids.ctx < -1 || ids.ctx >= a.V || ids.neg < 0 || ids.neg >= a.V) != 0ull ||
         ids.target < 0 || ids.target >= a.V;
}

}  // namespace w2v
