// What the split-K decode kernels (decode_stream.h for bf16 and FP8 caches,
// decode.hip for fp32 ones) and the merge of their records share.
#pragma once

#include "fdkv_common.h"
#include "fdkv_kernels.h"

namespace fdkv {

// Launch shapes of a chunk of 512 tokens (one split-K record) of an fp32 cache.
//  kFull   - one workgroup of 4 waves, 128 tokens a wave.
//  kWide   - one workgroup of 4 NGRP waves; a group of 4 waves takes
//            512 / NGRP consecutive tokens.  (d = 128: sixteen waves hold it to
//            128 VGPRs, 12 spilled at two query heads and 23 at four.)
//  kSpread - the groups of kWide as NGRP workgroups, each writing a record of
//            its own, which the merge folds into the chunk's record with
//            kWide's arithmetic (the two give the same bits).
// kFull and the other two differ by the rounding of fp32 sums.  bf16 and FP8
// caches have the one shape of decode_stream.h: their probabilities are rounded
// to bf16 against the reference max that a wave has reached, so another split of
// a chunk would give outputs that differ by 2e-3 of their norm.
enum Shape : int { kFull, kWide, kSpread };

// The unit arrays as constant memory, so that uniform reads are scalar loads
// (the kernel does not write them).
template <class X>
__device__ __forceinline__ const __attribute__((address_space(4))) X* as_const(const X* p) {
  return (const __attribute__((address_space(4))) X*)p;
}

// Weight of a partial sum with reference max m in a sum with reference max M.
__device__ __forceinline__ float merge_weight(float m, float M) {
  return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
}

}  // namespace fdkv
