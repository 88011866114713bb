// How a deviation Gram launch of the probe splits a unit's tokens over
// workgroups.  Plain C++, usable on the host.
#pragma once

#include <stdint.h>

namespace fdkv {

// Tokens per workgroup: at most kProbeMost, which is what is summed in fp32
// before the sums over a unit's workgroups (taken in fp64), and at least
// kProbeLeast, for which the workspace holds a partial each.
constexpr int kProbeMost = 1024, kProbeLeast = 256;

inline uint64_t probe_partials(int T, int tokens) { return ((uint64_t)T + tokens - 1) / tokens; }

struct ProbeSplit {
  int chunk_tokens, n_chunks;  // tokens per workgroup (the last one: the rest), workgroups per unit
};

// The split of `units` units of T >= 1 tokens, `rows` tokens a step (a divisor
// of kProbeLeast), for a chip that holds `at_once` workgroups and a workspace of
// `cap` >= probe_partials(T, kProbeMost) partials a unit.  The launch runs in
// rounds of `at_once` workgroups; of the counts that the bounds allow, the one
// of the least cost is taken: the steps over all rounds, a workgroup's start and
// its contraction with the probe Gram matrix counted as three, plus a quarter of
// a workgroup's steps, as they don't end together.  Against 1024 tokens a
// workgroup, probe of 32 layers of the 8B shape: default block setting 157 -> 98
// us at 500 tokens, 273 -> 128 at 2000, 715 -> 612 at 12345 (48 units of four:
// 624 workgroups of 1024 tokens, the third round nearly empty); pairs 353 -> 340
// at 12345, and the same where the rounds come out even (804 us at 32768).
// (Counted as one step: 633 at 12345 in the default setting.)
inline ProbeSplit probe_split(int units, int T, int rows, int at_once, int cap) {
  const int64_t steps = ((int64_t)T + rows - 1) / rows, least = (int64_t)probe_partials(T, kProbeMost);
  ProbeSplit s{};
  int64_t best = INT64_MAX;
  for (int64_t n = least; n <= cap && n <= least + 64; ++n) {  // past that the rounds are many and come out alike
    const int64_t each = (steps + n - 1) / n, used = (steps + each - 1) / each;
    const int64_t cost = 4 * ((units * used + at_once - 1) / at_once) * (each + 3) + each;
    if (cost <= best) {
      best = cost;
      s.chunk_tokens = (int)(each * rows);
      s.n_chunks = (int)used;
    }
  }
  return s;
}

}  // namespace fdkv
