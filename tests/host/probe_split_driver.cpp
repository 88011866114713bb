// Host driver for the probe's split of a unit over workgroups: checks, over
// units, lengths, steps, chips and workspaces, that every token is taken once, by
// at most 1024 a workgroup, in whole steps and within the workspace's partials,
// and prints the number of splits checked.
#include <cstdio>
#include <initializer_list>
#include "../../paper_2607_06519_amd/csrc/probe_split.h"

using namespace fdkv;

int main() {
  unsigned long long n_checked = 0;
  auto check = [&](int units, int T, int rows, int at_once, int cap) {
    const ProbeSplit s = probe_split(units, T, rows, at_once, cap);
    ++n_checked;
    const bool ok = s.n_chunks >= 1 && s.n_chunks <= cap && s.chunk_tokens >= rows && s.chunk_tokens <= kProbeMost &&
                    s.chunk_tokens % rows == 0 && (long long)s.n_chunks * s.chunk_tokens >= T &&
                    (long long)(s.n_chunks - 1) * s.chunk_tokens < T;
    if (!ok) printf("wrong: %d units of %d tokens, %d a step, %d at once, %d partials: %d x %d\n", units, T, rows, at_once, cap,
                    s.n_chunks, s.chunk_tokens);
    return ok;
  };
  auto all = [&](int T) {
    for (int units : {1, 2, 3, 8, 16, 48, 96, 128, 256, 320, 640, 5120})
      for (int rows : {32, 64})
        for (int at_once : {256, 512})
          for (int tokens : {kProbeMost, kProbeLeast})
            if (!check(units, T, rows, at_once, (int)probe_partials(T, tokens))) return false;
    return true;
  };
  for (int T = 1; T <= 5000; ++T)
    if (!all(T)) return 1;
  for (int T : {12345, 32767, 32768, 32769, 131071, 131072, 131073, 1000003, 8388607})
    if (!all(T)) return 1;
  printf("%llu\n", n_checked);
  return 0;
}
