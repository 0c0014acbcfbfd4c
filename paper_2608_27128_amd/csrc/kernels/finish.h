// The pair sweep's candidates to results: best_ret / arg_ret from plane 0 (S0 columns), best_all /
// arg_all from both planes.  Shared by the finish kernel and the repair of short sequences.
#pragma once
#include <hip/hip_runtime.h>

#include "../twinkv_internal.h"
#include "key_scale.h"

namespace twinkv {

// Where a problem's candidates and results lie.
struct FinishPlace {
  int64_t col, row;  // its first slot in the column arrays, its first token in the row arrays
  int ret_pad, nslots;
};
__device__ inline FinishPlace finish_place(const SimArgs& a, int head, const SeqInfo& si, const ProblemMeta& pm) {
  return {(int64_t)head * a.PT + si.perm_off, (int64_t)head * a.T + si.start, pm.ret_chunks * kChunk,
          pm.total_chunks * kChunk};
}

// Tokens i, i + step, .. (N of them; those past the problem's len tokens are left out), their loads in
// flight together; returns b_i(S0) of each.  A key with infinite elements makes NaN of a dropped block's zero r', in the row direction also
// of the zeros past the list's end: a candidate there names no token.
template <int N>
struct Scores {
  float b[N];
};
template <int N>
__device__ inline Scores<N> finish_tokens(const SimArgs& a, const FinishPlace& pl, int len, int i, int step) {
  const unsigned long long* best = a.best + pl.col;
  const int32_t* pc = a.pcol + pl.col;
  const int64_t plane = (int64_t)a.n_heads * a.PT;
  unsigned long long kr[N], ke[N];
  int jr[N], je[N];
  float ri[N];
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int t = min(i + n * step, len - 1);
    const int r0 = a.prank[pl.col + t], r1 = a.prank[pl.col + t + 1];
    const int slot = r1 > r0 ? r0 : pl.ret_pad + (t - r0);
    kr[n] = best[slot];
    ke[n] = best[plane + slot];
    ri[n] = a.rinv[pl.row + t];
  }
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const uint32_t sr = ~(uint32_t)kr[n], se = ~(uint32_t)ke[n];
    const bool any_r = (uint32_t)(kr[n] >> 32) >= kValidMin && sr < (uint32_t)pl.nslots;
    const bool any_e = (uint32_t)(ke[n] >> 32) >= kValidMin && se < (uint32_t)pl.nslots;
    jr[n] = any_r ? pc[sr] : -1;
    je[n] = any_e ? pc[se] : -1;
  }
  Scores<N> out;
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int64_t o = pl.row + i + n * step;
    const uint32_t vr = (uint32_t)(kr[n] >> 32), ve = (uint32_t)(ke[n] >> 32);
    out.b[n] = jr[n] >= 0 ? similarity(vr, ri[n]) : -1.0f;
    if (i + n * step >= len) continue;
    if (a.best_ret) a.best_ret[o] = out.b[n];
    if (a.arg_ret) a.arg_ret[o] = jr[n];
    const bool take_r = jr[n] >= 0 && (je[n] < 0 || vr > ve || (vr == ve && jr[n] < je[n]));
    const int j = take_r ? jr[n] : je[n];
    if (a.best_all) a.best_all[o] = j >= 0 ? similarity(take_r ? vr : ve, ri[n]) : -1.0f;
    if (a.arg_all) a.arg_all[o] = j;
  }
  return out;
}

}  // namespace twinkv
