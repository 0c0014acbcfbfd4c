// Which sweep a call takes that needs all columns (sweep_for), at shapes whose times are known.
// Prints "sweep rule ok".
#include <cstdint>
#include <cstdio>
#include <vector>

#include "twinkv.h"
#include "twinkv_internal.h"

using namespace twinkv;

namespace {
int g_fail = 0;

// n_seqs sequences spread evenly over [lo, hi] tokens.
void expect(int line, Sweep want, int dtype, int d, bool counts, int heads, int n_seqs, int lo, int hi) {
  std::vector<int64_t> cu(n_seqs + 1, 0);
  for (int s = 0; s < n_seqs; ++s) cu[s + 1] = cu[s] + lo + (n_seqs > 1 ? (int64_t)(hi - lo) * s / (n_seqs - 1) : 0);
  const Sweep got = sweep_for(dtype, d, counts, heads, n_seqs, cu.data());
  if (got != want) {
    std::fprintf(stderr, "line %d: sweep %d, expected %d\n", line, (int)got, (int)want);
    ++g_fail;
  }
}
#define EXPECT_SWEEP(...) expect(__LINE__, __VA_ARGS__)
}  // namespace

int main() {
  const int B = TWINKV_BF16, F = TWINKV_F32;
  // many short sequences: the rectangle
  EXPECT_SWEEP(kSweepAll, B, 128, false, 128, 16, 150, 300);
  EXPECT_SWEEP(kSweepAll, B, 128, false, 64, 16, 250, 500);
  EXPECT_SWEEP(kSweepAll, B, 128, false, 288, 1, 395, 395);
  EXPECT_SWEEP(kSweepAll, B, 64, false, 288, 16, 175, 700);
  EXPECT_SWEEP(kSweepAll, B, 64, true, 128, 1, 100, 100);
  EXPECT_SWEEP(kSweepAll, B, 128, true, 288, 1, 128, 128);
  EXPECT_SWEEP(kSweepAll, F, 64, false, 128, 32, 40, 64);
  EXPECT_SWEEP(kSweepAll, F, 128, false, 128, 32, 40, 64);
  // few problems or long ones: the pairs
  EXPECT_SWEEP(kSweepPairs, F, 64, false, 1, 1, 512, 512);
  EXPECT_SWEEP(kSweepPairs, B, 128, false, 8, 1, 4001, 4001);
  EXPECT_SWEEP(kSweepPairs, B, 128, false, 8, 8, 100, 200);
  EXPECT_SWEEP(kSweepPairs, B, 128, false, 288, 16, 64, 64);
  EXPECT_SWEEP(kSweepPairs, B, 128, false, 288, 1, 900, 900);
  EXPECT_SWEEP(kSweepPairs, B, 64, false, 288, 1, 400, 400);
  EXPECT_SWEEP(kSweepPairs, B, 64, true, 288, 16, 128, 128);
  EXPECT_SWEEP(kSweepPairs, F, 64, true, 128, 32, 40, 64);
  EXPECT_SWEEP(kSweepPairs, B, 128, false, 288, 64, 1024, 4096);
  EXPECT_SWEEP(kSweepPairs, B, 64, false, 128, 1, 8192, 8192);
  EXPECT_SWEEP(kSweepPairs, B, 128, true, 288, 1, 16384, 16384);
  EXPECT_SWEEP(kSweepPairs, F, 128, false, 32, 4, 1000, 5000);
  // the mean is over the tokens: a few long sequences among many short ones decide
  {
    std::vector<int64_t> cu{0};
    for (int s = 0; s < 60; ++s) cu.push_back(cu.back() + 200);
    cu.push_back(cu.back() + 30000);
    if (sweep_for(B, 128, false, 8, (int)cu.size() - 1, cu.data()) != kSweepPairs) ++g_fail;
    cu.pop_back();
    if (sweep_for(B, 128, false, 8, (int)cu.size() - 1, cu.data()) != kSweepAll) ++g_fail;
  }
  // empty sequences
  EXPECT_SWEEP(kSweepPairs, B, 128, false, 128, 4, 0, 0);
  EXPECT_SWEEP(kSweepAll, B, 64, false, 128, 4, 0, 0);
  if (g_fail) return 1;
  std::printf("sweep rule ok\n");
  return 0;
}
