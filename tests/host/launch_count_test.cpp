// Launches of a call (a short one is bound by them), counted at the launcher stand-ins: the sequence table
// goes with the partition, not in a launch of its own.  Prints "launch count ok".
#include <cstdint>
#include <cstdio>
#include <vector>

#include "twinkv.h"

namespace stub {
extern int64_t g_launches;
}

int main() {
  const int d = 64, n = 512;
  const int64_t cu[2] = {0, n}, budget[1] = {n / 2};
  std::vector<float> keys(n * d), b(n);
  std::vector<uint8_t> mask(n), out(n);
  std::vector<int32_t> arg(n), counts(n), stats(4);
  const int64_t nb = twinkv_workspace_bytes(TWINKV_OP_REPAIR, TWINKV_F32, d, 1, 1, cu);
  std::vector<char> ws(nb);
  int fail = 0;
  auto count = [&](int line, int64_t want, int rc) {
    if (rc != TWINKV_OK || stub::g_launches != want) {
      std::fprintf(stderr, "line %d: rc %d, %lld launches, expected %lld\n", line, rc,
                   (long long)stub::g_launches, (long long)want);
      fail = 1;
    }
    stub::g_launches = 0;
  };
  // partition, key preparation, similarity, repair
  count(__LINE__, 4, twinkv_repair(keys.data(), TWINKV_F32, d, 1, 1, cu, n * d, d, mask.data(), out.data(), budget,
                                   0.9f, 32, 4, 4, stats.data(), b.data(), arg.data(), nullptr, nullptr, ws.data(),
                                   nb, nullptr));
  count(__LINE__, 4, twinkv_repair(keys.data(), TWINKV_F32, d, 1, 1, cu, n * d, d, mask.data(), out.data(), budget,
                                   0.9f, 32, 4, 4, stats.data(), nullptr, nullptr, nullptr, nullptr, ws.data(), nb,
                                   nullptr));
  count(__LINE__, 3, twinkv_nn_scores(keys.data(), TWINKV_F32, d, 1, 1, cu, n * d, d, nullptr, 32, b.data(),
                                      arg.data(), nullptr, nullptr, nullptr, ws.data(), nb, nullptr));
  count(__LINE__, 3, twinkv_twin_counts(keys.data(), TWINKV_F32, d, 1, 1, cu, n * d, d, 0.9f, 32, counts.data(),
                                        nullptr, ws.data(), nb, nullptr));
  if (fail) return 1;
  std::printf("launch count ok\n");
  return 0;
}
