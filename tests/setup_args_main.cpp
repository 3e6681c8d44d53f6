// Arrays to be cleared by the first launch of a call: as many as the argument block holds, then one more.
#include <cstdio>

#include "plan_device.h"

int main() {
  unsigned char blob[16];
  uint32_t words[16];
  adwin::SetupArgs a(blob, 1);
  const int most = adwin::SetupArgs::kMaxZero;
  a.clear(nullptr, 5);          // an output that is not wanted takes no place
  a.clear(words, 0);
  for (int i = 0; i < most; ++i) a.clear(words + i, i + 1);
  bool kept = a.n_zero == most;
  a.clear(words + most, 77);
  for (int i = 0; i < most; ++i) kept = kept && a.zero[i] == words + i && a.zero_n[i] == i + 1;
  const bool refused = adwin::launch_setup(a, std::vector<unsigned char>(16), nullptr) == hipErrorInvalidValue;
  std::printf("%s %s\n", kept ? "kept" : "overwritten", refused ? "refused" : "accepted");
  return kept && refused ? 0 : 1;
}
