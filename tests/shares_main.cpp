// Shares against what they stand for, every number of parts up to kMaxShares: share i begins at floor(i total / parts),
// and by_length lists the longer shares and then the others, each in index order.
#include <cstdio>

#include "fused_shared.h"

int main() {
  using adwin::Shares;
  static_assert(adwin::kMaxShares >= adwin::kMaxSweepStrips && adwin::kMaxShares >= adwin::kMaxStrips, "parts in use");
  const int totals[] = {1, 2, 31, 94, 188, 1187, 2374, 65535, 1000003};
  long bad = 0, checked = 0;
  for (int parts = 1; parts <= adwin::kMaxShares; ++parts) {
    auto check = [&](int total) {
      Shares s;
      s.split(total, parts);
      for (int i = 0; i <= parts; ++i, ++checked) bad += s.first(i) != (int)((long long)i * total / parts);
      int at[2] = {0, s.longer};
      for (int i = 0; i < parts; ++i) {
        const bool longer = s.first(i + 1) - s.first(i) > s.each;
        bad += s.by_length(at[longer ? 0 : 1]++) != i;
      }
      bad += at[0] != s.longer || at[1] != parts;
    };
    for (int total : totals) check(total);
    for (int rest = 0; rest < parts; rest += 1 + parts / 64) check(3 * parts + rest);
    check(4 * parts - 1);
  }
  std::printf("%s %ld\n", bad ? "bad" : "ok", checked);
  return bad != 0;
}
