// The merge of a row's strips against the same fp32 sums on the host, in the order of 64 lanes: lane s takes the strips
// s, s + 64, ...; then lanes 32 apart are added, 16 apart, and so on.  1 / Z_s and A / Z_s, bit for bit.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "fused_shared.h"

#define TRY(x) do { hipError_t e = (x); if (e != hipSuccess) { std::printf("%s: %s\n", #x, hipGetErrorString(e)); return 2; } } while (0)

static float lanes_sum(const float* p, int strips, int n) {
  float lane[64] = {};
  for (int s = 0; s < strips; ++s) lane[s & 63] += p[(size_t)s * n];
  for (int o = 32; o > 0; o >>= 1)
    for (int l = 0; l < o; ++l) lane[l] += lane[l + o];
  return lane[0];
}

int main() {
  constexpr int n = adwin::kTileTokens, most = adwin::kMaxSweepStrips;
  std::vector<float> part((size_t)5 * most * n), zero(n, 0.f), mu(n), iz(n);
  std::vector<int32_t> idx(n);
  unsigned x = 1;
  for (auto& v : part) { x = x * 1664525u + 1013904223u; v = 0.25f + (float)(x >> 8) * 0x1p-24f; }
  for (int i = 0; i < n; ++i) idx[i] = i;
  float *d_part, *d_f;
  int32_t* d_idx;
  TRY(hipMalloc((void**)&d_part, part.size() * 4));
  TRY(hipMalloc((void**)&d_f, (size_t)8 * n * 4));
  TRY(hipMalloc((void**)&d_idx, (size_t)2 * n * 4));
  TRY(hipMemcpy(d_part, part.data(), part.size() * 4, hipMemcpyHostToDevice));
  TRY(hipMemcpy(d_idx, idx.data(), n * 4, hipMemcpyHostToDevice));
  TRY(hipMemset(d_idx + n, 0xff, n * 4));                   // no tokens
  TRY(hipMemset(d_f, 0, (size_t)8 * n * 4));
  const int strips[] = {1, 2, 3, 15, 16, 17, 31, 32, 33, 38, 47, 48, 49, 63, 64, 65, 127, 128, 129, 200, 238, 255, 256};
  for (int s : strips)
    for (int diag = 0; diag < 2; ++diag) {
      adwin::MergeSingleArgs a{};
      a.m.part = d_part; a.m.strips = s; a.m.n_pad = n; a.m.n_rows = n; a.m.row_idx = d_idx; a.m.diag = diag;
      a.m.klr = d_f; a.m.lse_s = d_f + n;
      a.mu_out = d_f + 2 * n; a.inv_z = d_f + 3 * n;
      a.ref.max[0] = d_f + 4 * n; a.ref.max[1] = d_f + 5 * n; a.ref.zy[0] = d_f + 6 * n; a.ref.zy[1] = d_f + 7 * n;
      a.ref.yid = d_idx + n; a.ref.n_pad = n; a.ref.parts = 1;
      a.row0 = 0; a.rows = n;
      std::printf("%d strips, diagnostics %d\n", s, diag);
      std::fflush(stdout);
      TRY(adwin::launch_merge_single(a, nullptr));
      TRY(hipDeviceSynchronize());
      TRY(hipMemcpy(mu.data(), a.mu_out, n * 4, hipMemcpyDeviceToHost));
      TRY(hipMemcpy(iz.data(), a.inv_z, n * 4, hipMemcpyDeviceToHost));
      for (int r = 0; r < n; ++r) {
        const float Z = lanes_sum(part.data() + r, s, n), A = lanes_sum(part.data() + (size_t)s * n + r, s, n);
        const float want_iz = 1.f / Z, want_mu = A / Z;
        if (std::memcmp(&want_iz, &iz[r], 4) || std::memcmp(&want_mu, &mu[r], 4)) {
          std::printf("row %d: %.9g %.9g, not %.9g %.9g\n", r, iz[r], mu[r], want_iz, want_mu);
          return 1;
        }
      }
    }
  std::puts("ok");
  return 0;
}
