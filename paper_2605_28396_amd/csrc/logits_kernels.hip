// Logits-given path: full-vocabulary log-softmax of student and teacher, per-token
// reverse KL (Eq. 2 at token level), sampled cost c_t (Sec. 2.3) and the logit gradient
// p_s((z_s - z_t) - mu) (Eq. 4 in expectation, App. A.1) on the admitted rows
// (Sec. 4.1), from HBM.  Which kernel a row takes follows its length and the number of rows.
#include <mutex>
#include <utility>
#include <vector>

#include "device_utils.h"
#include "plan_device.h"
#include "setup_device.h"
#include "tail_device.h"

namespace adwin {

constexpr int kRowThreads = 512;

struct LogitsArgs {
  DevicePlan pl;
  int64_t T;
  int32_t B, V;
  const uint4* z_s;
  const uint4* z_t;
  const int32_t* ids;
  float grad_scale;
  float* kl;
  float* c;
  uint4* dz;
  float* klr;          // [T] workspace copy of KL_t on computed rows (compact index)
  uint32_t* status;
  // teacher-side diagnostics (Sec. 3.1), each may be NULL
  float* t_logp; float* t_entropy; int32_t* t_rank;
  // few long rows, each cut into `splits` pieces: the pieces' sums [n_adm][splits][8]
  float* part; int splits; int64_t n_adm;
  int sampled;         // dz = scale c_t (e_y - p_s) (Eq. 4 on the sampled token) instead of scale p_s (Delta - KL_t)
  int tail_has_kl;     // split rows: the tail's workgroups, in the same launch as dz, write klr
  int mark;            // an excluded row leaves kExcludedRow in klr, for the tail to report (BatchArgs::status)
};

// The arguments of a launch that also sets up.  A launch costs about 2 us on the device and 4 on the host however
// little it does, and a call of few or short rows is little else: where the plan fits the arguments (up to about
// 90 rollouts) workgroup 0 of the rows' own launch writes it to the workspace, and the others read it
// from the arguments.  us per call, with a launch of its own / this: 60 rows of 1,000 logits 14.0 / 11.5, 416 rows
// of 8,000 17.8 / 15.2, 3,100 rows of 2,048 23.0 / 20.7, 12,000 rows of 16,000 150.1 / 147.7.
struct RowsLaunch {
  LogitsArgs a;
  SetupArgs setup;
  SetupBlob blob;
};
static_assert(sizeof(RowsLaunch) < 4096, "kernel arguments");
__device__ __forceinline__ DevicePlan plan_of(const RowsLaunch& l) {
  DevicePlan pl = l.a.pl;
  auto here = [&](const auto* q) {
    return (decltype(q))((const unsigned char*)l.blob.data + ((const unsigned char*)q - l.setup.plan));
  };
  pl.offsets = here(pl.offsets);
  pl.comp_off = here(pl.comp_off);
  pl.n = here(pl.n);
  pl.alpha_p = here(pl.alpha_p);
  return pl;
}

// The one-hot part of the sampled estimator: dz[y] = k (1 - p_s(y)), k = scale c_t, written
// over the -k p_s(y) the vector sweep stored there.
__device__ __forceinline__ void store_onehot(uint4* dzr, int y, float k, float zy_s, float lse_s) {
  const float v = k * (1.f - __expf(zy_s - lse_s));
  ((uint16_t*)dzr)[y] = (uint16_t)(pack_bf16(v, 0.f) & 0xffffu);
}

__device__ __forceinline__ void unpack8(const uint4& q, float (&f)[8]) {
  f[0] = bf16_lo(q.x); f[1] = bf16_hi(q.x);
  f[2] = bf16_lo(q.y); f[3] = bf16_hi(q.y);
  f[4] = bf16_lo(q.z); f[5] = bf16_hi(q.z);
  f[6] = bf16_lo(q.w); f[7] = bf16_hi(q.w);
}

// DIAG: also the teacher-side drift diagnostics of Sec. 3.1 for the row: entropy of the
// teacher distribution (H = lse_t - E_{p_t}[z_t]; the branching factor is exp(H)), the rank of
// y_t under the teacher (1 + number of entries with a strictly larger logit) and log p_t(y_t).
template <bool DIAG>
__global__ __launch_bounds__(kRowThreads) void logits_row_kernel(LogitsArgs a) {
  __shared__ float sh[7][kRowThreads / 64];
  __shared__ float bc[5];
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int nvec = a.V >> 3;
  const int i = last_le<int64_t>(a.pl.offsets, a.B + 1, t);
  const int64_t j = t - a.pl.offsets[i];
  uint4* dzr = a.dz ? a.dz + t * nvec : nullptr;
  if (j >= a.pl.n[i]) {   // outside the window: zero gradient row, zero KL
    if (dzr) {
      const uint4 z = {0u, 0u, 0u, 0u};
      for (int q = tid; q < nvec; q += kRowThreads) store16(dzr + q, z);
    }
    if (tid == 0) {
      if (a.kl) a.kl[t] = 0.f;
      if (a.c) a.c[t] = 0.f;
      if (DIAG) {
        if (a.t_logp) a.t_logp[t] = 0.f;
        if (a.t_entropy) a.t_entropy[t] = 0.f;
        if (a.t_rank) a.t_rank[t] = 0;
      }
    }
    return;
  }
  const uint4* zs = a.z_s + t * nvec;
  const uint4* zt = a.z_t + t * nvec;
  // sampled token and its teacher logit, for the rank
  int y = -1;
  float zy_rank = 0.f;
  if (DIAG && a.ids) {
    y = a.ids[t];
    if (y >= 0 && y < a.V) zy_rank = __uint_as_float((uint32_t)((const uint16_t*)zt)[y] << 16);
    else y = -1;
  }
  float Bt = 0.f;     // sum e^{z_t - m_t} z_t
  int cnt = 0;        // entries the teacher ranks strictly above y_t

  // ---- sweep 1: running max / sum-exp of both rows and A = sum e^{z_s-m}(z_s-z_t) ----
  float ms = kNegBig, Zs = 0.f, A = 0.f, mt = kNegBig, Zt = 0.f;
  for (int q = tid; q < nvec; q += kRowThreads) {
    const uint4 qs = zs[q], qt = zt[q];
    float s[8], u[8];
    unpack8(qs, s);
    unpack8(qt, u);
    float mx = s[0], mxt = u[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) { mx = fmaxf(mx, s[k]); mxt = fmaxf(mxt, u[k]); }
    if (mx > ms) {
      const float sc = fast_exp2((ms - mx) * kLog2e);
      Zs *= sc; A *= sc; ms = mx;
    }
    if (mxt > mt) {
      const float sc = fast_exp2((mt - mxt) * kLog2e);
      Zt *= sc; Bt *= sc; mt = mxt;
    }
    const float ms2 = ms * kLog2e, mt2 = mt * kLog2e;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float e = fast_exp2(fmaf(s[k], kLog2e, -ms2));
      Zs += e;
      A = fmaf(e, s[k] - u[k], A);
      const float et = fast_exp2(fmaf(u[k], kLog2e, -mt2));
      Zt += et;
      if (DIAG) {
        Bt = fmaf(et, u[k], Bt);
        cnt += (u[k] > zy_rank && q * 8 + k != y) ? 1 : 0;
      }
    }
  }
  // wave then block merge, fixed order
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    merge_mza(ms, Zs, A, __shfl_xor(ms, o, 64), __shfl_xor(Zs, o, 64), __shfl_xor(A, o, 64));
    if (DIAG) {
      merge_mza(mt, Zt, Bt, __shfl_xor(mt, o, 64), __shfl_xor(Zt, o, 64), __shfl_xor(Bt, o, 64));
      cnt += __shfl_xor(cnt, o, 64);
    } else {
      merge_mz(mt, Zt, __shfl_xor(mt, o, 64), __shfl_xor(Zt, o, 64));
    }
  }
  if (lane == 0) {
    sh[0][w] = ms; sh[1][w] = Zs; sh[2][w] = A; sh[3][w] = mt; sh[4][w] = Zt;
    if (DIAG) { sh[5][w] = Bt; sh[6][w] = __int_as_float(cnt); }
  }
  __syncthreads();
  if (tid == 0) {
    float m = sh[0][0], Z = sh[1][0], Aa = sh[2][0], m2 = sh[3][0], Z2 = sh[4][0];
    float B2 = DIAG ? sh[5][0] : 0.f;
    int rank = DIAG ? __float_as_int(sh[6][0]) : 0;
    for (int k = 1; k < kRowThreads / 64; ++k) {
      merge_mza(m, Z, Aa, sh[0][k], sh[1][k], sh[2][k]);
      if (DIAG) {
        merge_mza(m2, Z2, B2, sh[3][k], sh[4][k], sh[5][k]);
        rank += __float_as_int(sh[6][k]);
      } else {
        merge_mz(m2, Z2, sh[3][k], sh[4][k]);
      }
    }
    const float lse_s = m + logf(Z), lse_t = m2 + logf(Z2);
    const float mu = Aa / Z;                       // E_{p_s}[z_s - z_t]
    float kl = kl_from_sums(mu, m - m2, Z, Z2);
    float ent = DIAG ? lse_t - B2 / Z2 : 0.f;
    // a row without finite statistics is excluded: zeros in every output
    const bool dead = !(fabsf(lse_s) < 3.0e38f) || !(fabsf(lse_t) < 3.0e38f) || !(fabsf(kl) < 3.0e38f) ||
                      !(fabsf(mu) < 3.0e38f) || !(fabsf(ent) < 3.0e38f);
    float c = 0.f;
    uint32_t flag = dead ? ADWIN_DEV_NONFINITE : 0u;
    if (dead) { kl = 0.f; ent = 0.f; }
    if (a.ids && !dead) {
      const int y = a.ids[t];
      if (y >= 0 && y < a.V) {
        const uint16_t* ps = (const uint16_t*)zs;
        const uint16_t* pt = (const uint16_t*)zt;
        const float zy_s = __uint_as_float((uint32_t)ps[y] << 16);
        const float zy_t = __uint_as_float((uint32_t)pt[y] << 16);
        c = (zy_s - lse_s) - (zy_t - lse_t);
      } else {
        flag |= ADWIN_DEV_BAD_ID;
      }
    }
    if (flag && a.status) atomicOr(a.status, flag);
    if (a.kl) a.kl[t] = kl;
    if (a.c) a.c[t] = c;
    if (DIAG) {
      if (a.t_entropy) a.t_entropy[t] = ent;
      if (a.t_logp) a.t_logp[t] = (y >= 0 && !dead) ? zy_rank - lse_t : 0.f;
      if (a.t_rank) a.t_rank[t] = (y >= 0 && !dead) ? rank + 1 : 0;
    }
    a.klr[a.pl.comp_off[i] + j] = kl;
    bc[0] = lse_s * kLog2e;
    bc[1] = mu;
    bc[2] = c;
    bc[3] = lse_s;
    bc[4] = dead ? 1.f : 0.f;
  }
  __syncthreads();
  if (!dzr) return;
  if (bc[4] != 0.f) {
    const uint4 z = {0u, 0u, 0u, 0u};
    for (int q = tid; q < nvec; q += kRowThreads) store16(dzr + q, z);
    return;
  }
  // ---- sweep 2: dz = scale * p_s * ((z_s - z_t) - mu), or scale * c_t * (e_y - p_s) ---
  const float lse2 = bc[0];
  const float scale = a.grad_scale * a.pl.alpha_p[i];
  const float ca = a.sampled ? 0.f : 1.f, cb = a.sampled ? -bc[2] : -bc[1];
  for (int q = tid; q < nvec; q += kRowThreads) {
    const uint4 qs = zs[q], qt = zt[q];
    float s[8], u[8], d[8];
    unpack8(qs, s);
    unpack8(qt, u);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      d[k] = scale * fast_exp2(fmaf(s[k], kLog2e, -lse2)) * fmaf(s[k] - u[k], ca, cb);
    uint4 o;
    o.x = pack_bf16(d[0], d[1]);
    o.y = pack_bf16(d[2], d[3]);
    o.z = pack_bf16(d[4], d[5]);
    o.w = pack_bf16(d[6], d[7]);
    store16(dzr + q, o);
  }
  if (a.sampled) {
    __syncthreads();
    if (tid == 0 && a.ids) {
      const int yy = a.ids[t];
      if (yy >= 0 && yy < a.V)
        store_onehot(dzr, yy, scale * bc[2], __uint_as_float((uint32_t)((const uint16_t*)zs)[yy] << 16), bc[3]);
    }
  }
}

// ---------------------------------------------------------------------------------------
// Row-resident variant.  One 256-thread workgroup (one wave per SIMD, up to 512 registers
// per lane) per packed row keeps the whole row pair on chip between the two sweeps: z_s in
// registers, z_t partly in LDS and partly in registers, so HBM sees each logit once
// (4 B read + 2 B written per element).  Rows longer than kResVec vectors re-read the
// excess from memory.
// ---------------------------------------------------------------------------------------
constexpr int kResThreads = 256;
constexpr int kResIters = 75;                      // vectors of 8 logits per thread
constexpr int kResTLds = 39;                       // of which z_t vectors parked in LDS
constexpr int kResTReg = kResIters - kResTLds;     // and in registers
constexpr int kResBatch = 5;                       // iterations whose loads are issued together
constexpr int kResDepth = 1;                       // batches in flight ahead of the arithmetic (2 and 3: no faster)
constexpr int kResVec = kResIters * kResThreads;   // 19,200 vectors = 153,600 logits
constexpr int kResLdsBytes = kResTLds * kResThreads * 16 + 256;

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
// Calls f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop whose index
// is a compile-time constant, so that register arrays are never indexed dynamically.
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Row access through buffer descriptors: base = the row, extent = its bytes.  Every 16-byte
// load is then one instruction with a lane offset shared by all of them (16 * thread index)
// and a scalar offset per iteration (a store: one with their 32-bit sum), no 64-bit address per access to compute or to keep in
// vector registers (with 150 accesses per sweep those addresses, computed ahead by the
// compiler, crowded the row itself out of the register file); an access beyond the extent reads
// zeros / is dropped by the hardware, which is what the ragged last iteration needs.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* row, int bytes) {
  // flag word: the raw-buffer setting of the gfx9 family (32-bit data format, no swizzle)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), 0, bytes, 0x00020000);
}
// PAST: past the caches (non-temporal), see past_caches.
template <bool PAST = false>
__device__ __forceinline__ uint4 row_load16(__amdgpu_buffer_rsrc_t r, int lane_off, int iter_off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, iter_off, PAST ? 2 : 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}
// No scalar offset: the compiler puts two wait states between a 16-byte buffer store and an instruction that overwrites its
// data registers, but none if the store has one, and such stores of the sweep were seen to write the registers' next
// contents where two waves shared a SIMD.
template <bool PAST = false>
__device__ __forceinline__ void row_store16(__amdgpu_buffer_rsrc_t r, int lane_off, int iter_off, const uint4& v) {
  u32x4 x;
  x.x = v.x; x.y = v.y; x.z = v.z; x.w = v.w;
  __builtin_amdgcn_raw_buffer_store_b128(x, r, lane_off + iter_off, 0, PAST ? 2 : 0);
}

// Bt = sum e^{z_t - m_t} z_t and cnt = entries above zy, the teacher's logit of y_t: diagnostics only.
struct RowStats { float ms, Zs, A, mt, Zt, Bt; int cnt; };

__device__ __forceinline__ float max8(const float (&v)[8]) {
  return fmaxf(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7])));
}

// DIAG: the eight terms of a vector are summed by themselves first.  A thread adds up 600 logits of a row
// of 151,936, and as one chain the teacher entropy of such rows was 1.9 times as far from 64 bits as the
// streaming kernel's, whose 512 threads add up 300 (KL_t 1.3 times).
template <bool DIAG>
__device__ __forceinline__ void stats_update(RowStats& r, const uint4& qs, const uint4& qt, float zy, bool in) {
  float s[8], u[8];
  unpack8(qs, s);
  unpack8(qt, u);
  const float mx = max8(s), mxt = max8(u);
  if (mx > r.ms) {
    const float sc = fast_exp2((r.ms - mx) * kLog2e);
    r.Zs *= sc; r.A *= sc; r.ms = mx;
  }
  if (mxt > r.mt) {
    const float sc = fast_exp2((r.mt - mxt) * kLog2e);
    r.Zt *= sc;
    if (DIAG) r.Bt *= sc;
    r.mt = mxt;
  }
  const float ms2 = r.ms * kLog2e, mt2 = r.mt * kLog2e;
  float Zs = DIAG ? 0.f : r.Zs, A = DIAG ? 0.f : r.A, Zt = DIAG ? 0.f : r.Zt, Bt = 0.f;
  int above = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float e = fast_exp2(fmaf(s[k], kLog2e, -ms2));
    Zs += e;
    A = fmaf(e, s[k] - u[k], A);
    const float et = fast_exp2(fmaf(u[k], kLog2e, -mt2));
    Zt += et;
    if (DIAG) {
      Bt = fmaf(et, u[k], Bt);
      above += u[k] > zy ? 1 : 0;           // y_t itself is not above itself
    }
  }
  r.Zs = DIAG ? r.Zs + Zs : Zs;
  r.A = DIAG ? r.A + A : A;
  r.Zt = DIAG ? r.Zt + Zt : Zt;
  if (DIAG) {
    r.Bt += Bt;
    r.cnt += in ? above : 0;
  }
}

// dz = sgn * 2^(z_s*log2e - lse2s) * ((z_s - z_t) - mu), with |scale| folded into lse2s
__device__ __forceinline__ uint4 dz_vector(const uint4& qs, const uint4& qt, float lse2s, float sgn,
                                           float neg_sgn_mu) {
  float s[8], u[8], d[8];
  unpack8(qs, s);
  unpack8(qt, u);
#pragma unroll
  for (int k = 0; k < 8; ++k)
    d[k] = fast_exp2(fmaf(s[k], kLog2e, -lse2s)) * fmaf(s[k] - u[k], sgn, neg_sgn_mu);
  uint4 o;
  o.x = pack_bf16(d[0], d[1]);
  o.y = pack_bf16(d[2], d[3]);
  o.z = pack_bf16(d[4], d[5]);
  o.w = pack_bf16(d[6], d[7]);
  return o;
}

template <bool DIAG, bool PAST>
__global__ __launch_bounds__(kResThreads, 1) void logits_row_resident_kernel(LogitsArgs a) {
  extern __shared__ __align__(16) char lds_raw[];
  uint4* lds_t = (uint4*)lds_raw;
  float* sh = (float*)(lds_raw + kResTLds * kResThreads * 16);   // [7][4] + broadcast [5]
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int nvec = a.V >> 3;
  const int i = last_le<int64_t>(a.pl.offsets, a.B + 1, t);
  const int64_t j = t - a.pl.offsets[i];
  uint4* dzr = a.dz ? a.dz + t * nvec : nullptr;
  if (j >= a.pl.n[i]) {
    if (dzr) {
      const uint4 z = {0u, 0u, 0u, 0u};
      for (int q = tid; q < nvec; q += kResThreads) store16(dzr + q, z);
    }
    if (tid == 0) {
      if (a.kl) a.kl[t] = 0.f;
      if (a.c) a.c[t] = 0.f;
      if (DIAG) {
        if (a.t_logp) a.t_logp[t] = 0.f;
        if (a.t_entropy) a.t_entropy[t] = 0.f;
        if (a.t_rank) a.t_rank[t] = 0;
      }
    }
    return;
  }
  const uint4* zs = a.z_s + t * nvec;
  const uint4* zt = a.z_t + t * nvec;
  // bf16 -3.39e38 in every lane: neutral for max, exp and the difference
  const uint4 neutral = {0xff7fff7fu, 0xff7fff7fu, 0xff7fff7fu, 0xff7fff7fu};

  uint4 rs[kResIters];
  uint4 rt[kResTReg];
  RowStats st = {kNegBig, 0.f, 0.f, kNegBig, 0.f, 0.f, 0};
  float zy_rank = 0.f;            // teacher logit of the sampled token, for the rank
  if (DIAG && a.ids) {
    const int y = a.ids[t];
    if (y >= 0 && y < a.V) zy_rank = __uint_as_float((uint32_t)((const uint16_t*)zt)[y] << 16);
  }
  // ---- sweep 1: load the row pair once, keep it, accumulate the statistics ------------
  // Loads are issued kResDepth batches (of kResBatch iterations) ahead of the arithmetic, so
  // that the single wave per SIMD always has 2 * kResBatch 16-byte loads in flight per lane.
  // z_s vectors and the register-resident z_t vectors land in their final registers (the
  // loads write accumulation registers directly); the z_t vectors that go to the LDS pass
  // through a small staging ring.  Lanes beyond the row read zeros and take a neutral value.
  const int row_bytes = nvec * 16, lane_off = tid * 16;
  const __amdgpu_buffer_rsrc_t bs = row_rsrc(zs, row_bytes), bt = row_rsrc(zt, row_bytes);
  uint4 tb[kResDepth + 1][kResBatch];
  auto issue = [&](auto b_c) {
    constexpr int b = decltype(b_c)::value;
    if constexpr (b < kResIters / kResBatch) {
      static_for<kResBatch>([&](auto g_c) {
        constexpr int g = decltype(g_c)::value;
        constexpr int it = b * kResBatch + g;
        rs[it] = row_load16<PAST>(bs, lane_off, it * kResThreads * 16);
        if constexpr (it < kResTLds) tb[b % (kResDepth + 1)][g] = row_load16<PAST>(bt, lane_off, it * kResThreads * 16);
        else rt[it - kResTLds] = row_load16<PAST>(bt, lane_off, it * kResThreads * 16);
      });
    }
  };
  static_for<kResDepth>([&](auto b_c) { issue(b_c); });
  static_for<kResIters / kResBatch>([&](auto b_c) {
    constexpr int b = decltype(b_c)::value;
    issue(std::integral_constant<int, b + kResDepth>{});
    if (b * kResBatch * kResThreads < nvec) {
      static_for<kResBatch>([&](auto g_c) {
        constexpr int g = decltype(g_c)::value;
        constexpr int it = b * kResBatch + g;
        const bool in = it * kResThreads + tid < nvec;
        uint4 qs = rs[it], qt;
        if constexpr (it < kResTLds) qt = tb[b % (kResDepth + 1)][g]; else qt = rt[it - kResTLds];
        if (!in) { qs = neutral; qt = neutral; }
        if constexpr (it < kResTLds) lds_t[it * kResThreads + tid] = qt;
        stats_update<DIAG>(st, qs, qt, zy_rank, in);
      });
    }
  });
  for (int q = kResVec + tid; q < nvec; q += kResThreads) stats_update<DIAG>(st, zs[q], zt[q], zy_rank, true);
  float Zs = st.Zs, As = st.A, Zt = st.Zt;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    merge_mza(st.ms, Zs, As, __shfl_xor(st.ms, o, 64), __shfl_xor(Zs, o, 64), __shfl_xor(As, o, 64));
    if (DIAG) {
      merge_mza(st.mt, Zt, st.Bt, __shfl_xor(st.mt, o, 64), __shfl_xor(Zt, o, 64), __shfl_xor(st.Bt, o, 64));
      st.cnt += __shfl_xor(st.cnt, o, 64);
    } else {
      merge_mz(st.mt, Zt, __shfl_xor(st.mt, o, 64), __shfl_xor(Zt, o, 64));
    }
  }
  if (lane == 0) { sh[0 + w] = st.ms; sh[4 + w] = Zs; sh[8 + w] = As; sh[12 + w] = st.mt; sh[16 + w] = Zt; }
  if (DIAG && lane == 0) { sh[20 + w] = st.Bt; sh[24 + w] = __int_as_float(st.cnt); }
  __syncthreads();
  if (tid == 0) {
    float m = sh[0], Z = sh[4], Aa = sh[8], m2 = sh[12], Z2 = sh[16];
    float B2 = DIAG ? sh[20] : 0.f;
    int rank = DIAG ? __float_as_int(sh[24]) : 0;
    for (int k = 1; k < kResThreads / 64; ++k) {
      merge_mza(m, Z, Aa, sh[k], sh[4 + k], sh[8 + k]);
      if (DIAG) {
        merge_mza(m2, Z2, B2, sh[12 + k], sh[16 + k], sh[20 + k]);
        rank += __float_as_int(sh[24 + k]);
      } else {
        merge_mz(m2, Z2, sh[12 + k], sh[16 + k]);
      }
    }
    const float lse_s = m + logf(Z), lse_t = m2 + logf(Z2);
    const float mu = Aa / Z;                       // E_{p_s}[z_s - z_t]
    float kl = kl_from_sums(mu, m - m2, Z, Z2);
    float ent = DIAG ? lse_t - B2 / Z2 : 0.f;
    // a row without finite statistics is excluded: zeros in every output
    const bool dead = !(fabsf(lse_s) < 3.0e38f) || !(fabsf(lse_t) < 3.0e38f) || !(fabsf(kl) < 3.0e38f) ||
                      !(fabsf(mu) < 3.0e38f) || !(fabsf(ent) < 3.0e38f);
    float c = 0.f, logp_t = 0.f;
    bool have_y = false;
    uint32_t flag = dead ? ADWIN_DEV_NONFINITE : 0u;
    if (dead) { kl = 0.f; ent = 0.f; }
    if (a.ids && !dead) {
      const int y = a.ids[t];
      if (y >= 0 && y < a.V) {
        const float zy_s = __uint_as_float((uint32_t)((const uint16_t*)zs)[y] << 16);
        const float zy_t = __uint_as_float((uint32_t)((const uint16_t*)zt)[y] << 16);
        c = (zy_s - lse_s) - (zy_t - lse_t);
        logp_t = zy_t - lse_t;
        have_y = true;
      } else {
        flag |= ADWIN_DEV_BAD_ID;
      }
    }
    if (flag && a.status) atomicOr(a.status, flag);
    if (a.kl) a.kl[t] = kl;
    if (a.c) a.c[t] = c;
    if (DIAG) {
      if (a.t_entropy) a.t_entropy[t] = ent;
      if (a.t_logp) a.t_logp[t] = logp_t;
      if (a.t_rank) a.t_rank[t] = have_y ? rank + 1 : 0;
    }
    a.klr[a.pl.comp_off[i] + j] = kl;
    sh[28] = lse_s * kLog2e;
    sh[29] = mu;
    sh[30] = c;
    sh[31] = lse_s;
    sh[32] = dead ? 1.f : 0.f;
  }
  __syncthreads();
  if (!dzr) return;
  if (sh[32] != 0.f) {
    const uint4 z = {0u, 0u, 0u, 0u};
    for (int q = tid; q < nvec; q += kResThreads) store16(dzr + q, z);
    return;
  }
  // ---- sweep 2: dz from the resident copy ----------------------------------------------
  // expected: scale p_s ((z_s - z_t) - mu); sampled: -k p_s with k = scale c_t (the one-hot
  // term follows); |scale| resp. |k| is folded into the exponent, the sign into the factor
  const float scale = a.grad_scale * a.pl.alpha_p[i];
  const float k_s = a.sampled ? scale * sh[30] : scale;
  const float sg = k_s < 0.f ? -1.f : 1.f;
  const float sgn = a.sampled ? 0.f : sg;
  const float lse2 = sh[28] - log2f(fabsf(k_s)), nmu = a.sampled ? -sg : -sg * sh[29];
  const __amdgpu_buffer_rsrc_t bd = row_rsrc(dzr, row_bytes);
  static_for<kResIters>([&](auto it_c) {
    constexpr int it = decltype(it_c)::value;
    if (it * kResThreads < nvec) {
      uint4 qt;
      if constexpr (it < kResTLds) qt = lds_t[it * kResThreads + tid]; else qt = rt[it - kResTLds];
      row_store16<PAST>(bd, lane_off, it * kResThreads * 16, dz_vector(rs[it], qt, lse2, sgn, nmu));
    }
  });
  for (int q = kResVec + tid; q < nvec; q += kResThreads)
    store16(dzr + q, dz_vector(zs[q], zt[q], lse2, sgn, nmu));
  if (a.sampled) {
    __syncthreads();
    if (tid == 0 && a.ids) {
      const int yy = a.ids[t];
      if (yy >= 0 && yy < a.V)
        store_onehot(dzr, yy, k_s, __uint_as_float((uint32_t)((const uint16_t*)zs)[yy] << 16), sh[31]);
    }
  }
}

// ---------------------------------------------------------------------------------------
// Rows of up to 80 logits per thread, in registers alone: THREADS threads (64: a wave per row, four
// rows to a workgroup) load the whole row pair at once and keep it until dz is written, so HBM
// sees each logit once (6 B per element) and, at 4 waves per SIMD, one workgroup's reduction and
// stores run under the loads of others.  Memory bound: what counts is bytes in flight.  The
// kernel for long rows has 75 such vectors per thread, one workgroup per compute unit and most of
// its iterations empty on a shorter row; the streaming kernel reads the rows twice.
// Train call, us, long-row kernel / streaming / this one: V = 2,048 (25,600 of 32,768 rows)
// 942 / 158 / 97; V = 8,192 (16,384 rows) 522 / 166 / 150; V = 32,776 (3,584) 220 / 165 / 132 and
// with diagnostics - / 172 / 141; V = 65,536 (2,048) 193 / 209 / 172; V = 81,920 (1,536) 173 / 212 / 159.
// ---------------------------------------------------------------------------------------
constexpr int kShortIters = 10;
constexpr int short_row_limit(int threads) { return threads * kShortIters * 8; }

// What a launch does with its rows: all of it, or the two halves of a split row.  A row beyond the
// limit has a whole compute unit in the long-row kernel, 50 us however few rows there are.  A
// call of few such rows cuts each into pieces (<= 20,480 logits, 256 threads): one launch leaves the
// sums of every piece, the next combines them in piece order and writes dz, its second read of
// the logits coming from the caches.
constexpr int kWhole = 0, kPieceSums = 1, kPieceGrad = 2;

// A row's results from its sums.
struct RowResult { float lse_s, lse_t, mu, kl, ent; bool dead; };
template <bool DIAG>
__device__ __forceinline__ RowResult row_result(float ms, float Zs, float A, float mt, float Zt, float Bt) {
  RowResult r;
  r.lse_s = ms + logf(Zs);
  r.lse_t = mt + logf(Zt);
  r.mu = A / Zs;                       // E_{p_s}[z_s - z_t]
  r.kl = kl_from_sums(r.mu, ms - mt, Zs, Zt);
  r.ent = DIAG ? r.lse_t - Bt / Zt : 0.f;
  // a row without finite statistics is excluded: zeros in every output
  r.dead = !(fabsf(r.lse_s) < 3.0e38f) || !(fabsf(r.lse_t) < 3.0e38f) || !(fabsf(r.kl) < 3.0e38f) ||
           !(fabsf(r.mu) < 3.0e38f) || !(fabsf(r.ent) < 3.0e38f);
  if (r.dead) { r.kl = 0.f; r.ent = 0.f; }
  return r;
}

template <bool DIAG>
__device__ __forceinline__ void fold_sums(float& ms, float& Zs, float& A, float& mt, float& Zt, float& Bt, int& cnt, int o) {
  merge_mza(ms, Zs, A, __shfl_xor(ms, o, 64), __shfl_xor(Zs, o, 64), __shfl_xor(A, o, 64));
  if (DIAG) {
    merge_mza(mt, Zt, Bt, __shfl_xor(mt, o, 64), __shfl_xor(Zt, o, 64), __shfl_xor(Bt, o, 64));
    cnt += __shfl_xor(cnt, o, 64);
  } else {
    merge_mz(mt, Zt, __shfl_xor(mt, o, 64), __shfl_xor(Zt, o, 64));
  }
}

template <int THREADS, bool DIAG, int PHASE>
__device__ __forceinline__ void short_rows(const LogitsArgs& a, const DevicePlan& pl, unsigned block) {
  constexpr int kRows = THREADS == 64 ? 4 : 1, kWaves = THREADS / 64;
  static_assert(PHASE == kWhole || kRows == 1, "a piece is a workgroup's");
  __shared__ float sh[7][kWaves];
  const int lid = kRows > 1 ? threadIdx.x & 63 : threadIdx.x, lane = threadIdx.x & 63;
  // pieces come first, a workgroup each; kPieceSums has the T packed rows behind them, of which
  // those outside the windows are cleared
  const int64_t n_pieces = PHASE == kWhole ? 0 : a.n_adm * a.splits;
  const bool is_piece = PHASE != kWhole && (int64_t)block < n_pieces;
  int64_t t = kRows > 1 ? (int64_t)block * kRows + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)
                        : (int64_t)block - (is_piece ? 0 : n_pieces);
  if (t >= a.T && !is_piece) return;
  const int row_vec = a.V >> 3;
  int i, piece = 0, q0 = 0, nvec = row_vec;       // the vectors [q0, q0 + nvec) of the row
  int64_t j;
  if (is_piece) {
    const int64_t r = t / a.splits;               // the r-th admitted row
    piece = (int)(t % a.splits);
    i = wave_last_le(pl.comp_off, a.B + 1, r);
    j = r - pl.comp_off[i];
    t = pl.offsets[i] + j;
    q0 = (int)((int64_t)row_vec * piece / a.splits);
    nvec = (int)((int64_t)row_vec * (piece + 1) / a.splits) - q0;
  } else {
    i = wave_last_le(pl.offsets, a.B + 1, t);
    j = t - pl.offsets[i];
  }
  const int row_bytes = nvec * 16, lane_off = lid * 16;
  const __amdgpu_buffer_rsrc_t bd = row_rsrc(a.dz ? a.dz + t * row_vec + q0 : nullptr, a.dz ? row_bytes : 0);
  auto clear_row = [&]() {
    const uint4 z = {0u, 0u, 0u, 0u};
    for (int it = 0; it * THREADS < nvec; ++it) row_store16(bd, lane_off, it * THREADS * 16, z);
  };
  if (j >= pl.n[i]) {   // outside the window: zero gradient row, zero KL
    if (a.dz) clear_row();
    if (lid == 0) {
      if (a.kl) a.kl[t] = 0.f;
      if (a.c) a.c[t] = 0.f;
      if (DIAG) {
        if (a.t_logp) a.t_logp[t] = 0.f;
        if (a.t_entropy) a.t_entropy[t] = 0.f;
        if (a.t_rank) a.t_rank[t] = 0;
      }
    }
    return;
  }
  if (PHASE != kWhole && !is_piece) return;
  const uint4* zs = a.z_s + t * row_vec;
  const uint4* zt = a.z_t + t * row_vec;
  const __amdgpu_buffer_rsrc_t bs = row_rsrc(zs + q0, row_bytes), bt = row_rsrc(zt + q0, row_bytes);
  uint4 rs[kShortIters], rt[kShortIters];
  static_for<kShortIters>([&](auto it_c) {
    constexpr int it = decltype(it_c)::value;
    rs[it] = row_load16(bs, lane_off, it * THREADS * 16);      // zeros beyond the row
    rt[it] = row_load16(bt, lane_off, it * THREADS * 16);
  });
  int y = a.ids ? a.ids[t] : -1;
  const bool has_y = y >= 0 && y < a.V;
  if (!has_y) y = -1;
  float zy_s = 0.f, zy_t = 0.f;
  if (PHASE != kPieceGrad && has_y) {
    zy_s = __uint_as_float((uint32_t)((const uint16_t*)zs)[y] << 16);
    zy_t = __uint_as_float((uint32_t)((const uint16_t*)zt)[y] << 16);
  }
  // ---- statistics: the thread's maxima first, then its sums relative to them -------------
  float ms = kNegBig, mt = kNegBig, Zs = 0.f, A = 0.f, Zt = 0.f, Bt = 0.f;
  int cnt = 0;            // entries the teacher ranks strictly above y_t
  if constexpr (PHASE != kPieceGrad) static_for<kShortIters>([&](auto it_c) {
    constexpr int it = decltype(it_c)::value;
    if (it * THREADS + lid < nvec) {
      float s[8], u[8];
      unpack8(rs[it], s);
      unpack8(rt[it], u);
      ms = fmaxf(ms, max8(s));
      mt = fmaxf(mt, max8(u));
    }
  });
  const float ms2 = ms * kLog2e, mt2 = mt * kLog2e;
  if constexpr (PHASE != kPieceGrad) static_for<kShortIters>([&](auto it_c) {
    constexpr int it = decltype(it_c)::value;
    // unpacked again: kept from the maxima, the halves of all vectors are 80 registers more, and spilled
    asm volatile("" : "+v"(rs[it].x), "+v"(rs[it].y), "+v"(rs[it].z), "+v"(rs[it].w));
    asm volatile("" : "+v"(rt[it].x), "+v"(rt[it].y), "+v"(rt[it].z), "+v"(rt[it].w));
    if (it * THREADS + lid < nvec) {
      float s[8], u[8];
      unpack8(rs[it], s);
      unpack8(rt[it], u);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float e = fast_exp2(fmaf(s[k], kLog2e, -ms2));
        Zs += e;
        A = fmaf(e, s[k] - u[k], A);
        const float et = fast_exp2(fmaf(u[k], kLog2e, -mt2));
        Zt += et;
        if (DIAG) {
          Bt = fmaf(et, u[k], Bt);
          cnt += u[k] > zy_t ? 1 : 0;       // y_t itself is not above itself
        }
      }
    }
  });
  auto fold = [&](int o) __attribute__((always_inline)) { fold_sums<DIAG>(ms, Zs, A, mt, Zt, Bt, cnt, o); };
  float* part = PHASE == kWhole ? nullptr : a.part + (pl.comp_off[i] + j) * a.splits * 8;   // of the row's pieces
  if constexpr (PHASE == kPieceGrad) {
    // up to 64 pieces, one per lane; lanes without one hold the neutral element
    uint32_t zy = 0u;
    if (lane < a.splits) {
      const float4 x = *(const float4*)(part + lane * 8), x2 = *(const float4*)(part + lane * 8 + 4);
      ms = x.x; Zs = x.y; A = x.z; mt = x.w; Zt = x2.x; Bt = x2.y; cnt = __float_as_int(x2.z);
      zy = __float_as_uint(x2.w);
    }
    zy = (uint32_t)__shfl((int)zy, 0, 64);        // the token's logits, from piece 0
    zy_s = bf16_lo(zy); zy_t = bf16_hi(zy);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) fold(o);
  if constexpr (kWaves > 1 && PHASE != kPieceGrad) {
    if (lane == 0) {
      const int w = threadIdx.x >> 6;
      sh[0][w] = ms; sh[1][w] = Zs; sh[2][w] = A; sh[3][w] = mt; sh[4][w] = Zt;
      if (DIAG) { sh[5][w] = Bt; sh[6][w] = __int_as_float(cnt); }
    }
    __syncthreads();
    const int w = lane & (kWaves - 1);
    ms = sh[0][w]; Zs = sh[1][w]; A = sh[2][w]; mt = sh[3][w]; Zt = sh[4][w];
    if (DIAG) { Bt = sh[5][w]; cnt = __float_as_int(sh[6][w]); }
#pragma unroll
    for (int o = kWaves / 2; o > 0; o >>= 1) fold(o);
  }
  if constexpr (PHASE == kPieceSums) {
    if (lid == 0) {
      *(float4*)(part + piece * 8) = make_float4(ms, Zs, A, mt);
      // the token's two logits go along (exact: they are bf16): the launch that writes dz must not
      // read them from the rows, of which another piece's workgroup may hold dz by then (dz in place)
      const uint32_t zy = (__float_as_uint(zy_s) >> 16) | (__float_as_uint(zy_t) & 0xffff0000u);
      *(float4*)(part + piece * 8 + 4) = make_float4(Zt, Bt, __int_as_float(cnt), __uint_as_float(zy));
    }
    return;
  }
  // every thread has the row's sums
  const RowResult res = row_result<DIAG>(ms, Zs, A, mt, Zt, Bt);
  const float lse_s = res.lse_s, lse_t = res.lse_t, mu = res.mu, kl = res.kl, ent = res.ent;
  const bool dead = res.dead;
  const float c = has_y && !dead ? (zy_s - lse_s) - (zy_t - lse_t) : 0.f;
  if (lid == 0 && piece == 0) {
    const uint32_t flag = dead ? ADWIN_DEV_NONFINITE : (a.ids && !has_y ? ADWIN_DEV_BAD_ID : 0u);
    if (flag && a.status) atomicOr(a.status, flag);
    if (a.kl) a.kl[t] = kl;
    if (a.c) a.c[t] = c;
    if (DIAG) {
      if (a.t_entropy) a.t_entropy[t] = ent;
      if (a.t_logp) a.t_logp[t] = has_y && !dead ? zy_t - lse_t : 0.f;
      if (a.t_rank) a.t_rank[t] = has_y && !dead ? cnt + 1 : 0;
    }
    if (PHASE == kWhole || !a.tail_has_kl) a.klr[pl.comp_off[i] + j] = dead && a.mark ? __uint_as_float(kExcludedRow) : kl;
  }
  if (!a.dz) return;
  if (dead) return clear_row();
  // ---- dz from the registers (see logits_row_resident_kernel) ------------------------------
  const float scale = a.grad_scale * pl.alpha_p[i];
  const float k_s = a.sampled ? scale * c : scale;
  const float sg = k_s < 0.f ? -1.f : 1.f;
  const float sgn = a.sampled ? 0.f : sg;
  const float lse2 = lse_s * kLog2e - log2f(fabsf(k_s)), nmu = a.sampled ? -sg : -sg * mu;
  const bool onehot = a.sampled && has_y;
  const uint32_t vy = pack_bf16(k_s * (1.f - __expf(zy_s - lse_s)), 0.f) & 0xffffu;
  static_for<kShortIters>([&](auto it_c) {
    constexpr int it = decltype(it_c)::value;
    if (it * THREADS < nvec) {
      uint4 o = dz_vector(rs[it], rt[it], lse2, sgn, nmu);
      if (onehot && q0 + it * THREADS + lid == (y >> 3)) {      // the one-hot term: k (1 - p_s(y))
        const int word = (y >> 1) & 3;
        auto put = [&](uint32_t x) { return (y & 1) ? (x & 0xffffu) | (vy << 16) : (x & 0xffff0000u) | vy; };
        o.x = word == 0 ? put(o.x) : o.x;
        o.y = word == 1 ? put(o.y) : o.y;
        o.z = word == 2 ? put(o.z) : o.z;
        o.w = word == 3 ? put(o.w) : o.w;
      }
      row_store16(bd, lane_off, it * THREADS * 16, o);
    }
  });
}

// Workgroups in front of a launch's pieces, a multiple of the dies: workgroups go to them in turn, and a piece whose
// second launch is on the die of its first finds its logits in that die's L2 (120 rows of 120,000 logits
// in two pieces each, the second launch: 11.0 us, one workgroup further 13.2).
__host__ __device__ constexpr unsigned lead_blocks(unsigned n) { return (n + 7) / 8 * 8; }

template <int THREADS, bool DIAG, int PHASE = kWhole>
__global__ __launch_bounds__(THREADS < 256 ? 256 : THREADS, THREADS < 1024 ? 4 : 1)
void logits_row_short_kernel(LogitsArgs a) {
  short_rows<THREADS, DIAG, PHASE>(a, a.pl, blockIdx.x);
}
template <int THREADS, bool DIAG, int PHASE = kWhole>
__global__ __launch_bounds__(THREADS < 256 ? 256 : THREADS, THREADS < 1024 ? 4 : 1)
void logits_row_short_setup_kernel(RowsLaunch l) {
  if (blockIdx.x == 0)
    return setup_body(l.setup, &l.blob, (const unsigned char*)l.blob.data, 0, 1, THREADS < 256 ? 256 : THREADS);
  if (PHASE != kWhole && blockIdx.x < lead_blocks(1)) return;
  short_rows<THREADS, DIAG, PHASE>(l.a, plan_of(l), blockIdx.x - (PHASE == kWhole ? 1 : lead_blocks(1)));
}

// KL_t of rollout i's rows from the sums of their pieces, with the same merges as the workgroups that write dz:
// LANES (16 up to 16 pieces, or 64) to a row, the next row's sums on their way.
template <bool DIAG, int LANES>
__device__ __forceinline__ void rollout_kl(const LogitsArgs& a, int i) {
  const int64_t r0 = a.pl.comp_off[i];
  const int n = a.pl.n[i], g = threadIdx.x & (LANES - 1);
  constexpr int kRows = 256 / LANES;
  const float4 none = make_float4(kNegBig, 0.f, 0.f, kNegBig), none2 = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 x = none, x2 = none2;
  auto load = [&](int j) {
    if (g < a.splits && j < n) {
      const float* q = a.part + ((r0 + j) * a.splits + g) * 8;
      x = *(const float4*)q;
      x2 = *(const float4*)(q + 4);
    }
  };
  load(threadIdx.x / LANES);
  for (int first = 0; first < n; first += kRows) {
    const int j = first + threadIdx.x / LANES;
    float ms = x.x, Zs = x.y, A = x.z, mt = x.w, Zt = x2.x, Bt = x2.y;
    int cnt = 0;
    load(j + kRows);
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) fold_sums<DIAG>(ms, Zs, A, mt, Zt, Bt, cnt, o);
    const RowResult r = row_result<DIAG>(ms, Zs, A, mt, Zt, Bt);
    if (g == 0 && j < n) a.klr[r0 + j] = r.kl;
  }
  __syncthreads();
}

// The second launch of a call of split rows without summaries: its first workgroups end the call
// (tail_device.h), which then has two launches instead of four.  They need only KL_t, which they take from the
// sums of the pieces themselves instead of waiting for the workgroups that write dz.  us per call, four launches /
// two: V = 151,936, 29 rows 22.6 / 16.0, 8 rollouts of 10 to 30 rows 45.5 / 36.2; V = 100,000, 117 rows 24.5 / 17.4.
template <bool DIAG>
__global__ __launch_bounds__(256, 4) void logits_piece_grad_kernel(LogitsArgs a, TailArgs tail) {
  if ((int)blockIdx.x < tail.blocks) {
    __shared__ double sh[16];
    __shared__ int sh_first[4];
    if (a.splits <= 16) rollout_kl<DIAG, 16>(a, blockIdx.x);
    else rollout_kl<DIAG, 64>(a, blockIdx.x);
    return tail_body<false>(tail, blockIdx.x, sh, sh_first);
  }
  const unsigned lead = lead_blocks((unsigned)tail.blocks);
  if (blockIdx.x >= lead) short_rows<256, DIAG, kPieceGrad>(a, a.pl, blockIdx.x - lead);
}

// `blocks` workgroups of rows; with a plan in the arguments, and the one that sets up.
template <int THREADS, bool DIAG, int PHASE = kWhole>
static hipError_t launch_rows(const RowsLaunch& l, unsigned blocks, hipStream_t st) {
  constexpr int kThreads = THREADS < 256 ? 256 : THREADS;
  if (l.blob.n16) logits_row_short_setup_kernel<THREADS, DIAG, PHASE><<<blocks + (PHASE == kWhole ? 1 : lead_blocks(1)), kThreads, 0, st>>>(l);
  else logits_row_short_kernel<THREADS, DIAG, PHASE><<<blocks, kThreads, 0, st>>>(l.a);
  return hipGetLastError();
}

template <bool DIAG>
static hipError_t launch_short_rows(const RowsLaunch& l, hipStream_t st) {
  const unsigned T = (unsigned)l.a.T;
  if (l.a.V <= short_row_limit(64)) return launch_rows<64, DIAG>(l, (T + 3) / 4, st);
  if (l.a.V <= short_row_limit(256)) return launch_rows<256, DIAG>(l, T, st);
  if (l.a.V <= short_row_limit(512)) return launch_rows<512, DIAG>(l, T, st);
  return launch_rows<1024, DIAG>(l, T, st);
}

// Whether the long-row kernel reads the logits and writes dz past the caches: each of these arrays, T x V, is beyond the
// last-level cache of 256 MiB, so it is in memory again before anybody can find it there, and its lines displace those that
// other workgroups are about to complete.  us per call, kept / past: V = 151,936: 2,615 of 3,901 rows 624 / 581, with diagnostics
// 2,321 of 3,877 642 / 567, 6,505 of 9,708 1678 / 1426, 20,000 rows 4171 / 3787; V = 100,032: 911 / 861; few of the rows
// admitted, V = 151,936, 450 of 4,000 345 / 327; no dz, 1,110 rows 159 / 145.  The line was drawn by rows that are whole lines of
// an array that begins one.  Where the array begins is no part of it: the rule also decides which kernel serves calls with
// diagnostics, and the same logits give the same bits wherever they lie.  (16 bytes into a line: 1,110 rows 272 / 239,
// 20,000 rows 4117 / 3935, V = 82,048, 2,050 rows with diagnostics 333 / 275.)  Short rows, four waves to a SIMD, gain 0 to 2 % by it,
// dz alone, and lose up to 5 % with the logits.
static bool past_caches(int64_t T, int V) { return 2 * T * V > ((int64_t)320 << 20) && V % 64 == 0; }

// Whether a call with diagnostics takes the streaming kernel under ADWIN_LOGITS_AUTO.
// Diagnostics add arithmetic, which a workgroup that holds a row of more than 40,960 logits and has its
// compute unit to itself (1024 threads, or the long-row kernel's 256) hides less well than the streaming
// kernel's two workgroups; what that costs in return is the second read of the rows, which comes from
// the last-level cache while the row pairs of the call fit its 256 MiB.  us, row on chip / streaming, on
// both sides of that line: V = 90,000: 700 rows 131 / 121, 768 rows 131 / 144; V = 102,400: 600 rows
// 135 / 118, 700 rows 140 / 147; V = 136,000: 480 rows 128 / 125, 512 rows 132 / 143; V = 151,936: 400 rows
// 130 / 121, 480 rows 139 / 157.  The line of the 1024-thread kernel lies a
// little lower, and the two draw level as a row fills its registers: V = 60,000: 600 rows 77 / 68, 1,024
// rows 112 / 112; V = 65,536: 513 rows 72 / 65, 1,024 rows 122 / 130; V = 73,728: 512 rows 67 / 68.  Up to 256 rows
// each has a compute unit either way: V = 50,000: 256 rows 36 / 38; V = 122,880: 200 rows 61 / 59, 256 rows
// 65 / 66; V = 151,936: 200 rows 70 / 70, 256 rows 73 / 77.  A few rows more than two rounds cost a row on
// chip a third: V = 73,728: 513 rows 76 / 70; V = 131,072: 169 / 147; V = 176,000: 541 rows 238 / 227;
// V = 151,936: 520 rows 186 / 193.
// A kernel whose registers are half empty loses whatever the number of rows (V = 42,000: 16,384 rows
// 1066 / 988; V = 50,000: 700 rows 76 / 66, 2,048 rows 184 / 187, 8,192 rows 623 / 619; V = 81,928: 1,352 rows
// 230 / 227), and so does the long-row kernel far beyond the 153,600 logits that stay on chip, where it
// reads twice as well (V = 176,000: 1,024 rows 327 / 367; V = 200,000: 447 / 415; V = 262,144: 682 / 531).
// Past the caches (`past`) the long-row kernel is up to a sixth faster than that: V = 82,048: 3,542 rows 498 / 609, 15,847 rows
// 2000 / 2460; V = 86,016: 505 / 637; V = 102,400: 2,914 rows 452 / 633; V = 196,608: 2,346 rows 948 / 1013.
static bool streaming_suits_diagnostics(int V, int64_t n_adm, bool past) {
  const int64_t mib = 4 * n_adm * V >> 20;
  const bool third_round = n_adm > 512 && n_adm <= 560;
  if (V <= short_row_limit(1024))
    return V > short_row_limit(512) && n_adm > 256 && (V <= 51200 || third_round || (V <= 69632 && mib < 240));
  if ((V <= 86016 && !past) || V > (past ? 196608 : 180224)) return true;
  return n_adm <= 256 ? n_adm <= 216 : mib < 256 || third_round;
}

// Pieces per row of a call of few rows of more than 81,920 logits; 0: not split.  A piece fits the
// registers of a workgroup; a call of very few rows takes as many as give every compute unit one.  The
// pieces cost a time for every row, the long-row kernel one for every round of 256 rows, most of it in the
// first rows of the round: pieces serve the first part of a round, up to the rows where the two draw level.
// us, pieces / long-row: V = 82,000: 200 rows 37 / 42, 224 rows 42 / 42, 300 rows 51 / 67, 400 rows 64 / 69,
// 448 rows 69 / 70; V = 122,880: 200 rows 48 / 51, 224 rows 54 / 53, 300 rows 68 / 85, 400 rows 85 / 89;
// V = 151,936: 128 rows 41 / 57, 180 rows 55 / 58, 200 rows 60 / 59, 300 rows 80 / 103, 400 rows 111 / 113,
// 448 rows 136 / 119; V = 164,000: 180 rows 59 / 65, 224 rows 69 / 67, 400 rows 125 / 130.  The long-row kernel
// reads twice what it cannot hold: V = 180,000: 224 rows 72 / 76, 256 rows 80 / 79; V = 200,000: 224 rows
// 79 / 89, 256 rows 88 / 94, 300 rows 105 / 174, 400 rows 160 / 183; V = 300,000: 256 rows 155 / 220.  (211 to 256 rows
// of 172,001 to 190,000 logits go to the long-row kernel whole: it is 5 % behind at 224 rows and 1 % ahead at 256.)
// With diagnostics against the better of the streaming and the long-row kernel: V = 102,400: 128 rows 44 / 48,
// 156 rows 50 / 49; V = 122,880: 156 rows 52 / 55, 180 rows 58 / 57, 300 rows 81 / 79; V = 151,936: 156 rows 59 / 66,
// 180 rows 67 / 68, 200 rows 73 / 69, 300 rows 94 / 95, 352 rows 106 / 111, 400 rows 124 / 120; V = 200,000:
// 224 rows 92 / 93, 256 rows 102 / 108, 300 rows 119 / 140, 400 rows 172 / 178.
static int row_splits(int V, int64_t n_adm, bool diag, int64_t room) {
  if (n_adm <= 0 || V <= short_row_limit(1024)) return 0;
  const int64_t round = diag ? (V < 122880 ? 140 : 165) : V < 136000 || V > 172000 ? 210 : 185;
  const int64_t second = diag && V <= 190000 ? (V > 144000 ? 352 : 0) : 400;
  const bool rereads = V > 190000;
  if (n_adm > round && !(n_adm <= second && (n_adm > 256 || rereads))) return 0;
  int splits = (V + short_row_limit(256) - 1) / short_row_limit(256);
  const int64_t fill = 256 / n_adm < 16 ? 256 / n_adm : 16;
  if (splits < fill) splits = (int)fill;
  return splits <= 64 && n_adm * splits <= room ? splits : 0;
}

template <bool DIAG>
static hipError_t launch_split_rows(const RowsLaunch& l, const TailArgs& tail, hipStream_t st) {
  const unsigned pieces = (unsigned)(l.a.n_adm * l.a.splits);
  hipError_t e = launch_rows<256, DIAG, kPieceSums>(l, pieces + (unsigned)l.a.T, st);
  if (e != hipSuccess) return e;
  if (tail.blocks > 0) logits_piece_grad_kernel<DIAG><<<lead_blocks((unsigned)tail.blocks) + pieces, 256, 0, st>>>(l.a, tail);
  else logits_row_short_kernel<256, DIAG, kPieceGrad><<<pieces, 256, 0, st>>>(l.a);
  return hipGetLastError();
}

hipError_t logits_kernels_opt_in() {
  const void* kernels[] = {(const void*)logits_row_resident_kernel<false, false>, (const void*)logits_row_resident_kernel<false, true>,
                           (const void*)logits_row_resident_kernel<true, false>, (const void*)logits_row_resident_kernel<true, true>};
  for (const void* k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kResLdsBytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

constexpr size_t kPieceBytes = 32;       // the sums of one piece: 8 words
constexpr size_t kMaxPieces = 4096;

struct LogitsLayout {
  size_t o_plan, o_klr, o_seg, o_done, o_summ, total;
  LogitsLayout(int32_t B, int64_t T) {
    size_t o = 0;
    o_plan = o; o += PlanBlobLayout(B).bytes;
    o_klr = o;  o = align_up(o + sizeof(float) * (size_t)(T > 0 ? T : 1), 256);
    o_seg = o;  o = align_up(o + sizeof(double) * 4 * (size_t)B, 256);
    o_done = o; o = align_up(o + sizeof(double) * 4 * (size_t)B, 256);   // one word; the size is part of the interface's limit
    o_summ = o; o = align_up(o + sizeof(double) * kSummarySlots * (size_t)B, 256);
    total = o;
  }
  // Room for the pieces of split rows behind everything else; a call whose workspace lacks it
  // serves its rows whole.
  size_t with_pieces() const {
    const size_t all = total + kPieceBytes * kMaxPieces;
    // what fits the static scratch without them still does, with what is left of it
    if (total <= (size_t)ADWIN_STATIC_SCRATCH_BYTES && all > (size_t)ADWIN_STATIC_SCRATCH_BYTES)
      return (size_t)ADWIN_STATIC_SCRATCH_BYTES;
    return all;
  }
};

static int check_logits_problem(const adwin_opd_logits_problem* p) {
  if (!p) return ADWIN_E_NULL;
  if (p->struct_bytes != sizeof(adwin_opd_logits_problem)) return ADWIN_E_MODE;
  int st = validate_ragged(p->T, p->B, p->offsets, p->window);
  if (st != ADWIN_OK) return st;
  if (p->V <= 0 || (p->V & 7)) return ADWIN_E_SHAPE;
  if (p->reduction < ADWIN_RED_SEQ_MEAN || p->reduction > ADWIN_RED_TOKEN_MEAN) return ADWIN_E_MODE;
  if (p->estimator != ADWIN_EST_EXPECTED && p->estimator != ADWIN_EST_SAMPLED) return ADWIN_E_MODE;
  if (p->estimator == ADWIN_EST_SAMPLED && !p->ids) return ADWIN_E_NULL;
  if (p->scheme < ADWIN_LOGITS_AUTO || p->scheme > ADWIN_LOGITS_STREAMING) return ADWIN_E_MODE;
  if (p->t_first_reject && !p->t_rank) return ADWIN_E_NULL;
  if (p->t_first_reject && p->topk <= 0) return ADWIN_E_SHAPE;
  if (p->t_logp_mean && !p->t_logp) return ADWIN_E_NULL;
  return ADWIN_OK;
}

}  // namespace adwin

using namespace adwin;

extern "C" int adwin_opd_logits_workspace_bytes(const adwin_opd_logits_problem* p, size_t* bytes) {
  if (!bytes) return ADWIN_E_NULL;
  int st = check_logits_problem(p);
  if (st != ADWIN_OK) return st;
  *bytes = LogitsLayout(p->B, p->T).with_pieces();
  return ADWIN_OK;
}

static int logits_impl(const adwin_opd_logits_problem* p, void* workspace, size_t workspace_bytes,
                       void* hip_stream, PhaseTimer* timer) {
  int st = check_logits_problem(p);
  if (st != ADWIN_OK) return st;
  if (p->T > 0 && (!p->z_s || !p->z_t)) return ADWIN_E_NULL;
  const uintptr_t al = (uintptr_t)p->z_s | (uintptr_t)p->z_t | (uintptr_t)p->dz;
  if (al & 15) return ADWIN_E_ALIGN;
  LogitsLayout L(p->B, p->T);
  if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < L.total)
    return ADWIN_E_WORKSPACE;
  hipStream_t stream = (hipStream_t)hip_stream;
  unsigned char* ws = (unsigned char*)workspace;

  std::vector<unsigned char> blob;
  HostPlan hp = make_host_plan(p->T, p->B, p->offsets, p->window, /*probe=*/0, p->reduction, &blob);
  DevicePlan pl = device_plan_at(ws + L.o_plan, p->B, nullptr, nullptr);
  float* klr = (float*)(ws + L.o_klr);
  double* seg = (double*)(ws + L.o_seg);

  uint32_t* done = (uint32_t*)(ws + L.o_done);
  const size_t room = (workspace_bytes - L.total) / kPieceBytes;
  const bool diag = p->t_logp || p->t_entropy || p->t_rank;
  const bool automatic = p->scheme == ADWIN_LOGITS_AUTO;
  const int splits = automatic ? row_splits(p->V, hp.n_adm, diag, (int64_t)(room < kMaxPieces ? room : kMaxPieces)) : 0;
  const bool past = past_caches(p->T, p->V);
  const bool streaming = p->scheme == ADWIN_LOGITS_STREAMING ||
                         (automatic && diag && splits == 0 && streaming_suits_diagnostics(p->V, hp.n_adm, past));
  const bool shorts = !streaming && p->V <= short_row_limit(1024);

  SetupArgs setup(ws + L.o_plan, p->B);
  setup.clear(done, 1);
  setup.clear(p->status_dev, 1);
  RowsLaunch l{LogitsArgs{}, setup, SetupBlob{}};
  // setup in the first launch of the rows; the calls of the other two kernels take 60 us and more
  const bool together = p->T > 0 && (shorts || splits > 0) && l.blob.take(blob);
  if (!together) ADWIN_HIP_TRY(launch_setup(setup, blob, stream));
  BatchArgs b{};
  b.pl = pl; b.B = p->B; b.H = 0; b.probe = 0; b.zero_grad = 1;
  b.klr = klr; b.rownorm = nullptr; b.seg = seg; b.loss_prefix = p->loss_prefix; b.loss_full = nullptr;
  b.done = done;
  b.batch = p->batch; b.n_out = p->n_out; b.n_adm_out = p->n_adm_out; b.n_adm = hp.n_adm;
  SummaryArgs sa{};
  if (p->t_first_reject || p->t_logp_mean) {
    sa.pl = pl; sa.B = p->B; sa.probe = 0; sa.topk = p->topk; sa.K = 0;
    sa.t_rank = p->t_rank; sa.t_logp = p->t_logp;
    sa.acc = (double*)(ws + L.o_summ);
    sa.first_reject = p->t_first_reject; sa.logp_mean = p->t_logp_mean;
  }
  bool ended = false;
  if (p->T > 0) {
    LogitsArgs& a = l.a;
    a.pl = pl; a.T = p->T; a.B = p->B; a.V = p->V;
    a.z_s = (const uint4*)p->z_s; a.z_t = (const uint4*)p->z_t; a.ids = p->ids;
    a.grad_scale = p->grad_scale;
    a.kl = p->kl; a.c = p->c; a.dz = (uint4*)p->dz; a.klr = klr; a.status = p->status_dev;
    a.t_logp = p->t_logp; a.t_entropy = p->t_entropy; a.t_rank = p->t_rank;
    a.sampled = p->estimator == ADWIN_EST_SAMPLED;
    PhaseScope scope(timer, ADWIN_PHASE_STATS);
    a.part = (float*)(ws + L.total);
    a.n_adm = hp.n_adm;
    a.splits = splits;
    if (together && splits == 0 && a.status) {      // the launch that clears the status word cannot also set it
      a.mark = 1;
      a.status = nullptr;
      b.status = p->status_dev; b.ids = p->ids; b.V = p->V;
    }
    if (shorts) {
      ADWIN_HIP_TRY(diag ? launch_short_rows<true>(l, stream) : launch_short_rows<false>(l, stream));
    } else if (splits > 0) {
      TailArgs tail = make_tail(b, sa);
      // summaries need the rows' outputs, which the second launch writes; a profile times the reductions by themselves
      ended = !tail.with_summary && !timer;
      if (!ended) tail.blocks = 0;
      a.tail_has_kl = ended;
      ADWIN_HIP_TRY(diag ? launch_split_rows<true>(l, tail, stream) : launch_split_rows<false>(l, tail, stream));
    } else if (streaming) {
      if (diag) logits_row_kernel<true><<<(unsigned)p->T, kRowThreads, 0, stream>>>(a);
      else logits_row_kernel<false><<<(unsigned)p->T, kRowThreads, 0, stream>>>(a);
    } else {
      if (first_use_on_device(1)) ADWIN_HIP_TRY(logits_kernels_opt_in());
#define ADWIN_LAUNCH(...) logits_row_resident_kernel<__VA_ARGS__><<<(unsigned)p->T, kResThreads, kResLdsBytes, stream>>>(a)
      if (diag && past) ADWIN_LAUNCH(true, true);
      else if (diag) ADWIN_LAUNCH(true, false);
      else if (past) ADWIN_LAUNCH(false, true);
      else ADWIN_LAUNCH(false, false);
#undef ADWIN_LAUNCH
    }
    ADWIN_HIP_TRY(hipGetLastError());
  }
  PhaseScope scope(timer, ADWIN_PHASE_REDUCE);
  if (!ended) ADWIN_HIP_TRY(launch_tail(b, sa, CandArgs{}, nullptr, 0, stream));
  return ADWIN_OK;
}

extern "C" int adwin_opd_from_logits(const adwin_opd_logits_problem* p, void* workspace,
                                     size_t workspace_bytes, void* hip_stream) {
  return logits_impl(p, workspace, workspace_bytes, hip_stream, nullptr);
}

// ---------------------------------------------------------------------------------------
// The entry point that allocates nothing: the same call with its scratch (plan blob,
// per-row KL copy, per-rollout accumulators) in a fixed array inside the library.  Every GPU
// holds its own copy of the array at its own address; the name `static_scratch` is only the
// host-side handle of the symbol, so host code asks the runtime for the device address once per
// device and uses that pointer from then on.  (No `used` attribute on the array: the compiler
// makes a file-local device variable visible to the runtime's lookup by name only because host
// code refers to it, and that attribute switches this off.)
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char static_scratch[ADWIN_STATIC_SCRATCH_BYTES];

namespace adwin {

static std::mutex g_static_mu;
static void* g_static_ptr[64];          // device address of static_scratch, per device ordinal

// Address of the current device's copy of static_scratch (looked up on first use per device).
static hipError_t static_scratch_ptr(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (!g_static_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(static_scratch));
    if (e != hipSuccess) return e;
    if (!ptr || ((uintptr_t)ptr & 255)) return hipErrorInvalidSymbol;
    g_static_ptr[dev] = ptr;
  }
  *out = g_static_ptr[dev];
  return hipSuccess;
}

hipError_t logits_static_setup() {
  void* ptr = nullptr;
  return static_scratch_ptr(&ptr);
}

}  // namespace adwin

extern "C" int adwin_opd_from_logits_static(const adwin_opd_logits_problem* p, void* hip_stream) {
  int st = check_logits_problem(p);
  if (st != ADWIN_OK) return st;
  if (LogitsLayout(p->B, p->T).total > (size_t)ADWIN_STATIC_SCRATCH_BYTES) return ADWIN_E_WORKSPACE;
  void* ptr = nullptr;
  ADWIN_HIP_TRY(static_scratch_ptr(&ptr));
  // Nothing in the scratch has to start at zero: every kernel of the call writes what a later
  // one reads (the plan blob, KL of every admitted row, the per-rollout sums), so what the
  // previous call left behind is never read.
  return logits_impl(p, ptr, (size_t)ADWIN_STATIC_SCRATCH_BYTES, hip_stream, nullptr);
}

extern "C" int adwin_opd_from_logits_profile(const adwin_opd_logits_problem* p, void* workspace,
                                             size_t workspace_bytes, void* hip_stream,
                                             float* phase_ms) {
  if (!phase_ms) return ADWIN_E_NULL;
  PhaseTimer timer((hipStream_t)hip_stream);
  int st = logits_impl(p, workspace, workspace_bytes, hip_stream, &timer);
  if (st != ADWIN_OK) return st;
  ADWIN_HIP_TRY(timer.collect(phase_ms, ADWIN_N_PHASES));
  return ADWIN_OK;
}
