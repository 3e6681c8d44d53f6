// Plan expansion, fills and the deterministic segmented reductions over ragged
// windows: per-window losses (Sec. 4.1) and prefix-vs-full alignment (Sec. 4.2).
// No floating-point atomics: every sum has a fixed order.
#include <cmath>
#include <cstring>

#include "device_utils.h"
#include "plan_device.h"
#include "setup_device.h"
#include "tail_device.h"

namespace adwin {

DevicePlan device_plan_at(unsigned char* ws_plan, int32_t B, int32_t* row_idx, int32_t* row_seq) {
  PlanBlobLayout L(B);
  DevicePlan d;
  d.offsets = (const int64_t*)(ws_plan + L.o_offsets);
  d.comp_off = (const int64_t*)(ws_plan + L.o_comp_off);
  d.n = (const int32_t*)(ws_plan + L.o_n);
  d.chunk_off = (const int32_t*)(ws_plan + L.o_chunk_off);
  d.alpha_p = (const float*)(ws_plan + L.o_alpha_p);
  d.alpha_f = (const float*)(ws_plan + L.o_alpha_f);
  d.row_idx = row_idx;
  d.row_seq = row_seq;
  return d;
}

// ---------------------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------------------
__global__ void fill_f32_kernel(float* p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Column sums of g over the window and over the rollout, in two levels.  Both kernels add rows in
// index order; the rows of a step are loaded together first (added one by one as they arrived, a
// chunk of 128 rows was 128 dependent round trips: 37 us of a 400 us call, and now 8).
constexpr int kPoolStep = 16;

__global__ __launch_bounds__(256) void pool_partial_kernel(PoolArgs a) {
  const int ch = blockIdx.x;
  const int h = blockIdx.y * 256 + threadIdx.x;
  const int i = last_le<int32_t>(a.pl.chunk_off, a.B + 1, ch);
  const int64_t len = a.pl.offsets[i + 1] - a.pl.offsets[i];
  const int64_t ni = a.pl.n[i];
  const int64_t j0 = (int64_t)(ch - a.pl.chunk_off[i]) * kChunkRows;
  const int rows = (int)(j0 + kChunkRows < len ? (int64_t)kChunkRows : len - j0);
  const int in_window = (int)(ni - j0 < rows ? (ni > j0 ? ni - j0 : 0) : rows);
  if (h >= a.H) return;
  const float* g = a.g + (a.pl.comp_off[i] + j0) * a.H + h;
  float sp = 0.f, sf = 0.f;
  for (int j = 0; j < rows; j += kPoolStep) {
    float v[kPoolStep];
#pragma unroll
    for (int q = 0; q < kPoolStep; ++q) v[q] = j + q < rows ? g[(int64_t)(j + q) * a.H] : 0.f;
#pragma unroll
    for (int q = 0; q < kPoolStep; ++q) {
      sf += v[q];
      sp += j + q < in_window ? v[q] : 0.f;
    }
  }
  a.pp[(int64_t)ch * a.H + h] = sp;
  a.pf[(int64_t)ch * a.H + h] = sf;
}

// Slot 0: the pooled sums of the call's own windows and of whole rollouts, from the chunk sums.
// Slot 1 + k: the pooled prefix sum u_i(L_k) of candidate k, whole chunks from the chunk sums,
// the ragged rest row by row.
__global__ __launch_bounds__(256) void pool_kernel(PoolArgs a, CandArgs c) {
  const int slot = blockIdx.x / a.B, i = blockIdx.x % a.B;
  const int h = blockIdx.y * 256 + threadIdx.x;
  if (h >= a.H) return;
  const int64_t c0 = a.pl.chunk_off[i];
  const float* pf = a.pf + c0 * a.H + h;
  if (slot == 0) {
    const int nch = (int)(a.pl.chunk_off[i + 1] - c0);
    const float* pp = a.pp + c0 * a.H + h;
    float sp = 0.f, sf = 0.f;
#pragma unroll 8
    for (int q = 0; q < nch; ++q) {
      sp += pp[(int64_t)q * a.H];
      sf += pf[(int64_t)q * a.H];
    }
    a.up[(int64_t)i * a.H + h] = sp;
    a.uf[(int64_t)i * a.H + h] = sf;
    return;
  }
  const int k = slot - 1;
  const int64_t len = a.pl.offsets[i + 1] - a.pl.offsets[i];
  const int64_t n = c.L[k] < len ? (int64_t)c.L[k] : len;
  const int full = (int)(n / kChunkRows), rest = (int)(n - (int64_t)full * kChunkRows);
  float s = 0.f;
#pragma unroll 8
  for (int q = 0; q < full; ++q) s += pf[(int64_t)q * a.H];
  const float* g = a.g + (a.pl.comp_off[i] + (int64_t)full * kChunkRows) * a.H + h;
  for (int j = 0; j < rest; j += kPoolStep) {
    float v[kPoolStep];
#pragma unroll
    for (int q = 0; q < kPoolStep; ++q) v[q] = j + q < rest ? g[(int64_t)(j + q) * a.H] : 0.f;
#pragma unroll
    for (int q = 0; q < kPoolStep; ++q) s += v[q];
  }
  c.uc[((int64_t)k * a.B + i) * a.H + h] = s;
}

// ---------------------------------------------------------------------------------------
// Candidate-window audit (Sec. 4.2).  For candidate k every rollout uses the shared window
// L_k: n = min(L_k, len_i).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double cand_alpha_p(const CandArgs& a, int k, int64_t n) {
  if (n <= 0) return 0.0;
  if (a.reduction == ADWIN_RED_SEQ_MEAN) return 1.0 / ((double)a.B * (double)n);
  if (a.reduction == ADWIN_RED_SUM) return 1.0;
  return a.inv_nadm[k];
}

// Candidate k, rollout i: cosines of the pooled and of the field gradients.
__device__ __forceinline__ void cand_align_body(const CandArgs& a, int k, int i, double* sh) {
  const int64_t len = a.pl.offsets[i + 1] - a.pl.offsets[i];
  const int64_t n = a.L[k] < len ? (int64_t)a.L[k] : len;
  double v[4] = {0.0, 0.0, 0.0, 0.0};   // <u_p,u_f>, |u_p|^2, |u_f|^2, S_i(n)
  double Sf[1] = {0.0};                 // S_i(len), summed as in rollout_body
  if (!a.zero_grad) {
    const float* up = a.uc + ((int64_t)k * a.B + i) * a.H;
    const float* uf = a.uf + (int64_t)i * a.H;
#pragma unroll 4
    for (int h = threadIdx.x; h < a.H; h += 256) {
      const double p = up[h], f = uf[h];
      v[0] += p * f;
      v[1] += p * p;
      v[2] += f * f;
    }
    const float* rn = a.rownorm + a.pl.comp_off[i];
#pragma unroll 4
    for (int64_t j = threadIdx.x; j < len; j += 256) {
      const double s = (double)rn[j];
      if (j < n) v[3] += s;
      Sf[0] += s;
    }
  }
  block_sum256<4>(v, sh);
  block_sum256<1>(Sf, sh);
  if (threadIdx.x == 0) {
    double rp = 0.0, rf = 0.0, okp = 0.0, okf = 0.0;
    if (!a.zero_grad) {
      if (v[1] > 0.0 && v[2] > 0.0) { rp = v[0] / (sqrt(v[1]) * sqrt(v[2])); okp = 1.0; }
      if (v[3] > 0.0 && Sf[0] > 0.0) { rf = sqrt(v[3] / Sf[0]); okf = 1.0; }
    }
    const int64_t o = (int64_t)k * a.B + i;
    a.cacc[o * 4 + 0] = rp;
    a.cacc[o * 4 + 1] = okp;
    a.cacc[o * 4 + 2] = rf;
    a.cacc[o * 4 + 3] = okf;
    a.cS[o] = v[3];
    if (a.rho_pooled) a.rho_pooled[o] = (float)rp;
    if (a.rho_field) a.rho_field[o] = (float)rf;
  }
}

// Columns [256 col, 256 col + 256) of the gradients aggregated over the batch, <p, f>, |p|^2 and |f|^2: the
// batch aggregates are then sums over B and over these.  As one workgroup per slot they had all columns to
// themselves, one group after the other, behind the launch of the rollouts instead of beside it: batch_kernel of
// 30 rollouts with 7 candidates, H = 1536, 28.4 us (9 rollouts, H = 512: 9.8), now 7.0 and 6.1.  The weights
// of up to kCandLds rollouts are formed once (their divisions, repeated per column, were most of the time).
constexpr int kCandLds = 256;
__device__ __forceinline__ void micro_body(const BatchArgs& b, const CandArgs& c, int slot, int col, double* sh,
                                           double* alpha_lds /* [2 kCandLds] */) {
  if (b.zero_grad) return;
  const int B = b.B, h = col * 256 + threadIdx.x;
  auto alpha_p = [&](int i) -> double {
    if (slot == 0) return b.pl.alpha_p[i];
    const int64_t len = b.pl.offsets[i + 1] - b.pl.offsets[i];
    return cand_alpha_p(c, slot - 1, c.L[slot - 1] < len ? (int64_t)c.L[slot - 1] : len);
  };
  for (int i = threadIdx.x; i < B && i < kCandLds; i += 256) {
    alpha_lds[i] = alpha_p(i);
    alpha_lds[kCandLds + i] = b.pl.alpha_f[i];
  }
  __syncthreads();
  double m[3] = {0.0, 0.0, 0.0};
  if (h < b.H) {
    const float* up = (slot == 0 ? b.up : c.uc + (int64_t)(slot - 1) * B * b.H) + h;
    const float* uf = b.uf + h;
    double sp = 0.0, sf = 0.0;
    for (int i0 = 0; i0 < B; i0 += kBatchStep) {
      float p[kBatchStep], f[kBatchStep];
#pragma unroll
      for (int q = 0; q < kBatchStep; ++q) {
        const int64_t i = i0 + q < B ? i0 + q : B - 1;
        p[q] = up[i * b.H];
        f[q] = uf[i * b.H];
      }
#pragma unroll
      for (int q = 0; q < kBatchStep; ++q)
        if (i0 + q < B) {
          const int i = i0 + q;
          sp += (i < kCandLds ? alpha_lds[i] : alpha_p(i)) * (double)p[q];
          sf += (i < kCandLds ? alpha_lds[kCandLds + i] : (double)b.pl.alpha_f[i]) * (double)f[q];
        }
    }
    m[0] = sp * sf;
    m[1] = sp * sp;
    m[2] = sf * sf;
  }
  block_sum256<3>(m, sh);
  if (threadIdx.x == 0)
    for (int k = 0; k < 3; ++k) b.micro[((int64_t)slot * batch_columns(b.H) + col) * 3 + k] = m[k];
}

// Candidate k: micro (after batch aggregation) and macro cosines.
__device__ __forceinline__ void cand_batch_body(const BatchArgs& b, const CandArgs& a, int k, double* sh) {
  const int B = a.B;
  double w[4] = {0.0, 0.0, 0.0, 0.0};   // macro pooled sum, count, macro field sum, count
  double f[3] = {0.0, 0.0, 0.0};        // field: dot, |p|^2, |f|^2
  auto alpha = [&](int i) {
    const int64_t len = a.pl.offsets[i + 1] - a.pl.offsets[i];
    return cand_alpha_p(a, k, a.L[k] < len ? (int64_t)a.L[k] : len);
  };
  for (int i = threadIdx.x; i < B; i += 256) {
    const int64_t o = (int64_t)k * B + i;
    const double ap = alpha(i), af = a.pl.alpha_f[i];
    w[0] += a.cacc[o * 4 + 0] * a.cacc[o * 4 + 1];
    w[1] += a.cacc[o * 4 + 1];
    w[2] += a.cacc[o * 4 + 2] * a.cacc[o * 4 + 3];
    w[3] += a.cacc[o * 4 + 3];
    f[0] += ap * af * a.cS[o];
    f[1] += ap * ap * a.cS[o];
    f[2] += af * af * a.seg[i * 4 + 3];
  }
  block_sum256<4>(w, sh);
  block_sum256<3>(f, sh);
  double m[3] = {0.0, 0.0, 0.0};
  if (!a.zero_grad) {
    micro_sums(b, 1 + k, m);
  }
  block_sum256<3>(m, sh);
  if (threadIdx.x == 0 && a.batch) {
    float o[4] = {0.f, 0.f, 0.f, 0.f};
    if (!a.zero_grad) {
      if (m[1] > 0.0 && m[2] > 0.0) o[0] = (float)(m[0] / (sqrt(m[1]) * sqrt(m[2])));
      if (f[1] > 0.0 && f[2] > 0.0) o[1] = (float)(f[0] / (sqrt(f[1]) * sqrt(f[2])));
      if (w[1] > 0.0) o[2] = (float)(w[0] / w[1]);
      if (w[3] > 0.0) o[3] = (float)(w[2] / w[3]);
    }
    for (int q = 0; q < 4; ++q) a.batch[k * 4 + q] = o[q];
  }
}

// ---------------------------------------------------------------------------------------
// The end of a call in one launch (two with probe gradients), or in that of finalize_kernel
// (tail_device.h).  Workgroups [0, B): rollouts; the next B (with_summary): their summaries; the next
// K B: candidates; then, with probe gradients, the columns of the batch (micro_body).  Each of these used to be a
// launch of about 4.7 us, and so were the batch aggregates, which need all of them: without probe gradients
// (`fold`) the workgroup that finishes last takes them; with them a launch of 1 + K workgroups
// (batch_kernel) takes them side by side.  Logits of 24
// rollouts with diagnostics: 425 -> 412 us; one rollout of 37 rows 52.6 -> 49.5 us; the probe
// audit of 9 rollouts with 7 candidates, with the pooling above: 397 -> 333 us.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void tail_kernel(TailArgs a) {
  __shared__ double sh[4 * (ADWIN_MAX_CANDIDATES + 1)];
  __shared__ int sh_first[4];
  if (a.fold) return tail_body<true>(a, blockIdx.x, sh, sh_first);
  const int B = a.b.B, role = blockIdx.x / B, i = blockIdx.x % B, aligned = B * (1 + a.with_summary + a.c.K);
  if ((int)blockIdx.x >= aligned) {
    __shared__ double alpha[2 * kCandLds];
    const int cols = batch_columns(a.b.H), m = (int)blockIdx.x - aligned;
    micro_body(a.b, a.c, m / cols, m % cols, sh, alpha);
  } else if (role == 0) rollout_body<true>(a.b, i, sh);
  else if (role == 1 && a.with_summary) summary_rollout_body(a.s, i, sh, sh_first);
  else cand_align_body(a.c, role - 1 - a.with_summary, i, sh);
}

__global__ __launch_bounds__(256) void batch_kernel(TailArgs a) {
  __shared__ double sh[16];
  if (blockIdx.x == 0) {
    batch_body<true>(a.b, sh);
    if (a.with_summary) summary_batch_body(a.s);
  } else {
    cand_batch_body(a.b, a.c, blockIdx.x - 1, sh);
  }
}

// ---------------------------------------------------------------------------------------
// Cosine of two long fp32 arrays (the two head-weight gradients).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void cosine_partial_kernel(const float* x, const float* y, int64_t n,
                                                             double* partials) {
  __shared__ double sh[4];
  const int64_t per = (n + kCosineBlocks - 1) / kCosineBlocks;
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = lo + per < n ? lo + per : n;
  double xy = 0.0, xx = 0.0, yy = 0.0;
  for (int64_t q = lo + threadIdx.x; q < hi; q += 256) {
    const double a = (double)x[q], b = (double)y[q];
    xy += a * b; xx += a * a; yy += b * b;
  }
  xy = block_sum_256(xy, sh);
  xx = block_sum_256(xx, sh);
  yy = block_sum_256(yy, sh);
  if (threadIdx.x == 0) {
    partials[3 * blockIdx.x + 0] = xy;
    partials[3 * blockIdx.x + 1] = xx;
    partials[3 * blockIdx.x + 2] = yy;
  }
}

__global__ void cosine_final_kernel(const double* partials, float* out) {
  if (threadIdx.x != 0) return;
  double xy = 0.0, xx = 0.0, yy = 0.0;
  for (int b = 0; b < kCosineBlocks; ++b) {
    xy += partials[3 * b + 0]; xx += partials[3 * b + 1]; yy += partials[3 * b + 2];
  }
  *out = (xx > 0.0 && yy > 0.0) ? (float)(xy / (sqrt(xx) * sqrt(yy))) : 0.f;
}

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------
hipError_t launch_cosine(const float* x, const float* y, int64_t n, double* partials, float* out,
                         hipStream_t st) {
  cosine_partial_kernel<<<kCosineBlocks, 256, 0, st>>>(x, y, n, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  cosine_final_kernel<<<1, 64, 0, st>>>(partials, out);
  return hipGetLastError();
}
TailArgs make_tail(const BatchArgs& b, const SummaryArgs& s) {
  TailArgs a;
  a.b = b; a.s = s; a.c = CandArgs{};
  a.fold = 1;
  a.with_summary = s.first_reject || s.logp_mean || s.loss_share;
  a.blocks = b.B * (1 + a.with_summary);
  return a;
}
hipError_t launch_tail(const BatchArgs& b, const SummaryArgs& s, const CandArgs& c, const PoolArgs* pooled,
                       int64_t n_chunks, hipStream_t st) {
  TailArgs a = make_tail(b, s);
  hipError_t e;
  if (!pooled) {
    tail_kernel<<<(unsigned)a.blocks, 256, 0, st>>>(a);
    return hipGetLastError();
  }
  a.c = c;
  a.fold = 0;
  const unsigned B = (unsigned)b.B, K = (unsigned)c.K, cols = (unsigned)((pooled->H + 255) / 256);
  if (n_chunks > 0) {
    pool_partial_kernel<<<dim3((unsigned)n_chunks, cols), 256, 0, st>>>(*pooled);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  pool_kernel<<<dim3((1 + K) * B, cols), 256, 0, st>>>(*pooled, c);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  tail_kernel<<<B * (1 + (unsigned)a.with_summary + K) + (1 + K) * cols, 256, 0, st>>>(a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  batch_kernel<<<1 + K, 256, 0, st>>>(a);
  return hipGetLastError();
}
hipError_t launch_fill_f32(float* p, int64_t n, float v, hipStream_t st) {
  if (!p || n <= 0) return hipSuccess;
  fill_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, n, v);
  return hipGetLastError();
}
// Host -> device upload of a small blob through kernel arguments: the launch takes its copy
// of the bytes before it returns, so the host buffer may be pageable and may be freed or
// reused at once, whatever the stream still has to do, and the launch is an ordinary kernel
// node for a caller who captures the stream.
struct UploadArgs { uint4* dst; int n16; uint4 data[kUploadChunk / 16]; };
__global__ __launch_bounds__(256) void upload_kernel(const UploadArgs a) {
  const int q = threadIdx.x;
  if (q < a.n16) a.dst[q] = a.data[q];
}
hipError_t launch_upload(void* dst, const void* src_host, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  if (!dst || !src_host || (bytes & 15) || ((uintptr_t)dst & 15)) return hipErrorInvalidValue;
  static_assert(kUploadChunk / 16 <= 256, "one thread per 16 bytes");
  UploadArgs a;
  for (size_t at = 0; at < bytes; at += kUploadChunk) {
    const size_t nb = bytes - at < (size_t)kUploadChunk ? bytes - at : (size_t)kUploadChunk;
    a.dst = (uint4*)((unsigned char*)dst + at);
    a.n16 = (int)(nb / 16);
    memcpy(a.data, (const unsigned char*)src_host + at, nb);
    upload_kernel<<<1, 256, 0, st>>>(a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Setup in a launch of its own: calls whose plan does not fit a kernel's arguments, logits calls served by the
// long-row or the streaming kernel.
__global__ __launch_bounds__(256) void setup_inline_kernel(const SetupArgs a, const SetupBlob b) {
  setup_body(a, &b, (const unsigned char*)b.data, blockIdx.x, gridDim.x, 256);
}
__global__ __launch_bounds__(256) void setup_kernel(const SetupArgs a) {
  setup_body(a, nullptr, a.plan, blockIdx.x, gridDim.x, 256);
}

hipError_t launch_setup(const SetupArgs& a, const std::vector<unsigned char>& blob, hipStream_t st) {
  static_assert(sizeof(SetupArgs) + sizeof(SetupBlob) < 4096, "kernel arguments");
  if (a.n_zero > SetupArgs::kMaxZero) return hipErrorInvalidValue;
  const unsigned grid = setup_blocks(a, 256);
  SetupBlob b;
  if (b.take(blob)) {
    setup_inline_kernel<<<grid, 256, 0, st>>>(a, b);
  } else {
    hipError_t e = launch_upload(a.plan, blob.data(), blob.size(), st);
    if (e != hipSuccess) return e;
    setup_kernel<<<grid, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// phase timer
// ---------------------------------------------------------------------------------------
PhaseTimer::~PhaseTimer() {
  for (auto& s : spans_) {
    if (s.a) (void)hipEventDestroy(s.a);
    if (s.b) (void)hipEventDestroy(s.b);
  }
}
void PhaseTimer::begin(int phase) {
  open_ = false;
  if (err_ != hipSuccess) return;
  Span s{phase, nullptr, nullptr};
  err_ = hipEventCreate(&s.a);
  if (err_ != hipSuccess) return;
  err_ = hipEventCreate(&s.b);
  if (err_ != hipSuccess) { (void)hipEventDestroy(s.a); return; }
  spans_.push_back(s);
  err_ = hipEventRecord(s.a, st_);
  open_ = err_ == hipSuccess;
}
void PhaseTimer::end() {
  if (!open_) return;
  open_ = false;
  err_ = hipEventRecord(spans_.back().b, st_);
}
hipError_t PhaseTimer::collect(float* phase_ms, int n_phases) {
  if (err_ != hipSuccess) return err_;
  hipError_t e = hipStreamSynchronize(st_);
  if (e != hipSuccess) return e;
  for (int k = 0; k < n_phases; ++k) phase_ms[k] = 0.f;
  for (auto& s : spans_) {
    float ms = 0.f;
    e = hipEventElapsedTime(&ms, s.a, s.b);
    if (e != hipSuccess) return e;
    if (s.phase >= 0 && s.phase < n_phases) phase_ms[s.phase] += ms;
  }
  return hipSuccess;
}

}  // namespace adwin
