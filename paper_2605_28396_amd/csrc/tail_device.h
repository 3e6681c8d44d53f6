// The reductions that end a call, as device functions of a 256-thread workgroup (ALIGN: with probe
// gradients): per-rollout sums and losses, batch aggregates, rollout summaries.  Used by the launches of
// reduce_kernels.hip and, in calls without probe gradients or summaries, by workgroups of
// logits_piece_grad_kernel and of finalize_kernel: 224 rows, V = 4,096 60.4 -> 54.1 us per call, 256 rows, V = 151,936 772 -> 762.
#pragma once
#include "device_utils.h"
#include "plan_device.h"

namespace adwin {

// Fixed-order block sum of up to 4 doubles per thread (256 threads).
template <int K>
__device__ __forceinline__ void block_sum256(double (&v)[K], double* sh /* [K][4] */) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    v[k] = wave_sum(v[k]);
    if (lane == 0) sh[k * 4 + w] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = (sh[k * 4 + 0] + sh[k * 4 + 1]) + (sh[k * 4 + 2] + sh[k * 4 + 3]);
  __syncthreads();
}

// Sums that another workgroup of the same launch reads: past the L2 of the compute unit's die, which the
// others do not see.  A fence instead writes back all that this L2 holds of the launch's other outputs: with it 60
// rows of 1,000 logits 12.6 us per call, without 11.5; with summaries, 250 rows of 32,776 24.2 and 22.7.
__device__ __forceinline__ void store_shared(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_shared(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Rollout i: sums of KL_t and ||g_t||^2 over the window and the rollout, the window losses, and
// the cosines from the pooled sums and the norm sums.
template <bool ALIGN>
__device__ __forceinline__ void rollout_body(const BatchArgs& a, int i, double* sh) {
  const int64_t len = a.pl.offsets[i + 1] - a.pl.offsets[i];
  const int64_t ni = a.pl.n[i];
  const int64_t hi = a.probe ? len : ni;
  const int64_t r0 = a.pl.comp_off[i];
  double v[4] = {0.0, 0.0, 0.0, 0.0};   // kl prefix, kl full, norm prefix, norm full
  uint32_t flags = 0u;
#pragma unroll 4
  for (int64_t j = threadIdx.x; j < hi; j += 256) {
    float kl = a.klr[r0 + j];
    if (a.status) {
      if (__float_as_uint(kl) == kExcludedRow) { kl = 0.f; flags |= ADWIN_DEV_NONFINITE; }
      else if (a.ids && (uint32_t)a.ids[a.pl.offsets[i] + j] >= (uint32_t)a.V) flags |= ADWIN_DEV_BAD_ID;
    }
    const double k = kl;
    const double s = a.rownorm ? (double)a.rownorm[r0 + j] : 0.0;
    v[1] += k;
    v[3] += s;
    if (j < ni) { v[0] += k; v[2] += s; }
  }
  if (flags) atomicOr(a.status, flags);
  block_sum256<4>(v, sh);
  const bool align = ALIGN && a.probe && !a.zero_grad;
  double u[3] = {0.0, 0.0, 0.0};
  if (align) {
    const float* up = a.up + (size_t)i * a.H;
    const float* uf = a.uf + (size_t)i * a.H;
#pragma unroll 4
    for (int h = threadIdx.x; h < a.H; h += 256) {
      const double p = up[h], f = uf[h];
      u[0] += p * f;
      u[1] += p * p;
      u[2] += f * f;
    }
    block_sum256<3>(u, sh);
  }
  if (threadIdx.x == 0) {
    for (int k = 0; k < 4; ++k) store_shared(a.seg + i * 4 + k, v[k]);
    if (a.loss_prefix) a.loss_prefix[i] = ni > 0 ? (float)(v[0] / (double)ni) : 0.f;
    if (a.loss_full) a.loss_full[i] = (a.probe && len > 0) ? (float)(v[1] / (double)len) : 0.f;
    double rp = 0.0, rf = 0.0, okp = 0.0, okf = 0.0;
    if (align) {
      if (u[1] > 0.0 && u[2] > 0.0) { rp = u[0] / (sqrt(u[1]) * sqrt(u[2])); okp = 1.0; }
      if (v[2] > 0.0 && v[3] > 0.0) { rf = sqrt(v[2] / v[3]); okf = 1.0; }
      a.racc[i * 4 + 0] = rp;
      a.racc[i * 4 + 1] = okp;
      a.racc[i * 4 + 2] = rf;
      a.racc[i * 4 + 3] = okf;
    }
    if (a.rho_pooled) a.rho_pooled[i] = (float)rp;
    if (a.rho_field) a.rho_field[i] = (float)rf;
  }
}

// Rollouts whose terms of a sum in index order are loaded together: one round trip per rollout made the
// aggregates of 200 rollouts at H = 1536 635 us.
constexpr int kBatchStep = 16;

// The three sums over columns that micro_body leaves per 256 of them.  Slot 0: the call's windows, slot 1 + k: candidate k.
__device__ __forceinline__ void micro_sums(const BatchArgs& a, int slot, double (&m)[3]) {
  const int cols = batch_columns(a.H);
  for (int q = threadIdx.x; q < cols; q += 256) {
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k] += a.micro[((int64_t)slot * cols + q) * 3 + k];
  }
}

// One workgroup: batch objectives, micro (after aggregation) and macro (mean of
// per-rollout) alignment, integer outputs.  The sums over the rollouts run in index order.
template <bool ALIGN>
__device__ __forceinline__ void batch_body(const BatchArgs& a, double* sh) {
  const int B = a.B;
  const bool align = ALIGN && a.probe && !a.zero_grad;
  // batch objectives and field sums
  double w[4] = {0.0, 0.0, 0.0, 0.0};   // L^p, L^f, macro pooled sum, macro pooled count
  double f[4] = {0.0, 0.0, 0.0, 0.0};   // field: dot, |p|^2, |f|^2, unused
  double mf[2] = {0.0, 0.0};            // macro field sum, count
  for (int i = threadIdx.x; i < B; i += 256) {
    const double ap = a.pl.alpha_p[i], af = a.pl.alpha_f[i];
    w[0] += ap * load_shared(a.seg + i * 4 + 0);
    if (a.probe) w[1] += af * load_shared(a.seg + i * 4 + 1);
    if (align) {
      w[2] += a.racc[i * 4 + 0] * a.racc[i * 4 + 1];
      w[3] += a.racc[i * 4 + 1];
      mf[0] += a.racc[i * 4 + 2] * a.racc[i * 4 + 3];
      mf[1] += a.racc[i * 4 + 3];
      const double Sp = load_shared(a.seg + i * 4 + 2), Sf = load_shared(a.seg + i * 4 + 3);
      f[0] += ap * af * Sp;
      f[1] += ap * ap * Sp;
      f[2] += af * af * Sf;
    }
  }
  block_sum256<4>(w, sh);
  // micro pooled: aggregate the weighted pooled gradients over the batch, then one cosine
  double m[3] = {0.0, 0.0, 0.0};
  if (align) {
    block_sum256<4>(f, sh);
    block_sum256<2>(mf, sh);
    micro_sums(a, 0, m);
    block_sum256<3>(m, sh);
  }
  if (a.n_out)
    for (int i = threadIdx.x; i < B; i += 256) a.n_out[i] = a.pl.n[i];
  if (threadIdx.x == 0) {
    if (a.n_adm_out) *a.n_adm_out = a.n_adm;
    if (a.batch) {
      float o[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      o[0] = (float)w[0];
      if (a.probe) o[1] = (float)w[1];
      if (align) {
        if (m[1] > 0.0 && m[2] > 0.0) o[2] = (float)(m[0] / (sqrt(m[1]) * sqrt(m[2])));
        if (f[1] > 0.0 && f[2] > 0.0) o[3] = (float)(f[0] / (sqrt(f[1]) * sqrt(f[2])));
        if (w[3] > 0.0) o[4] = (float)(w[2] / w[3]);
        if (mf[1] > 0.0) o[5] = (float)(mf[0] / mf[1]);
      }
      for (int k = 0; k < 8; ++k) a.batch[k] = o[k];
    }
  }
}

// ---------------------------------------------------------------------------------------
// Rollout-level summaries of the per-row outputs.  One workgroup per rollout; every thread
// takes positions tid, tid + 256, ... in ascending order with double accumulators, and the
// 256 partials are folded in a fixed order, so the results do not depend on scheduling.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double block_sum_256(double v, double* sh) {
  double x[1] = {v};
  block_sum256<1>(x, sh);
  return x[0];
}

__device__ __forceinline__ void summary_rollout_body(const SummaryArgs& a, int i, double* sh /* [4 (ADWIN_MAX_CANDIDATES + 1)] */,
                                                     int* sh_first /* [4] */) {
  const int tid = threadIdx.x;
  const int64_t base = a.pl.offsets[i];
  const int64_t len = a.pl.offsets[i + 1] - base;
  const int64_t n = a.pl.n[i];
  const int64_t m = a.probe ? len : n;          // computed positions of this rollout
  double* acc = a.acc + (size_t)i * kSummarySlots;
  if (a.first_reject) {
    int64_t first = m;
    for (int64_t j = tid; j < m; j += 256)
      if (a.t_rank[base + j] > a.topk) { first = j; break; }
    int lowest = (int)first;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lowest = min(lowest, __shfl_xor(lowest, o, 64));
    if ((tid & 63) == 0) sh_first[tid >> 6] = lowest;
    __syncthreads();
    if (tid == 0) a.first_reject[i] = min(min(sh_first[0], sh_first[1]), min(sh_first[2], sh_first[3]));
  }
  if (a.logp_mean) {
    double sp = 0.0, ss = 0.0;
    for (int64_t j = tid; j < m; j += 256) {
      const double v = (double)a.t_logp[base + j];
      if (j < n) sp += v; else ss += v;
    }
    double both[2] = {sp, ss};
    block_sum256<2>(both, sh);
    sp = both[0]; ss = both[1];
    if (tid == 0) {
      store_shared(acc + ADWIN_MAX_CANDIDATES + 1, sp);
      store_shared(acc + ADWIN_MAX_CANDIDATES + 2, ss);
      a.logp_mean[2 * i + 0] = n > 0 ? (float)(sp / (double)n) : 0.f;
      a.logp_mean[2 * i + 1] = m > n ? (float)(ss / (double)(m - n)) : 0.f;
    }
  }
  if (a.loss_share) {
    double part[ADWIN_MAX_CANDIDATES + 1];       // per candidate, then the total
#pragma unroll
    for (int k = 0; k <= ADWIN_MAX_CANDIDATES; ++k) part[k] = 0.0;
    for (int64_t j = tid; j < m; j += 256) {
      const double v = (double)a.kl[base + j];
      part[ADWIN_MAX_CANDIDATES] += v;
#pragma unroll
      for (int k = 0; k < ADWIN_MAX_CANDIDATES; ++k)
        if (k < a.K && j < a.L[k]) part[k] += v;
    }
    block_sum256<ADWIN_MAX_CANDIDATES + 1>(part, sh);     // together: two barriers in all
    if (tid == 0) {
      store_shared(acc + ADWIN_MAX_CANDIDATES, part[ADWIN_MAX_CANDIDATES]);
#pragma unroll
      for (int k = 0; k < ADWIN_MAX_CANDIDATES; ++k)
        if (k < a.K) store_shared(acc + k, part[k]);
    }
  }
}

// Batch rows of the summaries: sums over rollouts in index order.
__device__ __forceinline__ void summary_batch_body(const SummaryArgs& a) {
  const int tid = threadIdx.x;
  if (a.loss_share && tid < a.K) {
    double part = 0.0, tot = 0.0;
    for (int i0 = 0; i0 < a.B; i0 += kBatchStep) {
      double p[kBatchStep], t[kBatchStep];
#pragma unroll
      for (int q = 0; q < kBatchStep; ++q) {
        const double* acc = a.acc + (size_t)(i0 + q < a.B ? i0 + q : a.B - 1) * kSummarySlots;
        p[q] = load_shared(acc + tid);
        t[q] = load_shared(acc + ADWIN_MAX_CANDIDATES);
      }
#pragma unroll
      for (int q = 0; q < kBatchStep; ++q)
        if (i0 + q < a.B) { part += p[q]; tot += t[q]; }
    }
    a.loss_share[tid] = tot != 0.0 ? (float)(part / tot) : 0.f;
  }
  if (a.logp_mean && tid >= 32 && tid < 34) {
    const int c = tid - 32;
    double sum = 0.0;
    int64_t cnt = 0;
    for (int i0 = 0; i0 < a.B; i0 += kBatchStep) {
      double v[kBatchStep];
      int64_t k[kBatchStep];
#pragma unroll
      for (int q = 0; q < kBatchStep; ++q) {
        const int i = i0 + q < a.B ? i0 + q : a.B - 1;
        const int64_t len = a.pl.offsets[i + 1] - a.pl.offsets[i];
        const int64_t n = a.pl.n[i], m = a.probe ? len : n;
        v[q] = load_shared(a.acc + (size_t)i * kSummarySlots + ADWIN_MAX_CANDIDATES + 1 + c);
        k[q] = c == 0 ? n : m - n;
      }
#pragma unroll
      for (int q = 0; q < kBatchStep; ++q)
        if (i0 + q < a.B) { sum += v[q]; cnt += k[q]; }
    }
    a.logp_mean[2 * a.B + c] = cnt > 0 ? (float)(sum / (double)cnt) : 0.f;
  }
}

// Workgroup `block` of the a.blocks that end a call without probe gradients: [0, B) rollouts, with SUMMARY
// the next B their summaries (a.with_summary).  The batch aggregates, a few sums over B, are taken by the workgroup that
// finishes last: it counts the finished ones in `done`, and adds in rollout order, so the result does not
// depend on which one it is.
template <bool SUMMARY>
__device__ __forceinline__ void tail_body(const TailArgs& a, int block, double* sh /* [4 (ADWIN_MAX_CANDIDATES + 1)] */,
                                          int* sh_first /* [4] */) {
  if (!SUMMARY || block < a.b.B) rollout_body<false>(a.b, block, sh);
  else summary_rollout_body(a.s, block - a.b.B, sh, sh_first);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the workgroup's sums have arrived (store_shared)
  __syncthreads();
  if (threadIdx.x == 0)
    sh_first[0] = __hip_atomic_fetch_add(a.b.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == (uint32_t)a.blocks;
  __syncthreads();
  if (!sh_first[0]) return;
  batch_body<false>(a.b, sh);
  if (SUMMARY && a.with_summary) summary_batch_body(a.s);
}

}  // namespace adwin
