// Per-call plan blob (host side) and the launchers of the small bookkeeping and
// reduction kernels shared by the fused and the logits-given path.
#pragma once
#include <vector>

#include "common.h"

namespace adwin {

DevicePlan device_plan_at(unsigned char* ws_plan, int32_t B, int32_t* row_idx, int32_t* row_seq);

// large dynamic LDS of the row-resident logits kernel, once per device (logits_kernels.hip)
hipError_t logits_kernels_opt_in();
// looks up the current device's address of the library's static scratch array (logits_kernels.hip)
hipError_t logits_static_setup();

// --- launchers (all asynchronous on `st`) ---------------------------------------------
// copies `bytes` (a multiple of 16) of host memory to `dst`; the host bytes are taken
// before the call returns
hipError_t launch_upload(void* dst, const void* src_host, size_t bytes, hipStream_t st);
hipError_t launch_fill_f32(float* p, int64_t n, float v, hipStream_t st);

// What a call sets up before its first real kernel, in one launch: the plan in the workspace, the
// rows of the plan's rollouts (row_idx, row_seq; padding repeats the last computed row) and
// arrays of 32-bit words that start at zero.
struct SetupArgs {
  unsigned char* plan;                  // in the workspace; PlanBlobLayout(B)
  int32_t B;
  int64_t o_comp_off;                   // PlanBlobLayout(B).o_comp_off (o_offsets is 0)
  int64_t n_rows = 0, n_pad = 0;        // 0: no rows wanted
  int32_t* row_idx = nullptr; int32_t* row_seq = nullptr;
  static constexpr int kMaxZero = 8;
  uint32_t* zero[kMaxZero]; int64_t zero_n[kMaxZero];
  int n_zero = 0;
  SetupArgs(unsigned char* ws_plan, int32_t rollouts)
      : plan(ws_plan), B(rollouts), o_comp_off((int64_t)PlanBlobLayout(rollouts).o_comp_off) {}
  void clear(void* words, int64_t n) {  // NULL: an output that is not wanted
    if (!words || n <= 0) return;
    if (n_zero < kMaxZero) {            // one too many is counted, and refused by launch_setup
      zero[n_zero] = (uint32_t*)words;
      zero_n[n_zero] = n;
    }
    ++n_zero;
  }
};
hipError_t launch_setup(const SetupArgs& a, const std::vector<unsigned char>& blob, hipStream_t st);

// Per-rollout sums of KL (and of ||g_t||^2 when `rownorm` is given) over the window and
// over the whole rollout, the window losses and the alignment of the two gradients, then the
// batch aggregates.
struct BatchArgs {
  DevicePlan pl;
  int32_t B;
  int32_t H;            // 0: no gradient statistics (logits-given path)
  int probe;
  int zero_grad;        // grad_scale == 0: every alignment is defined as 0
  const float* klr; const float* rownorm;   // per computed row; rownorm may be NULL
  double* seg;          // [B][4] scratch: KL prefix, KL full, ||g||^2 prefix, ||g||^2 full
  float* loss_prefix; float* loss_full;     // [B], may be NULL
  const float* up;      // [B][H] pooled prefix sums (unweighted)
  const float* uf;      // [B][H] pooled full-rollout sums
  double* racc;         // [B][4] scratch of the alignment (not used without probe gradients)
  uint32_t* done;       // a word that is zero when the call starts (not used with probe gradients)
  float* rho_pooled; float* rho_field; float* batch;
  int32_t* n_out; int64_t* n_adm_out; int64_t n_adm;
  // Not NULL: the rows' status bits are still to be reported, from klr (kExcludedRow) and the ids of
  // the rows [0, n_i) of every rollout (NULL: none); the word is zero, or holds other rollouts' bits.
  uint32_t* status; const int32_t* ids; int32_t V;
  double* micro;        // [1 + K][batch_columns(H)][3] scratch of the probe's batch aggregates (micro_body)
};
inline __host__ __device__ int batch_columns(int H) { return (H + 255) / 256; }
constexpr uint32_t kExcludedRow = 0x7fffffffu;   // a NaN; KL_t of every other row is finite
// Candidate-window audit (Sec. 4.2): alignment of the shared prefix window L_k, for every
// candidate k, with the full-rollout gradient, from the per-row gradients of one
// full-rollout pass.
struct CandArgs {
  DevicePlan pl;
  int32_t B, H, K;
  int reduction;
  int zero_grad;
  int32_t L[ADWIN_MAX_CANDIDATES];
  double inv_nadm[ADWIN_MAX_CANDIDATES];   // TOKEN_MEAN weight of candidate k: 1 / sum_i min(L_k, len_i)
  const float* uf;       // [B][H] pooled full-rollout sums
  const float* rownorm;  // [rows] ||g_t||^2
  const double* seg;     // [B][4]; seg[4 i + 3] = sum of ||g_t||^2 over rollout i
  float* uc;             // [K][B][H] scratch: pooled prefix sums
  double* cacc;          // [K][B][4] scratch: rho pooled, valid, rho field, valid
  double* cS;            // [K][B]   scratch: sum of ||g_t||^2 over the prefix
  float* rho_pooled; float* rho_field; float* batch;   // outputs, may be NULL
};

// Rollout-level summaries of per-row outputs (Sec. 3.1 top-k rejection; App. C loss
// distribution and prefix / suffix teacher log-probability).  Rows are packed positions;
// rollout i's computed positions are j < computed_i = (probe ? len_i : n_i).
struct SummaryArgs {
  DevicePlan pl;
  int32_t B, K;
  int probe;
  int32_t topk;
  int32_t L[ADWIN_MAX_CANDIDATES];
  const int32_t* t_rank;     // [T] or NULL
  const float* t_logp;       // [T] or NULL
  const float* kl;           // [T] or NULL
  double* acc;               // [B][kSummarySlots] scratch
  int32_t* first_reject;     // [B] or NULL (needs t_rank)
  float* logp_mean;          // [B + 1][2] or NULL (needs t_logp)
  float* loss_share;         // [K] or NULL (needs kl)
};
constexpr int kSummarySlots = ADWIN_MAX_CANDIDATES + 3;   // K candidate sums, total, logp prefix, logp suffix

// The reductions that end a call.  pooled: the probe's pooled gradients (PoolArgs) are wanted
// too; cand.K may be 0; a summary output that is NULL is not wanted.
struct PoolArgs {       // pooled gradients per rollout (see pool_partial_kernel, pool_kernel)
  DevicePlan pl; int B; int H;
  const float* g; float* pp; float* pf;   // partials [n_chunks][H]
  float* up; float* uf;                   // [B][H]
};
struct TailArgs { BatchArgs b; SummaryArgs s; CandArgs c; int fold, with_summary, blocks; };
// a tail without probe gradients: `blocks` workgroups (see tail_device.h)
TailArgs make_tail(const BatchArgs& b, const SummaryArgs& s);
hipError_t launch_tail(const BatchArgs& b, const SummaryArgs& s, const CandArgs& c, const PoolArgs* pooled,
                       int64_t n_chunks, hipStream_t st);

// Cosine of two fp32 arrays of n elements into *out (0 if either norm is 0): fixed partition
// into kCosineBlocks contiguous pieces, double sums, pieces added in index order.
constexpr int kCosineBlocks = 1024;
hipError_t launch_cosine(const float* x, const float* y, int64_t n, double* partials /* [kCosineBlocks][3] */,
                         float* out, hipStream_t st);

// Optional per-phase timing with HIP events on the caller's stream (profiling entry
// points only).  begin()/end() bracket one launch; collect() waits and sums per phase.
class PhaseTimer {
 public:
  explicit PhaseTimer(hipStream_t st) : st_(st) {}
  ~PhaseTimer();
  // begin/end keep the first error they meet; collect returns it instead of times
  void begin(int phase);
  void end();
  hipError_t collect(float* phase_ms, int n_phases);
 private:
  struct Span { int phase; hipEvent_t a, b; };
  hipStream_t st_;
  std::vector<Span> spans_;
  hipError_t err_ = hipSuccess;
  bool open_ = false;
};

// RAII helper: no-op when the timer is null.
struct PhaseScope {
  PhaseTimer* t;
  PhaseScope(PhaseTimer* timer, int phase) : t(timer) { if (t) t->begin(phase); }
  ~PhaseScope() { if (t) t->end(); }
};

}  // namespace adwin
