// Shared between the translation units of the fused path: tile geometry, the argument
// blocks of its kernels and the host-side launchers.  The kernels live in
// sweep_kernels.hip (LM-head projections, row statistics, gradient factors) and
// grad_kernels.hip (combine pass, gradient contractions, scale + scatter); fused_host.hip
// lays out the workspace and strings the launches together.
#ifndef ADWIN_FUSED_SHARED_H
#define ADWIN_FUSED_SHARED_H

#include "device_utils.h"
#include "plan_device.h"

namespace adwin {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowBytes = kBK * 2;   // 128 B of k per staged row

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of
// virtual ids so that the tiles sharing operands also share an L2.
__device__ __forceinline__ int xcd_contiguous_id(int bid, int nb) {
  const int xcd = bid & 7, loc = bid >> 3;
  const int base = nb >> 3, rem = nb & 7;
  return xcd * base + (xcd < rem ? xcd : rem) + loc;
}

// Quotients by a number that the host knows: with per = ceil(2^32 / d) the upper half of n per is n / d while
// n (per d - 2^32) < 2^32, for which n < 2^32 / d is enough.  On the device the division, with 64-bit operands,
// was 100 instructions in front of the first load of every workgroup.
struct Quotient {
  uint32_t per = 0;                // 0: d = 1
  void by(int d) { per = d > 0 ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u; }
  __host__ __device__ __forceinline__ int operator()(int n) const {
    return per ? (int)(((uint64_t)(uint32_t)n * per) >> 32) : n;
  }
};

// `total` things in `parts` contiguous shares: share i begins at floor(i total / parts), so that the longer ones,
// of one more, are spread evenly.  The boundaries enter the results (the running means of a strip, the order
// of the sums).  No quotient is taken of more than parts^2.
constexpr int kMaxShares = 1024;
struct Shares {
  int parts, each, longer;         // longer shares hold one more
  Quotient of_parts, of_longer, of_shorter;
  void split(int total, int n) {
    parts = n;
    each = total / n;
    longer = total % n;
    of_parts.by(n);
    of_longer.by(longer);
    of_shorter.by(n - longer);
  }
  __host__ __device__ __forceinline__ int first(int i) const { return i * each + of_parts(i * longer); }
  // the i-th share in the order: longer ones, then the others
  __host__ __device__ __forceinline__ int by_length(int i) const {
    return i < longer ? of_longer((i + 1) * parts - 1) : of_shorter((i - longer) * parts);
  }
};

// Workgroup `vid` of a logit pass -> (strip, token tile): groups of `tg` token tiles, inside a
// group strip-major, so that consecutive ids share a strip's W tiles and a group's h tiles.  The
// last group holds the tiles that remain: every workgroup of the grid (n_tiles x strips) has
// work.  With the last group padded to `tg` tiles instead, a call of one token tile left three
// of four workgroups empty and the XCDs of a 13-tile call unevenly loaded.
__device__ __forceinline__ void strip_and_tile(int vid, int tg, int strips, int n_tiles, int* strip, int* tile) {
  const int per_group = tg * strips, g = vid / per_group;
  const int within = vid - g * per_group, left = n_tiles - g * tg;
  const int h = left < tg ? left : tg;
  *strip = within / h;
  *tile = g * tg + within % h;
}

// One wave instruction of a direct global->LDS load: lane l moves the 16 bytes at
// sbase + voff(l) to LDS address lds_base + IMM + 16 l (M0 = LDS destination of the wave;
// scalar base + 32-bit lane offset).  Such loads return in order and are waited for with an
// explicit s_waitcnt vmcnt(N).  The destination is given as scalar base + literal and added
// straight into M0, and the callers keep the wave's share of both addresses in operands that
// are set up once, so that a load costs three instructions: a wave issues one instruction at a
// time and the loads share the shadow of an MFMA with LDS reads.
// ONCE: lines that nobody reads again, the first to be evicted.
template <int IMM, bool ONCE = false>
__device__ __forceinline__ void dma16_at(uint32_t lds_base, uint32_t voff, const char* sbase) {
  if constexpr (ONCE)
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :: "s"(lds_base), "v"(voff), "s"(sbase), "n"(IMM) : "memory", "scc");
  else
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(voff), "s"(sbase), "n"(IMM) : "memory", "scc");
}

// Wave-uniform bookkeeping of a k-step pipeline, written as instructions at a fixed place:
// plain scalar arithmetic has no place of its own in the pinned instruction order of a k-step
// and would be gathered in front of the k-step's first MFMA, where the wave, which issues one
// instruction at a time, keeps the matrix pipe waiting.
// Ring slot after slot x (LDS addresses; the ring is [begin, end), slots STEP bytes apart).
template <int STEP>
__device__ __forceinline__ uint32_t ring_next(uint32_t x, uint32_t ring_begin, uint32_t ring_end) {
  uint32_t y;
  asm volatile("s_add_u32 %0, %1, %4\n\ts_cmp_lg_u32 %0, %2\n\ts_cselect_b32 %0, %0, %3"
               : "=&s"(y) : "s"(x), "s"(ring_end), "s"(ring_begin), "n"(STEP) : "scc");
  return y;
}
// 64-bit address, kept as two halves, += BYTES.
template <int BYTES>
__device__ __forceinline__ void addr_advance(uint32_t& lo, uint32_t& hi) {
  asm volatile("s_add_u32 %0, %0, %2\n\ts_addc_u32 %1, %1, 0" : "+s"(lo), "+s"(hi) : "n"(BYTES) : "scc");
}
__device__ __forceinline__ void addr_advance(uint32_t& lo, uint32_t& hi, uint32_t bytes) {
  asm volatile("s_add_u32 %0, %0, %2\n\ts_addc_u32 %1, %1, 0" : "+s"(lo), "+s"(hi) : "s"(bytes) : "scc");
}
__device__ __forceinline__ const char* addr_of(uint32_t lo, uint32_t hi) {
  return (const char*)(((uint64_t)hi << 32) | lo);
}

// a fragment (8 bf16 of one row) in the LDS, addressed by its 32-bit LDS address
typedef const __attribute__((address_space(3))) bf16x8* LdsFragPtr;
__device__ __forceinline__ LdsFragPtr lds_frag(uint32_t addr) { return (LdsFragPtr)(uintptr_t)addr; }

// The same, 4 bytes per lane.
template <int IMM>
__device__ __forceinline__ void dma4_at(uint32_t lds_base, uint32_t voff, const char* sbase) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(lds_base), "v"(voff), "s"(sbase), "n"(IMM) : "memory", "scc");
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// Slab layout (the A operand of the gradient GEMM, see "Tile images" below): block
// (row tile, k-step) of 256 rows x 64 vocabulary entries, row r at r * 64 elements, its
// 8-entry chunk c at chunk position c ^ ((r >> 1) & 7).  A 256 x 128 logit tile covers the
// two consecutive blocks 2 vt and 2 vt + 1 of its row tile; `blk` points at the first.
constexpr int kSlabBlock = kTileTokens * kBK;   // elements per block
constexpr int kImgBytesSlab = kSlabBlock * 2;   // 32 KiB

// A staged block of either operand of the gradient GEMM: 256 x 64 entries (see grad_kernels.hip).
constexpr int kImgBytes = kGradTile * kBK * 2;        // 32 KiB

// Heavy entries.  The logit gradient dz = p_s ((z_s - z_t) - mu) is contracted with W_s as
// bf16.  On a peaked row a handful of entries carry the whole gradient row and their rounding
// (2^-9 relative each) does not average out, so every entry with p_s >= kHeavyP is taken out
// of the bf16 operand (stored as an exact zero) and listed per computed row instead; the
// scale-and-scatter kernel recomputes those few logits as fp32 dot products and adds
// dz W_s[v] in fp32.  Probabilities sum to 1, so a row has at most 1 / kHeavyP such entries;
// a flat row (the random-initialisation regime) has none.
constexpr float kHeavyP = 1.f / 32.f;
constexpr int kHeavySlots = 32;
struct HeavyList {
  int32_t* cnt;    // [n_pad] entries listed per computed row (zeroed at the start of a call)
  int32_t* v;      // [n_pad][kHeavySlots] vocabulary indices, in no particular order
};

// Lists entry v of computed row r; false when the row's list is full (the entry then stays in
// the bf16 operand).
__device__ __forceinline__ bool heavy_push(const HeavyList& hl, int64_t r, int v) {
  const int slot = atomicAdd(hl.cnt + r, 1);
  if (slot >= kHeavySlots) return false;
  hl.v[r * kHeavySlots + slot] = v;
  return true;
}

// x . y over H bf16 entries (H a multiple of 8), all 64 lanes of the wave; every lane gets the sum.
__device__ __forceinline__ float dot_bf16_row(const __bf16* x, const __bf16* y, int H, int lane) {
  float acc = 0.f;
  const uint4* px = (const uint4*)x;
  const uint4* py = (const uint4*)y;
  for (int q = lane; q < (H >> 3); q += 64) {
    const uint4 a = px[q], b = py[q];
    acc = fmaf(bf16_lo(a.x), bf16_lo(b.x), acc); acc = fmaf(bf16_hi(a.x), bf16_hi(b.x), acc);
    acc = fmaf(bf16_lo(a.y), bf16_lo(b.y), acc); acc = fmaf(bf16_hi(a.y), bf16_hi(b.y), acc);
    acc = fmaf(bf16_lo(a.z), bf16_lo(b.z), acc); acc = fmaf(bf16_hi(a.z), bf16_hi(b.z), acc);
    acc = fmaf(bf16_lo(a.w), bf16_lo(b.w), acc); acc = fmaf(bf16_hi(a.w), bf16_hi(b.w), acc);
  }
  return wave_sum(acc);
}

// References of the single sweep per computed row (see prepare_kernel): the larger of the maximum
// over vocabulary tile 0 and the logit of the sampled token, as the maximum over `parts` planes: one, or,
// in calls of few token tiles, the four blocks of 32 entries and the token (kMaxRefParts).
constexpr int kRefBlocks = kTileVocab / 32;
constexpr int kMaxRefParts = kRefBlocks + 1;
constexpr int kFineRefTiles = 5;           // see launch_prepare
struct References {
  float* max[2];            // [parts][n_pad] student, teacher; kNegBig: nothing to take the maximum of
  float* zy[2];             // [n_pad] logit of the sampled token (0: none)
  int32_t* yid;             // [n_pad] its id; -1: none, or out of range
  int64_t n_pad;
  int parts;
  // log2 e times the reference, rounded: the number that the sweep takes its exponentials against and that the merge
  // adds back.  Its rounding (2^-18 at 32 nats) is part of the reference and must be the same in both, or KL_t
  // errs by it: the product stays a product, whatever it is added to.
  static __device__ __forceinline__ float scaled(float m) {
    float s = m * kLog2e;
    asm("" : "+v"(s));
    return s;
  }
  __device__ __forceinline__ float of(int head, int64_t r) const {
    if (parts == 1) return scaled(max[head][r]);
    float v[kMaxRefParts];                  // loaded together
#pragma unroll
    for (int k = 0; k < kMaxRefParts; ++k) v[k] = max[head][(k < parts ? k : 0) * n_pad + r];
#pragma unroll
    for (int k = 1; k < kMaxRefParts; ++k) v[0] = fmaxf(v[0], v[k]);
    return scaled(v[0]);
  }
};

// ---------------------------------------------------------------------------------------
// Argument blocks
// ---------------------------------------------------------------------------------------
struct LogitPassArgs {
  const __bf16* h_s; const __bf16* h_t; const __bf16* W_s; const __bf16* W_t;
  int H_s, H_t, V;
  const int32_t* row_idx;      // [n_pad]
  int64_t n_pad;
  int tile0;                   // first token tile of this launch
  int n_tiles;                 // token tiles in this launch
  bool narrow;                 // one token tile, of which only the first 128 rows are wanted (see DmaTile)
  int strips;                  // vocabulary strips
  Shares strip_tiles;          // vocabulary tiles of each (set by launch_logit_pass)
  int long_first;              // the longer strips' workgroups of all token tiles come first (sweep_strips)
  int tg;                      // token tiles per workgroup group (share W tiles in one L2)
  int vt_total;                // vocabulary tiles (of 128)
  // pass 1 out: [5][strips][n_pad]
  float* part;
  // pass 2 in / out
  const float* lse2; const float* mu;
  __bf16* slab; int64_t Vp;    // slab blocks of the launch's token tiles, tile0 first
  // single-sweep mode: fixed per-row references and the offset of the second slab half
  References ref;
  int64_t e2_off;
  bool lines;                  // factors as whole lines, past the caches (sweep_whole_lines)
  // per-(vocabulary tile, slab row) reference mu0 of the D factor, written by the sweep
  float* mu0t; int64_t mu0t_stride;
  // direct-to-LDS kernel: tile images of the four operands (see row_image_kernel)
  const char* Wt_img; const char* Ws_img; const char* ht_img; const char* hs_img;
  int stage;                   // kStage*: where the W tiles come from
  bool rotate;                 // ... the heads of strip s from k-step s on, the first ones last (see rotate_k)
  HeavyList heavy;             // second sweep of the two-sweep scheme: entries taken out of dz
};

// Factors of a slab beyond this are in memory again by the time the next launch reads them, and go past the caches: a
// quarter more than the last-level cache of 256 MiB.  Combine pass, us, kept / past: 297 MiB 74 / 76, 451 MiB 138 / 121.
// The weights of a call likewise (sweep_stage).
constexpr int64_t kPastCacheBytes = (int64_t)320 << 20;

constexpr int kNarrowRows = kTileTokens / 2;

// Where the W tiles of the direct-to-LDS logit kernel come from: tile images; the row-major weights; those, of a single token
// tile, with all lines of W or the teacher's past the caches (sweep_stage).
constexpr int kStageImages = 0, kStageRows = 1, kStageRowsOnce = 2, kStageTeacherOnce = 3;

// Modes of the direct-to-LDS logit kernel.
constexpr int kModeStats = 0;   // online (running-max) statistics only
constexpr int kModeDz = 1;      // second sweep of the two-sweep scheme: dz tiles
constexpr int kModeSingle = 2;  // single sweep: fixed-reference statistics + D/E2 tiles
constexpr int kModeSingleDiag = 3;  // the same plus the teacher-side diagnostics of Sec. 3.1
constexpr int kModeSingleE2 = 4;      // single sweep that emits only the E2 factor (sampled estimator)
constexpr int kModeSingleE2Diag = 5;  // the same plus the diagnostics
constexpr int kModeSingleFwd = 6;     // single sweep, statistics only: nothing is written to the slab
constexpr int kModeSingleFwdDiag = 7; // the same plus the diagnostics

// Tile images of a row-major [rows, H] operand (see row_image_kernel).
struct RowImageArgs {
  const uint4* src; uint4* img;
  int64_t n_rows; int H, nk;
  int permute;     // rows of every group of 32 in the order the logit kernels' epilogues want (W tiles)
};

// Merge of the strip partials into lse, mu, KL_t and c_t.
struct MergeArgs {
  const float* part; int strips; int64_t n_pad; int64_t n_rows;
  const int32_t* row_idx;
  const __bf16* h_s; const __bf16* h_t; const __bf16* W_s; const __bf16* W_t;
  int H_s, H_t, V;
  const int32_t* ids;
  float* lse2; float* mu; float* klr;
  float* lse_s;                // [n_pad] student log-sum-exp in nats (for the heavy entries)
  float* alive;                // [n_pad] two-sweep merge: 1, or 0 for an excluded (non-finite) row
  float* kl; float* c;
  uint32_t* status;
  // teacher-side diagnostics (single-sweep merge only); part planes 3 and 4 hold
  // sum e_t z_t and the rank count when `diag` is set
  int diag;
  float* t_logp; float* t_entropy; int32_t* t_rank;
  float* cr;     // [n_pad] c_t per computed row, for the sampled estimator (else NULL)
};

struct MergeSingleArgs {
  MergeArgs m;                 // part: [3][strips][n_pad] sums Z_s, A, Z_t
  References ref;
  float* mu_out; float* inv_z;
  int64_t row0, rows;          // computed rows [row0, row0 + rows) of this launch (one slab)
};

// What a call prepares for its sweep (see prepare_kernel).
struct PrepareArgs {
  const int32_t* row_idx; const int32_t* ids;     // ids may be NULL
  const __bf16* h[2]; const __bf16* W[2];         // student, teacher
  int H[2]; int V;
  References ref;
  RowImageArgs img[2];                            // of the hidden states
  // workgroups: references (0: none wanted), logits of the sampled tokens, images of h_s, of h_t
  int ref_blocks, dot_blocks, img_blocks[2], setup_blocks;
};

// Combine pass over one slab (see combine_kernel).
struct CombineArgs {
  uint4* slab; int64_t e2_vec;          // E2 lies e2_vec 16-byte vectors after D
  bool past_cache;                      // the factors exceed kPastCacheBytes
  const float* mu; const float* inv_z;      // per computed row
  const float* mu0t; int64_t mu0t_stride;   // reference of D per (vocabulary tile, slab row)
  int64_t row0;                         // computed-row index of slab row 0
  int nk;                               // k-steps (blocks) per row tile
  // TR: also the transpose of w * dz as tile images for the head-weight GEMMs (rows =
  // vocabulary entries in tiles of 256, k = slab rows): block (vt, kr) with kr = 4 rt + j,
  // j = 0..3.  w = grad_scale * alpha of the row under the prefix objective (dzT_p; 0 outside
  // the window) and under the full-rollout objective (dzT_f); the weight is applied in fp32
  // before the one rounding to bf16.  Either image may be NULL.
  uint4* dzT_p; uint4* dzT_f; int nkr;  // k-steps (of 64 slab rows) per vocabulary tile
  DevicePlan pl; int64_t n_rows; float grad_scale;
  // SAMPLED (with TR): the slab holds only E2 and is left as it is; the transposed images take
  // Eq. 4's logit gradient c_t (e_{y_t} - p_s) = c_t (1[v = y_t] - E2 / Z_s), the one-hot term
  // entering before the rounding.  c_t and y_t per computed row (y_t = -1: none).
  const float* cr; const int32_t* yid;
  HeavyList heavy;             // entries with p_s >= kHeavyP leave the bf16 operand (expected estimator)
};

// h_s rows of one slab (see hs_gather_kernel).
struct HsGatherArgs {
  const uint4* h_s; const int32_t* row_idx;
  int64_t row0;
  int H;
  uint4* out;
  const float* alive;     // per computed row; 0: excluded row, written as zeros
};

// Gradient GEMM (see grad_gemm_kernel).
struct GradArgs {
  const __bf16* slab;       // A: tile images
  const __bf16* Bm;         // B: row-major [k_rows][H]
  int nk_total;             // A blocks per tile, k_rows of B rounded up
  int64_t k_rows;
  float* g;                 // [ksplit][g_rows][H]
  int64_t g_rows; int H;
  int64_t slab_row0;        // computed-row index of slab row 0
  int row_tiles, h_tiles, ksplit;
  Shares split_steps;       // k-steps of each piece that hold rows of B (set by launch_grad_gemm)
  int half_tiles;           // slab row tiles >= half_tiles hold the E2 factor: output rows
  int64_t half_off;         // half_off + slab_row0 + ... (single-sweep mode; else half_tiles = row_tiles)
  // Rows of g that are stored: whole blocks of 8, so a multiple of 8, up to 7 more than exist where g has room for them
  int64_t out_rows;
  int accumulate;           // add to g instead of overwriting it
  // A as the two factors of the single sweep: bytes from D to E2 (0: A is the operand itself), and what collapses
  // them (see CombineArgs)
  int64_t e2_bytes;
  const float* mu; const float* inv_z;      // per computed row
  const float* mu0t; int64_t mu0t_stride;   // reference of D per (vocabulary tile, slab row)
  HeavyList heavy;
  bool past_cache;                          // the factors exceed kPastCacheBytes
};

// Scale + scatter of the row gradients (see finalize_kernel).
struct FinalizeArgs {
  DevicePlan pl; int B; int64_t T; int probe; int64_t n_rows;
  float* g; int ksplit; int64_t n_pad; int H;
  int64_t g_rows;                          // rows per k-split plane of g
  const float* inv_z;                      // per computed row: 1 / Z_s (single sweep) or 1 (two sweeps);
                                           // 0 marks an excluded (non-finite) row: zeros everywhere
  // heavy entries: fp32 part of g, from the row's lse_s and mu and fresh dot products
  HeavyList heavy; const float* lse_s; const float* mu;
  const __bf16* h_s; const __bf16* h_t; const __bf16* W_t; int H_t;
  // sampled estimator (Eq. 4): g = c_t (W_s[y_t] - G2 inv_z), G2 = E2 W_s behind the n_pad rows of
  // g; cr NULL: g is the contraction of the logit gradient itself (plane 0 once summed)
  const float* cr; const int32_t* ids; const __bf16* W_s; int V;
  float grad_scale; int dh_bf16;
  void* dh_prefix; void* dh_full;
  float* rownorm;
};

// ---------------------------------------------------------------------------------------
// Launchers (asynchronous on `st`; the return value is that of the launch)
// ---------------------------------------------------------------------------------------
// fused_host.hip
int sweep_strips(int n_tiles, int vt_total, int* long_first);   // vocabulary strips of a sweep, and their order
// sweep_kernels.hip
hipError_t sweep_kernels_opt_in();       // large dynamic LDS of the logit kernels, once per device
hipError_t launch_row_image(const RowImageArgs& a, unsigned tiles, hipStream_t st);
// mode: one of kMode*; dma false selects the register-staged kernel (kModeStats, kModeDz only)
hipError_t launch_logit_pass(int mode, bool dma, const LogitPassArgs& a, hipStream_t st);
// the call's setup and what its sweep needs prepared; `refs`: with the references of the single sweep
hipError_t launch_prepare(const PrepareArgs& a, bool refs, int n_tiles, const SetupArgs& setup,
                          const std::vector<unsigned char>& plan, hipStream_t st);
hipError_t launch_merge_stats(const MergeArgs& a, hipStream_t st);
hipError_t launch_merge_single(const MergeSingleArgs& a, hipStream_t st);
// grad_kernels.hip
hipError_t grad_kernels_opt_in();
hipError_t launch_hs_gather(const HsGatherArgs& a, int64_t rows, hipStream_t st);
hipError_t launch_combine(bool transposed, bool sampled, const CombineArgs& a, int row_tiles, hipStream_t st);
hipError_t launch_grad_gemm(const GradArgs& a, hipStream_t st);
// `tail`: the reductions that end a call without probe gradients, in the same launch (or NULL)
hipError_t launch_finalize(const FinalizeArgs& a, const TailArgs* tail, hipStream_t st);

}  // namespace adwin

#endif  // ADWIN_FUSED_SHARED_H
