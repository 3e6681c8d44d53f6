// Fused path, second half: from the stored gradient factors to dL/dh_s and dL/dW_s.
//
// Combine  : once a slab's rows have their mu, the two factors the sweep stored collapse
//            in place into the logit gradient dz = p_s ((z_s - z_t) - mu) (Eq. 4 in
//            expectation, App. A.1); optionally also the transposed, weighted copies that
//            the head-weight contraction needs.
// GEMM     : g = dz W_s (and dW_s = (w dz)^T h_s) as bf16 MFMA GEMMs over tile images.
// Finalize : scale by grad_scale * alpha, scatter to dh_prefix / dh_full, row norms.
#include "fused_shared.h"
#include "tail_device.h"
#include <utility>

namespace adwin {

// ---------------------------------------------------------------------------------------
// Tile images.  The A operand of the gradient GEMM lives in memory as the exact LDS images
// of its k-steps: block (tile, kt) is 256 rows x 64 k-entries = 32 KiB, row r at r * 128 B,
// its 16-byte chunk c (k-entries 8 c .. 8 c + 7) at chunk position c ^ ((r >> 1) & 7).
// Blocks of one tile are consecutive in kt, so a workgroup streams the operand as one
// sequential run and every wave-load moves 1 KiB of consecutive bytes.  The B operand is read
// from its row-major rows (one row per k-entry) and transposed on the way out of the LDS.
// ---------------------------------------------------------------------------------------

// ---------------------------------------------------------------------------------------
// Combine.  Once a slab's rows have their mu (all strips merged), the two stored factors
// collapse into the logit gradient itself, dz = E2 (D - (mu - mu0)) / Z_s = p_s (d - mu),
// written over D in the same image order, and the gradient GEMM runs on one factor.  A
// streaming pass: 4 B read + 2 B written per slab element.
// PAST: all of that past the caches (non-temporal), for slabs that exceed the last-level one (kPastCacheBytes): whatever
// line is kept for the factors or for dz is evicted before anything asks for it.  us per pass, kept / past: 4,096
// rows of V = 151,936 760 / 635 (4.9 and 5.9 TB/s), 24,000 rows 4540 / 3760, 1,286 rows 242 / 198; with the transposed copy,
// 8,192 rows, 2050 / 1859; the GEMM that reads dz next 4090 / 4020 for the 24,000 rows (with the loads alone past the caches
// the pass takes 4180 and the GEMM is 2 % slower).  3,139 rows of V = 11,912, a slab of 150 MB: 37 / 41.
// ---------------------------------------------------------------------------------------
template <bool PAST>
__device__ __forceinline__ uint4 slab_load(const uint4* p) {
  if constexpr (!PAST) return *p;
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool PAST>
__device__ __forceinline__ void slab_store(uint4* p, const uint4& v) {
  if constexpr (!PAST) { *p = v; return; }
  const u32x4 x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, (u32x4*)p);
}

template <bool TR, bool SAMPLED, bool PAST>
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a) {
  // one workgroup per block (row tile rt = blockIdx.y, kt = blockIdx.x): 2048 vectors of 8
  // entries; vector q holds row q / 8, chunk position q % 8
  __shared__ __align__(16) uint16_t tile[TR ? kTileTokens : 1][TR ? kBK + 8 : 1];   // [row][entry], padded
  __shared__ float wrow[2][TR ? kTileTokens : 1];
  const int kt = blockIdx.x, rt = blockIdx.y;
  const int64_t blk = (int64_t)rt * a.nk + kt;
  uint4* p1 = a.slab + blk * (kImgBytesSlab / 16);
  const uint4* p2 = p1 + a.e2_vec;
  const int64_t rbase = a.row0 + (int64_t)rt * kTileTokens;
  if (TR) {
    const int64_t r = rbase + threadIdx.x;
    float wp = 0.f, wf = 0.f;
    if (r < a.n_rows && a.inv_z[r] != 0.f) {     // excluded rows carry weight 0
      const int i = a.pl.row_seq[r];
      wf = a.grad_scale * a.pl.alpha_f[i];
      wp = (r - a.pl.comp_off[i]) < a.pl.n[i] ? a.grad_scale * a.pl.alpha_p[i] : 0.f;
    }
    wrow[0][threadIdx.x] = wp;
    wrow[1][threadIdx.x] = wf;
    __syncthreads();
  }
  float dz[TR ? 8 : 1][8];
  // kTogether vectors of each factor and what belongs to their rows are loaded before the first is looked at:
  // in a call of few rows nothing else covers the round trips (118 rows of V = 4,096: 44.1 -> 42.6 us per
  // call; large calls, where waves are many: the same within 0.3 %)
  constexpr int kTogether = TR ? 2 : 4;
  // Rows that do not exist, of a call of few rows most of its only tile, are left as they are: what the GEMM makes
  // of them nobody reads.  (The transposed operand is contracted over the rows, and has zeros there.)
  // 128 rows of V = 151,936: combine pass 35 -> 19 us; 16 rows 35 -> 7.
  const int64_t left = TR ? kTileTokens : a.n_rows - rbase;
#pragma unroll
  for (int i0 = 0; i0 < 8; i0 += kTogether) {
    if (!TR && i0 * 32 >= left) break;
    uint4 xs[kTogether], ys[kTogether];
    float izs[kTogether], ms[kTogether], m0s[kTogether];
    int ids[kTogether];
#pragma unroll
    for (int j = 0; j < kTogether; ++j) {
      const int q = (i0 + j) * 256 + threadIdx.x;
      const int64_t r = rbase + (q >> 3);
      if (!TR && (i0 + j) * 32 >= left) continue;
      ys[j] = slab_load<PAST>(p2 + q);
      izs[j] = a.inv_z[r];
      if (SAMPLED) {
        ms[j] = a.cr[r];
        ids[j] = a.yid[r];
      } else {
        xs[j] = slab_load<PAST>(p1 + q);
        ms[j] = a.mu[r];
        m0s[j] = a.mu0t[(int64_t)(kt >> 1) * a.mu0t_stride + rt * kTileTokens + (q >> 3)];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kTogether; ++j) {
      const int i = i0 + j, q = i * 256 + threadIdx.x;
      const int64_t r = rbase + (q >> 3);
      if (!TR && i * 32 >= left) continue;
      const float iz = izs[j];
      const uint4 y = ys[j];
      float d[8];
      if (SAMPLED) {
        const float c = ms[j], ciz = -c * iz;
        d[0] = bf16_lo(y.x) * ciz; d[1] = bf16_hi(y.x) * ciz; d[2] = bf16_lo(y.y) * ciz; d[3] = bf16_hi(y.y) * ciz;
        d[4] = bf16_lo(y.z) * ciz; d[5] = bf16_hi(y.z) * ciz; d[6] = bf16_lo(y.w) * ciz; d[7] = bf16_hi(y.w) * ciz;
        // entries of this vector: 64 kt + 8 (logical chunk) + e
        const int rl = q >> 3, v0 = kt * kBK + (((q & 7) ^ ((rl >> 1) & 7)) << 3);
        const int e_y = ids[j] - v0;
#pragma unroll
        for (int e = 0; e < 8; ++e) d[e] += (e == e_y) ? c : 0.f;
        if (TR) {
#pragma unroll
          for (int e = 0; e < 8; ++e) dz[i][e] = d[e];
        }
      } else {
        const float dl = ms[j] - m0s[j];
        const uint4 x = xs[j];
        float pv[8], xv[8];                      // p_s and the stored D of the vector's 8 entries
        pv[0] = bf16_lo(y.x) * iz; pv[1] = bf16_hi(y.x) * iz; pv[2] = bf16_lo(y.y) * iz; pv[3] = bf16_hi(y.y) * iz;
        pv[4] = bf16_lo(y.z) * iz; pv[5] = bf16_hi(y.z) * iz; pv[6] = bf16_lo(y.w) * iz; pv[7] = bf16_hi(y.w) * iz;
        xv[0] = bf16_lo(x.x); xv[1] = bf16_hi(x.x); xv[2] = bf16_lo(x.y); xv[3] = bf16_hi(x.y);
        xv[4] = bf16_lo(x.z); xv[5] = bf16_hi(x.z); xv[6] = bf16_lo(x.w); xv[7] = bf16_hi(x.w);
        const bool dead = iz == 0.f;             // excluded row: its factors may hold inf / NaN
        float pmax = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          d[e] = dead ? 0.f : (xv[e] - dl) * pv[e];
          pmax = fmaxf(pmax, pv[e]);
        }
        if (TR) {                                // the head-weight operand keeps every entry in bf16
#pragma unroll
          for (int e = 0; e < 8; ++e) dz[i][e] = d[e];
        }
        if (__builtin_expect(pmax >= kHeavyP && !dead, 0)) {
          // entries of this vector: 64 kt + 8 (logical chunk) + e
          const int rl = q >> 3, v0 = kt * kBK + (((q & 7) ^ ((rl >> 1) & 7)) << 3);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (pv[e] >= kHeavyP && heavy_push(a.heavy, r, v0 + e)) d[e] = 0.f;
        }
        uint4 o;
        o.x = pack_bf16(d[0], d[1]); o.y = pack_bf16(d[2], d[3]);
        o.z = pack_bf16(d[4], d[5]); o.w = pack_bf16(d[6], d[7]);
        slab_store<PAST>(p1 + q, o);
      }
    }
  }
  if (TR) {
    // this block's 64 entries are image rows (kt % 4) * 64 .. + 64 of vocabulary tile kt / 4;
    // its 256 slab rows are the k-steps 4 rt .. 4 rt + 3.  Vector u: k-step u / 512, image
    // row (u / 8) % 64, chunk position u % 8 -> one wave instruction writes 8 whole rows.
    const int vt = kt >> 2, row0 = (kt & 3) * kBK;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      uint4* dst = which == 0 ? a.dzT_p : a.dzT_f;
      if (!dst) continue;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int q = i * 256 + threadIdx.x;
        const int rl = q >> 3;
        const float w = wrow[which][rl];
        const int c = (q & 7) ^ ((rl >> 1) & 7);             // logical chunk: entries 8 c .. 8 c + 7
        uint4 o = make_uint4(0u, 0u, 0u, 0u);     // rows of weight zero (padding too) are exact zeros
        if (w != 0.f) {
          o.x = pack_bf16(w * dz[i][0], w * dz[i][1]); o.y = pack_bf16(w * dz[i][2], w * dz[i][3]);
          o.z = pack_bf16(w * dz[i][4], w * dz[i][5]); o.w = pack_bf16(w * dz[i][6], w * dz[i][7]);
        }
        *(uint4*)&tile[rl][c * 8] = o;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int u = i * 256 + threadIdx.x;
        const int j = u >> 9, vl = (u >> 3) & 63, pos = u & 7;
        const int imgrow = row0 + vl;
        const int c = pos ^ ((imgrow >> 1) & 7);             // slab rows 64 j + 8 c .. + 7
        const int rl = j * kBK + c * 8;
        uint4 o;
        o.x = tile[rl + 0][vl] | ((uint32_t)tile[rl + 1][vl] << 16);
        o.y = tile[rl + 2][vl] | ((uint32_t)tile[rl + 3][vl] << 16);
        o.z = tile[rl + 4][vl] | ((uint32_t)tile[rl + 5][vl] << 16);
        o.w = tile[rl + 6][vl] | ((uint32_t)tile[rl + 7][vl] << 16);
        slab_store<PAST>(dst + (((int64_t)vt * a.nkr + 4 * rt + j) * kGradTile + imgrow) * 8 + pos, o);
      }
    }
  }
}

// The student hidden states of one slab, the B operand of the head-weight GEMMs: row r =
// h_s[row_idx[row0 + r]], zeros for an excluded row (it carries weight 0 in the other operand;
// its own entries, possibly inf or NaN, must not meet that 0 in the product).  One wave per row.
__global__ __launch_bounds__(256) void hs_gather_kernel(HsGatherArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), r = a.row0 + k;   // rows: a multiple of 4
  const bool alive = a.alive[r] != 0.f;
  const uint4* src = a.h_s + (int64_t)a.row_idx[r] * (a.H >> 3);
  uint4* dst = a.out + k * (a.H >> 3);
  for (int q = lane; q < (a.H >> 3); q += 64) {
    uint4 v = src[q];                      // (a choice between src[q] and a zero vector puts that vector into scratch memory)
    if (!alive) v = make_uint4(0u, 0u, 0u, 0u);
    dst[q] = v;
  }
}

// ---------------------------------------------------------------------------------------
// Pass 3: g[r][h] = sum_v dz[r][v] W_s[v][h].  256 x 256 output tile, 2 x 2 waves of
// 128 x 128.  A = slab rows (i = row), B = columns of W_s (j = hidden column, contiguous in
// g).  B stays row-major: a k-step stages 64 rows of W_s x 256 columns, 512 B of a row at a time,
// and the fragments (one column, 8 consecutive rows) come out of the LDS by transposing reads
// (ds_read_b64_tr_b16: each group of 16 lanes reads a 4 x 16 block and lane i receives its
// column i).  No transposed copy of W_s exists: building one took 730 us of every call at
// V = 151,936, H_s = 2048 (1.25 GB) and a workspace of the size of W_s.
// Row v of a staged block lies at 512 v, its 16-byte chunk c (columns 8 c .. 8 c + 7) at chunk
// position c ^ (4 (v & 3)): the four rows that 16 lanes read then fall on four different
// 64-byte quarters of the 256 bytes that the 64 banks cover (SQ_LDS_BANK_CONFLICT reads 0 over a
// launch of 16,384 rows at V = 151,936, H_s = 2048; matrix pipe busy 92 %, 7.0 ms).
// The k-steps (one 32 KiB block of each operand) go through five block buffers in the
// LDS, three for B and two for A, by direct global->LDS loads.  Per k-step a wave issues
// its 16 wave-loads of the k-step after next in the shadow of MFMAs (see grad_kstep), so
// that they have a k-step or more (upwards of 2000 matrix-pipe cycles) to land.  The one
// barrier per k-step sits before the last of the four k16 sub-steps: by then every fragment
// of the current blocks is in registers, so the last sub-step's MFMAs cover the LDS reads of
// the next blocks' first fragments and the matrix pipe never waits for LDS after a barrier.
// ---------------------------------------------------------------------------------------

// Five block buffers fill the 160 KiB of LDS: a ring of three for the B operand and a ring
// of two for the A operand.
constexpr int kGradRing3 = 3;
constexpr int kGradRing2Off = kGradRing3 * kImgBytes;         // the ring of two follows
constexpr int kGradLds = (kGradRing3 + 2) * kImgBytes;        // 160 KiB
constexpr int kGradRowBytes = kGradTile * 2;                  // a staged row of B: 256 columns
constexpr int kGradSubBytes = 16 * kGradRowBytes;             // the 16 rows of a sub-step

// A B fragment: 8 consecutive rows (k-entries) of one column, as two transposing reads of four.
// addr: the lane's address in rows 0..3 of its half of sub-step 0; OFF: the sub-step.
typedef short s16x4 __attribute__((ext_vector_type(4)));
template <int OFF>
__device__ __forceinline__ s16x4 lds_read_tr(uint32_t addr) {
  typedef __attribute__((address_space(3))) s16x4* Ptr;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((Ptr)(uintptr_t)addr + OFF / 8);
}
__device__ __forceinline__ bf16x8 tr_frag(s16x4 lo, s16x4 hi) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x8 f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, f);
}
template <int OFF>
__device__ __forceinline__ bf16x8 lds_frag_tr(uint32_t addr) {
  return tr_frag(lds_read_tr<OFF>(addr), lds_read_tr<OFF + 4 * kGradRowBytes>(addr));
}

// LOADS: in k-step s the B block of k-step s + 2 is loaded in sub-steps 1 and 2, four
// wave-loads behind the last MFMAs of each (`early`: into the third buffer of its ring, which
// no wave reads any more once it has passed the previous step's barrier; all eight in one
// sub-step, whichever, is 1 % slower) and the A block of k-step s + 2 in sub-step 3 (`late`: after this step's
// barrier, into the buffer of the ring of two that this step has just finished reading).
// The early operand has a lead of a k-step and a quarter to a half, the late one of one k-step.  Which
// operand gets which was measured: in `dz W_s` every XCD streams all of W_s^T (B) once per
// round of tiles while a slab block (A) is fetched by one XCD only, and the deeper lead on
// B is worth 2 % (on A 4 % against no third buffer at all).  Loads return in order: the wait
// before the barrier leaves the youngest eight, this step's early loads, in flight.
// Ring state (wave-uniform, LDS addresses that include the wave's KiB, which the loads want and
// the fragment offsets swA/swB take out again): r_a, r_b = the A and B buffers this k-step
// reads, on return those of the next k-step.  (pa, pb) = the blocks loaded by the previous
// k-step, on return those loaded by this one.  voffd[d] = 16 lane + 1024 wave + 4096 d.  The
// ring and address arithmetic sits in the shadows of the first MFMAs (see ring_next).
template <bool LOADS, bool LAST>
__device__ __forceinline__ void grad_kstep(f32x16 (&acc)[4][4], bf16x8 (&fa)[2][4], bf16x8 (&fb)[2][4],
                                           uint32_t& r_a, uint32_t& r_b, uint32_t a_begin, uint32_t a_end,
                                           uint32_t b_begin, uint32_t b_end, const uint32_t (&swA)[4],
                                           const uint32_t (&swB)[4], const uint32_t (&voffd)[8],
                                           const uint32_t (&voffb)[8], uint32_t b_step,
                                           uint32_t& pa_lo, uint32_t& pa_hi, uint32_t& pb_lo, uint32_t& pb_hi) {
  uint32_t r_a_nx = 0, r_b_nx = 0, r_b_wr = 0;
  uint32_t xa = 0;              // the lane's LDS address of its first A fragment of a sub-step
  uint32_t xb[4];               // ... and of its part of the four B fragments of a sub-step
#define ADWIN_FENCE __builtin_amdgcn_sched_barrier(0);
#define ADWIN_MM(KK, I, J)                                                                    \
  acc[I][J] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[(KK) & 1][I], fb[(KK) & 1][J],       \
                                                      acc[I][J], 0, 0, 0);                    \
  ADWIN_FENCE
  // side operation M (0..15) in the shadow of MFMA M of sub-step KK: fragment reads of the
  // next sub-step (from this step's buffers, in sub-step 3 from the next step's; a B fragment is
  // two transposing reads, k-entries 0..3 and 4..7 of the lane's eight), the ring and
  // address arithmetic (sub-step 0), then (sub-steps 1, 2 and 3) the wave-loads of the k-step
  // after next: 4 KiB groups d = 0..7 of the early block, then of the late block
#define ADWIN_SIDE(KK, M)                                                                           \
  if constexpr ((M) < 8 && ((KK) < 3 || !LAST)) {                                                   \
    constexpr int ad_n = ((KK) + 1) & 3, ad_f = ((M) >> 1) & 3;                                     \
    if constexpr ((M) == 0) {                                                                       \
      xa = ((KK) < 3 ? r_a : r_a_nx) + swA[ad_n];                                                   \
      asm volatile("" : "+v"(xa));                                                                  \
    }                                                                                               \
    if constexpr (((M) & 1) == 0) {                                                                 \
      fa[ad_n & 1][ad_f] = lds_frag(xa)[ad_f * 32 * kRowBytes / 16];                                \
      if constexpr ((KK) == 0 || (KK) == 3) {                                                       \
        xb[ad_f] = ((KK) < 3 ? r_b : r_b_nx) + swB[ad_f];                                           \
        asm volatile("" : "+v"(xb[ad_f]));                                                          \
      }                                                                                             \
    } else {                                                                                        \
      fb[ad_n & 1][ad_f] = lds_frag_tr<ad_n * kGradSubBytes>(xb[ad_f]);                             \
    }                                                                                               \
    if constexpr ((KK) == 0 && (M) == 0 && !LAST) r_b_nx = ring_next<kImgBytes>(r_b, b_begin, b_end); \
    if constexpr ((KK) == 0 && (M) == 1 && !LAST) r_a_nx = ring_next<kImgBytes>(r_a, a_begin, a_end); \
    if constexpr ((KK) == 0 && (M) == 2 && LOADS) r_b_wr = ring_next<kImgBytes>(r_b_nx, b_begin, b_end); \
    if constexpr ((KK) == 0 && (M) == 3 && LOADS) addr_advance(pb_lo, pb_hi, b_step);               \
    if constexpr ((KK) == 0 && (M) == 4 && LOADS) addr_advance<kImgBytes>(pa_lo, pa_hi);            \
    ADWIN_FENCE                                                                                     \
  } else if constexpr (((KK) == 1 || (KK) == 2) && (M) >= 12 && LOADS) {                            \
    dma16_at<(((KK) - 1) * 4 + (M) - 12) * 4096>(r_b_wr, voffb[(((KK) - 1) * 4 + (M) - 12) & 7], addr_of(pb_lo, pb_hi)); \
    ADWIN_FENCE                                                                                     \
  } else if constexpr ((KK) == 3 && (M) >= 8 && LOADS) {                                            \
    dma16_at<((M) - 8) * 4096>(r_a, voffd[((M) - 8) & 7], addr_of(pa_lo, pa_hi));                         \
    ADWIN_FENCE                                                                                     \
  }
#define ADWIN_ROW(KK, I, M0)                                                    \
  ADWIN_MM(KK, I, 0) ADWIN_SIDE(KK, (M0) + 0) ADWIN_MM(KK, I, 1) ADWIN_SIDE(KK, (M0) + 1) \
  ADWIN_MM(KK, I, 2) ADWIN_SIDE(KK, (M0) + 2) ADWIN_MM(KK, I, 3) ADWIN_SIDE(KK, (M0) + 3)
#define ADWIN_SUB(KK) ADWIN_ROW(KK, 0, 0) ADWIN_ROW(KK, 1, 4) ADWIN_ROW(KK, 2, 8) ADWIN_ROW(KK, 3, 12)
  ADWIN_FENCE
  ADWIN_SUB(0)
  ADWIN_SUB(1)
  ADWIN_SUB(2)
  // every fragment of this stage is in registers; the next stage's loads must have landed
  // before its first fragments are read in the shadow of the last sub-step
  if constexpr (!LAST) {
    if constexpr (LOADS) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
  }
  ADWIN_FENCE
  ADWIN_SUB(3)
  if constexpr (!LAST) { r_a = r_a_nx; r_b = r_b_nx; }
#undef ADWIN_SUB
#undef ADWIN_ROW
#undef ADWIN_SIDE
#undef ADWIN_MM
#undef ADWIN_FENCE
}

// The factors D and E2 of a k-step on their way to an A block (grad_gemm_kernel<true>, which has no combine pass before
// it): they are loaded into registers, asked for a k-step ahead of their conversion, and dz = E2 (D - (mu - mu0)) / Z_s
// goes into the LDS two k-steps ahead of its use.  Each of the eight vectors that a lane has in flight is loaded again as soon
// as it has been converted.  The compiler's waits for them do not count the eight loads of the B block (inline assembly) that
// are asked for between them: vmcnt(21) before vector 0 and vmcnt(18) before the others stand where 29 and 26 loads are
// younger, so that each also waits for up to eight younger loads, vector 0 for those of vector 3, and the time that a load
// has is two sub-steps, half a k-step.  Vector j of a lane belongs at byte 4096 j + 1024 wave + 16 lane of the block, i.e. to
// row 8 (4 j + wave) + lane / 8.  PAST: the lines of the factors past the caches, where one column tile reads them once.
template <bool PAST>
struct FactorLoads {
  uint4 x[8], y[8];            // D and E2
  float m0[8];                 // the reference of D: one per row and vocabulary tile
  float mu[8], iz[8];          // of the row, the whole piece long; iz = inf: a row that is excluded or not there
  __amdgpu_buffer_rsrc_t rx, ry, rm;
  uint32_t off_m;              // of the lane's first row in the references
  uint32_t soff;               // of the k-step that is loaded next
  int kt; uint32_t m0_step;    // its number in the contraction, bytes per vocabulary tile in the references

  __device__ __forceinline__ void load_part(int part, int j, uint32_t voff) {
    if (part == 1) x[j] = row_load(rx, voff);
    else if (part == 2) y[j] = row_load(ry, voff);
    else m0[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rm, (int)(off_m + j * 128), (int)((uint32_t)(kt >> 1) * m0_step), 0));
  }
  __device__ __forceinline__ void load(int j, uint32_t voff) {
    load_part(1, j, voff); load_part(2, j, voff); load_part(3, j, voff);
  }
  __device__ __forceinline__ uint4 row_load(__amdgpu_buffer_rsrc_t r, uint32_t voff) const {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, PAST ? 2 : 0);
    return make_uint4(v.x, v.y, v.z, v.w);
  }
  __device__ __forceinline__ void next() { soff += kImgBytes; ++kt; }
};

// Entries of a vector that do not go into the product: those of a row that is excluded, and the heavy ones, which
// the workgroups of the first column tile list.  (The others need not ask whether the list had room: 33 entries of
// p >= 1/32, each up to 2^-9 too large as a bf16, would add up to more than 1.)
__device__ __forceinline__ void collapse_rare(const GradArgs& a, const uint4& y, float iz, int64_t row, int v0, bool list, uint32_t (&o)[4]) {
  int r = (int)row;
  asm volatile("" : "+v"(r));        // the addresses of the lists are formed here: kept by the loop, they spilled
  if (iz == __builtin_inff()) {
    o[0] = o[1] = o[2] = o[3] = 0u;
    return;
  }
#pragma unroll 1
  for (int w = 0; w < 4; ++w) {
    const uint32_t yw = w == 0 ? y.x : w == 1 ? y.y : w == 2 ? y.z : y.w;
    uint32_t keep = 0xffffffffu;
    if (bf16_lo(yw) * iz >= kHeavyP && (!list || heavy_push(a.heavy, r, v0 + 2 * w))) keep &= 0xffff0000u;
    if (bf16_hi(yw) * iz >= kHeavyP && (!list || heavy_push(a.heavy, r, v0 + 2 * w + 1))) keep &= 0x0000ffffu;
    if (w == 0) o[0] &= keep; else if (w == 1) o[1] &= keep; else if (w == 2) o[2] &= keep; else o[3] &= keep;
  }
}

// A k-step of grad_gemm_kernel<true>.  LOADS: load the factors of k-step s + 3.  MORE: convert those of k-step s + 2 behind
// the MFMAs, and load its B block.  The A blocks are written from sub-step 0 on, into the third buffer of
// their ring, so it is the B blocks that have the ring of two here and are loaded behind the barrier.
// What bounds it, 4,000 rows of V = 151,936, H_s = 512 (2,500 rows, H_s = 768 the same): the wave, alone on its SIMD, issues
// 62 % of the time (SQ_ACTIVE_INST_ANY; 650 instructions in a k-step, 370 of them convert), waits 24 % for loads and LDS reads
// (SQ_WAIT_ANY; 9 % in the GEMM on dz) and 14 % for its turn to issue; the matrix pipe is busy half of the time, and
// a k-step takes 2.3 us for 1.4 after a combine pass.  3,139 rows of V = 11,912, 21 k-steps to a workgroup: 49, 36 and 15 %, pipe
// 32 %: prologue and epilogue.  4,096 rows of V = 50,000, H_s = 256, past the caches: 49, 27 and 24 %, pipe 37 %.  Touching
// the factors' lines a k-step or two ahead made it 11 % slower, in the same queue of loads.  Two entries at a time, their last products
// behind the MFMA after the one that covers the first ones, the loads behind three MFMAs and one fragment read
// to each of twelve: 2,500 rows of V = 151,936, H_s = 768 724 -> 696 us, 1,000 rows, H_s = 512 207 -> 200, against an entry
// at a time from end to end.  Combine pass and GEMM / this: 4,096 rows of V = 50,000, H_s = 256 305 / 170 us (180 with the
// factors' lines kept); 6,000 rows of V = 151,936, H_s = 512 1645 / 1172.
template <bool LOADS, bool MORE, bool LAST, bool PAST>
__device__ __forceinline__ void grad_kstep_factors(const GradArgs& a, FactorLoads<PAST>& f, f32x16 (&acc)[4][4], bf16x8 (&fa)[2][4], bf16x8 (&fb)[2][4],
                                           uint32_t& r_a, uint32_t& r_b, uint32_t a_begin, uint32_t a_end,
                                           uint32_t b_begin, uint32_t b_end, const uint32_t (&swA)[4],
                                           const uint32_t (&swB)[4], const uint32_t (&voffd)[8],
                                           const uint32_t (&voffb)[8], uint32_t b_step,
                                           uint32_t& pb_lo, uint32_t& pb_hi, int64_t row0, int v0, bool list) {
  uint32_t r_a_nx = 0, r_b_nx = 0, r_a_wr = 0;
  uint32_t xa = 0, xb[4];
  float ndl = 0.f, pm = 0.f, x_lo = 0.f, x_hi = 0.f, y_lo = 0.f, y_hi = 0.f;
  s16x4 tr_lo;
  uint32_t o[4];
  const uint32_t lane16 = (threadIdx.x & 63) * 16u;
#define ADWIN_FENCE __builtin_amdgcn_sched_barrier(0);
#define ADWIN_MM(KK, I, J)                                                                    \
  acc[I][J] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[(KK) & 1][I], fb[(KK) & 1][J],       \
                                                      acc[I][J], 0, 0, 0);                    \
  ADWIN_FENCE
#define ADWIN_SIDE(KK, M)                                                                           \
  if constexpr ((M) < 12 && ((KK) < 3 || !LAST)) {                                                  \
    /* one read of a fragment of the next sub-step: A 0, the two halves of B 0 .. 3, A 1 .. 3 */    \
    constexpr int ad_n = ((KK) + 1) & 3;                                                            \
    if constexpr ((M) == 0) {                                                                       \
      xa = ((KK) < 3 ? r_a : r_a_nx) + swA[ad_n];                                                   \
      asm volatile("" : "+v"(xa));                                                                  \
    }                                                                                               \
    if constexpr ((M) == 0 || (M) > 8) {                                                            \
      constexpr int ad_f = (M) == 0 ? 0 : (M) & 3;                                                  \
      fa[ad_n & 1][ad_f] = lds_frag(xa)[ad_f * 32 * kRowBytes / 16];                                \
    } else {                                                                                        \
      constexpr int ad_f = (((M) - 1) >> 1) & 3;                                                    \
      if constexpr (((M) & 1) == 1) {                                                               \
        if constexpr ((KK) == 0 || (KK) == 3) {                                                     \
          xb[ad_f] = ((KK) < 3 ? r_b : r_b_nx) + swB[ad_f];                                         \
          asm volatile("" : "+v"(xb[ad_f]));                                                        \
        }                                                                                           \
        tr_lo = lds_read_tr<ad_n * kGradSubBytes>(xb[ad_f]);                                        \
      } else {                                                                                      \
        fb[ad_n & 1][ad_f] = tr_frag(tr_lo, lds_read_tr<ad_n * kGradSubBytes + 4 * kGradRowBytes>(xb[ad_f])); \
      }                                                                                             \
    }                                                                                               \
    if constexpr ((KK) == 0 && (M) == 0 && !LAST) r_b_nx = ring_next<kImgBytes>(r_b, b_begin, b_end); \
    if constexpr ((KK) == 0 && (M) == 1 && !LAST) r_a_nx = ring_next<kImgBytes>(r_a, a_begin, a_end); \
    if constexpr ((KK) == 0 && (M) == 2 && MORE) r_a_wr = ring_next<kImgBytes>(r_a_nx, a_begin, a_end); \
    if constexpr ((KK) == 0 && (M) == 3 && MORE) addr_advance(pb_lo, pb_hi, b_step);               \
  }                                                                                                 \
  if constexpr (MORE) {                                                                             \
    if constexpr ((KK) == 3 && (M) >= 8)                                                            \
      dma16_at<((M) - 8) * 4096>(r_b, voffb[((M) - 8) & 7], addr_of(pb_lo, pb_hi));                 \
    constexpr int ad_j = 2 * (KK) + ((M) >> 3), ad_e = (M) & 7, ad_w = ad_e >> 1;                   \
    /* the pair before: the products of an entry wait for no result that was only just asked for */ \
    if constexpr ((ad_e & 1) == 0 && (ad_j > 0 || ad_e > 0)) ADWIN_PAIR_END((ad_w + 3) & 3)         \
    if constexpr (ad_e == 0 && ad_j > 0) ADWIN_VECTOR_END((ad_j + 7) & 7)                           \
    if constexpr (LOADS && ad_j > 0 && ad_e >= 1 && ad_e <= 3) f.load_part(ad_e, (ad_j + 7) & 7, voffd[(ad_j + 7) & 7]); \
    const uint32_t ad_x = ad_w == 0 ? f.x[ad_j].x : ad_w == 1 ? f.x[ad_j].y : ad_w == 2 ? f.x[ad_j].z : f.x[ad_j].w; \
    const uint32_t ad_y = ad_w == 0 ? f.y[ad_j].x : ad_w == 1 ? f.y[ad_j].y : ad_w == 2 ? f.y[ad_j].z : f.y[ad_j].w; \
    if constexpr ((ad_e & 1) == 0) {                                                                \
      if constexpr (ad_e == 0) { ndl = (f.m0[ad_j] - f.mu[ad_j]) * f.iz[ad_j]; pm = 0.f; }          \
      x_lo = bf16_lo(ad_x); x_hi = bf16_hi(ad_x);                                                   \
    } else {                                                                                        \
      y_lo = bf16_lo(ad_y); y_hi = bf16_hi(ad_y);                                                   \
      x_lo = fmaf(x_lo, f.iz[ad_j], ndl); x_hi = fmaf(x_hi, f.iz[ad_j], ndl);                       \
      pm = fmaxf(fmaxf(pm, y_lo), y_hi);                                                            \
    }                                                                                               \
    if constexpr (ad_j == 7 && ad_e == 7) {                                                         \
      ADWIN_PAIR_END(3)                                                                             \
      ADWIN_VECTOR_END(7)                                                                           \
      if constexpr (LOADS) f.load(7, voffd[7]);                                                     \
    }                                                                                               \
  }                                                                                                 \
  ADWIN_FENCE
#define ADWIN_PAIR_END(W) {                                                                         \
    asm volatile("" : "+v"(x_lo), "+v"(x_hi));      /* here, not right behind what they wait for */  \
    o[W] = pack_bf16(y_lo * x_lo, y_hi * x_hi);                                                     \
  }
#define ADWIN_VECTOR_END(J) {                                                                       \
    if (__builtin_expect(__any(!(pm * f.iz[J] < kHeavyP)), 0)) {                                    \
      if (!(pm * f.iz[J] < kHeavyP)) collapse_rare(a, f.y[J], f.iz[J], row0 + (J) * 32, v0, list, o); \
    }                                                                                               \
    u32x4 ad_o; ad_o.x = o[0]; ad_o.y = o[1]; ad_o.z = o[2]; ad_o.w = o[3];                         \
    *((__attribute__((address_space(3))) u32x4*)(uintptr_t)(r_a_wr + lane16) + (J) * 4096 / 16) = ad_o; \
  }
#define ADWIN_ROW(KK, I, M0)                                                    \
  ADWIN_MM(KK, I, 0) { ADWIN_SIDE(KK, (M0) + 0) } ADWIN_MM(KK, I, 1) { ADWIN_SIDE(KK, (M0) + 1) } \
  ADWIN_MM(KK, I, 2) { ADWIN_SIDE(KK, (M0) + 2) } ADWIN_MM(KK, I, 3) { ADWIN_SIDE(KK, (M0) + 3) }
#define ADWIN_SUB(KK) ADWIN_ROW(KK, 0, 0) ADWIN_ROW(KK, 1, 4) ADWIN_ROW(KK, 2, 8) ADWIN_ROW(KK, 3, 12)
  ADWIN_FENCE
  ADWIN_SUB(0)
  ADWIN_SUB(1)
  ADWIN_SUB(2)
  if constexpr (!LAST) {
    // The B block of the next k-step was asked for in the last sub-step of the previous one; behind it came the
    // loads of six vectors, three each.
    if constexpr (LOADS) asm volatile("s_waitcnt vmcnt(18) lgkmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
  }
  ADWIN_FENCE
  ADWIN_SUB(3)
  if constexpr (!LAST) { r_a = r_a_nx; r_b = r_b_nx; }
#undef ADWIN_SUB
#undef ADWIN_ROW
#undef ADWIN_VECTOR_END
#undef ADWIN_PAIR_END
#undef ADWIN_SIDE
#undef ADWIN_MM
#undef ADWIN_FENCE
}

// A whole A block from its factors: the first two of a piece.
template <class F>
__device__ __forceinline__ void collapse_block(const GradArgs& a, const F& f, const uint4 (&x)[8], const uint4 (&y)[8], const float (&m0)[8],
                                               uint32_t lds, int64_t row0, int v0, bool list) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float iz = f.iz[j], ndl = (m0[j] - f.mu[j]) * iz;
    const uint32_t xw[4] = {x[j].x, x[j].y, x[j].z, x[j].w}, yw[4] = {y[j].x, y[j].y, y[j].z, y[j].w};
    uint32_t o[4];
    float pm = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float lo = bf16_lo(yw[w]), hi = bf16_hi(yw[w]);
      o[w] = pack_bf16(lo * fmaf(bf16_lo(xw[w]), iz, ndl), hi * fmaf(bf16_hi(xw[w]), iz, ndl));
      pm = fmaxf(pm, fmaxf(lo, hi));
    }
    if (__builtin_expect(!(pm * iz < kHeavyP), 0)) collapse_rare(a, y[j], iz, row0 + j * 32, v0, list, o);
    u32x4 v; v.x = o[0]; v.y = o[1]; v.z = o[2]; v.w = o[3];
    *((__attribute__((address_space(3))) u32x4*)(uintptr_t)lds + j * 4096 / 16) = v;
  }
}

// The eight wave-loads of one 32 KiB block into the buffer at lds_wave (its address + 1024 wave).
template <int... D>
__device__ __forceinline__ void dma_block(uint32_t lds_wave, const uint32_t (&voffd)[8], const char* blk,
                                          std::integer_sequence<int, D...>) {
  (dma16_at<D * 4096>(lds_wave, voffd[D], blk), ...);
}

// FACTORS: A is the two factors of the single sweep, collapsed on their way into the LDS (FactorLoads; collapse_in_gemm says
// when).
template <bool FACTORS, bool PAST = false>
__global__ __launch_bounds__(256) void grad_gemm_kernel(GradArgs a) {
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int vid = xcd_contiguous_id(blockIdx.x, gridDim.x);
  const int tiles = a.row_tiles * a.h_tiles;
  const int nth = vid / tiles, split = a.split_steps.by_length(nth);
  vid -= nth * tiles;
  const int rt = vid / a.h_tiles, ht = vid % a.h_tiles;
  // k-steps that hold rows of B: the A blocks are padded to whole vocabulary tiles, of which the
  // last k-step may lie beyond k_rows altogether (its A entries are exact zeros)
  const int k_begin = a.split_steps.first(split), k_end = a.split_steps.first(split + 1);
  const int nk = k_end - k_begin;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

  // wave-load d of a block covers its bytes [4096 d + 1024 wave, + 1024): lane l moves the
  // 16 bytes at offset 16 l of that KiB to the same place of the LDS stage
  uint32_t voffd[8];
  const int64_t out_row0 = rt < a.half_tiles ? a.slab_row0 + (int64_t)rt * kGradTile
                                             : a.half_off + a.slab_row0 + (int64_t)(rt - a.half_tiles) * kGradTile;
  const int64_t rows_left = a.out_rows - out_row0;       // >= 1
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    // rows that do not exist re-read the first eight (16 rows of V = 151,936, H = 3584: 234 -> 224 us)
    const int kib = (4 * d + wave) * 8 < rows_left ? 4 * d + wave : 0;
    voffd[d] = (uint32_t)lane * 16u + (uint32_t)kib * 1024u;
    asm volatile("" : "+v"(voffd[d]));   // kept in registers, not recomputed at every load
  }
  const char* sA = (const char*)a.slab + ((int64_t)rt * a.nk_total + k_begin) * kImgBytes;
  // the B rows: wave-load d moves rows 2 wave + 8 d and the next, lane l the chunk that belongs at
  // position l % 32 of row l / 32 of the two.  Columns at or beyond H (their output does not
  // exist) re-read the row's first chunk; rows at or beyond k_rows (their A entries are zero)
  // re-read its last row.
  const uint32_t ldb = (uint32_t)a.H * 2u, b_step = kBK * ldb;
  const char* sB = (const char*)a.Bm + (int64_t)k_begin * b_step + ht * kGradRowBytes;
  uint32_t voffb[8];
  auto b_rows = [&](int kt) __attribute__((always_inline)) {
    const int row = 2 * wave + (lane >> 5);
    int c = (lane & 31) ^ ((row & 3) << 2);
    if (ht * kGradTile + c * 8 >= a.H) c = 0;
    const int64_t left = a.k_rows - (int64_t)kt * kBK;      // >= 1
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      int v = row + 8 * d;
      if (v >= left) v = (int)left - 1;
      voffb[d] = (uint32_t)v * ldb + (uint32_t)c * 16u;
      asm volatile("" : "+v"(voffb[d]));
    }
  };
  b_rows(k_begin);
  const uint32_t ldsw = lds0 + (uint32_t)wave * 1024u;
  // the ring of three (offset 0) holds the B blocks, the ring of two the slab blocks; FACTORS: the other way round
  const uint32_t ring3 = ldsw, ring3_end = ldsw + kGradRing3 * kImgBytes, ring2 = ldsw + kGradRing2Off, ring2_end = ring2 + 2 * kImgBytes;
  const uint32_t b_begin = FACTORS ? ring2 : ring3, b_end = FACTORS ? ring2_end : ring3_end;
  const uint32_t a_begin = FACTORS ? ring3 : ring2, a_end = FACTORS ? ring3_end : ring2_end;
  const std::make_integer_sequence<int, 8> all8{};

  f32x16 acc[4][4];
  FactorLoads<PAST> f;
  const int64_t row0 = a.slab_row0 + (int64_t)rt * kGradTile + 8 * wave + (lane >> 3);   // of the lane's first vector
  const int chunk = 8 * ((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7));                   // its entry in the k-step
  if constexpr (FACTORS) {
    const int64_t tile_bytes = (int64_t)a.nk_total * kImgBytes;
    f.rx = __builtin_amdgcn_make_buffer_rsrc((char*)a.slab + rt * tile_bytes, 0, (int)tile_bytes, 0x00020000);
    f.ry = __builtin_amdgcn_make_buffer_rsrc((char*)a.slab + a.e2_bytes + rt * tile_bytes, 0, (int)tile_bytes, 0x00020000);
    f.m0_step = (uint32_t)a.mu0t_stride * 4u;
    f.rm = __builtin_amdgcn_make_buffer_rsrc((char*)(a.mu0t + (int64_t)rt * kGradTile), 0,
                                             (int)(((uint32_t)(a.nk_total / 2 - 1)) * f.m0_step + kGradTile * 4), 0x00020000);
    f.off_m = (uint32_t)(8 * wave + (lane >> 3)) * 4u;
    f.kt = k_begin; f.soff = (uint32_t)k_begin * kImgBytes;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      f.mu[j] = a.mu[row0 + j * 32];
      f.iz[j] = a.inv_z[row0 + j * 32];
      if (f.iz[j] == 0.f || (4 * j + wave) * 8 >= rows_left) f.iz[j] = __builtin_inff();
    }
  }
  if (nk > 0) {
    // first the blocks of k-step 0, then its first fragments
    uint64_t pb = (uint64_t)sB;
    dma_block(b_begin, voffb, sB, all8);
    if constexpr (FACTORS) {
      uint4 x[8], y[8];
      float m0[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) { f.load(j, voffd[j]); x[j] = f.x[j]; y[j] = f.y[j]; m0[j] = f.m0[j]; }
      f.next();
      if (nk > 1) {
#pragma unroll
        for (int j = 0; j < 8; ++j) { f.load(j, voffd[j]); __builtin_amdgcn_sched_barrier(0); }
        f.next();
        pb += b_step;
        if (nk == 2) b_rows(k_end - 1);
        dma_block(b_begin + kImgBytes, voffb, (const char*)pb, all8);
      }
      __builtin_amdgcn_sched_barrier(0);
      collapse_block(a, f, x, y, m0, a_begin + (uint32_t)lane * 16u, row0, k_begin * kBK + chunk, ht == 0);
      __builtin_amdgcn_sched_barrier(0);
      if (nk > 1) {
        collapse_block(a, f, f.x, f.y, f.m0, a_begin + kImgBytes + (uint32_t)lane * 16u, row0, (k_begin + 1) * kBK + chunk, ht == 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (nk > 2) {
#pragma unroll
        for (int j = 0; j < 8; ++j) { f.load(j, voffd[j]); __builtin_amdgcn_sched_barrier(0); }
        f.next();
      }
      __builtin_amdgcn_sched_barrier(0);
      if (nk > 2) asm volatile("s_waitcnt vmcnt(24) lgkmcnt(0)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    } else {
      dma_block(a_begin, voffd, sA, all8);
      wait_vm<0>();
    }
    __syncthreads();
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < 4; ++fn)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[fm][fn][e] = 0.f;
    bf16x8 fa[2][4], fb[2][4];
    uint32_t swA[4], swB[4];
    {
      const int key = (lane >> 1) & 7, half = lane >> 5;
      const uint32_t rowoff = (uint32_t)(lane & 31) * kRowBytes - (uint32_t)wave * 1024u;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const uint32_t x = rowoff + (uint32_t)(((kk * 2 + half) ^ key) << 4);
        swA[kk] = x + (uint32_t)(wm * 128 * kRowBytes);
      }
      // B fragment fn: the lane reads row q = (lane % 16) / 4 (+ 8 for the upper half of the wave) and
      // 8 bytes of columns 128 wn + 32 fn + 16 ((lane / 16) % 2) + 4 (lane % 4); the chunk swizzle
      // moves the fragment's 64 bytes
      const int q = (lane & 15) >> 2;
      const uint32_t rowb = (uint32_t)(8 * half + q) * kGradRowBytes - (uint32_t)wave * 1024u +
                            (uint32_t)(wn * 256 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8);
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) swB[fn] = rowb + (uint32_t)((fn ^ q) << 6);
    }
    uint32_t r_a = a_begin, r_b = b_begin;     // k-step s reads B buffer s % 3 and A buffer s % 2
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[0][i] = lds_frag(r_a + swA[0])[i * 32 * kRowBytes / 16];
      fb[0][i] = lds_frag_tr<0>(r_b + swB[i]);
    }
    int s = 0;
    if constexpr (FACTORS) {
      uint32_t pb_lo = (uint32_t)pb, pb_hi = (uint32_t)(pb >> 32);
#define ADWIN_KSTEP(...) grad_kstep_factors<__VA_ARGS__>(a, f, acc, fa, fb, r_a, r_b, a_begin, a_end, b_begin, b_end, swA, swB, voffd, voffb, \
                                                        b_step, pb_lo, pb_hi, row0, (k_begin + s + 2) * kBK + chunk, ht == 0)
      for (; s + 3 < nk; ++s) {
        ADWIN_KSTEP(true, true, false, PAST);
        f.next();
      }
      if (s + 2 < nk) {           // the step that loads the last k-step, which may hold fewer rows
        b_rows(k_end - 1);
        ADWIN_KSTEP(false, true, false, PAST);
        ++s;
      }
      if (s + 1 < nk) ADWIN_KSTEP(false, false, false, PAST);
      ADWIN_KSTEP(false, false, true, PAST);
#undef ADWIN_KSTEP
    } else {
      // blocks of k-step 1 (k-step s of the loop loads those of k-step s + 2)
      uint64_t pa = (uint64_t)sA;
      if (nk > 1) {
        pa += kImgBytes; pb += b_step;
        if (nk == 2) b_rows(k_end - 1);
        dma_block(b_begin + kImgBytes, voffb, (const char*)pb, all8);
        dma_block(a_begin + kImgBytes, voffd, (const char*)pa, all8);
      }
      uint32_t pa_lo = (uint32_t)pa, pa_hi = (uint32_t)(pa >> 32), pb_lo = (uint32_t)pb, pb_hi = (uint32_t)(pb >> 32);
      for (; s + 3 < nk; ++s)
        grad_kstep<true, false>(acc, fa, fb, r_a, r_b, a_begin, a_end, b_begin, b_end, swA, swB, voffd, voffb, b_step,
                                pa_lo, pa_hi, pb_lo, pb_hi);
      if (s + 2 < nk) {           // the step that loads the last k-step, which may hold fewer rows
        b_rows(k_end - 1);
        grad_kstep<true, false>(acc, fa, fb, r_a, r_b, a_begin, a_end, b_begin, b_end, swA, swB, voffd, voffb, b_step,
                                pa_lo, pa_hi, pb_lo, pb_hi);
        ++s;
      }
      if (s + 1 < nk)
        grad_kstep<false, false>(acc, fa, fb, r_a, r_b, a_begin, a_end, b_begin, b_end, swA, swB, voffd, voffb, b_step,
                                 pa_lo, pa_hi, pb_lo, pb_hi);
      grad_kstep<false, true>(acc, fa, fb, r_a, r_b, a_begin, a_end, b_begin, b_end, swA, swB, voffd, voffb, b_step,
                              pa_lo, pa_hi, pb_lo, pb_hi);
    }
  } else {
    for (auto& row : acc) for (auto& tile : row) tile = f32x16{};
  }
  // Epilogue.  H and out_rows end on whole blocks of 32 columns and 8 rows (H is a multiple of 64; the rows of a
  // dW are V, a multiple of 8, those of g are rounded up to one within its padded planes), so every bound is wave-uniform and a store takes one 32-bit lane offset, a scalar
  // and an immediate: 256 stores in 320 instructions.  With a 64-bit address and two lane bounds per
  // store it was 4,700 instructions in 780 blocks, fetched from a cold instruction cache by every
  // workgroup.  us per call: V = 4,096, H = 256 + 384, 224 rows 75.5 -> 63.3; V = 32,776, H = 1024 + 1024,
  // 1,000 rows with the head gradient 506 -> 466; V = 11,912, H = 512 + 640, 3,139 rows 294 -> 280;
  // 8,192 rows of V = 151,936 with the head gradient (19 tiles per compute unit) 23,200 -> 23,028.
  char* g = (char*)(a.g + ((int64_t)split * a.g_rows + out_row0) * a.H + ht * kGradTile);
  const uint32_t ldg = (uint32_t)a.H * 4u;
  const int rows = (int)(rows_left < kGradTile ? rows_left : kGradTile) - wm * 128, cols = a.H - ht * kGradTile - wn * 128;
  const uint32_t lane_off = (uint32_t)(wm * 128 + 4 * (lane >> 5)) * ldg + (uint32_t)(wn * 128 + (lane & 31)) * 4u;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(g, 0, (int)(kGradTile * ldg) - ht * kGradTile * 4, 0x00020000);
  auto write_tile = [&](auto accumulate) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (fm * 32 + 8 * q >= rows) continue;
#pragma unroll
        for (int fn = 0; fn < 4; ++fn) {
          if (fn * 32 >= cols) continue;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t row_off = (uint32_t)(fm * 32 + 8 * q + e) * ldg, off = lane_off + (uint32_t)fn * 128u;
            const float v = acc[fm][fn][4 * q + e];
            // accumulate: every element is added to by exactly one lane of this launch and
            // launches are ordered on the stream, so the hardware add keeps the sum
            // deterministic while sparing the lane the round trip of a load
            if constexpr (accumulate) unsafeAtomicAdd((float*)(g + row_off + off), v);
            else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, (int)off, (int)row_off, 0);
          }
        }
      }
  };
  if (a.accumulate) write_tile(std::true_type{});
  else write_tile(std::false_type{});
}

// ---------------------------------------------------------------------------------------
// Finalize.  TPR threads per computed row sum the k-split planes, add the heavy entries, write
// the row norm, scale by grad_scale*alpha and scatter to dh_prefix / dh_full; the workgroups
// behind those clear the rows outside the windows, kZeroRows packed rows each, and the first
// tail.blocks take the reductions that end the call, which need nothing of the rest.
// Memory bound, if enough is in flight: a wave per row added up to 32 planes of 8 KB one load
// after the other (97 us for 337 rows, H = 2048) and looked every packed row up for itself before
// it wrote 8 bytes per lane (291,000 rows cleared at 3.4 TB/s, 350 us).  A row of more than 512
// columns with several planes takes 256 threads, its planes are loaded eight at a time and the
// dot products of its heavy entries are split over all of them.  Narrower rows take a wave, and so do
// rows of one plane: 256 threads for two 16-byte loads each spend their time at the barriers
// (65,536 rows, H = 2048, with 212,000 cleared: the reductions of the call 882 -> 735 us on one GPU).
// 337 rows of 32 planes: 98 -> 19 us; 4,096 computed and 291,000 cleared rows: 350 -> 209 us.
// ---------------------------------------------------------------------------------------
constexpr int kZeroRows = 32;
constexpr int kPlaneStep = 8;

__device__ __forceinline__ void store_dh(void* base, int bf16, int64_t t, int H, int h, float4 v) {
  if (!base) return;
  if (bf16) {
    uint2 o;
    o.x = pack_bf16(v.x, v.y);
    o.y = pack_bf16(v.z, v.w);
    *(uint2*)((uint16_t*)base + t * H + h) = o;
  } else {
    *(float4*)((float*)base + t * H + h) = v;
  }
}

// Clears dh_prefix on the packed rows [t0, t1) that lie outside their rollout's window.
__device__ __forceinline__ void clear_rows(const FinalizeArgs& a, int64_t t0, int64_t t1) {
  const int64_t row_vec = (int64_t)a.H * (a.dh_bf16 ? 2 : 4) / 16;     // H is a multiple of 64
  const uint4 zero = {0u, 0u, 0u, 0u};
  for (int i = last_le<int64_t>(a.pl.offsets, a.B + 1, t0); i < a.B && a.pl.offsets[i] < t1; ++i) {
    const int64_t first = a.pl.offsets[i] + a.pl.n[i], end = a.pl.offsets[i + 1];
    const int64_t lo = first > t0 ? first : t0, hi = end < t1 ? end : t1;
    for (int64_t q = lo * row_vec + threadIdx.x; q < hi * row_vec; q += 256) store16((uint4*)a.dh_prefix + q, zero);
  }
}

template <int TPR>
__global__ __launch_bounds__(256) void finalize_kernel(FinalizeArgs a, TailArgs tail) {
  constexpr int kRows = 256 / TPR, kWaves = TPR / 64;
  __shared__ int heavy_v[kRows][kHeavySlots];
  __shared__ float heavy_d[kRows][kHeavySlots];
  __shared__ float part[kRows][kHeavySlots][kWaves][2];
  __shared__ double sh[16];
  __shared__ int sh_first[4];
  if ((int)blockIdx.x < tail.blocks) return tail_body<false>(tail, blockIdx.x, sh, sh_first);
  const int64_t block = (int64_t)blockIdx.x - tail.blocks;
  const int64_t row_blocks = (a.n_rows + kRows - 1) / kRows;
  if (block >= row_blocks) {
    const int64_t t0 = (block - row_blocks) * kZeroRows;
    return clear_rows(a, t0, t0 + kZeroRows < a.T ? t0 + kZeroRows : a.T);
  }
  const int sub = threadIdx.x / TPR, lid = threadIdx.x % TPR, lane = threadIdx.x & 63, w = lid >> 6;
  const int64_t r = block * kRows + sub;
  const bool have = r < a.n_rows;
  const int i = have ? a.pl.row_seq[r] : 0;
  const int64_t t = have ? a.pl.row_idx[r] : 0;
  const float iz = have ? a.inv_z[r] : 0.f;
  // 0: excluded row (no finite statistics): zeros in both gradients, in g (the pooled sums
  // read it) and in the row norm
  const bool dead = iz == 0.f;
  const bool admitted = have && t - a.pl.offsets[i] < a.pl.n[i];
  // Heavy entries of the row (those the bf16 operand holds as zeros): heavy_v[k] is the k-th
  // smallest listed vocabulary index and heavy_d[k] that entry's logit gradient, taken in fp32
  // from fresh dot products.  The list is filled in no particular order; adding the entries in
  // index order keeps the result the same from call to call.
  int nh = have && !dead && a.heavy.cnt ? a.heavy.cnt[r] : 0;
  nh = nh < kHeavySlots ? nh : kHeavySlots;
  if (nh > 0 && lid < 64) {
    const int mine = lane < nh ? a.heavy.v[r * kHeavySlots + lane] : 0x7fffffff;
    int rank = 0;                                  // indices of one row are distinct
    for (int k = 0; k < nh; ++k) rank += (__shfl(mine, k, 64) < mine) ? 1 : 0;
    if (lane < nh) heavy_v[sub][rank] = mine;
  }
  __syncthreads();
  for (int k = 0; k < nh; ++k) {
    const int64_t v = heavy_v[sub][k];
    auto dot = [&](const __bf16* x, const __bf16* y, int H) __attribute__((always_inline)) {
      float acc = 0.f;
#pragma unroll 2
      for (int q = lid; q < (H >> 3); q += TPR) {
        const uint4 p = ((const uint4*)x)[q], o = ((const uint4*)y)[q];
        acc = fmaf(bf16_lo(p.x), bf16_lo(o.x), acc); acc = fmaf(bf16_hi(p.x), bf16_hi(o.x), acc);
        acc = fmaf(bf16_lo(p.y), bf16_lo(o.y), acc); acc = fmaf(bf16_hi(p.y), bf16_hi(o.y), acc);
        acc = fmaf(bf16_lo(p.z), bf16_lo(o.z), acc); acc = fmaf(bf16_hi(p.z), bf16_hi(o.z), acc);
        acc = fmaf(bf16_lo(p.w), bf16_lo(o.w), acc); acc = fmaf(bf16_hi(p.w), bf16_hi(o.w), acc);
      }
      return wave_sum(acc);
    };
    const float zt = dot(a.h_t + t * a.H_t, a.W_t + v * a.H_t, a.H_t);
    const float zs = dot(a.h_s + t * a.H, a.W_s + v * a.H, a.H);
    if (lane == 0) { part[sub][k][w][0] = zs; part[sub][k][w][1] = zt; }
  }
  __syncthreads();
  if (lid < nh) {
    float zs = 0.f, zt = 0.f;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) { zs += part[sub][lid][q][0]; zt += part[sub][lid][q][1]; }
    heavy_d[sub][lid] = __expf(zs - a.lse_s[r]) * ((zs - zt) - a.mu[r]);
  }
  __syncthreads();
  const float sp = admitted ? a.grad_scale * a.pl.alpha_p[i] : 0.f;
  const float sf = a.grad_scale * a.pl.alpha_f[i];
  // sampled estimator: g = c (W_s[y] - G2 / Z_s), G2 in the planes, which lie behind the n_pad rows of g
  const float c = a.cr && have ? a.cr[r] : 0.f;
  const int64_t src = (a.cr ? a.n_pad + r : r) * a.H;
  int64_t y = 0;
  if (a.cr && have) {
    y = a.ids[t];
    if (y < 0 || y >= a.V) y = 0;                  // c is 0 then
  }
  float nrm = 0.f;
  for (int h = have ? lid * 4 : a.H; h < a.H; h += TPR * 4) {
    float4 g = {0.f, 0.f, 0.f, 0.f};
    if (!dead) {
      g = *(const float4*)(a.g + src + h);
      for (int s = 1; s < a.ksplit; s += kPlaneStep) {
        float4 q[kPlaneStep];
#pragma unroll
        for (int u = 0; u < kPlaneStep; ++u) {
          q[u] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (s + u < a.ksplit) q[u] = *(const float4*)(a.g + (int64_t)(s + u) * a.g_rows * a.H + src + h);
        }
#pragma unroll
        for (int u = 0; u < kPlaneStep; ++u) { g.x += q[u].x; g.y += q[u].y; g.z += q[u].z; g.w += q[u].w; }
      }
      if (a.cr) {
        const uint2 wy = *(const uint2*)(a.W_s + y * a.H + h);
        g.x = c * (bf16_lo(wy.x) - g.x * iz); g.y = c * (bf16_hi(wy.x) - g.y * iz);
        g.z = c * (bf16_lo(wy.y) - g.z * iz); g.w = c * (bf16_hi(wy.y) - g.w * iz);
      }
      for (int k = 0; k < nh; ++k) {
        const float dzv = heavy_d[sub][k];
        const uint2 wv = *(const uint2*)(a.W_s + (int64_t)heavy_v[sub][k] * a.H + h);
        g.x = fmaf(dzv, bf16_lo(wv.x), g.x); g.y = fmaf(dzv, bf16_hi(wv.x), g.y);
        g.z = fmaf(dzv, bf16_lo(wv.y), g.z); g.w = fmaf(dzv, bf16_hi(wv.y), g.w);
      }
    }
    // the pooled sums of the probe read g
    if (a.probe && (a.ksplit > 1 || nh > 0 || a.cr || dead)) *(float4*)(a.g + r * a.H + h) = g;
    nrm = fmaf(g.x, g.x, fmaf(g.y, g.y, fmaf(g.z, g.z, fmaf(g.w, g.w, nrm))));
    const float4 p = {g.x * sp, g.y * sp, g.z * sp, g.w * sp};
    store_dh(a.dh_prefix, a.dh_bf16, t, a.H, h, p);
    if (a.probe) {
      const float4 f = {g.x * sf, g.y * sf, g.z * sf, g.w * sf};
      store_dh(a.dh_full, a.dh_bf16, t, a.H, h, f);
    }
  }
  nrm = wave_sum(nrm);
  if constexpr (kWaves > 1) {
    if (lane == 0) part[0][0][w][0] = nrm;         // last read before the barrier above
    __syncthreads();
    nrm = (part[0][0][0][0] + part[0][0][1][0]) + (part[0][0][2][0] + part[0][0][3][0]);
  }
  if (have && lid == 0) a.rownorm[r] = nrm;
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
hipError_t grad_kernels_opt_in() {
  for (const void* k : {(const void*)grad_gemm_kernel<false>, (const void*)grad_gemm_kernel<true>, (const void*)grad_gemm_kernel<true, true>}) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kGradLds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_hs_gather(const HsGatherArgs& a, int64_t rows, hipStream_t st) {
  hs_gather_kernel<<<(unsigned)(rows / 4), 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_combine(bool transposed, bool sampled, const CombineArgs& a, int row_tiles, hipStream_t st) {
  const dim3 grid((unsigned)a.nk, (unsigned)row_tiles);
  if (sampled && !transposed) return hipErrorInvalidValue;   // the sampled estimator contracts E2 as stored
#define ADWIN_LAUNCH(TR, SAMPLED)                                                  \
  if (a.past_cache) combine_kernel<TR, SAMPLED, true><<<grid, 256, 0, st>>>(a);    \
  else combine_kernel<TR, SAMPLED, false><<<grid, 256, 0, st>>>(a);
  if (sampled) { ADWIN_LAUNCH(true, true) }
  else if (transposed) { ADWIN_LAUNCH(true, false) }
  else { ADWIN_LAUNCH(false, false) }
#undef ADWIN_LAUNCH
  return hipGetLastError();
}

hipError_t launch_grad_gemm(const GradArgs& p, hipStream_t st) {
  if (p.out_rows & 7) return hipErrorInvalidValue;       // rows are stored by eights
  GradArgs a = p;
  a.split_steps.split((int)((a.k_rows + kBK - 1) / kBK), a.ksplit);
  const unsigned grid = (unsigned)(a.row_tiles * a.h_tiles * a.ksplit);
  if (a.e2_bytes && a.past_cache && a.h_tiles == 1) grad_gemm_kernel<true, true><<<grid, 256, kGradLds, st>>>(a);
  else if (a.e2_bytes) grad_gemm_kernel<true><<<grid, 256, kGradLds, st>>>(a);
  else grad_gemm_kernel<false><<<grid, 256, kGradLds, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeArgs& a, const TailArgs* end, hipStream_t st) {
  // one plane: thousands of rows, or a vocabulary so small that a row has nothing to add up; a wave each
  const bool wide = a.H > 512 && a.ksplit > 1;
  const int64_t row_blocks = wide ? a.n_rows : (a.n_rows + 3) / 4;
  const int64_t zero_blocks = !a.probe && a.dh_prefix ? (a.T + kZeroRows - 1) / kZeroRows : 0;
  TailArgs tail{};
  if (end) tail = *end;
  const unsigned grid = (unsigned)(row_blocks + zero_blocks + tail.blocks);
  if (grid == 0) return hipSuccess;
  if (wide) finalize_kernel<256><<<grid, 256, 0, st>>>(a, tail);
  else finalize_kernel<64><<<grid, 256, 0, st>>>(a, tail);
  return hipGetLastError();
}

}  // namespace adwin
