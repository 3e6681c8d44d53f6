// Fused path, first half: LM-head projections on bf16 MFMA and everything that is taken
// from the logits while they sit in registers -- full-vocabulary log-sum-exp, per-token
// reverse KL (Eq. 2 at token level) and the factors of the logit gradient (Eq. 4 in
// expectation, App. A.1).  The logits themselves are never written anywhere.
//
// Single sweep (the default): per-row references are fixed in advance (the largest logit
// of vocabulary tile 0 and the sampled token), so one pass over the vocabulary
// yields the sums Z_s, A = sum e_s (z_s - z_t), Z_t and two bf16 gradient factors
// D = (z_s - z_t) - mu0 and E2 = e_s per logit, written as tile images into a bounded row
// slab; the merge gives lse, mu, KL_t, c_t per row, and the combine pass (grad_kernels.hip)
// turns the factors into dz = p_s ((z_s - z_t) - mu).
// Two sweeps (fallback): running-max statistics, merge, then the logits again for dz.
//
// For a token tile (256, or the 128 of a call of few rows) a workgroup walks vocabulary tiles of 128; per tile two MFMA GEMMs
// (teacher, then student) into fp32 accumulators, then the epilogue on the registers.
// MFMA operand roles: v_mfma_f32_32x32x16_bf16 computes D[i][j] += sum_k A[i][k] B[k][j]
// with i in registers and j = lane % 32.  A = W tile (i = vocabulary) and B = h tile
// (j = token), so each lane owns one token column and the reduction over the vocabulary
// runs down its own registers with no cross-lane traffic.
// A lane holds rows i = 8 (e / 4) + 4 (lane / 32) + e % 4 of a 32 x 32 block, e = 0..15.  The
// W tiles are staged with their rows permuted inside every group of 32 (entry_of_tile_row), so
// that these are 16 consecutive vocabulary entries, 16 (lane / 32) + e: a lane then owns 32
// consecutive bytes of a slab row per block and writes them with two 16-byte stores, where the
// natural order gives it four separate 8-byte pieces.
#include "fused_shared.h"
#include "setup_device.h"

namespace adwin {

// ---------------------------------------------------------------------------------------
// Staging of [ROWS x 64] bf16 tiles: global -> registers -> LDS.  Thread t moves the
// 16-byte chunk (t & 7) of rows (t >> 3) + 32 i.  Chunk c of row r is stored at chunk
// position c ^ ((r >> 1) & 7): two 128-byte rows span all 64 LDS banks, so the 16 rows
// that 16 consecutive lanes of an MFMA fragment read touch land on 16 distinct
// (row parity, position) pairs, i.e. on distinct banks.
// ---------------------------------------------------------------------------------------
template <int ROWS>
struct RowStager {
  static constexpr int N = ROWS / 32;
  const uint4* p[N];
  uint4 v[N];
  __device__ __forceinline__ void issue(int kt) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[i][kt * 8];
  }
  __device__ __forceinline__ void commit(char* tile, int thread_off) const {
#pragma unroll
    for (int i = 0; i < N; ++i) *(uint4*)(tile + thread_off + i * 32 * kRowBytes) = v[i];
  }
};

__device__ __forceinline__ int stage_thread_off(int tid) {
  const int r = tid >> 3, c = tid & 7;
  return r * kRowBytes + ((c ^ ((r >> 1) & 7)) << 4);
}

// Row order of the staged W tiles: tile row 8 q + 4 h + r of a group of 32 holds vocabulary entry
// 16 h + 4 q + r of the group (q = 0..3, h = 0..1, r = 0..3).
__device__ __forceinline__ int entry_of_tile_row(int i) {
  return (i & ~31) + 16 * ((i >> 2) & 1) + 4 * ((i >> 3) & 3) + (i & 3);
}

// acc[FM][FN] += A_tile(wave rows) * B_tile(wave rows)^T for one staged k-step of 64.
template <int FM, int FN>
__device__ __forceinline__ void mma_stage(f32x16 (&acc)[FM][FN], const char* tA, const char* tB,
                                          int lane) {
  const int row_off = (lane & 31) * kRowBytes;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int sw = ((kk * 2 + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4;
    bf16x8 a[FM], b[FN];
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
      a[fm] = *(const bf16x8*)(tA + fm * 32 * kRowBytes + row_off + sw);
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
      b[fn] = *(const bf16x8*)(tB + fn * 32 * kRowBytes + row_off + sw);
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[fm], b[fn], acc[fm][fn], 0, 0, 0);
  }
}

// Double-buffered k loop.  ldsA/ldsB: stage 0 tiles; stage 1 follows at `stage_bytes`.
// waveA/waveB: byte offset of this wave's rows inside the A/B tile.
template <int RA, int RB, int FM, int FN>
__device__ __forceinline__ void gemm_kloop(f32x16 (&acc)[FM][FN], RowStager<RA>& sa,
                                           RowStager<RB>& sb, int kt0, int nk, char* lds,
                                           int stage_bytes, int waveA, int waveB, int tid) {
  constexpr int kOffB = RA * kRowBytes;
  const int toff = stage_thread_off(tid);
  const int lane = tid & 63;
  sa.issue(kt0);
  sb.issue(kt0);
  sa.commit(lds, toff);
  sb.commit(lds + kOffB, toff);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    char* cur = lds + (kt & 1) * stage_bytes;
    char* nxt = lds + ((kt + 1) & 1) * stage_bytes;
    const bool more = kt + 1 < nk;
    if (more) {
      sa.issue(kt0 + kt + 1);
      sb.issue(kt0 + kt + 1);
    }
    mma_stage<FM, FN>(acc, cur + waveA, cur + kOffB + waveB, lane);
    if (more) {
      sa.commit(nxt, toff);
      sb.commit(nxt + kOffB, toff);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------
// Logit passes
// ---------------------------------------------------------------------------------------

// Running per-token statistics held by one lane for its two token columns.
struct LaneStats { float m_s[2], Z_s[2], A_s[2], m_t[2], Z_t[2]; };

// Element e of block fm is vocabulary entry v0 + fm*32 + 16*(lane/32) + e.
// Online update of (m_s, Z_s, A, m_t, Z_t) with one 128 x 64 logit tile per wave.
__device__ __forceinline__ void stats_epilogue(const f32x16 (&zs)[4][2], const f32x16 (&zt)[4][2],
                                               LaneStats& st, int v0, int V, bool tail, int lane) {
  const int vlane = v0 + 16 * (lane >> 5);
#pragma unroll
  for (int fn = 0; fn < 2; ++fn) {
    float mxs = st.m_s[fn], mxt = st.m_t[fn];
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const bool ok = !tail || (vlane + fm * 32 + e) < V;
        if (ok) { mxs = fmaxf(mxs, zs[fm][fn][e]); mxt = fmaxf(mxt, zt[fm][fn][e]); }
      }
    const float scs = fast_exp2((st.m_s[fn] - mxs) * kLog2e);
    const float sct = fast_exp2((st.m_t[fn] - mxt) * kLog2e);
    float Zs = st.Z_s[fn] * scs, As = st.A_s[fn] * scs, Zt = st.Z_t[fn] * sct;
    const float ms2 = mxs * kLog2e, mt2 = mxt * kLog2e;
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const bool ok = !tail || (vlane + fm * 32 + e) < V;
        const float s = zs[fm][fn][e], t = zt[fm][fn][e];
        float es = fast_exp2(fmaf(s, kLog2e, -ms2));
        float et = fast_exp2(fmaf(t, kLog2e, -mt2));
        float d = s - t;
        if (!ok) { es = 0.f; et = 0.f; d = 0.f; }
        Zs += es;
        As = fmaf(es, d, As);
        Zt += et;
      }
    st.m_s[fn] = mxs; st.m_t[fn] = mxt; st.Z_s[fn] = Zs; st.A_s[fn] = As; st.Z_t[fn] = Zt;
  }
}

// dz = p_s ((z_s - z_t) - mu), rounded to bf16, into rows wrow + fn*32 + lane%32 of the tile.
// Entries with p_s >= kHeavyP are listed for computed row crow + fn*32 + lane%32 and stored as 0.
__device__ __forceinline__ void dz_epilogue(const f32x16 (&zs)[4][2], const f32x16 (&zt)[4][2],
                                            const float (&lse2)[2], const float (&mu)[2], __bf16* blk,
                                            int wrow, int v0, int V, bool tail, int lane,
                                            const HeavyList& heavy, int64_t crow) {
  // chunk c = 4 (fm & 1) + 2 half + p of slab block fm / 2 holds the lane's entries 8 p .. 8 p + 7
  // of block fm; its position in the row is c ^ key = (4 (fm & 1) + p) ^ key2
  const int half = lane >> 5, vlane = v0 + 16 * half, key2 = ((lane >> 1) & 7) ^ (2 * half);
#pragma unroll
  for (int fn = 0; fn < 2; ++fn) {
    __bf16* out = blk + (wrow + fn * 32 + (lane & 31)) * kBK;
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        float d[8];
        const bool in = !tail || vlane + fm * 32 + 8 * p < V;      // V is a multiple of 8
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float s = zs[fm][fn][p * 8 + e], t = zt[fm][fn][p * 8 + e];
          const float pr = fast_exp2(fmaf(s, kLog2e, -lse2[fn]));
          d[e] = in ? pr * ((s - t) - mu[fn]) : 0.f;
          if (__builtin_expect(pr >= kHeavyP && in, 0)) {
            if (heavy_push(heavy, crow + fn * 32 + (lane & 31), vlane + fm * 32 + 8 * p + e)) d[e] = 0.f;
          }
        }
        uint4 o;
        o.x = pack_bf16(d[0], d[1]); o.y = pack_bf16(d[2], d[3]);
        o.z = pack_bf16(d[4], d[5]); o.w = pack_bf16(d[6], d[7]);
        *(uint4*)(out + (fm >> 1) * kSlabBlock + ((((fm & 1) * 4 + p) ^ key2) << 3)) = o;
      }
  }
}

// Single-sweep epilogue.  With per-row references fixed in advance (rs2 = m_ref_s*log2e,
// rt2 = m_ref_t*log2e, mu0 ~ E_{p_s}[z_s - z_t]) every exponential is taken relative to the
// same reference in every tile, so the statistics are plain sums,
//   Z_s = sum e_s,  A = sum e_s d,  Z_t = sum e_t,   e_s = exp(z_s - m_ref_s), d = z_s - z_t,
// and two bf16 factors of the unnormalised gradient can be emitted at once, D = d - mu0 and
// E2 = e_s: dz = E2 (D - (mu - mu0)) / Z_s.  mu0 is a per-(row, vocabulary tile) reference
// kept for the combine pass.  D goes to slab rows row0.., E2 to the same rows e2_off elements
// further on.
// B_t = sum e_t z_t (teacher entropy) and cnt = entries ranked above the sampled token are
// only maintained in diagnostics mode.
struct LaneSums { float Z_s[2], A_s[2], Z_t[2], B_t[2]; int cnt[2]; };

// One accumulator element for vector arithmetic.  The operand constraint keeps the accumulators
// in their registers up to the read: left alone, the register allocator moves blocks of them
// about (and one into scratch memory) during the epilogue, and every reload from scratch waits
// for all the stores in flight.
__device__ __forceinline__ float acc_read(const float& a) {
  float v;
  asm("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
  return v;
}

// The two slab blocks of a logit tile through a buffer descriptor: the lane's offset is one
// 32-bit register, so the stores need no 64-bit address registers.  No part of it is given as the instruction's scalar
// offset: the compiler puts two wait states between a 16-byte buffer store and an instruction that overwrites its
// data registers, but none if the store has one, and stores of this epilogue were seen to write the register's next
// contents (an accumulator read right behind the store) once a second wave shared the SIMD.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slab_rsrc(__bf16* blk) {
  // extent: the tile's two blocks; flag word: the raw-buffer setting of the gfx9 family
  // (32-bit data format, no swizzle)
  return __builtin_amdgcn_make_buffer_rsrc(blk, 0, 2 * kImgBytesSlab, 0x00020000);
}
__device__ __forceinline__ u32x4 pack_chunk(const float (&x)[8]) {
  u32x4 o;
  o.x = pack_bf16(x[0], x[1]); o.y = pack_bf16(x[2], x[3]);
  o.z = pack_bf16(x[4], x[5]); o.w = pack_bf16(x[6], x[7]);
  return o;
}
__device__ __forceinline__ void slab_store16(__amdgpu_buffer_rsrc_t r, int off, const float (&x)[8]) {
  __builtin_amdgcn_raw_buffer_store_b128(pack_chunk(x), r, off, 0, 0);
}

// LINES: the factors as whole lines, past the caches (sweep_whole_lines says when).  A lane has 16 bytes of one row at a time,
// so that a store as above is 64 pieces of 16 bytes in 32 lines, which only the L2 can put together.  Here the wave lays the
// chunks of 32 rows x 64 entries (a group, 4 KiB) into the LDS, in image order, and stores it as four instructions of
// 1 KiB in one piece, 8 lines each; the operations of a wave on the LDS take effect in order, so the next group may be
// written over it at once.  What gains is not the fewer pieces (kept in the caches, whole lines take as long as
// pieces) but that the lines of a slab that the caches cannot hold no longer push W and h out of the L2; non-temporal pieces
// take up to 1.8 times as long as plain ones.
typedef __attribute__((address_space(3))) u32x4* LdsVecPtr;
__device__ __forceinline__ LdsVecPtr lds_vec(uint32_t addr) { return (LdsVecPtr)(uintptr_t)addr; }
constexpr int kGroupBytes = 32 * kRowBytes;

template <bool TAIL, bool DIAG, bool WRITE_D, bool WRITE_E2, int FN, bool LINES>
__device__ __forceinline__ void single_epilogue(const f32x16 (&zs)[4][FN], const f32x16 (&zt)[4][FN],
                                                LaneSums& sm, const float (&rs2)[2],
                                                const float (&rt2)[2], float (&mu0)[2],
                                                const float (&zyt)[2], const int (&yid)[2],
                                                __bf16* blk, int64_t e2_off, int wrow,
                                                int v0, int V, int lane, float* mu0_out, uint32_t side) {
  // lane's entries of block fm: v0 + fm*32 + 16*half + e, e = 0..15; chunk positions as in dz_epilogue
  const int half = lane >> 5, vlane = v0 + 16 * half, key2 = ((lane >> 1) & 7) ^ (2 * half);
  // byte offset of chunk cb of the lane's row (fn = 0, first block): rowb ^ (cb << 4)
  const int rowb = (wrow + (lane & 31)) * kRowBytes + (key2 << 4);
  // with diagnostics formed again for every store: kept, the sixteen offsets made the kernel spill
  auto offset = [&](int fn, int fm, int p) __attribute__((always_inline)) {
    int b = rowb;
    if (DIAG) asm volatile("" : "+v"(b));
    return (b ^ (((fm & 1) * 4 + p) << 4)) + (fm >> 1) * kImgBytesSlab + fn * 32 * kRowBytes;
  };
  const __amdgpu_buffer_rsrc_t rd = slab_rsrc(blk), re = slab_rsrc(blk + e2_off);
  // chunk cb of the lane's row in the LDS: row_lds ^ (cb << 4)
  const uint32_t row_lds = side + (uint32_t)((lane & 31) * kRowBytes + (key2 << 4));
  u32x4 group[4];                          // a group out of the LDS, stored when the next one is under way
  int group_off = -1;
  bool group_is_d = false;
  auto store_group = [&]() __attribute__((always_inline)) {
    if (group_off < 0) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(group[j], group_is_d ? rd : re,
                                             wrow * kRowBytes + lane * 16 + group_off + j * 1024, 0, 2);
    group_off = -1;
  };
  auto fetch_group = [&](bool d, int fn, int pair) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) group[j] = *lds_vec(side + (uint32_t)(j * 1024 + lane * 16));
    group_is_d = d;
    group_off = pair * kImgBytesSlab + fn * kGroupBytes;
  };
  auto put = [&](bool d, int fn, int fm, int p, const float (&x)[8]) __attribute__((always_inline)) {
    if constexpr (LINES) *lds_vec(row_lds ^ (uint32_t)(((fm & 1) * 4 + p) << 4)) = pack_chunk(x);
    else slab_store16(d ? rd : re, offset(fn, fm, p), x);
  };
  float Zs[2], As[2], Zt[2], Bt[2];
  int cnt[2], vy[2];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    Zs[fn] = sm.Z_s[fn]; As[fn] = sm.A_s[fn]; Zt[fn] = sm.Z_t[fn]; Bt[fn] = sm.B_t[fn];
    cnt[fn] = sm.cnt[fn];
    vy[fn] = yid[fn] - vlane;              // position of the sampled token among this lane's entries
  }
  // first pass over 8 entries of token column fn: sums and the E2 factor
  auto sums8 = [&](int fn, int fm, int p) __attribute__((always_inline)) {
    float e2[8];
    const bool ok = !TAIL || (vlane + fm * 32 + 8 * p) < V;      // V is a multiple of 8
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float s = acc_read(zs[fm][fn][p * 8 + e]), t = acc_read(zt[fm][fn][p * 8 + e]);
      float es = fast_exp2(fmaf(s, kLog2e, -rs2[fn]));
      float et = fast_exp2(fmaf(t, kLog2e, -rt2[fn]));
      float d = s - t;
      if (TAIL && !ok) { es = 0.f; et = 0.f; d = 0.f; }
      Zs[fn] += es;
      As[fn] = fmaf(es, d, As[fn]);
      Zt[fn] += et;
      if (DIAG) {
        Bt[fn] = fmaf(et, t, Bt[fn]);
        cnt[fn] += (t > zyt[fn] && (fm * 32 + 8 * p + e) != vy[fn] && ok) ? 1 : 0;
      }
      e2[e] = es;
    }
    if (WRITE_E2) put(false, fn, fm, p, e2);
  };
  // Second factor: D = d - mu0 with mu0 the strip's running mean of d = z_s - z_t under the
  // student weights, this tile included (both half-columns of the row).  A heavy entry
  // dominates the mean of its own tile, so its D is stored small and the correction
  // (mu - mu0) carries its gradient: the rounding of both factors stays proportional to
  // p_s |d - mu| even when the row is peaked and the first vocabulary entries say nothing
  // about mu.  The masked entries of a tail tile have E2 = 0; their D is immaterial.
  auto mean_of = [&](int fn) __attribute__((always_inline)) {
    const float Zr = Zs[fn] + __shfl_xor(Zs[fn], 32, 64), Ar = As[fn] + __shfl_xor(As[fn], 32, 64);
    if (Zr > 0.f) mu0[fn] = Ar / Zr;
    if (mu0_out && lane < 32) mu0_out[fn * 32 + lane] = mu0[fn];
    return mu0[fn];
  };
  auto factor8 = [&](int fn, int fm, int p, float m0) __attribute__((always_inline)) {
    float dd[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      dd[e] = (acc_read(zs[fm][fn][p * 8 + e]) - m0) - acc_read(zt[fm][fn][p * 8 + e]);
    put(true, fn, fm, p, dd);
  };
  if constexpr (LINES) {
    float m0[2] = {0.f, 0.f};
    auto group_e = [&](int fn, int pair) __attribute__((always_inline)) {
      sums8(fn, 2 * pair, 0);
      store_group();
      sums8(fn, 2 * pair, 1); sums8(fn, 2 * pair + 1, 0); sums8(fn, 2 * pair + 1, 1);
      fetch_group(false, fn, pair);
    };
    auto group_d = [&](int fn, int pair) __attribute__((always_inline)) {
      if (!WRITE_D) return;
      factor8(fn, 2 * pair, 0, m0[fn]);
      store_group();
      factor8(fn, 2 * pair, 1, m0[fn]); factor8(fn, 2 * pair + 1, 0, m0[fn]); factor8(fn, 2 * pair + 1, 1, m0[fn]);
      fetch_group(true, fn, pair);
    };
    // column 0's second pass between column 1's groups of the first (as below)
    group_e(0, 0); group_e(0, 1);
    if (WRITE_D) m0[0] = mean_of(0);
    group_e(FN - 1, 0); group_d(0, 0);
    group_e(FN - 1, 1); group_d(0, 1);
    if (WRITE_D) m0[FN - 1] = mean_of(FN - 1);
    group_d(FN - 1, 0); group_d(FN - 1, 1);
    store_group();
  } else {
    // The stores of D have little arithmetic of their own to hide behind, so column 0's second
    // pass is interleaved with column 1's first pass, whose exponentials cover them.
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int p = 0; p < 2; ++p) sums8(0, fm, p);
    float m0 = 0.f;
    if (WRITE_D) m0 = mean_of(0);
    if constexpr (FN == 2) {
#pragma unroll
      for (int fm = 0; fm < 4; ++fm)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          sums8(1, fm, p);
          if (WRITE_D) factor8(0, fm, p, m0);
        }
      if (WRITE_D) m0 = mean_of(1);
    }
    if (WRITE_D) {
#pragma unroll
      for (int fm = 0; fm < 4; ++fm)
#pragma unroll
        for (int p = 0; p < 2; ++p) factor8(FN - 1, fm, p, m0);
    }
  }
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    sm.Z_s[fn] = Zs[fn]; sm.A_s[fn] = As[fn]; sm.Z_t[fn] = Zt[fn];
    if (DIAG) { sm.B_t[fn] = Bt[fn]; sm.cnt[fn] = cnt[fn]; }
  }
}

template <bool DIAG, int FN>
__device__ __forceinline__ void write_sums(LaneSums& sm, float* part, int strips, int strip,
                                           int64_t n_pad, int64_t row0, int lane) {
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const float Zs = sm.Z_s[fn] + __shfl_xor(sm.Z_s[fn], 32, 64);
    const float As = sm.A_s[fn] + __shfl_xor(sm.A_s[fn], 32, 64);
    const float Zt = sm.Z_t[fn] + __shfl_xor(sm.Z_t[fn], 32, 64);
    const float Bt = DIAG ? sm.B_t[fn] + __shfl_xor(sm.B_t[fn], 32, 64) : 0.f;
    const int cnt = DIAG ? sm.cnt[fn] + __shfl_xor(sm.cnt[fn], 32, 64) : 0;
    if (lane < 32) {
      const int64_t plane = (int64_t)strips * n_pad;
      float* o = part + (int64_t)strip * n_pad + row0 + fn * 32 + lane;
      o[0 * plane] = Zs;
      o[1 * plane] = As;
      o[2 * plane] = Zt;
      if (DIAG) {
        o[3 * plane] = Bt;
        o[4 * plane] = (float)cnt;     // at most V < 2^24: exact
      }
    }
  }
}

// Merge the two half-columns held by lanes l and l^32 and write one strip's partials.
__device__ __forceinline__ void write_partials(LaneStats& st, float* part, int strips, int strip,
                                               int64_t n_pad, int64_t row0, int lane) {
#pragma unroll
  for (int fn = 0; fn < 2; ++fn) {
    merge_mza(st.m_s[fn], st.Z_s[fn], st.A_s[fn], __shfl_xor(st.m_s[fn], 32, 64),
              __shfl_xor(st.Z_s[fn], 32, 64), __shfl_xor(st.A_s[fn], 32, 64));
    merge_mz(st.m_t[fn], st.Z_t[fn], __shfl_xor(st.m_t[fn], 32, 64), __shfl_xor(st.Z_t[fn], 32, 64));
    if (lane < 32) {
      const int64_t plane = (int64_t)strips * n_pad;
      float* o = part + (int64_t)strip * n_pad + row0 + fn * 32 + lane;
      o[0 * plane] = st.m_s[fn];
      o[1 * plane] = st.Z_s[fn];
      o[2 * plane] = st.A_s[fn];
      o[3 * plane] = st.m_t[fn];
      o[4 * plane] = st.Z_t[fn];
    }
  }
}

constexpr int kLogitStage = (kTileVocab + kTileTokens) * kRowBytes;   // 48 KiB
constexpr int kLogitLds = 2 * kLogitStage;

template <bool PASS2>
__global__ __launch_bounds__(256) void logit_pass_kernel(LogitPassArgs a) {
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int strip, tt_local;
  strip_and_tile(xcd_contiguous_id(blockIdx.x, gridDim.x), a.tg, a.strips, a.n_tiles, &strip, &tt_local);
  const int tt = a.tile0 + tt_local;
  const int vt_begin = a.strip_tiles.first(strip), vt_end = a.strip_tiles.first(strip + 1);

  // token-row stagers (rows fixed for the whole vocabulary walk)
  RowStager<kTileTokens> hs, ht;
  RowStager<kTileVocab> ws, wt;
  {
    const int r = tid >> 3, c = tid & 7;
#pragma unroll
    for (int i = 0; i < kTileTokens / 32; ++i) {
      const int64_t row = a.row_idx[(int64_t)tt * kTileTokens + r + 32 * i];
      hs.p[i] = (const uint4*)(a.h_s + row * a.H_s) + c;
      ht.p[i] = (const uint4*)(a.h_t + row * a.H_t) + c;
    }
  }
  const int waveB = wave * 64 * kRowBytes;   // this wave's 64 token rows in the B tile

  LaneStats st;
  float lse2[2], mu[2];
#pragma unroll
  for (int fn = 0; fn < 2; ++fn) {
    st.m_s[fn] = kNegBig; st.Z_s[fn] = 0.f; st.A_s[fn] = 0.f; st.m_t[fn] = kNegBig; st.Z_t[fn] = 0.f;
    lse2[fn] = 0.f; mu[fn] = 0.f;
    if (PASS2) {
      const int64_t r = (int64_t)tt * kTileTokens + wave * 64 + fn * 32 + (lane & 31);
      lse2[fn] = a.lse2[r];
      mu[fn] = a.mu[r];
    }
  }

  for (int vt = vt_begin; vt < vt_end; ++vt) {
    const int v0 = vt * kTileVocab;
    {
      const int r = tid >> 3, c = tid & 7;
#pragma unroll
      for (int i = 0; i < kTileVocab / 32; ++i) {
        int v = v0 + entry_of_tile_row(r + 32 * i);   // staged row order, see entry_of_tile_row
        v = v < a.V ? v : a.V - 1;               // tail rows: load a valid row, masked below
        ws.p[i] = (const uint4*)(a.W_s + (int64_t)v * a.H_s) + c;
        wt.p[i] = (const uint4*)(a.W_t + (int64_t)v * a.H_t) + c;
      }
    }
    f32x16 zt[4][2], zs[4][2];
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < 2; ++fn)
#pragma unroll
        for (int e = 0; e < 16; ++e) { zt[fm][fn][e] = 0.f; zs[fm][fn][e] = 0.f; }
    gemm_kloop<kTileVocab, kTileTokens, 4, 2>(zt, wt, ht, 0, a.H_t / kBK, lds, kLogitStage, 0, waveB, tid);
    gemm_kloop<kTileVocab, kTileTokens, 4, 2>(zs, ws, hs, 0, a.H_s / kBK, lds, kLogitStage, 0, waveB, tid);

    const bool tail = v0 + kTileVocab > a.V;
    if (!PASS2) stats_epilogue(zs, zt, st, v0, a.V, tail, lane);
    else dz_epilogue(zs, zt, lse2, mu, a.slab + ((int64_t)tt_local * (a.Vp / kBK) + 2 * vt) * kSlabBlock,
                     wave * 64, v0, a.V, tail, lane, a.heavy, (int64_t)tt * kTileTokens + wave * 64);
  }
  if (!PASS2)
    write_partials(st, a.part, a.strips, strip, a.n_pad, (int64_t)tt * kTileTokens + wave * 64, lane);
}

// ---------------------------------------------------------------------------------------
// Logit passes, direct global->LDS staging.
//
// Same tile, MFMA roles and epilogues as logit_pass_kernel, but the k-tiles are moved by
// global_load_lds_dwordx4 (no register staging) into an LDS ring of kStages stages, kAhead
// k-steps ahead of the MFMAs (DmaTile), from tile images that already have the LDS layout (row_image_kernel
// below): one wave instruction moves 1 KiB of consecutive bytes, lane l its 16 bytes at 16 l.
// The teacher and student k-loops form one pipeline of H_t/64 + H_s/64 steps per vocabulary
// tile.
//
// The loads are written as inline assembly (M0 = LDS destination of the wave, 64-bit scalar
// base + 32-bit lane offset within the block) and waited for with explicit
// s_waitcnt vmcnt(N): the loads return in order, so "at most the loads of the kAhead - 1 later stages
// outstanding", kPerWave each, means this stage has landed.  Compiler-issued loads in between only make the
// count larger, i.e. the wait longer.
// ---------------------------------------------------------------------------------------
// FN = 2: tiles of 256 tokens, 64 to a wave, and a ring of three stages.  FN = 1, for calls of up to 128 rows:
// the first half of the one token tile, 32 tokens to a wave, and a ring of four.  With one token tile the
// sweep streams W from memory, and what bounds it is the bytes of W that are in flight per compute unit
// (16 KiB per stage and 1.5 us a round trip); the matrix work of the other half, all padding, is left out.
// 128 rows, V = 151,936, H = 2048 + 4096: sweep 497 -> 414 us (W at 4.5 TB/s), call 741 -> 648; 16 rows,
// H = 3584 + 4608: 986 -> 856; 100 rows, H = 1024 + 1024: 359 -> 318.  256 rows as two such tiles: 500 -> 650 us (the two
// workgroups that share W do not stay in step and fetch it twice).
template <int FN>
struct DmaTile {
  static constexpr int kTokens = 128 * FN, kStages = FN == 2 ? 3 : 4;
  static constexpr int kStage = (kTileVocab + kTokens) * kRowBytes;     // 48 KiB, 32 KiB
  static constexpr int kRing = kStages * kStage;                        // 144 KiB, 128 KiB
  // behind the ring, 4 KiB to a wave: the references of the single sweep, then (LINES) rows on their way to the slab
  static constexpr int kSideLds = 4096;
  static_assert(2 * kMaxRefParts * 256 <= kSideLds, "the references of a wave");
  static constexpr int kRefLds = kRing + 4 * kSideLds;
  static constexpr int kPerWave = (kTileVocab + kTokens) / 8 / 4;       // wave-loads per stage: 12, 8
  static constexpr int kAhead = kStages - 1;                            // k-steps from a load to its use
};

// Row images.  The direct-to-LDS logit kernel reads all four operands as LDS images of its
// k-steps: [rows, H] row-major (optionally gathered through row_idx) is re-laid as tiles of
// `th` consecutive rows; block (tile, kt) holds their k-entries 64 kt .. 64 kt + 63, row r at
// r * 128 B, its 16-byte chunk c at chunk position c ^ ((r >> 1) & 7); rows >= n_rows are
// zero.  Blocks of one tile are consecutive in kt.  Every wave-load then moves 1 KiB of
// consecutive bytes and no operand needs 32-bit lane offsets from its base.  With `permute`
// (the W operands) tile row r holds source row entry_of_tile_row(r) of the tile.

// `rows`: source rows of the tile (NULL: tile rows are source rows).
template <int THREADS, int TH>
__device__ __forceinline__ void image_block(const RowImageArgs& a, const int32_t* rows, int64_t tile, int kt) {
  constexpr int N = TH * 8 / THREADS;      // 16-byte chunks per thread, loaded together
  uint4* blk = a.img + ((tile * a.nk + kt) * TH) * 8;
  uint4 v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int q = threadIdx.x + i * THREADS;
    const int r = q >> 3, pos = q & 7, c = pos ^ ((r >> 1) & 7);
    const int64_t row = tile * TH + (a.permute ? entry_of_tile_row(r) : r);
    v[i] = make_uint4(0u, 0u, 0u, 0u);
    if (row < a.n_rows) {
      const int64_t src_row = rows ? (int64_t)rows[r] : row;
      v[i] = a.src[src_row * (a.H >> 3) + kt * 8 + c];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) blk[threadIdx.x + i * THREADS] = v[i];
}

// vocabulary tiles of 128 rows
__global__ __launch_bounds__(256) void row_image_kernel(RowImageArgs a) {
  image_block<256, kTileVocab>(a, nullptr, blockIdx.y, blockIdx.x);
}

constexpr int kImgABytes = kTileVocab * kRowBytes;    // 16 KiB: one W block
constexpr int kImgBBytes = kTileTokens * kRowBytes;   // 32 KiB: one h block

// Wave-load I (0 .. kPerWave - 1) of this wave for one stage: KiB (wave + 4 I) of the A block, then of
// the B block; lane l moves bytes 16 l .. 16 l + 15 of that KiB.  lds_wave = the stage's LDS
// address + 1024 wave; voffw[j] = 16 lane + 1024 (wave + 4 j): the wave's part of both addresses
// is folded into operands that are set up once, the rest is a literal.  voffa: the same for the
// A block, or the lane's offsets in the row-major W (direct staging).
template <int I, bool ONCE>
__device__ __forceinline__ void dma_one(uint32_t lds_wave, const uint32_t (&voffa)[4], const uint32_t (&voffw)[8],
                                        const char* sA, const char* sB) {
  if constexpr (I < kTileVocab / 32)
    dma16_at<4 * I * 1024, ONCE>(lds_wave, voffa[I], sA);
  else
    dma16_at<(kTileVocab / 8 + 4 * (I - kTileVocab / 32)) * 1024>(lds_wave, voffw[I - kTileVocab / 32], sB);
}

// One staged k-step (4 sub-steps of 4 FN MFMAs) of the 128 x 32 FN wave tile.  On entry fa[0],
// fb[0] hold the fragments of sub-step 0.  The instruction order is pinned: after each MFMA
// one or two side operations are issued in its shadow -- an LDS read of a fragment of the
// next sub-step (fragments are double-buffered), one of the kPerWave global->LDS loads of the
// stage kAhead k-steps on (every k-step loads) or a piece of the pipeline's bookkeeping -- so
// that neither the LDS latency nor the vector-memory issue holds up the matrix pipe.  The one
// barrier of the k-step sits before the last sub-step: by then every fragment of this stage is
// in registers, and the last sub-step's MFMAs cover the reads of the next stage's first
// fragments (the following ring slot, whose loads were issued kAhead - 1 k-steps earlier and are waited
// for here: kYounger younger ones may be outstanding).  LAST: no next stage in this vocabulary tile; no barrier and no fragment reads.
// FRESH: the k-step starts a new accumulation (first k-step of a head): its first MFMA on each
// block takes a zero addend, so the accumulators are never cleared.
// RELAXED > 0 (with `relaxed` set): the wait before the barrier lets RELAXED more operations
// stay in flight.  The counter takes loads and stores in the order of issue; the first k-step
// of a tile follows an epilogue that issued at least RELAXED stores after the loads this wait is
// for, and waiting for "all but the kYounger youngest" would mean waiting for every one of them.
// Ring and load state: r_rd = address (LDS base + 1024 wave + slot) of the slot consumed, on
// return that of the next k-step; swA/swB = the lane's fragment offsets from such an address
// per sub-step; (a_lo, a_hi), (b_lo, b_hi) = the blocks that the previous k-step loaded, on
// return those that this one loaded.
// A_STEP: bytes from one A block to the next (a W image's block, or a row-major W's 64 entries).
template <bool LAST, bool FRESH, int RELAXED, int A_STEP, int FN, bool ONCE>
__device__ __forceinline__ void sweep_kstep(f32x16 (&acc)[4][FN], bf16x8 (&fa)[2][4], bf16x8 (&fb)[2][FN],
                                            uint32_t& r_rd, uint32_t ring_begin, uint32_t ring_end,
                                            const uint32_t (&swA)[4], const uint32_t (&swB)[4],
                                            const uint32_t (&voffa)[4], const uint32_t (&voffw)[8],
                                            uint32_t& a_lo, uint32_t& a_hi,
                                            uint32_t& b_lo, uint32_t& b_hi, bool relaxed = false) {
  typedef DmaTile<FN> Tile;
  // loads issued after those of the next stage, up to the wait: whole stages, and three quarters of one
  constexpr int kYounger = (Tile::kAhead - 2) * Tile::kPerWave + Tile::kPerWave / 4 * 3;
  static_assert(kYounger + RELAXED <= 63, "the wait count has six bits");
  const f32x16 kZeroTile = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  uint32_t r_nx, r_wr;
#define ADWIN_FENCE __builtin_amdgcn_sched_barrier(0);
#define ADWIN_RA(KK, I) fa[((KK) + 1) & 1][I] = lds_frag(xa)[(I) * 32 * kRowBytes / 16]; ADWIN_FENCE
#define ADWIN_RB(KK, I) fb[((KK) + 1) & 1][I] = lds_frag(xb)[(I) * 32 * kRowBytes / 16]; ADWIN_FENCE
#define ADWIN_MM(KK, FMI, FNI)                                                                  \
  acc[FMI][FNI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[(KK) & 1][FMI], fb[(KK) & 1][FNI], \
                                                          (FRESH && (KK) == 0) ? kZeroTile : acc[FMI][FNI], 0, 0, 0); \
  ADWIN_FENCE
#define ADWIN_DMA(I) dma_one<I, ONCE>(r_wr, voffa, voffw, addr_of(a_lo, a_hi), addr_of(b_lo, b_hi)); ADWIN_FENCE
  // sub-step KK: 8 MFMAs; reads of the next sub-step's fragments from slot R when READ; H0..H3:
  // bookkeeping in the shadows of the first four MFMAs.  xa, xb: the lane's LDS addresses of its
  // first A and B fragment, formed once (and kept from being re-associated with the fragments'
  // constant offsets, which belong in the read instructions).
#define ADWIN_SUB(KK, READ, R, D0, D1, D2, H0, H1, H2, H3)                    \
  {                                                                     \
    uint32_t xa = 0, xb = 0;                                            \
    ADWIN_MM(KK, 0, 0)                                                  \
    if constexpr (READ) {                                               \
      xa = (R) + swA[((KK) + 1) & 3]; xb = (R) + swB[((KK) + 1) & 3];   \
      asm volatile("" : "+v"(xa), "+v"(xb));                            \
      ADWIN_RA(KK, 0)                                                   \
    }                                                                   \
    H0 ADWIN_FENCE                                                      \
    ADWIN_MM(KK, 0, 1) if constexpr (READ) { ADWIN_RB(KK, 0) } H1 ADWIN_FENCE \
    ADWIN_MM(KK, 1, 0) if constexpr (READ) { ADWIN_RA(KK, 1) } H2 ADWIN_FENCE \
    ADWIN_MM(KK, 1, 1) if constexpr (READ) { ADWIN_RB(KK, 1) } H3 ADWIN_FENCE \
    ADWIN_MM(KK, 2, 0) if constexpr (READ) { ADWIN_RA(KK, 2) }          \
    ADWIN_MM(KK, 2, 1) if constexpr (READ) { ADWIN_RA(KK, 3) } ADWIN_DMA(D0) \
    ADWIN_MM(KK, 3, 0) ADWIN_DMA(D1)                                    \
    ADWIN_MM(KK, 3, 1) ADWIN_DMA(D2)                                    \
  }
  // 4 MFMAs a sub-step with one token column
#define ADWIN_SUB1(KK, READ, R, D0, D1, H0, H1, H2, H3)                       \
  {                                                                     \
    uint32_t xa = 0, xb = 0;                                            \
    ADWIN_MM(KK, 0, 0)                                                  \
    if constexpr (READ) {                                               \
      xa = (R) + swA[((KK) + 1) & 3]; xb = (R) + swB[((KK) + 1) & 3];   \
      asm volatile("" : "+v"(xa), "+v"(xb));                            \
      ADWIN_RA(KK, 0) ADWIN_RB(KK, 0)                                   \
    }                                                                   \
    H0 ADWIN_FENCE                                                      \
    ADWIN_MM(KK, 1, 0) if constexpr (READ) { ADWIN_RA(KK, 1) } H1 ADWIN_FENCE \
    ADWIN_MM(KK, 2, 0) if constexpr (READ) { ADWIN_RA(KK, 2) } H2 ADWIN_FENCE ADWIN_DMA(D0) \
    ADWIN_MM(KK, 3, 0) if constexpr (READ) { ADWIN_RA(KK, 3) } H3 ADWIN_FENCE ADWIN_DMA(D1) \
  }
#define ADWIN_NEXT(X) ring_next<Tile::kStage>(X, ring_begin, ring_end)
  ADWIN_FENCE
  if constexpr (FN == 1) {
    ADWIN_SUB1(0, true, r_rd, 0, 1, { r_nx = ADWIN_NEXT(r_rd); }, { r_wr = ADWIN_NEXT(ADWIN_NEXT(r_nx)); addr_advance<A_STEP>(a_lo, a_hi); },
               { addr_advance<kImgBBytes>(b_lo, b_hi); }, {})
    ADWIN_SUB1(1, true, r_rd, 2, 3, {}, {}, {}, {})
    ADWIN_SUB1(2, true, r_rd, 4, 5, {}, {}, {}, {})
  } else {
  ADWIN_SUB(0, true, r_rd, 0, 1, 2,
            { r_nx = ADWIN_NEXT(r_rd); }, { r_wr = ADWIN_NEXT(r_nx); },
            { addr_advance<A_STEP>(a_lo, a_hi); }, { addr_advance<kImgBBytes>(b_lo, b_hi); })
  ADWIN_SUB(1, true, r_rd, 3, 4, 5, {}, {}, {}, {})
  ADWIN_SUB(2, true, r_rd, 6, 7, 8, {}, {}, {}, {})
  }
  if constexpr (!LAST) {
    if constexpr (RELAXED > 0) {
      if (relaxed) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kYounger + RELAXED) : "memory");
      else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kYounger) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kYounger) : "memory");
    }
    __syncthreads();
  }
  ADWIN_FENCE
  if constexpr (FN == 1) {
    ADWIN_SUB1(3, !LAST, r_nx, 6, 7, {}, {}, {}, {})
  } else {
  ADWIN_SUB(3, !LAST, r_nx, 9, 10, 11, {}, {}, {}, {})
  }
  r_rd = r_nx;
#undef ADWIN_NEXT
#undef ADWIN_SUB1
#undef ADWIN_SUB
#undef ADWIN_DMA
#undef ADWIN_MM
#undef ADWIN_RB
#undef ADWIN_RA
#undef ADWIN_FENCE
}

// STAGE, where the W tiles come from.  Rows: the row-major weights instead of their images: wave-load I
// takes its 8 rows' 128 bytes from 8 rows of W, the lane offsets following the image's row
// permutation and chunk swizzle, so that the LDS holds the same bytes; rows beyond V repeat the
// last one (their logits are masked like the image's zero rows).  Rows once: the same, of a single token tile, whose lines
// of W go past the L2; or those of the teacher only (sweep_stage).
template <int MODE, int STAGE, int FN = 2, bool LINES = false>
__global__ __launch_bounds__(256) void logit_pass_dma_kernel(LogitPassArgs a) {
  extern __shared__ __align__(16) char lds[];
  typedef DmaTile<FN> Tile;
  constexpr bool DIRECT = STAGE != kStageImages, kOnce = STAGE >= kStageRowsOnce;
  static_assert(!LINES || FN == 2, "groups of two token columns");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int strip, tt_local;
  {
    int block = blockIdx.x, blocks = gridDim.x, strips = a.strips, first = 0;
    if (a.long_first) {                       // the longer strips of all token tiles, then the others
      const int n = a.strip_tiles.longer * a.n_tiles;
      if (block < n) { blocks = n; strips = a.strip_tiles.longer; }
      else { block -= n; blocks -= n; first = a.strip_tiles.longer; strips -= first; }
    }
    strip_and_tile(xcd_contiguous_id(block, blocks), a.tg, strips, a.n_tiles, &strip, &tt_local);
    // the longer strips of a group of token tiles first: in index order, where they are spread, the last ones to start are
    // longer ones (4,096 rows of V = 151,936, H = 2048 + 4096 9205 us per call, so 9110; statistics 1 % as well)
    strip = a.strip_tiles.by_length(strip + first);
  }
  const int tt = a.tile0 + tt_local;
  const int64_t row_tile = (int64_t)tt * kTileTokens;
  const int vt_begin = a.strip_tiles.first(strip), vt_end = a.strip_tiles.first(strip + 1);
  if (vt_begin >= vt_end) return;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

  uint32_t voffw[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    voffw[j] = (uint32_t)lane * 16u + (uint32_t)(wave + 4 * j) * 1024u;
    asm volatile("" : "+v"(voffw[j]));   // kept in registers, not recomputed at every load
  }
  // ring slot addresses carry the wave's KiB (for the loads); the fragment offsets take it out again
  const uint32_t ring_begin = lds0 + (uint32_t)wave * 1024u, ring_end = ring_begin + Tile::kRing;
  uint32_t swA[4], swB[4];
  {
    const int key = (lane >> 1) & 7, half = lane >> 5;
    const uint32_t rowoff = (uint32_t)(lane & 31) * kRowBytes - (uint32_t)wave * 1024u;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      swA[kk] = rowoff + (uint32_t)(((kk * 2 + half) ^ key) << 4);
      swB[kk] = swA[kk] + (uint32_t)(kTileVocab * kRowBytes + wave * 32 * FN * kRowBytes);
    }
  }
  const int nk_t = a.H_t / kBK, nk_s = a.H_s / kBK, nk = nk_t + nk_s;   // each >= 2 on this path
  // blocks of this token tile (fixed) and of vocabulary tile vt, teacher and student
  const char* sHt = a.ht_img + (int64_t)tt * nk_t * kImgBBytes;
  const char* sHs = a.hs_img + (int64_t)tt * nk_s * kImgBBytes;
  constexpr int kAStep = DIRECT ? kRowBytes : kImgABytes;
  uint32_t voffa[4];
  // lane offsets of the wave's four A loads for the rows of vocabulary tile vt of a [V, H] operand:
  // tile row 8 wave + 32 I + lane / 8 holds entry 32 I + e0 (entry_of_tile_row)
  const int e0 = 16 * (lane >> 5) + 4 * wave + ((lane >> 3) & 3);
  const uint32_t chunk = (uint32_t)((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7)) * 16u;
  const uint32_t row0_t = (uint32_t)e0 * (uint32_t)a.H_t * 2u + chunk, row0_s = (uint32_t)e0 * (uint32_t)a.H_s * 2u + chunk;
  auto rows_w = [&](int vt, int H, uint32_t row0) __attribute__((always_inline)) {
    if constexpr (DIRECT) {
      const int left = a.V - vt * kTileVocab;
      if constexpr (MODE == kModeSingleDiag) {
        // The sweep with the most state: e0, the chunk and both row0 are formed from the lane number
        // again for each head of a tile (the asm hides that they could be kept).  Kept, they were the
        // registers that made it spill 13: V = 32,776, H = 1024 + 1024, 28 token tiles 1842 -> 1808 us
        // per call, H = 512 + 640 (V = 11,912, 13 tiles) 287 -> 278.  The others have the registers
        // and lose up to 1 % this way.
        int l = lane;
        asm volatile("" : "+v"(l));
        const int e = 16 * (l >> 5) + 4 * wave + ((l >> 3) & 3);
        const uint32_t c = (uint32_t)((l & 7) ^ ((4 * wave + (l >> 4)) & 7)) * 16u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = 32 * i + e < left ? 32 * i + e : left - 1;
          voffa[i] = (uint32_t)v * ((uint32_t)H * 2u) + c;
        }
      } else if (left >= kTileVocab) {
#pragma unroll
        for (int i = 0; i < 4; ++i) voffa[i] = row0 + (uint32_t)(i * 64 * H);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = 32 * i + e0 < left ? 32 * i + e0 : left - 1;
          voffa[i] = (uint32_t)v * ((uint32_t)H * 2u) + chunk;
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(voffa[i]));
    }
  };
  if constexpr (!DIRECT) {
#pragma unroll
    for (int i = 0; i < 4; ++i) voffa[i] = voffw[i];
  }
  auto blocks_wt = [&](int vt) {
    return DIRECT ? (const char*)a.W_t + (int64_t)vt * kTileVocab * a.H_t * 2 : a.Wt_img + (int64_t)vt * nk_t * kImgABytes;
  };
  auto blocks_ws = [&](int vt) {
    return DIRECT ? (const char*)a.W_s + (int64_t)vt * kTileVocab * a.H_s * 2 : a.Ws_img + (int64_t)vt * nk_s * kImgABytes;
  };

  LaneStats st;
  LaneSums sm;
  constexpr bool kDiag = MODE == kModeSingleDiag || MODE == kModeSingleE2Diag || MODE == kModeSingleFwdDiag;
  constexpr bool kWriteE2 = MODE < kModeSingleFwd;
  constexpr bool kWriteD = MODE == kModeSingle || MODE == kModeSingleDiag;
  constexpr bool kSingle = MODE >= kModeSingle;
  float lse2[2], mu[2], rs2[2], rt2[2];   // per-row inputs of the dz / single-sweep epilogues
  float zyt[2];
  int yid[2];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    st.m_s[fn] = kNegBig; st.Z_s[fn] = 0.f; st.A_s[fn] = 0.f; st.m_t[fn] = kNegBig; st.Z_t[fn] = 0.f;
    sm.Z_s[fn] = 0.f; sm.A_s[fn] = 0.f; sm.Z_t[fn] = 0.f; sm.B_t[fn] = 0.f; sm.cnt[fn] = 0;
    lse2[fn] = 0.f; mu[fn] = 0.f; rs2[fn] = 0.f; rt2[fn] = 0.f; zyt[fn] = 0.f; yid[fn] = -1;
    const int64_t r = row_tile + wave * (32 * FN) + fn * 32 + (lane & 31);
    if (MODE == kModeDz) {
      lse2[fn] = a.lse2[r];
      mu[fn] = a.mu[r];
    } else if (kSingle) {
      if (kDiag) { zyt[fn] = a.ref.zy[1][r]; yid[fn] = a.ref.yid[r]; }
    }
  }
  // The references go into the LDS behind the ring, ahead of the first stages: loaded into registers they
  // made every workgroup wait for one more round trip before it asked for its first stage.
  const uint32_t side_lds = lds0 + Tile::kRing + (uint32_t)wave * Tile::kSideLds;
  if (kSingle) {
    const uint32_t row = (uint32_t)(lane & (32 * FN - 1)) * 4u;
    for (int k = 0; k < 2 * a.ref.parts; ++k) {
      const int head = k >= a.ref.parts, plane = head ? k - a.ref.parts : k;
      dma4_at<0>(side_lds + (uint32_t)k * 256u, row,
                 (const char*)(a.ref.max[head] + plane * a.ref.n_pad + row_tile + wave * (32 * FN)));
    }
  }

  // The k-steps of all vocabulary tiles of the strip form one pipeline: per tile nk_t
  // teacher steps, then nk_s student steps; step g is staged into ring slot g % kStages kAhead steps
  // before it is consumed, also across head and tile boundaries (the next tile's first kAhead steps
  // are loaded during this tile's last ones, i.e. before and under the epilogue).  ld*: the step
  // whose loads were issued last; past the strip's last step the walk wraps to the strip's first
  // tile, so that every k-step loads (those last blocks land in slots nobody reads any more).
  // (a, b) = the blocks of that step; a k-step moves them on by one block before it loads, so
  // at the start of a head they are set one block in front of it.  A head that begins at k-step k0
  // comes back to 0 after its last: ld_lim steps, then the ld_rest others.
  uint32_t r_rd = ring_begin;  // ring slot (address) of the next step to consume
  // the k-step a head of a tile begins with: its own for every strip if there is one token tile (see
  // LogitPassArgs::rotate), else 0
  const int k0_t = DIRECT && a.rotate ? strip % nk_t : 0, k0_s = DIRECT && a.rotate ? strip % nk_s : 0;
  int ld_vt = vt_begin, ld_k = 0, ld_lim = nk_t - k0_t, ld_rest = k0_t;
  bool ld_student = false;
  uint32_t a_lo, a_hi, b_lo, b_hi;
#define ADWIN_SET_BLOCKS(A, B, K0)                                         \
  {                                                                        \
    const uint64_t pa = (uint64_t)(A) + (int64_t)((K0) - 1) * kAStep;      \
    const uint64_t pb = (uint64_t)(B) + (int64_t)((K0) - 1) * kImgBBytes;  \
    a_lo = (uint32_t)pa; a_hi = (uint32_t)(pa >> 32);                      \
    b_lo = (uint32_t)pb; b_hi = (uint32_t)(pb >> 32);                      \
  }
#define ADWIN_COUNT_LOADS()                                                \
  {                                                                        \
    if (++ld_k == ld_lim) {                                                \
      ld_k = 0;                                                            \
      if (DIRECT && ld_rest) {          /* the head's first k-steps, which come last */ \
        ld_lim = ld_rest; ld_rest = 0;                                     \
        if (ld_student) ADWIN_SET_BLOCKS(blocks_ws(ld_vt), sHs, 0)         \
        else ADWIN_SET_BLOCKS(blocks_wt(ld_vt), sHt, 0)                    \
      } else if (!ld_student) {                                            \
        ld_student = true; ld_lim = nk_s - k0_s; ld_rest = k0_s;           \
        ADWIN_SET_BLOCKS(blocks_ws(ld_vt), sHs, k0_s)                      \
        rows_w(ld_vt, a.H_s, row0_s);                                      \
      } else {                                                             \
        ld_student = false; ld_lim = nk_t - k0_t; ld_rest = k0_t;          \
        ld_vt = ld_vt + 1 < vt_end ? ld_vt + 1 : vt_begin;                 \
        ADWIN_SET_BLOCKS(blocks_wt(ld_vt), sHt, k0_t)                      \
        rows_w(ld_vt, a.H_t, row0_t);                                      \
      }                                                                    \
    }                                                                      \
  }
  ADWIN_SET_BLOCKS(blocks_wt(vt_begin), sHt, k0_t)
  rows_w(vt_begin, a.H_t, row0_t);
#pragma unroll
  for (int i = 0; i < Tile::kAhead; ++i) {
    const uint32_t dst = ring_begin + (uint32_t)i * Tile::kStage;
    addr_advance<kAStep>(a_lo, a_hi);
    addr_advance<kImgBBytes>(b_lo, b_hi);
    const char* ldA = addr_of(a_lo, a_hi);
    const char* ldB = addr_of(b_lo, b_hi);
    dma_one<0, kOnce>(dst, voffa, voffw, ldA, ldB); dma_one<1, kOnce>(dst, voffa, voffw, ldA, ldB);
    dma_one<2, kOnce>(dst, voffa, voffw, ldA, ldB); dma_one<3, kOnce>(dst, voffa, voffw, ldA, ldB);
    dma_one<4, kOnce>(dst, voffa, voffw, ldA, ldB); dma_one<5, kOnce>(dst, voffa, voffw, ldA, ldB);
    dma_one<6, kOnce>(dst, voffa, voffw, ldA, ldB); dma_one<7, kOnce>(dst, voffa, voffw, ldA, ldB);
    if constexpr (FN == 2) {
      dma_one<8, kOnce>(dst, voffa, voffw, ldA, ldB); dma_one<9, kOnce>(dst, voffa, voffw, ldA, ldB);
      dma_one<10, kOnce>(dst, voffa, voffw, ldA, ldB); dma_one<11, kOnce>(dst, voffa, voffw, ldA, ldB);
    }
    ADWIN_COUNT_LOADS()
  }
  if (kSingle) {
    typedef const __attribute__((address_space(3))) float* LdsFloat;
    wait_vm<Tile::kAhead * Tile::kPerWave>();  // all but the stages
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const LdsFloat p = (LdsFloat)(uintptr_t)(side_lds + (uint32_t)(fn * 32 + (lane & 31)) * 4u);
      float m[2] = {p[0], p[a.ref.parts * 64]};
      for (int k = 1; k < a.ref.parts; ++k) { m[0] = fmaxf(m[0], p[k * 64]); m[1] = fmaxf(m[1], p[(a.ref.parts + k) * 64]); }
      rs2[fn] = References::scaled(m[0]);
      rt2[fn] = References::scaled(m[1]);
    }
  }
  // 16-byte stores a wave issues per tile in its epilogue, at the least (see sweep_kstep, RELAXED)
  constexpr int kEpilogueStores = MODE == kModeDz ? 16 : (kWriteE2 && kSingle ? 8 * FN : 0) + (kWriteD ? 8 * FN : 0);
  f32x16 zt[4][FN], zs[4][FN];
  bf16x8 fa[2][4], fb[2][FN];
  // one k-step: consume slot r_rd, prefetch fragments from the following slot, load into the one after
  auto step = [&](auto last_c, auto fresh_c, auto relaxed_c, auto once_c, f32x16 (&acc)[4][FN], bool relaxed)
                  __attribute__((always_inline)) {
    constexpr bool kLast = decltype(last_c)::value, kFresh = decltype(fresh_c)::value;
    constexpr int kRelaxed = decltype(relaxed_c)::value;
    sweep_kstep<kLast, kFresh, kRelaxed, kAStep, FN, decltype(once_c)::value>(acc, fa, fb, r_rd, ring_begin, ring_end, swA, swB, voffa, voffw,
                                         a_lo, a_hi, b_lo, b_hi, relaxed);
    ADWIN_COUNT_LOADS()
  };
  const std::true_type yes{};
  const std::false_type no{};
  const std::integral_constant<int, 0> strict{};
  // the loads of a head's steps, of which the last kAhead already ask for the other's blocks
  const std::integral_constant<bool, kOnce> once_t{};
  const std::integral_constant<bool, STAGE == kStageRowsOnce> once_s{};
  const std::integral_constant<int, kEpilogueStores> after_epilogue{};
  for (int vt = vt_begin; vt < vt_end; ++vt) {
    const int v0 = vt * kTileVocab;
    // Step 0 of this tile has landed once at most the loads of the steps after it are outstanding.  For
    // the strip's first tile that is waited for here; for every later tile it was waited for
    // before the previous tile's epilogue (below): the counter takes loads and stores in order,
    // so a wait placed here would also wait for nearly all of that epilogue's stores.
    if (vt == vt_begin) wait_vm<(Tile::kAhead - 1) * Tile::kPerWave>();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[0][i] = lds_frag(r_rd + swA[0])[i * 32 * kRowBytes / 16];
#pragma unroll
    for (int i = 0; i < FN; ++i) fb[0][i] = lds_frag(r_rd + swB[0])[i * 32 * kRowBytes / 16];
    // teacher: nk_t k-steps (the first on a zero addend; after an epilogue its wait leaves that
    // epilogue's stores in flight), then student: nk_s k-steps, the last without a barrier
    step(no, yes, after_epilogue, once_t, zt, vt != vt_begin);
    for (int s = 1; s < nk_t; ++s) step(no, no, strict, once_t, zt, false);
    step(no, yes, strict, once_s, zs, false);
    for (int s = 1; s + 1 < nk_s; ++s) step(no, no, strict, once_s, zs, false);
    step(yes, no, strict, once_s, zs, false);
    wait_vm<(Tile::kAhead - 1) * Tile::kPerWave>();      // the next tile's step 0 (see the top of the loop)
    const bool tail = v0 + kTileVocab > a.V;
    const int wave_row = wave * (32 * FN);                // of the 256-row image
    __bf16* blk = a.slab + ((int64_t)(tt - a.tile0) * (a.Vp / kBK) + 2 * vt) * kSlabBlock;
    if constexpr (MODE == kModeStats) {
      stats_epilogue(zs, zt, st, v0, a.V, tail, lane);
    } else if constexpr (MODE == kModeDz) {
      dz_epilogue(zs, zt, lse2, mu, blk, wave_row, v0, a.V, tail, lane, a.heavy, row_tile + wave * (32 * FN));
    } else {
      float* m0t = a.mu0t ? a.mu0t + (int64_t)vt * a.mu0t_stride + (int64_t)(tt - a.tile0) * kTileTokens + wave_row : nullptr;
      if (tail) {
        single_epilogue<true, kDiag, kWriteD, kWriteE2, FN, LINES>(zs, zt, sm, rs2, rt2, mu, zyt, yid, blk, a.e2_off, wave_row, v0, a.V, lane, m0t, side_lds);
      } else {
        single_epilogue<false, kDiag, kWriteD, kWriteE2, FN, LINES>(zs, zt, sm, rs2, rt2, mu, zyt, yid, blk, a.e2_off, wave_row, v0, a.V, lane, m0t, side_lds);
      }
    }
  }
#undef ADWIN_COUNT_LOADS
#undef ADWIN_SET_BLOCKS
  wait_vm<0>();      // the strip's last kAhead k-steps loaded blocks nobody reads: landed before the LDS is released
  const int64_t row0 = row_tile + wave * (32 * FN);
  if (MODE == kModeStats) write_partials(st, a.part, a.strips, strip, a.n_pad, row0, lane);
  else if (kSingle) write_sums<kDiag, FN>(sm, a.part, a.strips, strip, a.n_pad, row0, lane);
}

// ---------------------------------------------------------------------------------------
// Merge of the strip partials, KL_t and c_t.  One wave per computed row.
// ---------------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void merge_stats_kernel(MergeArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= a.n_pad) return;
  const int64_t plane = (int64_t)a.strips * a.n_pad;
  float ms = kNegBig, Zs = 0.f, A = 0.f, mt = kNegBig, Zt = 0.f;
  if (lane < a.strips) {
    const float* p = a.part + (int64_t)lane * a.n_pad + r;
    ms = p[0]; Zs = p[plane]; A = p[2 * plane]; mt = p[3 * plane]; Zt = p[4 * plane];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    merge_mza(ms, Zs, A, __shfl_xor(ms, o, 64), __shfl_xor(Zs, o, 64), __shfl_xor(A, o, 64));
    merge_mz(mt, Zt, __shfl_xor(mt, o, 64), __shfl_xor(Zt, o, 64));
  }
  const float lse_s = ms + logf(Zs), lse_t = mt + logf(Zt);
  const float mu = A / Zs;                  // E_{p_s}[z_s - z_t]
  float kl = kl_from_sums(mu, ms - mt, Zs, Zt);
  // a row without a finite log-sum-exp, mean or KL is excluded: zeros in every output
  const bool dead = !(fabsf(lse_s) < 3.0e38f) || !(fabsf(lse_t) < 3.0e38f) || !(fabsf(kl) < 3.0e38f) ||
                    !(fabsf(mu) < 3.0e38f);
  if (dead) kl = 0.f;
  if (lane == 0) {
    a.lse2[r] = dead ? 0.f : lse_s * kLog2e;
    a.mu[r] = dead ? 0.f : mu;
    a.klr[r] = kl;
    a.lse_s[r] = dead ? 0.f : lse_s;
    a.alive[r] = dead ? 0.f : 1.f;
  }
  if (r >= a.n_rows) return;                // padding rows feed pass 2 only
  const int64_t t = a.row_idx[r];
  float c = 0.f;
  uint32_t flag = dead ? ADWIN_DEV_NONFINITE : 0u;
  if (a.ids && a.c && !dead) {
    const int y = a.ids[t];
    if (y >= 0 && y < a.V) {
      const float zy_s = dot_bf16_row(a.h_s + t * a.H_s, a.W_s + (int64_t)y * a.H_s, a.H_s, lane);
      const float zy_t = dot_bf16_row(a.h_t + t * a.H_t, a.W_t + (int64_t)y * a.H_t, a.H_t, lane);
      c = (zy_s - lse_s) - (zy_t - lse_t);
    } else {
      flag |= ADWIN_DEV_BAD_ID;
    }
  }
  if (lane == 0) {
    if (flag && a.status) atomicOr(a.status, flag);
    if (a.kl) a.kl[t] = kl;
    if (a.c) a.c[t] = c;
  }
}

// ---------------------------------------------------------------------------------------
// Single-sweep mode: what a call prepares for its sweep, in one launch: the references of every row
// (maxima over vocabulary tile 0, 128 entries, under both models), the logits of its sampled token,
// z_s[y_t] = h_s . W_s[y_t] and z_t[y_t] = h_t . W_t[y_t], which the merge and the diagnostics sweep
// use again, and the hidden states as tile images.
// The references are bound by latency, in two forms (the line between them: see launch_prepare).
//
// Calls of few token tiles: cut as finely as the maxima allow.  A workgroup takes 32 rows, one model and
// one block of 32 entries, its waves an eighth of the k-blocks each, straight from the row-major operands
// into the fragments: no staging, no barrier before the partial sums meet.  The order of k is free, so
// a lane takes 64 consecutive bytes of its row per k-block of 64 (lane / 32 picks the half), four
// fragments of either operand.  (A lane's 16 bytes of a fragment in its place, k = 8 (lane / 32) .. + 7
// of 16, costs the L1 a line each, in kilobyte strides.)  256 rows at H = 2048 + 4096, with the images: 48 us
// as eight workgroups of the other form, 17 as these 64; 800 rows at H = 2048 + 3072 32.5 -> 18.5.
//
// Others: 32 rows, one model and all four blocks to a workgroup of 8 waves, one per block and half of every
// k-step, loads kRefLead k-steps ahead.  Stages of 20 KiB: 60 KiB of LDS, so that a compute unit holds two
// workgroups, which hide each other's barriers: with one of six stages and both models 13 token tiles at H = 512 + 640
// took 17.0 us against 13.2, 30 tiles at H = 1536 + 2048 54.9 against 46.5 (both with the images), 134 tiles at
// H = 2048 + 4096 330 against 304.  Every operand line is moved into the LDS once; read into registers by the
// waves that use it, it goes through the L1 up to five times, which is what bounds the form above (13
// token tiles: 20.6 us).
// ---------------------------------------------------------------------------------------
constexpr int kPrepThreads = 512, kPrepWaves = kPrepThreads / 64;
constexpr int kRefRows = 32, kRefLead = 2;
constexpr int kRefStage = (kTileVocab + kRefRows) * kRowBytes;          // 20 KiB
constexpr int kRefLds = (kRefLead + 1) * kRefStage;                     // 60 KiB
constexpr int kOneLaunchTiles = 32;
constexpr int kRefFineLds = kPrepWaves * 17 * 64 * 4;                   // 34 KiB

// As dma16_at, from a 64-bit address per lane.
__device__ __forceinline__ void dma16_from(uint32_t lds, const char* src) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(src) : "memory");
}

// Four computed rows of a wave: their packed positions and sampled tokens (-1: none, or out of range).
constexpr int kTokenRows = 4;
struct TokenRows {
  int64_t row0, t[kTokenRows];
  int y[kTokenRows];
  bool any;
  __device__ __forceinline__ TokenRows(const PrepareArgs& a, const int32_t* rows, int64_t first) : row0(first), any(false) {
#pragma unroll
    for (int i = 0; i < kTokenRows; ++i) t[i] = rows[i];
#pragma unroll
    for (int i = 0; i < kTokenRows; ++i) {
      y[i] = a.ids ? a.ids[t[i]] : -1;
      if (y[i] < 0 || y[i] >= a.V) y[i] = -1;
      any |= y[i] >= 0;
    }
  }
};

// The sampled tokens' logits under one model, by one wave, the loads of all four rows together.  Lane i < 4
// returns that of row i, kNegBig without a token.
__device__ __forceinline__ float token_logits(const PrepareArgs& a, const TokenRows& r, int head, int lane) {
  const int H = a.H[head];
  const uint4 *x[kTokenRows], *w[kTokenRows];
  float z[kTokenRows], mine = kNegBig;
#pragma unroll
  for (int i = 0; i < kTokenRows; ++i) {
    x[i] = (const uint4*)(a.h[head] + r.t[i] * H);
    w[i] = (const uint4*)(a.W[head] + (int64_t)(r.y[i] >= 0 ? r.y[i] : 0) * H);
    z[i] = 0.f;
  }
  if (r.any) {                                      // uniform: the rows are the wave's
#pragma unroll 2
    for (int q = lane; q < (H >> 3); q += 64) {
      uint4 p[kTokenRows], o[kTokenRows];
#pragma unroll
      for (int i = 0; i < kTokenRows; ++i) { p[i] = x[i][q]; o[i] = w[i][q]; }
#pragma unroll
      for (int i = 0; i < kTokenRows; ++i) {        // as in dot_bf16_row
        z[i] = fmaf(bf16_lo(p[i].x), bf16_lo(o[i].x), z[i]); z[i] = fmaf(bf16_hi(p[i].x), bf16_hi(o[i].x), z[i]);
        z[i] = fmaf(bf16_lo(p[i].y), bf16_lo(o[i].y), z[i]); z[i] = fmaf(bf16_hi(p[i].y), bf16_hi(o[i].y), z[i]);
        z[i] = fmaf(bf16_lo(p[i].z), bf16_lo(o[i].z), z[i]); z[i] = fmaf(bf16_hi(p[i].z), bf16_hi(o[i].z), z[i]);
        z[i] = fmaf(bf16_lo(p[i].w), bf16_lo(o[i].w), z[i]); z[i] = fmaf(bf16_hi(p[i].w), bf16_hi(o[i].w), z[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kTokenRows; ++i) {
    z[i] = wave_sum(z[i]);
    if (lane == i) {
      a.ref.zy[head][r.row0 + i] = r.y[i] >= 0 ? z[i] : 0.f;
      if (head == 0) a.ref.yid[r.row0 + i] = r.y[i];
      if (r.y[i] >= 0) mine = z[i];
    }
  }
  return mine;
}

// References of 32 rows under one model, the tokens of four of them by each wave.
__device__ __forceinline__ void refs_staged_block(const PrepareArgs& a, const int32_t* rows, int64_t row0, int head, char* lds) {
  __shared__ float token[kRefRows];
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int H = a.H[head], nk = H / kBK;
  // A stage: 128 rows of W (tile 0; rows beyond V repeat the last, masked below), then 32 of h, row r
  // at 128 r, chunk c at position c ^ ((r >> 1) & 7).  Wave-load i < 2 of a wave: W rows
  // 16 wave + 8 i .. + 7; the third, of waves 0 to 3 only: h rows 8 wave .. + 7.
  const char* src[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int m = i < 2 ? 2 * wave + i : (wave & 3), r = 8 * m + (lane >> 3);
    const uint32_t chunk = (uint32_t)((lane & 7) ^ ((r >> 1) & 7)) * 16u;
    const int64_t row = i < 2 ? (r < a.V ? r : a.V - 1) : rows[r];
    src[i] = (const char*)((i < 2 ? a.W[head] : a.h[head]) + row * H) + chunk;
  }
  auto load = [&](int s) __attribute__((always_inline)) {      // past the last k-step: that one again
    const uint32_t slot = lds0 + (uint32_t)(s % (kRefLead + 1)) * kRefStage;
    const int64_t off = (int64_t)(s < nk ? s : nk - 1) * kRowBytes;
    dma16_from(slot + (uint32_t)(2 * wave) * 1024u, src[0] + off);
    dma16_from(slot + (uint32_t)(2 * wave + 1) * 1024u, src[1] + off);
    if (wave < 4) dma16_from(slot + (uint32_t)(16 + wave) * 1024u, src[2] + off);
  };
  for (int s = 0; s < kRefLead; ++s) load(s);
  {
    const TokenRows four(a, rows + wave * kTokenRows, row0 + wave * kTokenRows);
    const float y = token_logits(a, four, head, lane);
    if (lane < kTokenRows) token[wave * kTokenRows + lane] = y;
  }
  // wave = vocabulary block vb, half kq of every k-step; A = W rows, B = h rows as in the sweep
  const int vb = wave & 3, kq = wave >> 2;
  f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const uint32_t key = (uint32_t)(lane >> 1) & 7u, frag = (uint32_t)(lane & 31) * kRowBytes;
  for (int s = 0; s < nk; ++s) {
    // stage s has landed once at most the loads of the kRefLead - 1 later ones are outstanding;
    // past the barrier every wave is done with stage s - 1, whose slot the next load takes
    if (wave < 4) wait_vm<3 * (kRefLead - 1)>();
    else wait_vm<2 * (kRefLead - 1)>();
    __syncthreads();
    const uint32_t slot = lds0 + (uint32_t)(s % (kRefLead + 1)) * kRefStage + frag;
    bf16x8 fa[2], fb[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t sw = ((uint32_t)(4 * kq + 2 * j + half) ^ key) << 4;
      fa[j] = *lds_frag(slot + (uint32_t)(vb * 32 * kRowBytes) + sw);
      fb[j] = *lds_frag(slot + (uint32_t)(kTileVocab * kRowBytes) + sw);
    }
    load(s + kRefLead);
#pragma unroll
    for (int j = 0; j < 2; ++j) z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[j], fb[j], z, 0, 0, 0);
  }
  wait_vm<0>();
  __syncthreads();                                 // the ring is free from here on
  float(*half_sum)[16][64] = (float(*)[16][64])lds;                // [4]: of the second halves
  float(*top)[kRefRows] = (float(*)[kRefRows])(lds + 4 * 16 * 64 * 4);    // [4]: maxima
  if (kq) {
#pragma unroll
    for (int e = 0; e < 16; ++e) half_sum[vb][e][lane] = z[e];
  }
  __syncthreads();
  if (!kq) {
    float m = kNegBig;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      z[e] += half_sum[vb][e][lane];
      if (vb * 32 + 8 * (e >> 2) + 4 * half + (e & 3) < a.V) m = fmaxf(m, z[e]);
    }
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if (lane < 32) top[vb][lane] = m;
  }
  __syncthreads();
  const int r = threadIdx.x;
  if (r < kRefRows) a.ref.max[head][row0 + r] = fmaxf(fmaxf(fmaxf(top[0][r], top[1][r]), fmaxf(top[2][r], top[3][r])), token[r]);
}

// References of 32 rows, one model, one vocabulary block.
__device__ __forceinline__ void refs_fine_block(const PrepareArgs& a, const int32_t* rows, int blk, char* lds) {
  float(*part)[16][64] = (float(*)[16][64])lds;     // [kPrepWaves] a wave's partial logits
  float(*top)[64] = (float(*)[64])(lds + kPrepWaves * 16 * 64 * 4);   // [kPrepWaves]
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int head = blk & 1, vb = (blk >> 1) % kRefBlocks;
  const int64_t row0 = (int64_t)((blk >> 1) / kRefBlocks) * kRefRows;
  const int H = a.H[head], nb = H / kBK;
  const int v = vb * 32 + (lane & 31);
  const uint4* ph = (const uint4*)(a.h[head] + (int64_t)rows[lane & 31] * H) + half * 4;
  const uint4* pw = (const uint4*)(a.W[head] + (int64_t)(v < a.V ? v : a.V - 1) * H) + half * 4;   // masked below
  f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int U = 2;                              // k-blocks loaded together
  for (int b = wave; b < nb; b += U * kPrepWaves) {
    uint4 x[U][4], w[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (b + u * kPrepWaves < nb ? b + u * kPrepWaves : b) * (kBK / 8);
#pragma unroll
      for (int c = 0; c < 4; ++c) { x[u][c] = ph[k + c]; w[u][c] = pw[k + c]; }
    }
    __builtin_amdgcn_sched_barrier(0);              // the loads stay together
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (b + u * kPrepWaves >= nb) break;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[u][c]), __builtin_bit_cast(bf16x8, x[u][c]),
                                                    z, 0, 0, 0);
    }
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) part[wave][e][lane] = z[e];
  __syncthreads();
  // wave w adds up elements 2 w and 2 w + 1 of every lane: entries 8 (e / 4) + 4 half + e % 4 of the block
  float m = kNegBig;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = 2 * wave + q;
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < kPrepWaves; ++k) s += part[k][e][lane];
    if (vb * 32 + 8 * (e >> 2) + 4 * half + (e & 3) < a.V) m = fmaxf(m, s);
  }
  top[wave][lane] = m;
  __syncthreads();
  if (threadIdx.x >= kRefRows) return;
#pragma unroll
  for (int k = 0; k < kPrepWaves; ++k) m = fmaxf(m, fmaxf(top[k][threadIdx.x], top[k][threadIdx.x + 32]));
  a.ref.max[head][(int64_t)vb * a.ref.n_pad + row0 + threadIdx.x] = m;
}

constexpr int kTokenBlockRows = kPrepWaves / 2 * kTokenRows;
__device__ __forceinline__ void token_block(const PrepareArgs& a, const int32_t* rows, int blk) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int head = wave & 1, first = (wave >> 1) * kTokenRows;
  const TokenRows four(a, rows + first, (int64_t)blk * kTokenBlockRows + first);
  const float z = token_logits(a, four, head, lane);
  if (lane < kTokenRows) a.ref.max[head][kRefBlocks * a.ref.n_pad + four.row0 + lane] = z;
}

// Without INLINE a.row_idx is there already; with it, `setup` is done by the last workgroups of this launch and the
// others take their rows from the plan in the arguments.
template <bool FINE, bool INLINE>
__device__ __forceinline__ void prepare_body(const PrepareArgs& a, const SetupArgs* setup, const SetupBlob* blob, char* lds) {
  __shared__ int32_t table[INLINE ? kTileTokens : 1];
  int b = (int)blockIdx.x, role = 0;
  const int blocks[4] = {a.ref_blocks, a.dot_blocks, a.img_blocks[0], a.img_blocks[1]};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (role == k && b >= blocks[k]) { b -= blocks[k]; ++role; }
  if (role == 4) {
    if constexpr (INLINE)
      setup_body(*setup, blob, (const unsigned char*)blob->data, b, a.setup_blocks, kPrepThreads);
    return;
  }
  const int n = role == 0 ? kRefRows : role == 1 ? kTokenBlockRows : kTileTokens;
  const int unit = role == 0 ? (FINE ? b / (2 * kRefBlocks) : b >> 1) : role == 1 ? b : b / a.img[role - 2].nk;
  const int64_t row0 = (int64_t)unit * n;
  const int32_t* rows;
  if constexpr (INLINE) {
    plan_rows(*setup, (const unsigned char*)blob->data, row0, n, table);
    rows = table;
  } else {
    rows = a.row_idx + row0;
  }
  if (role == 0) return FINE ? refs_fine_block(a, rows, b, lds) : refs_staged_block(a, rows, row0, b & 1, lds);
  if (role == 1) return token_block(a, rows, b);
  const RowImageArgs& im = a.img[role - 2];
  image_block<kPrepThreads, kTileTokens>(im, rows, unit, b % im.nk);
}
template <bool FINE>
__global__ __launch_bounds__(kPrepThreads) void prepare_kernel(PrepareArgs a) {
  extern __shared__ __align__(16) char lds[];
  prepare_body<FINE, false>(a, nullptr, nullptr, lds);
}
template <bool FINE>
__global__ __launch_bounds__(kPrepThreads) void prepare_inline_kernel(PrepareArgs a, const SetupArgs setup, const SetupBlob blob) {
  extern __shared__ __align__(16) char lds[];
  prepare_body<FINE, true>(a, &setup, &blob, lds);
}

// ROWS rows to a workgroup.  The strips of a row are added in the order of 64 lanes, whatever ROWS is: lane s takes
// the strips s, s + 64, ...; then the lanes 32 apart are added, 16 apart, and so on.  A thread holds kLanes of these
// lanes, kStep apart, its wave does the next halvings and the four waves leave the last two.
// Bound by round trips: 16 rows read 64 bytes of a plane together, where a wave to a row read 4 bytes of 64 lines, and the
// strips of a thread are loaded together, so that up to kMergeStrips take one trip.  3,139 rows of 38 strips 7.4 -> 5.6 us
// (the call, V = 11,912, 257.8 -> 255.9).  More strips belong to a call of one token tile, whose 256 rows are too few
// for that (238 strips: 16 rows 11.6 us, four rows 9).
constexpr int kMergeStrips = 64;
template <int ROWS>
__global__ __launch_bounds__(256) void merge_single_kernel(MergeSingleArgs b) {
  static_assert(ROWS == 4 || ROWS == 16, "a wave's part of 64 lanes");
  constexpr int kStep = 256 / ROWS, kLanes = 64 / kStep, kGroupBits = ROWS == 16 ? 2 : 4;     // kStep = 4 << kGroupBits
  constexpr int kTogether = ROWS == 16 ? 1 : 4;       // with kLanes: four strips
  const MergeArgs& a = b.m;
  __shared__ float sums[4][5][ROWS];
  const int row = threadIdx.x % ROWS, wave = threadIdx.x >> 6;
  const int64_t r = b.row0 + (int64_t)blockIdx.x * ROWS + row;
  const int64_t plane = (int64_t)a.strips * a.n_pad;
  const float ref_s2 = b.ref.of(0, r), ref_t2 = b.ref.of(1, r);
  const int planes = a.diag ? 5 : 3;
  // the thread's first lane: neighbouring groups of a wave hold those that are farthest apart (bits reversed)
  const int first = wave + 4 * (int)(__brev((threadIdx.x & 63u) / ROWS) >> (32 - kGroupBits));
  float x[kLanes][5], y[kLanes][5];           // Z_s, A, Z_t, B_t, count
#pragma unroll
  for (int j = 0; j < kLanes; ++j)
#pragma unroll
    for (int k = 0; k < 5; ++k) x[j][k] = 0.f;
#pragma unroll kTogether
  for (int s0 = first; s0 < a.strips; s0 += 64) {
#pragma unroll
    for (int j = 0; j < kLanes; ++j) {
      const int s = s0 + j * kStep;
#pragma unroll
      for (int k = 0; k < 5; ++k) y[j][k] = 0.f;
      if (s < a.strips) {
        const float* p = a.part + (int64_t)s * a.n_pad + r;
        y[j][0] = p[0]; y[j][1] = p[plane]; y[j][2] = p[2 * plane];
        if (a.diag) { y[j][3] = p[3 * plane]; y[j][4] = p[4 * plane]; }
      }
    }
#pragma unroll
    for (int j = 0; j < kLanes; ++j)          // behind all of the loads
#pragma unroll
      for (int k = 0; k < 5; ++k) x[j][k] += y[j][k];
  }
  float v[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    v[k] = x[0][k];
    if constexpr (kLanes == 4) v[k] = (x[0][k] + x[2][k]) + (x[1][k] + x[3][k]);
    if (k >= planes) break;
#pragma unroll
    for (int o = ROWS; o < 64; o <<= 1) v[k] += __shfl_xor(v[k], o, 64);
    if ((threadIdx.x & 63) < ROWS) sums[wave][k][row] = v[k];
  }
  __syncthreads();
  if (threadIdx.x >= ROWS) return;
#pragma unroll
  for (int k = 0; k < 5; ++k)
    v[k] = k < planes ? (sums[0][k][row] + sums[2][k][row]) + (sums[1][k][row] + sums[3][k][row]) : 0.f;
  const float Zs = v[0], A = v[1], Zt = v[2], Bt = v[3], cnt = v[4];
  const float lse_s = ref_s2 * kLn2 + logf(Zs), lse_t = ref_t2 * kLn2 + logf(Zt);
  const float mu = A / Zs;                  // E_{p_s}[z_s - z_t]
  float kl = kl_from_sums(mu, (ref_s2 - ref_t2) * kLn2, Zs, Zt);
  const float iz = 1.f / Zs;
  float ent = lse_t - Bt / Zt;              // H[p_t] = lse_t - E_{p_t}[z_t]; both sums share the reference
  // a row without a finite log-sum-exp, mean or KL (logits beyond the range the fixed
  // references cover, or non-finite inputs) is excluded: zeros in every output
  const bool bad = !(fabsf(lse_s) < 3.0e38f) || !(fabsf(lse_t) < 3.0e38f) || !(fabsf(kl) < 3.0e38f) ||
                    !(fabsf(A) < 3.0e38f) || !(fabsf(mu) < 3.0e38f) || !(iz > 0.f) || !(iz < 3.0e38f) ||
                    (a.diag && !(fabsf(ent) < 3.0e38f));
  // padding rows are excluded too: the sweep of a narrow tile leaves them out, and what their slab rows hold
  // must not reach the lists of heavy entries
  const bool dead = bad || r >= a.n_rows;
  if (dead) { kl = 0.f; ent = 0.f; }
  b.mu_out[r] = dead ? 0.f : mu;
  b.inv_z[r] = dead ? 0.f : iz;
  a.klr[r] = kl;
  a.lse_s[r] = dead ? 0.f : lse_s;
  if (r >= a.n_rows) return;
  const int64_t t = a.row_idx[r];
  float c = 0.f, logp_t = 0.f;
  bool have_y = false;
  uint32_t flag = dead ? ADWIN_DEV_NONFINITE : 0u;
  if (a.ids && (a.c || a.t_logp || a.t_rank || a.cr) && !dead) {
    if (b.ref.yid[r] >= 0) {
      const float zy_s = b.ref.zy[0][r], zy_t = b.ref.zy[1][r];     // taken with the references
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
  if (a.t_logp) a.t_logp[t] = logp_t;
  if (a.t_entropy) a.t_entropy[t] = ent;
  if (a.t_rank) a.t_rank[t] = have_y ? (int32_t)cnt + 1 : 0;
  if (a.cr) a.cr[r] = c;
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
hipError_t sweep_kernels_opt_in() {
  hipError_t e;
#define ADWIN_OPT_IN(KERNEL, BYTES)                                                              \
  e = hipFuncSetAttribute((const void*)KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize, BYTES); \
  if (e != hipSuccess) return e;
  ADWIN_OPT_IN(prepare_kernel<false>, kRefLds)
  ADWIN_OPT_IN(prepare_inline_kernel<false>, kRefLds)
  ADWIN_OPT_IN(logit_pass_kernel<false>, kLogitLds)
  ADWIN_OPT_IN(logit_pass_kernel<true>, kLogitLds)
#define ADWIN_OPT_IN_MODE(M)                                                  \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageImages>), DmaTile<2>::kRefLds) \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageRows>), DmaTile<2>::kRefLds)
  ADWIN_OPT_IN_MODE(kModeStats)
  ADWIN_OPT_IN_MODE(kModeDz)
#undef ADWIN_OPT_IN_MODE
#define ADWIN_OPT_IN_MODE(M)                                                  \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageImages>), DmaTile<2>::kRefLds) \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageRows>), DmaTile<2>::kRefLds)   \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageRowsOnce>), DmaTile<2>::kRefLds)    \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageRows, 1>), DmaTile<1>::kRefLds)     \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageRowsOnce, 1>), DmaTile<1>::kRefLds)
  ADWIN_OPT_IN_MODE(kModeSingle)
  ADWIN_OPT_IN_MODE(kModeSingleDiag)
  ADWIN_OPT_IN_MODE(kModeSingleE2)
  ADWIN_OPT_IN_MODE(kModeSingleE2Diag)
  ADWIN_OPT_IN_MODE(kModeSingleFwd)
  ADWIN_OPT_IN_MODE(kModeSingleFwdDiag)
#undef ADWIN_OPT_IN_MODE
#define ADWIN_OPT_IN_MODE(M)                                                          \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageImages, 2, true>), DmaTile<2>::kRefLds) \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageRows, 2, true>), DmaTile<2>::kRefLds)
  ADWIN_OPT_IN_MODE(kModeSingle)
  ADWIN_OPT_IN_MODE(kModeSingleE2)
  ADWIN_OPT_IN_MODE(kModeSingleE2Diag)
#undef ADWIN_OPT_IN_MODE
#define ADWIN_OPT_IN_MODE(M)                                                          \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageTeacherOnce>), DmaTile<2>::kRefLds)    \
  ADWIN_OPT_IN((logit_pass_dma_kernel<M, kStageTeacherOnce, 1>), DmaTile<1>::kRefLds)
  ADWIN_OPT_IN_MODE(kModeSingle)
  ADWIN_OPT_IN_MODE(kModeSingleDiag)
  ADWIN_OPT_IN_MODE(kModeSingleE2)
  ADWIN_OPT_IN_MODE(kModeSingleE2Diag)
#undef ADWIN_OPT_IN_MODE
#undef ADWIN_OPT_IN
  return hipSuccess;
}

hipError_t launch_row_image(const RowImageArgs& a, unsigned tiles, hipStream_t st) {
  row_image_kernel<<<dim3((unsigned)a.nk, tiles), 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_logit_pass(int mode, bool dma, const LogitPassArgs& p, hipStream_t st) {
  LogitPassArgs a = p;
  a.strip_tiles.split(a.vt_total, a.strips);
  const unsigned grid = (unsigned)a.n_tiles * (unsigned)a.strips;
  if (!dma) {
    if (mode == kModeStats) logit_pass_kernel<false><<<grid, 256, kLogitLds, st>>>(a);
    else if (mode == kModeDz) logit_pass_kernel<true><<<grid, 256, kLogitLds, st>>>(a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  if (a.narrow && (a.stage == kStageImages || a.n_tiles != 1)) return hipErrorInvalidValue;
  // a kernel for each mode and staging that fused_host.hip may ask for
#define ADWIN_LAUNCH(FN, ...) logit_pass_dma_kernel<__VA_ARGS__><<<grid, 256, DmaTile<FN>::kRefLds, st>>>(a)
#define ADWIN_ROWS(M, S)                                                       \
  if (a.stage == S) {                                                          \
    if (a.narrow) ADWIN_LAUNCH(1, M, S, 1);                                    \
    else ADWIN_LAUNCH(2, M, S);                                                \
    return hipGetLastError();                                                  \
  }
#define ADWIN_STAGES(M)                                                        \
  ADWIN_ROWS(M, kStageRows)                                                    \
  ADWIN_ROWS(M, kStageRowsOnce)                                                \
  if (a.stage != kStageImages) return hipErrorInvalidValue;                    \
  ADWIN_LAUNCH(2, M, kStageImages);                                            \
  return hipGetLastError();
#define ADWIN_STAGES_GRADIENT(M)                                               \
  ADWIN_ROWS(M, kStageTeacherOnce)                                             \
  ADWIN_STAGES(M)
#define ADWIN_STAGES_LINES(M)                                                  \
  if (a.lines && !a.narrow && a.stage <= kStageRows) {                         \
    if (a.stage == kStageImages) ADWIN_LAUNCH(2, M, kStageImages, 2, true);    \
    else ADWIN_LAUNCH(2, M, kStageRows, 2, true);                              \
    return hipGetLastError();                                                  \
  }                                                                            \
  ADWIN_STAGES_GRADIENT(M)
#define ADWIN_STAGES_TWO_SWEEP(M)                                              \
  if (a.narrow || a.stage > kStageRows) return hipErrorInvalidValue;           \
  if (a.stage == kStageImages) ADWIN_LAUNCH(2, M, kStageImages);               \
  else ADWIN_LAUNCH(2, M, kStageRows);                                         \
  return hipGetLastError();
  switch (mode) {
    case kModeStats: ADWIN_STAGES_TWO_SWEEP(kModeStats)
    case kModeDz: ADWIN_STAGES_TWO_SWEEP(kModeDz)
    case kModeSingle: ADWIN_STAGES_LINES(kModeSingle)
    case kModeSingleDiag: ADWIN_STAGES_GRADIENT(kModeSingleDiag)
    case kModeSingleE2: ADWIN_STAGES_LINES(kModeSingleE2)
    case kModeSingleE2Diag: ADWIN_STAGES_LINES(kModeSingleE2Diag)
    case kModeSingleFwd: ADWIN_STAGES(kModeSingleFwd)
    case kModeSingleFwdDiag: ADWIN_STAGES(kModeSingleFwdDiag)
    default: return hipErrorInvalidValue;
  }
#undef ADWIN_STAGES_TWO_SWEEP
#undef ADWIN_STAGES_LINES
#undef ADWIN_STAGES_GRADIENT
#undef ADWIN_STAGES
#undef ADWIN_ROWS
#undef ADWIN_LAUNCH
}

// The finely cut references serve calls of up to kFineRefTiles token tiles (References::parts is set by the
// same rule).  us per call, fine / staged: three tiles at H = 1024 + 2048 169.4 / 174.3, five 598.9 / 603.2
// (V = 50,000); five at H = 1024 + 1024 441.0 / 441.2, seven at H = 512 + 768 130.9 / 127.5.
// A plan that fits the arguments is expanded here too, in calls whose preparation is one launch.
hipError_t launch_prepare(const PrepareArgs& p, bool refs, int n_tiles, const SetupArgs& setup,
                          const std::vector<unsigned char>& plan, hipStream_t st) {
  static_assert(sizeof(PrepareArgs) + sizeof(SetupArgs) + sizeof(SetupBlob) < 4096, "kernel arguments");
  PrepareArgs a = p;
  const int rows = n_tiles * kTileTokens;
  const bool fine = a.ref.parts > 1;
  a.ref_blocks = !refs ? 0 : rows / kRefRows * 2 * (fine ? kRefBlocks : 1);
  a.dot_blocks = refs && fine ? rows / kTokenBlockRows : 0;
  for (int m = 0; m < 2; ++m) a.img_blocks[m] = n_tiles * a.img[m].nk;
  const int rest = a.dot_blocks + a.img_blocks[0] + a.img_blocks[1];
  const unsigned lds = fine ? kRefFineLds : a.ref_blocks ? kRefLds : 0;
  SetupBlob blob;
  hipError_t e;
  if (n_tiles <= kOneLaunchTiles && blob.take(plan)) {
    if (setup.n_zero > SetupArgs::kMaxZero) return hipErrorInvalidValue;
    a.setup_blocks = (int)setup_blocks(setup, kPrepThreads);
    const unsigned grid = (unsigned)(a.ref_blocks + rest + a.setup_blocks);
    if (fine) prepare_inline_kernel<true><<<grid, kPrepThreads, lds, st>>>(a, setup, blob);
    else prepare_inline_kernel<false><<<grid, kPrepThreads, lds, st>>>(a, setup, blob);
    return hipGetLastError();
  }
  if ((e = launch_setup(setup, plan, st)) != hipSuccess) return e;
  if (fine) {
    prepare_kernel<true><<<(unsigned)(a.ref_blocks + rest), kPrepThreads, lds, st>>>(a);
    return hipGetLastError();
  }
  // a workgroup of a launch with staged references holds their LDS as well, two workgroups per compute
  // unit, so that the others of a large call, 155 us of copying for 34,000 rows, go by themselves
  if (a.ref_blocks && n_tiles > kOneLaunchTiles) {
    prepare_kernel<false><<<(unsigned)a.ref_blocks, kPrepThreads, lds, st>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    a.ref_blocks = 0;
  }
  prepare_kernel<false><<<(unsigned)(a.ref_blocks + rest), kPrepThreads, a.ref_blocks ? lds : 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_merge_stats(const MergeArgs& a, hipStream_t st) {
  merge_stats_kernel<<<(unsigned)((a.n_pad + 3) / 4), 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_merge_single(const MergeSingleArgs& a, hipStream_t st) {
  // slabs are whole token tiles
  if (a.m.strips <= kMergeStrips) merge_single_kernel<16><<<(unsigned)(a.rows / 16), 256, 0, st>>>(a);
  else merge_single_kernel<4><<<(unsigned)(a.rows / 4), 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace adwin
