// Fused path, host side: argument checks, workspace layout and the sequence of launches
// that makes one call (Sec. 4.1: supervision on the admitted prefix; Sec. 4.2: the probe
// audit against the full-rollout gradient).  The kernels are in sweep_kernels.hip,
// grad_kernels.hip and reduce_kernels.hip; nothing here touches device memory itself.
#include <cmath>
#include <optional>
#include <utility>
#include <vector>

#include "fused_shared.h"

namespace adwin {

// ---------------------------------------------------------------------------------------
// Workspace layout and the entry point
// ---------------------------------------------------------------------------------------
struct FusedLayout {
  bool use_dma;      // logit passes staged by direct global->LDS loads
  bool single;       // single-sweep scheme (needs use_dma)
  bool direct_w;     // ... whose W tiles come from the row-major weights, not from images
  size_t o_wt_img, o_ws_img, o_ht_img, o_hs_img;   // tile images of the logit operands (use_dma)
  size_t o_ref, o_delta, o_invz, o_mu0t;
  int strips, ksplit;
  int64_t slab_rows, Vp;
  size_t o_plan, o_row_idx, o_row_seq, o_part, o_lse2, o_mu, o_klr, o_rownorm, o_slab, o_g,
      o_pp, o_pf, o_up, o_uf, o_seg, o_racc, o_uc, o_cacc, o_cS, o_cr, o_zy_s, o_zy_t, o_yid, o_dzT_p, o_dzT_f, o_hsg, o_summ, o_cosp,
      o_lse_s, o_heavy_cnt, o_heavy_v, total;
};

// Which kernels a scheme selects for this shape: the direct-to-LDS logit kernel pipelines at
// least two k-steps per head, so it needs both hidden sizes >= 128.  False: the scheme is not
// available for the shape.
static bool resolve_scheme(const adwin_opd_problem* p, bool* use_dma, bool* single) {
  const bool dma_ok = p->H_s >= 2 * kBK && p->H_t >= 2 * kBK;
  switch (p->scheme) {
    case ADWIN_SCHEME_AUTO: *use_dma = dma_ok; *single = dma_ok; return true;
    case ADWIN_SCHEME_SINGLE: *use_dma = true; *single = true; return dma_ok;
    case ADWIN_SCHEME_TWO_SWEEP: *use_dma = dma_ok; *single = false; return true;
    case ADWIN_SCHEME_TWO_SWEEP_REG: *use_dma = false; *single = false; return true;
    default: *use_dma = false; *single = false; return false;
  }
}

static int env_int(const char* name, int dflt) {
  const char* s = getenv(name);
  if (!s || !*s) return dflt;
  const int v = atoi(s);
  return v > 0 ? v : dflt;
}

// Whether any requested output depends on the per-row gradients.  Without one the single
// sweep runs in its statistics-only mode (KL, c, losses, the diagnostics and their summaries):
// no gradient factors are stored, combined or contracted.
static bool needs_gradient(const adwin_opd_problem* p) {
  const bool probe = p->mode == ADWIN_PREFIX_AND_FULL;
  return p->dh_prefix || p->dh_full || p->rho_pooled || p->rho_field || p->dW_prefix || p->dW_full ||
         (probe && (p->batch || (p->candidates && p->n_candidates > 0 &&
                                 (p->cand_rho_pooled || p->cand_rho_field || p->cand_batch))));
}

// Vocabulary strips of a sweep over `n_tiles` token tiles: the grid is n_tiles x strips
// workgroups, one per compute unit at a time, dealt in equal shares to the 8 XCDs of 32, so a
// sweep costs rounds x (vocabulary tiles of the longest strip + a start, taken as a quarter of a
// tile).  32 strips is what the large slabs were tuned with (64 token tiles: 16 and 64 strips
// are 1 to 4 % slower although 16 has the better-filled rounds) and stays wherever it is within
// 5 % of the cheapest count; a call of few token tiles, which left most of the chip without
// work, takes more strips, and so does one whose rounds more strips fill better.  256 rows,
// V = 151,936, H = 2048 + 4096: 2612 us with 32 strips, 420 with 238.
// Never fewer: a strip's sums are fp32 chains of its length.  28 token tiles of V = 50,000 in the
// 18 strips that fill the chip: error of KL_t 2.9 times that of 32 strips (2-norm, against 64 bits),
// of c_t 1.2, of the gradient 1.03.  More cost none: 256 rows of V = 151,936 in 238 strips, the error of
// the gradient is 0.97 of that with 32 (three inputs), within 3 % either way at V = 32,776 and 50,000.
// Strips of two lengths fill the rounds better when the longer ones of all token tiles come first and a
// compute unit that ends one takes a shorter one next (long_first): a die's 32 units then need what the lengths
// add up to instead of rounds of the longer one.  13 token tiles of 94 vocabulary tiles: 18 strips of 3 and 20 of
// 2 end after 5, 32 strips of 3 and 2 after 6.  It is taken where it saves 3 % (at 0.5 % the gain is in the noise, and 16 token
// tiles of 1187 lost 1.5 %).  us per call, without / with: 3,300 rows, V = 12,000, H = 512 + 640 271 / 263 (probe),
// 143.5 / 135.0 (statistics); 5,100 rows, V = 16,600, H = 1024 + 1024 statistics 380 / 362; V = 50,000,
// H = 512 + 512 1250 / 1226; 7,600 rows, H = 512 + 1024 2137 / 2124.
int sweep_strips(int n_tiles, int vt_total, int* long_first) {
  const int most = vt_total < kMaxSweepStrips ? vt_total : kMaxSweepStrips;
  auto cost = [&](int s) {
    const int per_xcd = (n_tiles * s + 7) / 8, rounds = (per_xcd + 31) / 32;
    return rounds * ((vt_total + s - 1) / s + 0.25);
  };
  // where the last workgroup of a die that takes the longer ones first ends, in the same unit, or `least`
  auto cost_long_first = [&](int s, double least) {
    const int each = vt_total / s, longer = vt_total % s;
    const int n_long = (longer * n_tiles + 7) / 8, n_short = ((s - longer) * n_tiles + 7) / 8;
    const double b = each + 0.25, a = b + 1.0;
    if ((n_long * a + n_short * b) / 32 >= least) return least;
    const int q = n_long / 32, r = n_long % 32;              // r units begin with q + 1 of them, the others with q
    double best = least;
    for (int begin = 0; begin < 2; ++begin) {                // a unit of either kind ends last, after k shorter ones
      if (begin && !r) continue;
      for (int k = 0; (q + begin) * a + k * b < best; ++k) {
        const double end = (q + begin) * a + k * b + 1e-6;
        if (r && end < (q + 1) * a) continue;
        const int fits = r * (int)((end - (q + 1) * a) / b) + (32 - r) * (int)((end - q * a) / b);
        if (fits >= n_short) { best = end; break; }
      }
    }
    return best;
  };
  *long_first = 0;
  int tuned = env_int("ADWIN_STRIPS2", 32);
  if (tuned > most) tuned = most;
  if (getenv("ADWIN_STRIPS2")) return tuned;
  int best = tuned;
  double least = 0.95 * cost(tuned);
  for (int s = tuned + 1; s <= most; ++s)
    if (cost(s) < least) { best = s; least = cost(s); }
  if (n_tiles == 1) return best;           // one round
  least = 0.97 * cost(best);
  for (int s = tuned; s <= most; ++s) {
    const double c = cost_long_first(s, least);
    if (c < least) { best = s; least = c; *long_first = 1; }
  }
  return best;
}

// Rows per slab and k-splits of the gradient GEMM.  Its 256 x 256 output tiles run in rounds of
// 256 compute units; with ksplit > 1 the contraction over the vocabulary is cut into ksplit
// pieces, one workgroup each, whose partial planes of g finalize_kernel adds in index order.
// Cost in k-steps (1.6 us): rounds x (k-steps of a piece + 20 for the start and the epilogue of a
// tile, from 256-step and 2374-step launches), and per piece the partial plane written and read
// once at 4 TB/s plus 0.2 for the load of one more plane in finalize_kernel.  Slabs are
// multiples of 8 token tiles between 4,096 and 16,384 rows; ties go to the larger slab (fewer
// launches, each of which ends in a partly idle round) and to fewer pieces.  Up to 128 pieces: one
// output tile of 2374 k-steps (256 rows, H_s = 256) takes 95, call 250 -> 214 us against
// 32; two tiles 489 -> 458 us; 3,100 rows of 188 k-steps and H_s = 512 take 9, 302 -> 290 us.
constexpr int kMaxSplit = 128;
constexpr int64_t kMaxSlab = 16384;

// What bounds the pieces and sizes the workspace for them: pieces times token tiles, for a call of up
// to `n_tiles` tiles.  It grows with n_tiles, which the number of pieces that suits a call does not (64
// tiles of H_s = 2048 take 2, 36 tiles 8), so that a workspace for the largest call of a program holds
// every smaller one.  The optimum lies below 1.9 sqrt(nk) pieces (the cost of a piece is at least 0.28
// k-steps), below one round of output tiles, or, where a few rounds are filled, below 12 pieces;
// calls of several slabs take what fills a round.
static int64_t most_split_tiles(int64_t n_tiles, int h_tiles, int nk) {
  const int root = 2 + (int)(2.0 * sqrt((double)nk));
  int64_t pieces = root < kMaxSplit ? root : kMaxSplit;
  if (pieces > nk) pieces = nk;
  const int64_t slab_tiles = n_tiles < kMaxSlab / kTileTokens ? n_tiles : kMaxSlab / kTileTokens;
  int64_t most = 256 / h_tiles > 12 * slab_tiles ? 256 / h_tiles : 12 * slab_tiles;
  if (most > pieces * slab_tiles) most = pieces * slab_tiles;
  int64_t fill = 16 / h_tiles < 12 ? 16 / h_tiles : 12;          // slabs of 4,096 rows: 16 tiles
  if (fill > pieces) fill = pieces;
  const int64_t several = n_tiles * (fill > 1 ? fill : 1);
  return several > most ? several : most;
}

struct GradGeometry { int64_t slab_rows; int ksplit; };
static GradGeometry grad_geometry(int64_t n_pad, int h_tiles, int nk, double head_steps) {
  GradGeometry best{0, 1};
  double least = -1.0;
  const bool forced = getenv("ADWIN_SLAB_ROWS") != nullptr;
  const int64_t room = most_split_tiles(n_pad / kTileTokens, h_tiles, nk) / (n_pad / kTileTokens);
  int64_t first = forced ? (int64_t)align_up((size_t)env_int("ADWIN_SLAB_ROWS", 8192), kTileTokens) : kMaxSlab;
  // one size that holds every row is enough: the larger ones are the same slab (seven searches of up
  // to 128 pieces each made a layout of 256 rows 4.7 us of host time, of which one leaves 1.9)
  while (!forced && first > 4096 && first - 2048 >= n_pad) first -= 2048;
  for (int64_t r = first; r >= (forced ? first : 4096); r -= 2048) {
    const int64_t slab = r < n_pad ? r : n_pad;
    // the partial planes hold all rows of the call, so a call of several slabs takes no more pieces than
    // fill one round.  us per call, whole tiles / pieces: 18,000 rows, H_s = 128, V = 50,000 4585 / 3376;
    // 20,000 rows, H_s = 256, V = 151,936 18582 / 14667; H_s = 512, V = 11,912 1553 / 1259
    const int64_t fill = 256 / ((slab / kGradTile) * h_tiles);
    int64_t limit = slab == n_pad ? kMaxSplit : forced ? 1 : fill;
    if (limit > room) limit = room;
    const int most = (int)(limit > nk ? nk : limit > 1 ? limit : 1);
    // with the head gradient each slab beyond those that whole tiles need is one more pass over it.  V = 32,776,
    // H = 1024 + 1024, us without / with this term: 16,640 rows 6012 / 5887, 51,200 rows 16745 / 16605
    const double more_slabs = (double)((n_pad + slab - 1) / slab - (n_pad + kMaxSlab - 1) / kMaxSlab);
    for (int ks = 1; ks <= most; ++ks) {
      double cost = ks > 1 ? (double)ks * ((double)n_pad * h_tiles * kGradTile * 8.0 / 6.4e6 + 0.2) +
                                 more_slabs * head_steps : 0.0;
      for (int64_t r0 = 0; r0 < n_pad; r0 += slab) {
        const int64_t rows = n_pad - r0 < slab ? n_pad - r0 : slab;
        const int64_t rounds = ((rows / kGradTile) * h_tiles * ks + 255) / 256;
        cost += (double)rounds * ((nk + ks - 1) / ks + 20);
      }
      if (least < 0.0 || cost < least) { least = cost; best = GradGeometry{slab, ks}; }
    }
  }
  return best;
}

// Whether the logit passes stage their W tiles from the row-major weights rather than from tile
// images.  The images cost a pass over both weights (0.75 ms at V = 151,936, H = 2048 + 4096); a
// tile pair staged from them is faster by about the same amount at every hidden size (eight
// 128-byte pieces per wave-load against 1 KiB in one piece: 0.4 to 2 % of a sweep).  The line
// lies where the two meet.  us per call, direct against images: H = 2048 + 4096, 64 token tiles
// 35620 / 35884, 128 tiles 70313 / 70595, 256 tiles 140609 / 140325; H = 256 + 384, 16 tiles
// 2359 / 2387, 64 tiles 9396 / 9357; H = 1024 + 1024 (V = 32,776), 16 tiles 1062 / 1112, 64 tiles
// 3800 / 3781.
// The two-sweep scheme walks W twice and stages the same tiles: 54628 / 54634 at 64 tiles, 109372 /
// 110366 at 128 and 136430 / 138157 at 160 of H = 2048 + 4096; 3376 / 3358 at 16 and 4119 / 4130 at 24 of
// H = 256 + 384: within 1 % of each other on both sides of the line.
// The statistics-only sweep writes no factors, so its loads are a larger share of its time and the
// images are worth 2.4 % of it (64 tiles, H = 2048 + 4096: 23.3 against 23.9 ms): `loads_bound`
// moves the line to where that meets the 0.75 ms.  134 tiles, statistics: 50.9 -> 50.4 ms.  The
// diagnostics sweep that writes both factors shares it, direct against images, ms: H = 2048 + 4096, 64
// tiles 36.44 / 36.53, 85 tiles 49.31 / 49.15, 128 tiles 73.03 / 72.58; H = 1024 + 1024 (V = 32,776), 28
// tiles 1.785 / 1.826; H = 256 + 384, 9 tiles 1.508 / 1.559, 32 tiles 5.140 / 5.134.
static bool stage_w_directly(int64_t n_tiles, int H_s, int H_t, bool loads_bound) {
  return n_tiles * (loads_bound ? 72 : 40) <= H_s + H_t;
}

// Whether the strips of a sweep begin the contraction at different k-steps.  With one token tile every
// strip streams its own rows of W from memory, 128 bytes of each row per k-step, and rows of 4 KiB and more put
// the same 128 bytes of all rows into a few of the memory channels: a read-only copy of this pattern
// reaches 4.05 TB/s in step and 4.75 with the strips spread over the rows (V = 151,936, H = 4096).  256 rows,
// H = 2048 + 4096: 774 -> 747 us per call; 16 rows, H = 3584 + 4608: 995 -> 978; H = 1024 + 1024: the same, 355.
// With several token tiles the strips share their blocks of h in the L2 because they run in step:
// 512 rows 1243 -> 1289, 2,000 rows 4498 -> 4780 (spread by 5 k-steps a strip).
static bool rotate_k(int64_t n_tiles, int H_s, int H_t) {
  return n_tiles == 1 && (H_s > H_t ? H_s : H_t) >= 2048;
}

// Where the sweep of `n_tiles` token tiles gets W from.  With one token tile no other workgroup asks for its lines of W, and
// they displace the hidden states (3 MB at H = 2048 + 4096) that every workgroup of a die reads again for every tile: 20 %
// of those reads missed the L2.  Lines of W past the caches: us per sweep, kept / past, V = 151,936: 256 rows, H = 2048 + 4096
// 525 / 496; 100 rows 423 / 406; 230 rows, 1024 + 1024 208 / 190; statistics of 60 rows, 2048 + 2048 256 / 245.
// Not where both weights fit the last-level cache, which may hold them from the call before (100 rows of V = 100,000,
// 512 + 512 134 / 138 per call, statistics with 512 + 768 71 / 87); and W_s, which the gradient GEMM reads again, only
// if that exceeds the cache (per call, W_t past / both: 16,000 entries of 3584 + 4608 152 / 158, 60 rows of V = 151,936,
// 512 + 768 182 / 182; 230 rows of 1024 + 1024, 297 MiB of W_s, 363 / 353).  With two token tiles and more, whose workgroups
// share the lines, nothing or up to 10 % worse (4,096 rows).  A row of W is whole lines (H is a multiple of 64) if
// the first one begins a line; else neighbouring pieces of a row share lines, which would be fetched twice.
static int sweep_stage(const adwin_opd_problem* p, bool direct_w, int n_tiles, bool need_g) {
  if (!direct_w) return kStageImages;
  const int64_t student = 2 * (int64_t)p->V * p->H_s, teacher = 2 * (int64_t)p->V * p->H_t;
  if (n_tiles > 1 || student + teacher <= kPastCacheBytes || (((uintptr_t)p->W_s | (uintptr_t)p->W_t) & 127)) return kStageRows;
  return !need_g || student > ((int64_t)256 << 20) ? kStageRowsOnce : kStageTeacherOnce;
}

// Whether a sweep whose slab exceeds the caches stores the factors as whole lines past them (single_epilogue).  The shorter
// the contraction, the more of a sweep are its stores.  us per sweep, plain pieces / lines, V = 151,936: H = 640 + 256,
// 24,000 rows 8710 / 7790; 1536 + 1536, 16,384 rows 13830 / 13320; 8,192 rows of 1152 + 1792 (V = 124,200) 5515 / 5215, of
// 1536 + 2048 7940 / 7640, of 2048 + 2048 8730 / 8430.  The gain shrinks with the length, 2.2 % of 2560 + 2560 (10880 / 10640), and
// with 2048 + 4096 it depends on the GPU, 24.8 / 24.6 ms to 24.6 / 25.6 for 16,384 rows: the line lies below both.  The sweep
// with both factors and diagnostics has no registers for the group on its way and loses (2800 / 3070).
static bool sweep_whole_lines(int H) { return H <= 4096; }

// Whether the gradient GEMM takes the two factors themselves and collapses them on their way into the LDS, instead of dz from
// a combine pass.  That spares a pass of 6 bytes per entry, and costs every column tile the conversion: a k-step
// takes 2.3 us for 1.4 (grad_kstep_factors).  us per call, combine pass / none, H_t = 256, rows x V:
//   H_s = 256:  700 x 50,000 152 / 140; 3,000 x 50,000 514 / 397; 1,500 x 151,936 783 / 583; 16,000 x 11,912 680 / 560;
//               16,000 x 4,096 326 / 315; 8,000 x 4,096 168 / 171; 1,500 x 11,912 97 / 101
//   H_s = 512:  3,000 x 151,936 1782 / 1555; 700 x 50,000 194 / 185; 16,000 x 11,912 822 / 767; 8,000 x 8,192 330 / 326;
//               16,000 x 4,096 378 / 396; 1,500 x 11,912 115 / 126
//   H_s = 768:  3,000 x 151,936 2186 / 2009; 1,500 x 32,776 295 / 278; 8,000 x 20,000 849 / 873; 16,000 x 11,912 999 / 1072
//   H_s = 1024: 3,000 x 151,936 2498 / 2454; 8,000 x 32,776 1464 / 1470.  H_s = 1280: 3,000 x 151,936 2876 / 2920
// So for up to three column tiles, each number from a length of the contraction on (k-steps of the whole vocabulary, of which a
// piece takes its share: below it the longer prologue of the pieces weighs too much), and from 32 Mi entries on.
// (The descriptors of the kernel address a row tile of up to 1 GiB.)
static bool collapse_in_gemm(int64_t rows, int V, int h_tiles, int nk) {
  const int least = h_tiles == 1 ? 64 : h_tiles == 2 ? 128 : 512;
  return h_tiles <= 3 && nk >= least && nk <= 32768 && rows * V >= (int64_t)32 << 20;
}

static FusedLayout fused_layout(const adwin_opd_problem* p, const HostPlan& hp) {
  FusedLayout L;
  const int64_t n_pad = hp.n_pad > 0 ? hp.n_pad : kTileTokens;
  const int vt_total = (p->V + kTileVocab - 1) / kTileVocab;
  L.Vp = (int64_t)vt_total * kTileVocab;
  int strips = env_int("ADWIN_STRIPS", 8);
  if (strips > vt_total) strips = vt_total;
  if (strips > kMaxStrips) strips = kMaxStrips;
  L.strips = strips;
  (void)resolve_scheme(p, &L.use_dma, &L.single);     // validity was checked with the problem
  const int halves = L.single ? 2 : 1;     // the single sweep stores two factors per logit
  const int h_tiles = (p->H_s + kGradTile - 1) / kGradTile;
  // the head gradients of a slab after the first are read and written once more; k-steps of 1.6 us at 4 TB/s
  const double head_steps = ((p->dW_prefix ? 1 : 0) + (p->dW_full ? 1 : 0)) * (double)p->V * p->H_s * 8.0 / 6.4e6;
  const GradGeometry gg = grad_geometry(n_pad, h_tiles, (int)(L.Vp / kBK), head_steps);
  const int64_t slab = gg.slab_rows;
  const int ks = gg.ksplit;
  L.slab_rows = slab;
  L.ksplit = ks;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
  L.o_plan = take(PlanBlobLayout(p->B).bytes);
  L.o_row_idx = take(sizeof(int32_t) * (size_t)n_pad);
  L.o_row_seq = take(sizeof(int32_t) * (size_t)n_pad);
  // A program that sizes its workspace for its largest call, or with other outputs than the diagnostics,
  // uses it for the others: no part may be larger in a smaller call.  The slab, the strips and the
  // pieces that suit a call are not monotone in its rows, so their arrays are sized by bounds that are.
  const int64_t bound_slab = n_pad < kMaxSlab ? n_pad : slab > kMaxSlab ? slab : kMaxSlab;
  // strip partials: of one slab after the other (single sweep), or of all rows (two sweeps)
  const int most_strips = vt_total < kMaxSweepStrips ? vt_total : kMaxSweepStrips;
  L.o_part = take(sizeof(float) * 5 * (L.single ? (size_t)most_strips * (size_t)bound_slab
                                                : (size_t)strips * (size_t)n_pad));
  L.o_ref = take(L.single ? sizeof(float) * 2 * kMaxRefParts * (size_t)n_pad : 0);
  L.o_delta = take(sizeof(float) * (size_t)n_pad);
  L.o_mu0t = take((L.single && p->estimator != ADWIN_EST_SAMPLED)
                      ? sizeof(float) * (size_t)vt_total * (size_t)bound_slab : 0);
  L.o_invz = take(sizeof(float) * (size_t)n_pad);
  L.o_lse2 = take(L.single ? 0 : sizeof(float) * (size_t)n_pad);
  L.o_mu = take(L.single ? 0 : sizeof(float) * (size_t)n_pad);
  L.o_klr = take(sizeof(float) * (size_t)n_pad);
  L.o_rownorm = take(sizeof(float) * (size_t)n_pad);
  const bool both_factors_diag = (p->t_entropy || p->t_rank) && p->estimator != ADWIN_EST_SAMPLED;
  L.direct_w = stage_w_directly(n_pad / kTileTokens, p->H_s, p->H_t,
                                (L.single && !needs_gradient(p)) || both_factors_diag);
  // room for the images from the lower of the two lines on, whichever this call goes by
  const bool w_images = L.use_dma && !stage_w_directly(n_pad / kTileTokens, p->H_s, p->H_t, true);
  L.o_wt_img = take(w_images ? 2 * (size_t)L.Vp * (size_t)p->H_t : 0);
  L.o_ws_img = take(w_images ? 2 * (size_t)L.Vp * (size_t)p->H_s : 0);
  L.o_ht_img = take(L.use_dma ? 2 * (size_t)n_pad * (size_t)p->H_t : 0);
  L.o_hs_img = take(L.use_dma ? 2 * (size_t)n_pad * (size_t)p->H_s : 0);
  // statistics-only calls (no output depends on the gradients) need neither the slab nor g
  const bool need_g = needs_gradient(p) || !L.single;
  L.o_slab = take(need_g ? 2 * (size_t)halves * (size_t)bound_slab * (size_t)L.Vp : 0);
  // the planes of the pieces; with the sampled estimator behind n_pad rows for g itself, which
  // finalize_kernel forms from the contracted E2
  const bool sampled = L.single && p->estimator == ADWIN_EST_SAMPLED;
  int64_t g_tiles = most_split_tiles(n_pad / kTileTokens, h_tiles, (int)(L.Vp / kBK));
  if (g_tiles < ks * (n_pad / kTileTokens)) g_tiles = ks * (n_pad / kTileTokens);
  L.o_g = take(need_g ? sizeof(float) * ((size_t)g_tiles * kTileTokens + (sampled ? (size_t)n_pad : 0)) * (size_t)p->H_s : 0);
  const size_t nch = (size_t)(hp.n_chunks > 0 ? hp.n_chunks : 1);
  L.o_pp = take(sizeof(float) * nch * (size_t)p->H_s);
  L.o_pf = take(sizeof(float) * nch * (size_t)p->H_s);
  L.o_up = take(sizeof(float) * (size_t)p->B * (size_t)p->H_s);
  L.o_uf = take(sizeof(float) * (size_t)p->B * (size_t)p->H_s);
  L.o_seg = take(sizeof(double) * 4 * (size_t)p->B);
  L.o_racc = take(sizeof(double) * 4 * (size_t)p->B);
  const size_t kc = (p->candidates && p->n_candidates > 0) ? (size_t)p->n_candidates : 0;
  L.o_uc = take(sizeof(float) * kc * (size_t)p->B * (size_t)p->H_s);
  L.o_cacc = take(sizeof(double) * 4 * kc * (size_t)p->B);
  L.o_cS = take(sizeof(double) * kc * (size_t)p->B);
  L.o_cr = take(sizeof(float) * (size_t)n_pad);
  L.o_zy_s = take(sizeof(float) * (size_t)n_pad);
  L.o_zy_t = take(sizeof(float) * (size_t)n_pad);
  L.o_yid = take(sizeof(int32_t) * (size_t)n_pad);
  const bool head = p->dW_prefix || p->dW_full;       // transposed slab + gathered h_s rows
  // vocabulary tiles of 256 image rows: the last one may be half used (its upper rows are
  // never written, and their output rows do not exist)
  const size_t v_img = align_up((size_t)L.Vp, (size_t)kGradTile);
  L.o_dzT_p = take(p->dW_prefix ? 2 * (size_t)bound_slab * v_img : 0);
  L.o_dzT_f = take(p->dW_full ? 2 * (size_t)bound_slab * v_img : 0);
  L.o_hsg = take(head ? 2 * (size_t)bound_slab * (size_t)p->H_s : 0);
  L.o_cosp = take((p->dW_prefix && p->dW_full) ? sizeof(double) * 3 * kCosineBlocks : 0);
  L.o_summ = take((p->t_first_reject || p->t_logp_mean || p->cand_loss_share)
                      ? sizeof(double) * (size_t)p->B * kSummarySlots : 0);
  L.o_lse_s = take(sizeof(float) * (size_t)n_pad);
  L.o_heavy_cnt = take(sizeof(int32_t) * (size_t)n_pad);
  L.o_heavy_v = take(need_g ? sizeof(int32_t) * (size_t)kHeavySlots * (size_t)n_pad : 0);
  L.total = o;
  return L;
}

static int check_problem(const adwin_opd_problem* p) {
  if (!p) return ADWIN_E_NULL;
  if (p->struct_bytes != sizeof(adwin_opd_problem)) return ADWIN_E_MODE;
  int st = validate_ragged(p->T, p->B, p->offsets, p->window);
  if (st != ADWIN_OK) return st;
  if (p->V <= 0 || (p->V & 7) || p->H_s <= 0 || (p->H_s % kBK) || p->H_t <= 0 || (p->H_t % kBK))
    return ADWIN_E_SHAPE;
  if (p->mode != ADWIN_PREFIX_ONLY && p->mode != ADWIN_PREFIX_AND_FULL) return ADWIN_E_MODE;
  if (p->reduction < ADWIN_RED_SEQ_MEAN || p->reduction > ADWIN_RED_TOKEN_MEAN) return ADWIN_E_MODE;
  if (p->dh_dtype != ADWIN_DT_BF16 && p->dh_dtype != ADWIN_DT_F32) return ADWIN_E_MODE;
  if (p->estimator != ADWIN_EST_EXPECTED && p->estimator != ADWIN_EST_SAMPLED) return ADWIN_E_MODE;
  {
    bool use_dma, single;
    if (!resolve_scheme(p, &use_dma, &single)) return ADWIN_E_MODE;
  }
  if (p->n_candidates < 0 || p->n_candidates > ADWIN_MAX_CANDIDATES) return ADWIN_E_SHAPE;
  if (p->candidates && p->n_candidates > 0) {
    if (p->mode != ADWIN_PREFIX_AND_FULL) return ADWIN_E_MODE;
    for (int k = 0; k < p->n_candidates; ++k)
      if (p->candidates[k] <= 0) return ADWIN_E_WINDOW;
  }
  if (p->t_first_reject && !p->t_rank) return ADWIN_E_NULL;
  if (p->t_first_reject && p->topk <= 0) return ADWIN_E_SHAPE;
  if (p->t_logp_mean && !p->t_logp) return ADWIN_E_NULL;
  if (p->cand_loss_share && !(p->candidates && p->n_candidates > 0)) return ADWIN_E_NULL;
  return ADWIN_OK;
}

static hipError_t ensure_lds_opt_in() {
  if (!first_use_on_device(0)) return hipSuccess;
  hipError_t e = sweep_kernels_opt_in();
  if (e != hipSuccess) return e;
  return grad_kernels_opt_in();
}

}  // namespace adwin

using namespace adwin;

extern "C" int adwin_opd_init(void) {
  ADWIN_HIP_TRY(sweep_kernels_opt_in());
  ADWIN_HIP_TRY(grad_kernels_opt_in());
  ADWIN_HIP_TRY(logits_kernels_opt_in());
  ADWIN_HIP_TRY(logits_static_setup());
  (void)first_use_on_device(0);      // the calls need not repeat it on this device
  (void)first_use_on_device(1);
  return ADWIN_OK;
}

extern "C" int adwin_opd_workspace_bytes(const adwin_opd_problem* p, size_t* bytes) {
  if (!bytes) return ADWIN_E_NULL;
  int st = check_problem(p);
  if (st != ADWIN_OK) return st;
  HostPlan hp = make_host_plan(p->T, p->B, p->offsets, p->window,
                               p->mode == ADWIN_PREFIX_AND_FULL, p->reduction, nullptr);
  *bytes = fused_layout(p, hp).total;
  return ADWIN_OK;
}

extern "C" int adwin_opd_fused_launch_info(const adwin_opd_problem* p, int64_t info[4]) {
  if (!info) return ADWIN_E_NULL;
  int st = check_problem(p);
  if (st != ADWIN_OK) return st;
  HostPlan hp = make_host_plan(p->T, p->B, p->offsets, p->window,
                               p->mode == ADWIN_PREFIX_AND_FULL, p->reduction, nullptr);
  FusedLayout L = fused_layout(p, hp);
  info[0] = hp.n_rows;
  info[1] = hp.n_pad;
  info[2] = L.slab_rows;
  info[3] = hp.n_pad > 0 ? (hp.n_pad + L.slab_rows - 1) / L.slab_rows : 0;
  return ADWIN_OK;
}

static int fused_impl(const adwin_opd_problem* p, void* workspace, size_t workspace_bytes,
                      void* hip_stream, PhaseTimer* timer) {
  int st = check_problem(p);
  if (st != ADWIN_OK) return st;
  if (!p->W_s || !p->W_t) return ADWIN_E_NULL;
  if (p->T > 0 && (!p->h_s || !p->h_t)) return ADWIN_E_NULL;
  const uintptr_t al = (uintptr_t)p->h_s | (uintptr_t)p->h_t | (uintptr_t)p->W_s |
                       (uintptr_t)p->W_t | (uintptr_t)p->dh_prefix | (uintptr_t)p->dh_full;
  if (al & 15) return ADWIN_E_ALIGN;
  const int probe = p->mode == ADWIN_PREFIX_AND_FULL;
  std::vector<unsigned char> blob;
  HostPlan hp = make_host_plan(p->T, p->B, p->offsets, p->window, probe, p->reduction, &blob);
  FusedLayout L = fused_layout(p, hp);
  if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < L.total)
    return ADWIN_E_WORKSPACE;
  const bool diag = p->t_entropy || p->t_rank;          // need the diagnostics sweep
  const bool sampled = p->estimator == ADWIN_EST_SAMPLED;
  // the diagnostics and the sampled estimator ride on the single-sweep kernels
  const bool head = p->dW_prefix || p->dW_full;
  const bool need_g = needs_gradient(p) || !L.single;   // the statistics-only mode is a single-sweep mode
  if ((diag || p->t_logp || sampled || head) && !L.single) return ADWIN_E_MODE;
  if (sampled && !p->ids) return ADWIN_E_NULL;
  if (p->dW_full && p->mode != ADWIN_PREFIX_AND_FULL) return ADWIN_E_MODE;
  if (((uintptr_t)p->dW_prefix | (uintptr_t)p->dW_full) & 15) return ADWIN_E_ALIGN;
  hipStream_t stream = (hipStream_t)hip_stream;
  unsigned char* ws = (unsigned char*)workspace;
  ADWIN_HIP_TRY(ensure_lds_opt_in());

  // one timed span at a time: starting a phase ends the previous one (no-ops without a timer)
  std::optional<PhaseScope> scope;
  auto phase = [&](int ph) { scope.reset(); scope.emplace(timer, ph); };
  phase(ADWIN_PHASE_SETUP);
  DevicePlan pl = device_plan_at(ws + L.o_plan, p->B, (int32_t*)(ws + L.o_row_idx),
                                 (int32_t*)(ws + L.o_row_seq));
  float* klr = (float*)(ws + L.o_klr);
  float* rownorm = (float*)(ws + L.o_rownorm);
  float* gws = (float*)(ws + L.o_g);
  double* seg = (double*)(ws + L.o_seg);
  const int64_t n_pad = hp.n_pad;

  HeavyList heavy;
  heavy.cnt = (int32_t*)(ws + L.o_heavy_cnt); heavy.v = (int32_t*)(ws + L.o_heavy_v);
  SetupArgs setup(ws + L.o_plan, p->B);
  setup.n_rows = hp.n_rows; setup.n_pad = n_pad;
  setup.row_idx = pl.row_idx; setup.row_seq = pl.row_seq;
  setup.clear(p->status_dev, 1);
  setup.clear(heavy.cnt, n_pad);
  uint32_t* done = (uint32_t*)(ws + L.o_racc);      // racc is not used when `done` is
  setup.clear(done, 1);
  if (!probe) {   // rows outside the windows report zero KL, cost and diagnostics
    setup.clear(p->kl, p->T);
    setup.clear(p->c, p->T);
    setup.clear(p->t_logp, p->T);
    setup.clear(p->t_entropy, p->T);
    setup.clear(p->t_rank, p->T);
  } else if (!p->ids) {
    setup.clear(p->c, p->T);
  }
  const bool prepares = hp.n_rows > 0 && L.use_dma;       // launch_prepare does the setup too
  if (!prepares) ADWIN_HIP_TRY(launch_setup(setup, blob, stream));

  if (hp.n_rows > 0) {
    const int vt_total = (int)(L.Vp / kTileVocab);
    const int n_tiles = (int)(n_pad / kTileTokens);
    const int h_tiles = (p->H_s + kGradTile - 1) / kGradTile;
    const bool use_dma = L.use_dma;
    References ref;
    ref.n_pad = n_pad; ref.parts = n_tiles <= kFineRefTiles ? kMaxRefParts : 1; ref.yid = (int32_t*)(ws + L.o_yid);
    for (int m = 0; m < 2; ++m) ref.max[m] = (float*)(ws + L.o_ref) + (int64_t)m * kMaxRefParts * n_pad;
    ref.zy[0] = (float*)(ws + L.o_zy_s); ref.zy[1] = (float*)(ws + L.o_zy_t);
    if (use_dma) {
      // tile images of the logit operands: vocabulary tiles of 128 rows (zero beyond V),
      // token tiles of 256 computed rows gathered through row_idx
      RowImageArgs ia;
      if (!L.direct_w) {
        ia.n_rows = p->V; ia.permute = 1;
        ia.src = (const uint4*)p->W_t; ia.img = (uint4*)(ws + L.o_wt_img); ia.H = p->H_t; ia.nk = p->H_t / kBK;
        ADWIN_HIP_TRY(launch_row_image(ia, (unsigned)vt_total, stream));
        ia.src = (const uint4*)p->W_s; ia.img = (uint4*)(ws + L.o_ws_img); ia.H = p->H_s; ia.nk = p->H_s / kBK;
        ADWIN_HIP_TRY(launch_row_image(ia, (unsigned)vt_total, stream));
      }
      PrepareArgs pr{};
      pr.row_idx = pl.row_idx; pr.ids = p->ids; pr.V = p->V; pr.ref = ref;
      pr.h[0] = (const __bf16*)p->h_s; pr.W[0] = (const __bf16*)p->W_s; pr.H[0] = p->H_s;
      pr.h[1] = (const __bf16*)p->h_t; pr.W[1] = (const __bf16*)p->W_t; pr.H[1] = p->H_t;
      ia.n_rows = n_pad; ia.permute = 0;
      for (int m = 0; m < 2; ++m) {
        ia.src = (const uint4*)pr.h[m]; ia.img = (uint4*)(ws + (m ? L.o_ht_img : L.o_hs_img));
        ia.H = pr.H[m]; ia.nk = pr.H[m] / kBK;
        pr.img[m] = ia;
      }
      // single sweep: the fixed references of every row, from vocabulary tile 0 and the sampled
      // token (without ids: id -1 on every row, which the diagnostics sweep expects)
      ADWIN_HIP_TRY(launch_prepare(pr, L.single, n_tiles, setup, blob, stream));
    }
    LogitPassArgs la{};
    la.h_s = (const __bf16*)p->h_s; la.h_t = (const __bf16*)p->h_t;
    la.W_s = (const __bf16*)p->W_s; la.W_t = (const __bf16*)p->W_t;
    la.H_s = p->H_s; la.H_t = p->H_t; la.V = p->V;
    la.row_idx = pl.row_idx; la.n_pad = n_pad;
    la.vt_total = vt_total;
    la.part = (float*)(ws + L.o_part);
    la.slab = (__bf16*)(ws + L.o_slab); la.Vp = L.Vp;
    la.ref = ref; la.e2_off = 0;
    la.mu0t = (L.single && !sampled && need_g) ? (float*)(ws + L.o_mu0t) : nullptr; la.mu0t_stride = L.slab_rows;
    la.tg = env_int("ADWIN_TG", 4);      // tuning override
    la.Wt_img = (const char*)(ws + L.o_wt_img); la.Ws_img = (const char*)(ws + L.o_ws_img);
    la.ht_img = (const char*)(ws + L.o_ht_img); la.hs_img = (const char*)(ws + L.o_hs_img);
    la.long_first = 0;
    la.heavy = heavy; la.narrow = false; la.stage = L.direct_w ? kStageRows : kStageImages; la.rotate = rotate_k(n_tiles, p->H_s, p->H_t);
    MergeArgs m{};
    m.part = la.part; m.strips = L.strips; m.n_pad = n_pad; m.n_rows = hp.n_rows;
    m.row_idx = pl.row_idx;
    m.h_s = la.h_s; m.h_t = la.h_t; m.W_s = la.W_s; m.W_t = la.W_t;
    m.H_s = p->H_s; m.H_t = p->H_t; m.V = p->V; m.ids = p->ids;
    m.klr = klr;
    m.lse_s = (float*)(ws + L.o_lse_s); m.alive = (float*)(ws + L.o_invz);
    m.kl = p->kl; m.c = p->c; m.status = p->status_dev;
    m.diag = diag ? 1 : 0; m.t_logp = p->t_logp; m.t_entropy = p->t_entropy; m.t_rank = p->t_rank;
    m.cr = sampled ? (float*)(ws + L.o_cr) : nullptr;
    GradArgs ga;
    ga.slab = la.slab; ga.Bm = (const __bf16*)p->W_s; ga.nk_total = (int)(L.Vp / kBK); ga.k_rows = p->V;
    ga.g = gws; ga.H = p->H_s; ga.h_tiles = h_tiles; ga.ksplit = L.ksplit;
    ga.out_rows = (int64_t)1 << 62; ga.accumulate = 0; ga.e2_bytes = 0; ga.past_cache = false;
    if (L.single) {
      // Single sweep, the references fixed: per row slab one sweep over the vocabulary producing
      // the strip sums and the gradient factors, the merge of the slab's rows, the combine pass
      // over the factors and the GEMM of dz with W_s.
      la.vt_total = vt_total;
      ga.g_rows = n_pad; ga.half_off = n_pad;
      for (int64_t r0 = 0; r0 < n_pad; r0 += L.slab_rows) {
        const int64_t rows = (n_pad - r0 < L.slab_rows) ? n_pad - r0 : L.slab_rows;
        la.tile0 = (int)(r0 / kTileTokens); la.n_tiles = (int)(rows / kTileTokens);
        la.e2_off = rows * L.Vp;
        const bool past_cache = rows * L.Vp * 2 * (sampled ? 1 : 2) > kPastCacheBytes;
        la.lines = past_cache && sweep_whole_lines(p->H_s + p->H_t);
        la.strips = sweep_strips(la.n_tiles, vt_total, &la.long_first);
        la.part = (float*)(ws + L.o_part) - r0; la.n_pad = rows;       // partials of this slab's rows
        la.stage = sweep_stage(p, L.direct_w, la.n_tiles, need_g);
        la.narrow = L.direct_w && la.n_tiles == 1 && hp.n_rows - r0 <= kNarrowRows;
        phase(ADWIN_PHASE_STATS);
        const int sweep_mode = !need_g ? (diag ? kModeSingleFwdDiag : kModeSingleFwd)
                               : sampled ? (diag ? kModeSingleE2Diag : kModeSingleE2)
                                         : (diag ? kModeSingleDiag : kModeSingle);
        ADWIN_HIP_TRY(launch_logit_pass(sweep_mode, true, la, stream));
        // this slab's rows are complete: KL_t, c_t, mu; then the logit gradient proper
        phase(ADWIN_PHASE_MERGE);
        MergeSingleArgs ms;
        ms.m = m; ms.m.strips = la.strips; ms.m.part = la.part; ms.m.n_pad = la.n_pad;
        ms.ref = ref;
        ms.mu_out = (float*)(ws + L.o_delta); ms.inv_z = (float*)(ws + L.o_invz);
        ms.row0 = r0; ms.rows = rows;
        ADWIN_HIP_TRY(launch_merge_single(ms, stream));
        if (!need_g) continue;
        ga.slab_row0 = r0;
        ga.row_tiles = (int)(rows / kGradTile);
        CombineArgs ca;
        ca.slab = (uint4*)la.slab; ca.e2_vec = la.e2_off / 8;
        ca.past_cache = past_cache;
        ca.mu = ms.mu_out; ca.inv_z = ms.inv_z; ca.row0 = r0; ca.nk = ga.nk_total;
        ca.mu0t = la.mu0t; ca.mu0t_stride = la.mu0t_stride;
        ca.dzT_p = p->dW_prefix ? (uint4*)(ws + L.o_dzT_p) : nullptr;
        ca.dzT_f = p->dW_full ? (uint4*)(ws + L.o_dzT_f) : nullptr;
        ca.nkr = (int)(rows / kBK); ca.pl = pl; ca.n_rows = hp.n_rows; ca.grad_scale = p->grad_scale;
        ca.cr = (const float*)(ws + L.o_cr); ca.yid = (const int32_t*)(ws + L.o_yid);
        ca.heavy = heavy;
        if (sampled) {       // contract the E2 factor; c_t and W_s[y_t] enter in finalize_kernel
          ga.slab = la.slab + la.e2_off;
          ga.half_tiles = 0;                       // output rows behind the n_pad of g
          ga.out_rows = n_pad + (int64_t)align_up((size_t)hp.n_rows, 8);   // n_pad, whole tiles, holds them
          if (head) {        // the transposed operand of the head-weight GEMMs; the slab stays as it is
            phase(ADWIN_PHASE_DZ);
            ADWIN_HIP_TRY(launch_combine(true, true, ca, ga.row_tiles, stream));
          }
        } else {
          const int64_t left = hp.n_rows - r0;
          if (!head && collapse_in_gemm(left < rows ? left : rows, p->V, h_tiles, ga.nk_total)) {
            ga.e2_bytes = 2 * la.e2_off; ga.past_cache = past_cache; ga.heavy = heavy;
            ga.mu = ms.mu_out; ga.inv_z = ms.inv_z; ga.mu0t = la.mu0t; ga.mu0t_stride = la.mu0t_stride;
          } else {
            ga.e2_bytes = 0;
            phase(ADWIN_PHASE_DZ);
            ADWIN_HIP_TRY(launch_combine(head, false, ca, ga.row_tiles, stream));
          }
          ga.half_tiles = ga.row_tiles;            // output rows are those of g
          ga.out_rows = (int64_t)align_up((size_t)hp.n_rows, 8);
        }
        phase(ADWIN_PHASE_GRAD);
        ADWIN_HIP_TRY(launch_grad_gemm(ga, stream));
        if (head) {
          // head-weight gradient of this slab: dW += dz^T (w h_s), k = the slab's rows
          GradArgs wa = ga;
          wa.Bm = (const __bf16*)(ws + L.o_hsg);
          wa.nk_total = (int)(rows / kBK); wa.k_rows = rows;
          wa.H = p->H_s; wa.h_tiles = h_tiles; wa.ksplit = 1;
          wa.slab_row0 = 0; wa.row_tiles = (int)((L.Vp + kGradTile - 1) / kGradTile); wa.half_tiles = wa.row_tiles;
          wa.half_off = 0; wa.g_rows = 0; wa.out_rows = p->V; wa.accumulate = r0 > 0;
          HsGatherArgs ha;
          ha.h_s = (const uint4*)p->h_s; ha.row_idx = pl.row_idx; ha.row0 = r0; ha.H = p->H_s;
          ha.out = (uint4*)(ws + L.o_hsg); ha.alive = (const float*)(ws + L.o_invz);
          ADWIN_HIP_TRY(launch_hs_gather(ha, rows, stream));
          for (int which = 0; which < 2; ++which) {
            float* out = which == 0 ? p->dW_prefix : p->dW_full;
            if (!out) continue;
            wa.slab = (const __bf16*)(ws + (which == 0 ? L.o_dzT_p : L.o_dzT_f));
            wa.g = out;
            ADWIN_HIP_TRY(launch_grad_gemm(wa, stream));
          }
        }
      }
    } else {
      // Two sweeps: statistics over all token tiles, merge, then per row slab the dz sweep
      // and its GEMM with W_s.
      m.lse2 = (float*)(ws + L.o_lse2); m.mu = (float*)(ws + L.o_mu);
      la.lse2 = m.lse2; la.mu = m.mu;
      phase(ADWIN_PHASE_STATS);
      {
        la.tile0 = 0; la.n_tiles = n_tiles; la.strips = L.strips;
        ADWIN_HIP_TRY(launch_logit_pass(kModeStats, use_dma, la, stream));
      }
      phase(ADWIN_PHASE_MERGE);
      ADWIN_HIP_TRY(launch_merge_stats(m, stream));
      ga.g_rows = n_pad; ga.half_off = 0;
      for (int64_t r0 = 0; r0 < n_pad; r0 += L.slab_rows) {
        const int64_t rows = (n_pad - r0 < L.slab_rows) ? n_pad - r0 : L.slab_rows;
        la.tile0 = (int)(r0 / kTileTokens); la.n_tiles = (int)(rows / kTileTokens);
        la.strips = sweep_strips(la.n_tiles, vt_total, &la.long_first);
        phase(ADWIN_PHASE_DZ);
        ADWIN_HIP_TRY(launch_logit_pass(kModeDz, use_dma, la, stream));
        phase(ADWIN_PHASE_GRAD);
        ga.slab_row0 = r0;
        ga.row_tiles = (int)(rows / kGradTile); ga.half_tiles = ga.row_tiles;
        ADWIN_HIP_TRY(launch_grad_gemm(ga, stream));
      }
    }
  }
  if (hp.n_rows == 0) {     // nothing computed: the head-weight gradients are zero
    ADWIN_HIP_TRY(launch_fill_f32(p->dW_prefix, (int64_t)p->V * p->H_s, 0.f, stream));
    ADWIN_HIP_TRY(launch_fill_f32(p->dW_full, (int64_t)p->V * p->H_s, 0.f, stream));
  }
  const bool pooled = probe && need_g;
  PoolArgs pa{};
  pa.pl = pl; pa.B = p->B; pa.H = p->H_s; pa.g = gws;
  pa.pp = (float*)(ws + L.o_pp); pa.pf = (float*)(ws + L.o_pf);
  pa.up = (float*)(ws + L.o_up); pa.uf = (float*)(ws + L.o_uf);
  BatchArgs b{};
  b.pl = pl; b.B = p->B; b.H = need_g ? p->H_s : 0; b.probe = probe;
  b.zero_grad = (p->grad_scale == 0.f) || !need_g;
  b.klr = klr; b.rownorm = pooled ? rownorm : nullptr;     // only the alignment reads their sums
  b.loss_prefix = p->loss_prefix; b.loss_full = p->loss_full;
  b.seg = seg; b.up = pa.up; b.uf = pa.uf; b.racc = (double*)(ws + L.o_racc); b.done = done;
  // in pp and pf, which lie together and were read for the last time by pool_kernel: per 256 columns (64 at least)
  // 1 + K sums of three doubles against twice those columns of floats
  static_assert((1 + ADWIN_MAX_CANDIDATES) * 3 * sizeof(double) <= 2 * 64 * sizeof(float), "micro fits");
  b.micro = (double*)(ws + L.o_pp);
  b.rho_pooled = p->rho_pooled; b.rho_field = p->rho_field; b.batch = p->batch;
  b.n_out = p->n_out; b.n_adm_out = p->n_adm_out; b.n_adm = hp.n_adm;
  CandArgs ca{};
  if (pooled && p->candidates && p->n_candidates > 0) {
    ca.pl = pl; ca.B = p->B; ca.H = p->H_s; ca.K = p->n_candidates;
    ca.reduction = p->reduction; ca.zero_grad = (p->grad_scale == 0.f);
    for (int k = 0; k < ca.K; ++k) {
      ca.L[k] = p->candidates[k];
      int64_t nadm = 0;
      for (int32_t i = 0; i < p->B; ++i) {
        const int64_t len = p->offsets[i + 1] - p->offsets[i];
        nadm += ca.L[k] < len ? (int64_t)ca.L[k] : len;
      }
      ca.inv_nadm[k] = nadm > 0 ? 1.0 / (double)nadm : 0.0;
    }
    ca.uf = pa.uf; ca.rownorm = rownorm; ca.seg = seg;
    ca.uc = (float*)(ws + L.o_uc); ca.cacc = (double*)(ws + L.o_cacc); ca.cS = (double*)(ws + L.o_cS);
    ca.rho_pooled = p->cand_rho_pooled; ca.rho_field = p->cand_rho_field; ca.batch = p->cand_batch;
  }
  SummaryArgs sa{};
  if (p->t_first_reject || p->t_logp_mean || p->cand_loss_share) {
    sa.pl = pl; sa.B = p->B; sa.probe = probe; sa.topk = p->topk;
    sa.K = p->cand_loss_share ? p->n_candidates : 0;
    for (int k = 0; k < sa.K; ++k) sa.L[k] = p->candidates[k];
    sa.t_rank = p->t_rank; sa.t_logp = p->t_logp;
    sa.kl = klr;             // per computed row = per packed row in the full-rollout mode
    sa.acc = (double*)(ws + L.o_summ);
    sa.first_reject = p->t_first_reject; sa.logp_mean = p->t_logp_mean; sa.loss_share = p->cand_loss_share;
  }
  // finalize over every packed row (also zero-fills rows outside the windows).  Without probe gradients the
  // reductions that end the call need nothing of it and share its launch (but for the rollout summaries,
  // whose registers would cost it waves).
  phase(ADWIN_PHASE_REDUCE);
  const TailArgs tail = make_tail(b, sa);
  const bool finalize = p->T > 0 && need_g, together = finalize && !pooled && !tail.with_summary;
  if (finalize) {
    FinalizeArgs f;
    f.pl = pl; f.B = p->B; f.T = p->T; f.probe = probe; f.n_rows = hp.n_rows;
    f.g = gws; f.ksplit = L.ksplit; f.n_pad = n_pad; f.H = p->H_s;
    f.g_rows = n_pad;
    f.inv_z = (const float*)(ws + L.o_invz);
    // the fp32 part of g; the sampled estimator contracts E2 as stored and lists nothing
    f.heavy = heavy;
    if (p->estimator == ADWIN_EST_SAMPLED) f.heavy.cnt = nullptr;
    f.lse_s = (const float*)(ws + L.o_lse_s);
    f.mu = (const float*)(ws + (L.single ? L.o_delta : L.o_mu));
    f.h_s = (const __bf16*)p->h_s; f.h_t = (const __bf16*)p->h_t; f.W_t = (const __bf16*)p->W_t; f.H_t = p->H_t;
    f.cr = (L.single && p->estimator == ADWIN_EST_SAMPLED) ? (const float*)(ws + L.o_cr) : nullptr;
    f.ids = p->ids; f.W_s = (const __bf16*)p->W_s; f.V = p->V;
    f.grad_scale = p->grad_scale; f.dh_bf16 = p->dh_dtype == ADWIN_DT_BF16;
    f.dh_prefix = p->dh_prefix; f.dh_full = p->dh_full; f.rownorm = rownorm;
    ADWIN_HIP_TRY(launch_finalize(f, together ? &tail : nullptr, stream));
  }
  if (!together) ADWIN_HIP_TRY(launch_tail(b, sa, ca, pooled ? &pa : nullptr, hp.n_chunks, stream));
  // alignment of the two objectives in the LM-head parameter block: batch[6]
  if (p->dW_prefix && p->dW_full && p->batch)
    ADWIN_HIP_TRY(launch_cosine(p->dW_prefix, p->dW_full, (int64_t)p->V * p->H_s,
                                (double*)(ws + L.o_cosp), p->batch + 6, stream));
  return ADWIN_OK;
}

extern "C" int adwin_opd_fused(const adwin_opd_problem* p, void* workspace, size_t workspace_bytes,
                               void* hip_stream) {
  return fused_impl(p, workspace, workspace_bytes, hip_stream, nullptr);
}

extern "C" int adwin_opd_fused_profile(const adwin_opd_problem* p, void* workspace,
                                       size_t workspace_bytes, void* hip_stream, float* phase_ms) {
  if (!phase_ms) return ADWIN_E_NULL;
  PhaseTimer timer((hipStream_t)hip_stream);
  int st = fused_impl(p, workspace, workspace_bytes, hip_stream, &timer);
  if (st != ADWIN_OK) return st;
  ADWIN_HIP_TRY(timer.collect(phase_ms, ADWIN_N_PHASES));
  return ADWIN_OK;
}
