// C ABI of libgecc: argument checking, workspace layout and the stream-ordered launch
// sequences.  Host code only; all arithmetic of the path runs in the kernels.
#include <algorithm>
#include <cstdlib>
#include <mutex>
#include <new>
#include "gecc_internal.h"

using namespace gecc;

namespace {

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

size_t elem_size(int dtype) { return dtype == GECC_BF16 ? 2 : 4; }

bool blocked(const gecc_ctx* c) { return c->nbi > 0; }
int items_of(const gecc_ctx* c) { return blocked(c) ? c->nbi * c->nbj : c->p.batch; }

// Workgroups per tile of a product whose tiles alone would leave compute units idle: as many as give `want`
// workgroups in all, each with at least `least` terms of k.
int ksplit_of(int64_t tiles, int want, int k, int least = 128) {
  int s = (int)(want / tiles);
  if (s < 1) s = 1;
  if (s > 8) s = 8;
  while (s > 1 && k / s < least) --s;
  return s;
}
int ksplit_128(int64_t tiles, int k) { return ksplit_of(tiles, 256, k); }

void make_layout(gecc_ctx* c) {
  const gecc_params& p = c->p;
  const size_t b = p.batch, n = p.n, k = p.k, m = p.m;
  const size_t ni = blocked(c) ? c->nbi : 1, nj = blocked(c) ? c->nbj : 1;   // (blocked mode has batch 1)
  Layout& L = c->lay;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
  L.done = take(SCAN_DONE_WORDS * sizeof(uint32_t));
  L.rowpart = take(b * c->ntn * (size_t)c->rp_ld * 2 * sizeof(float));
  L.colpart = take(b * c->ntm * (size_t)c->cp_ld * 2 * sizeof(float));
  // (blocked mode: one record per block, nj * 2n + ni * 2m doubles in all; audits per operand line)
  L.synd = take(b * (nj * 2 * n + ni * 2 * m) * sizeof(double));
  L.allow = take(b * (nj * 2 * n + ni * 2 * m) * sizeof(double));
  L.state = take(b * ni * nj * sizeof(DecodeState));
  L.audit_a = take(b * ni * 2 * k * sizeof(double));
  L.audit_b = take(b * nj * 2 * k * sizeof(double));
  L.blockmax = take(b * (((n + m + 63) / 64) + ni * nj) * 4 * sizeof(double));
  // column reductions: A side reduces over n (A stored n x k) or over k (P_r with A stored
  // k x n); B side over k (P_c with B stored k x m) or over m (B stored m x k)
  const size_t sa = p.trans_a ? coldot_scratch_doubles(p.k, p.n, p.batch)
                              : coldot_scratch_doubles(p.n, p.k, p.batch);
  const size_t sb = p.trans_b ? coldot_scratch_doubles(p.m, p.k, p.batch)
                              : coldot_scratch_doubles(p.k, p.m, p.batch);
  L.scan_a = take(sa * sizeof(double));
  L.scan_b = take(sb * sizeof(double));
  // the operand that gets the one-pass tile scan, as stored: rows x contiguous columns
  const size_t ra = tile_scan_row_scratch_doubles(p.trans_a ? p.k : p.n, p.trans_a ? p.n : p.k, p.dtype, p.batch);
  const size_t rb = tile_scan_row_scratch_doubles(p.trans_b ? p.m : p.k, p.trans_b ? p.k : p.m, p.dtype, p.batch);
  L.scan_row = take((ra > rb ? ra : rb) * sizeof(double));
  L.ksplit = take(c->ksplit > 1 ? b * c->ntm * c->ntn * (size_t)c->ksplit * c->tile_m * c->tile_n * sizeof(float) : 0);
  L.w_a = L.w_b = L.side_r = L.side_c = L.gate = 0;
  if (blocked(c)) {
    const size_t esz = p.dtype == GECC_BF16 ? 2 : 4;
    L.w_a = take((size_t)c->w_cols_a * k * esz);
    L.w_b = take((size_t)c->w_cols_b * k * esz);
    L.side_r = take(n * (size_t)c->w_cols_b * sizeof(float));
    L.side_c = take((size_t)c->w_cols_a * m * sizeof(float));
    L.gate = take(256);
  }
  L.total = off;
}

// Tile of the product kernel (= granularity of the partial sums), workgroups per tile, and whether the bf16
// kernel with 256 x 256 tiles may take the product.  All figures: microseconds, product kernel alone.
struct ProductPlan { int tile, ksplit; bool fast, fold; };

// 128 x 128 tiles of a bf16 product, k split so that few compute units idle: the number of ranges with the
// least (rounds of workgroups) / (ranges), at most 512 workgroups.  0: fewer than 384 workgroups, or
// ranges below 512 terms (1920 x 2176 x 512, 60 tiles: eight ranges 35 us, 64 x 64 tiles 23).
int ksplit_bf16_128(int64_t t128, int k) {
  int best = 0;
  double cost = 1e30;
  for (int s = 1; s <= 8 && t128 * s <= 512 && k / s >= 512; ++s) {
    const int64_t per_cu = (t128 * s + 255) / 256;
    const double c = (double)per_cu * (per_cu == 1 ? 1.25 : 1.0) / s + 0.02 * s;
    if (t128 * s >= 384 && c < cost) { cost = c; best = s; }
  }
  return best;
}

// Times of bf16 products in gemm_tile, product alone, as fitted to measurements (aligned rows, NN; us): what a
// workgroup needs per term of k with as many beside it on its compute unit, and the exchange between s ranges (C goes
// out and in s times).
double exchange(int64_t symbols, int s) { return s > 1 ? 1.8e-6 * (double)symbols * s : 0.0; }
double time_128(int64_t k, int64_t t128, int s) {
  const int64_t per_cu = (t128 * s + 255) / 256;
  if (per_cu > 3) return 6.0 + 2e-9 * (double)t128 * 16384.0 * (double)k / 0.66 + exchange(t128 * 16384, s);
  return 5.4 + (double)k / s * (per_cu == 1 ? 0.0153 : per_cu == 2 ? 0.0175 : 0.0265) + exchange(t128 * 16384, s);
}
double time_64(int64_t k, int64_t t64, int s) {
  const int64_t per_cu = (t64 * s + 255) / 256;
  const double per_term = per_cu == 1 ? 0.0087 : per_cu == 2 ? 0.0105 : per_cu == 3 ? 0.0135 : 0.0043 * (double)per_cu;
  return 4.0 + (double)k / s * per_term + exchange(t64 * 4096, s);
}
// the number of ranges with the least time: an exchange of up to 38 MB (the static scratch has 48)
int ranges_128(int64_t k, int64_t t128) {
  int best = 1;
  for (int s = 2; s <= 8 && t128 * s <= 576 && k / s >= 512; ++s)
    if (time_128(k, t128, s) < time_128(k, t128, best)) best = s;
  return best;
}

// 128 x 128 tiles: products with tiles enough for every compute unit, as long as tiles that hang over the edge do not
// eat up what the larger tile gains (a saturated chip does a 128 x 128 tile in the time of three 64 x 64 ones), and
// bf16 products of long k.  64 x 64 tiles: the rest.  Products alone, us, tiles of 64 (ranges of k) / of 128:
//   fp32  128^3          7.2  / 13.1              bf16  1500 x 1000 x 1100       14.1 / 21.6
//         1024^3         25.7 (3) / 34.2 (4)            16384 x 4096 x 88        39.9 (2) / 38.8 (4)
//         64 x 300^3     42.0 / 60.3              whole call 1536 x 4224 x 768   53.1 (2) / 50.9 (7)
//         256 x 512^3    536  / 400 (gemm_f32_wide)
//
// Workgroups of fp32 tiles of 64: four per compute unit keep it busy (1024^3, when it took 28 us: one workgroup per
// tile 40, two 31, four 28, eight 38); up to one tile per compute unit three are enough, and leave the fourth place to
// the scans that ride along (whole calls at 800 and 1024 workgroups: 1024^3 40.2 and 41.5; with more tiles 800 are too
// few, 1300^3, 441 tiles in one range 72.2, in two 65.1).  fp32 tiles of 128: two ranges below 512 tiles (whole call
// 2000 x 1000 x 2000: one 106.7, two 83.1).
//
// What the ranges of a tile exchange takes 3 to 4 us, so they have to be worth it.  fp32: 128 terms, of few tiles,
// whose compute units have nothing else to do, fewer (whole calls, ranges of 128 -> 64: 128^3 20.9 -> 20.2, 256^3
// 23.1 -> 21.7).
//
// bf16 tiles of 64: two workgroups per compute unit and ranges of 450 terms, where that is one range two and a half
// and 600; up to 20 tiles two and a half and 128.  Where ranges of 128 terms would be more, or those of tiles of 128
// shorter than half of these (which have two chains), the sums are put aside every so often, which keeps the error
// (GemmArgs::fold; 1258 x 2122 x 1110 in one range 1.90e-7 from the fp64 product, in four of tiles of 128 1.36e-7).  Whole calls with ranges of 128 terms / with these:
//   36 tiles    102 x 1542 x 1096 TT  28.5 / 25.6        140 tiles  448 x 920 x 1248 TT   28.7 / 26.6
//   72 tiles    1152 x 704 x 256      24.9 / 22.7        270 tiles  916 x 1817 x 1137     44.4 (in one range 46.9)
//   104 tiles   256 x 512 x 1664      26.6 / 21.2        315 tiles  4017 x 1020 x 282     35.3 / 34.3
// and up to 20 tiles, with 450 terms / with these: 128 x 896 x 128 TT 20.7 / 19.7, 211 x 447 x 232 21.1 / 21.0.
//
// bf16 tiles of 128 have one chain of sums over their range and no registers for another, so they are not taken where
// tiles of 64 would be but for the time (3440 x 240 x 2496: 34.5 us a call and 8.3e-8 from the fp64 product, tiles of
// 64 49.8 and 6.4e-8), nor in fewer ranges.  Tiles of 64 replace them, closer to the fp64 product as well, where the
// fitted times say so (144 x 3176 x 4952 NT 60.3 -> 52.9), and in place of eight ranges, the most a tile is cut into
// (960 x 4352 x 960 NT 54.7 -> 43.9, 3328 x 4544 x 192 58.5 -> 49.3).
// Two ranges of tiles of 128 and one of more than 512 tiles of 64 are as far from the fp64 product: by the fitted times
// (tiles of 64 / of 128, whole calls: 395 x 6072 x 5383 144.8 / 111.2, 1504 x 3076 x 1797 77.2 / 66.4, 2778 x 2582 x 909 TT
// 59.0 / 61.7; 43 such 1.12 times as fast).  Single products: of narrow items tiles of 128 may fill half, and what they
// exchange beside the batch's own scratch can be too much (232 x 5024 x 104 x 91 NT 88.3 / 129.5).
//
// narrow: a side product of blocked mode, a few columns (rows) beside a whole operand; its bf16 ranges are as they were
// measured, two and a half workgroups and 128 terms.
int most_ranges_64(int64_t t64, int k) { return ksplit_of(t64, 512 + (int)(t64 < 512 ? t64 / 2 : 0), k); }
int ranges_64(int64_t t64, int k) {
  if (t64 <= 20) return most_ranges_64(t64, k);
  const int two = ksplit_of(t64, 512, k, 450);
  return two > 1 ? two : ksplit_of(t64, 512 + (int)(t64 < 512 ? t64 / 2 : 0), k, 600);
}
ProductPlan plan_tiles(int dtype, int64_t n, int64_t k, int64_t m, int64_t batch, bool narrow = false) {
  const int64_t t128 = ((n + 127) / 128) * ((m + 127) / 128) * batch, t64 = ((n + 63) / 64) * ((m + 63) / 64) * batch;
  const bool many = t128 >= 256 && k >= 256 && 3 * t128 < t64;
  const int s_long = dtype == GECC_BF16 ? ksplit_bf16_128(t128, (int)k) : 0;
  const int most = most_ranges_64(t64, (int)k), s64 = narrow ? most : ranges_64(t64, (int)k);
  if (s_long > 0 && (narrow || (s_long < 8 && time_128(k, t128, ranges_128(k, t128)) <= time_64(k, t64, s64))))
    return {128, s_long, false, false};
  if (s_long == 0 && many) return {128, dtype == GECC_F32 && t128 < 512 ? 2 : 1, false, false};
  // tiles of 64 that fill a compute unit three times over without being split: two ranges of tiles of 128 have chains
  // no longer than their two
  if (dtype == GECC_BF16 && !narrow && batch == 1 && t64 > 512) {
    const int s128 = ranges_128(k, t128);
    if (s128 > 1 && time_128(k, t128, s128) < time_64(k, t64, s64)) return {128, s128, false, false};
  }
  if (dtype == GECC_F32)
    return {64, ksplit_of(t64, t64 > 256 ? 1024 : 800, (int)k, t64 <= 64 ? 64 : t64 <= 128 ? 96 : 128), false, false};
  return {64, s64, false, s64 < most || s_long > 0 || (!narrow && ranges_128(k, t128) > 2 * s64)};
}

double time_256(int64_t k, int64_t t256) { return 6.0 + (0.0148 + 0.009 * (double)t256 / 256.0) * (double)k; }

// Whether the 256 x 256-tile kernel is worth a thought at all: it needs a workgroup per compute unit to show its rate
// (1300 TFLOP/s; gemm_tile comes to 660), and has no k-split for fewer tiles.
bool fast_may_pay(int64_t n, int64_t k, int64_t m, int64_t batch) {
  const int64_t t256 = ((n + 255) / 256) * ((m + 255) / 256) * batch;
  if (t256 > 128) return true;
  const ProductPlan g = plan_tiles(GECC_BF16, n, k, m, batch, true);
  const int64_t rows = (n + g.tile - 1) / g.tile * g.tile, cols = (m + g.tile - 1) / g.tile * g.tile;
  const double gf = 2e-9 * (double)rows * (double)k * (double)cols * (double)batch;
  const double t_gen = g.tile == 64 ? 6.0 + gf / 0.33 + 0.006 * (double)(k / g.ksplit) : 8.0 + gf / 0.42;
  const double t_fast = time_256(k, t256);
  // (by less than that the fit cannot tell them apart)
  return t_fast - t_gen < 5.0 || t_gen > 0.85 * t_fast;
}
// gemm_tile's plan for a product of which that is so: whichever tile and ranges the fitted times say.  (The other
// kernel has one chain of sums over all of k: none of these is longer.)  Whole calls, one range of 128 x 128 tiles ->
// two: 2048 x 1024 x 2048 38.5 -> 44.3, 2048 x 4096 x 2048 94.5 -> 81.4; tiles of 64 -> of 128: 1024^3 28.7 -> 35.5.
ProductPlan plan_beside_256(int64_t n, int64_t k, int64_t m, int64_t batch) {
  const int64_t t128 = ((n + 127) / 128) * ((m + 127) / 128) * batch, t64 = ((n + 63) / 64) * ((m + 63) / 64) * batch;
  const int s64 = ranges_64(t64, (int)k), s128 = ranges_128(k, t128);
  const bool large = t128 >= 256 && k >= 256 && 3 * t128 < t64;
  if (large || (t128 <= 576 && time_128(k, t128, s128) < time_64(k, t64, s64))) return {128, s128, false, false};
  return {64, s64, false, s128 > 2 * s64};
}
double time_of(const ProductPlan& g, int64_t n, int64_t k, int64_t m, int64_t batch) {
  const int64_t tiles = ((n + g.tile - 1) / g.tile) * ((m + g.tile - 1) / g.tile) * batch;
  return g.tile == 128 ? time_128(k, tiles, g.ksplit) : time_64(k, tiles, g.ksplit);
}
// bonus: what gemm_tile saves a protected product beyond its own time (fast_protected).  Whole calls, us, 256 x 256
// tiles -> gemm_tile (product alone):
//   2048 x 1024 x 2048   54.9 -> 39.2  (23.4 -> 21.1)      2560^3               84.3 -> 76.4  (46.0 -> 52.4)
//   2048^3               72.0 -> 56.5  (38.3 -> 36.6)      3072 x 1024 x 3072   57.1 -> 50.3  (26.0 -> 34.2)
//   2816 x 704 x 2816    51.2 -> 38.4  (19.7 -> 21.4)      1280 x 7296 x 2304   171.6 -> 109.8 (113 -> 73.7)
//   4096 x 512 x 2048    49.4 -> 35.3  (18.2 -> 18.1)      1024 x 4096 x 4096 NT 109.0 -> 80.2
// and on either side of the line 3584 x 1536 x 2560 67.8 -> 67.6, 3072 x 2048 x 3072 76.7 -> 81.6.
bool fast_pays(int64_t n, int64_t k, int64_t m, int64_t batch, double bonus) {
  const int64_t t256 = ((n + 255) / 256) * ((m + 255) / 256) * batch;
  if (t256 > 256) return true;
  return fast_may_pay(n, k, m, batch) && time_256(k, t256) + bonus < time_of(plan_beside_256(n, k, m, batch), n, k, m, batch);
}
// The same for a product on its own.  Beside tiles of 64 the fit is good to a tenth (us, 256 x 256 tiles / tiles of 64:
// 1000 x 512 x 776 14.7 / 8.0, 776 x 2048 x 1032 36.9 / 17.1, 1504 x 1024 x 1504 21.8 / 17.7, 4096 x 192 x 4096
// 18.4 / 23.0, 3072 x 128 x 4096 13.8 / 16.0); beside tiles of 128 they have to be a quarter apart, for what it does
// not know (2560^3 46.0 / 52.4 where it says 52.9 / 50.2).
bool fast_alone(int64_t n, int64_t k, int64_t m, int64_t batch) {
  const int64_t t256 = ((n + 255) / 256) * ((m + 255) / 256) * batch;
  const bool close = plan_beside_256(n, k, m, batch).tile == 128;
  return fast_pays(n, k, m, batch, close ? -0.25 * time_256(k, t256) : 0.0);
}
// Whether the scans of the parity blocks (`scans`: their workgroups) ride in the launch of gemm_tile.  Two launches
// saved are 9 us and more (128^3 fp32 44 -> 31 us, bf16 1500 x 1501 x 1500 75 -> 61), but a scan's workgroup there takes
// the place of a product's, with fewer rows in flight than in a launch of its own.  Clean passes, one after the other
// -> in one launch, over 2300 products of all layouts (this rule 13 to 23 % faster on average, riding
// whenever the product has at most 2048 workgroups 12 to 22 %, with products that took twice as long):
//   - many rounds of workgroups hide nothing (256 x 512^3 fp32 603 -> 608 us), and scans of more than 16 workgroups per
//     compute unit take longer than the product (bf16 307 x 503 x 301 x 94 193 -> 313);
//   - bf16 gains whatever the ranges of k, now that the scans come behind the product's workgroups where not all run
//     at once (before, long ranges and more than 5 scan workgroups per compute unit lost): 5064 x 3680 x 1752
//     157.5 -> 145.6 us, 3500^3 215.5 -> 202.4, 5001 x 700 x 5001 105.7 -> 96.2, 2500^3 89.9 -> 78.9;
//   - fp32 keeps four workgroups of 64 x 64 tiles on a compute unit: scans that find no place beside them delay a
//     product of long k (3904 x 5888 x 448 289 -> 323), and many of them one of more than 512 terms (8 x 600^3 NT
//     81 -> 143).  Of 128 x 128 tiles it keeps two: both scans together, if they are few, beside short ranges of k (68 x
//     512 x 256 x 128 TN 90 -> 73; 2048^3 143 -> 190, 253 x 256 x 640 x 128 TN, where a tile scan has left one, 170 -> 327).
bool scans_ride(const gecc_params& p, int tile, int ksplit, int64_t scans, bool both) {
  const int64_t own = (int64_t)((p.n + tile - 1) / tile) * ((p.m + tile - 1) / tile) * p.batch * ksplit;
  const int k_per = p.k / ksplit;
  const bool small = tile == 64;
  if (own > 2048 || scans > 4096) return false;
  if (p.dtype == GECC_BF16) return true;
  if (!small) return both && k_per <= 640 && scans <= 1024;
  return own + scans <= 1536 || (k_per <= 640 && (scans <= 1792 || k_per <= 512));
}

// Whether the 256 x 256-tile kernel takes a protected product.  Where the parity scans ride in gemm_tile's launch, that
// saves the launches that they have of their own beside the other kernel, two for NN and TT, 12 us; one for NT and TN,
// which small products feel (256^3 NT), and above 2^19 symbols the fit has to be 6 us apart.  An operand that is read
// once for both of its scans has one of them fewer to ride.  Tiles that hang over the edge are in the fitted times of
// both kernels.  Where the scans do not ride, the faster product it is; of single NT and TN products the fit has to be
// 6 us apart there too (5056 x 64 x 2176 TN 32.6 / 36.1), while batches would lose by that (3 to 16 %).  Whole calls, us, 256 x 256 tiles / gemm_tile:
//   ride       2000 x 1024 x 2000   54.6 / 41.6      do not   4096 x 192 x 4096     47.5 / 55.5 (NT 45.0 / 51.7)
//              3000 x 512 x 3000    52.5 / 40.1               3072 x 128 x 4096     40.7 / 46.5
//              2504 x 2496 x 2504   84.0 / 77.7               128 x 1280 x 512 x 100   103.6 / 85.3
//              1000 x 512 x 776     45.6 / 23.5               512 x 2432 x 128 x 53 NT 118.0 / 96.9
//              520 x 256 x 264      40.6 / 22.1
bool fast_protected(const gecc_params& p, int64_t tile_min) {
  const ProductPlan g = plan_beside_256(p.n, p.k, p.m, p.batch);
  // (their workgroups as plan_riders counts them)
  const int64_t chunks = (p.k + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS;
  const int64_t pr = p.trans_a ? (p.n + 511) / 512 * chunks : (p.n + 3) / 4;
  const int64_t pc = p.trans_b ? (p.m + 3) / 4 : (p.m + 511) / 512 * chunks;
  double bonus;
  if (!scans_ride(p, g.tile, g.ksplit, (1 + pr + pc) * p.batch, true)) bonus = p.trans_a != p.trans_b && p.batch == 1 ? -6.0 : 0.0;
  else if ((int64_t)p.n * p.k * p.batch >= tile_min || (int64_t)p.k * p.m * p.batch >= tile_min) bonus = 0.0;
  else bonus = p.trans_a == p.trans_b ? 12.0 : (int64_t)p.n * p.m * p.batch < (1 << 19) ? 9.0 : -6.0;
  return fast_pays(p.n, p.k, p.m, p.batch, bonus);
}

// compact: 128 x 128 tiles and 256 workgroups, the plan that needs the least workspace.
void plan_product(gecc_ctx* c, bool compact) {
  const gecc_params& p = c->p;
  const bool may_be_fast = p.dtype == GECC_BF16 && p.k % 64 == 0 && p.lda % 8 == 0 && p.ldb % 8 == 0 &&
                           (!p.trans_a || p.n % 8 == 0) && (p.trans_b || p.m % 8 == 0) && (int64_t)p.n * p.m >= 256 * 256;
  const int64_t t128 = (int64_t)((p.n + 127) / 128) * ((p.m + 127) / 128) * p.batch;
  ProductPlan pl = {128, ksplit_128(t128, p.k), true, false};
  if (blocked(c)) pl.ksplit = 1;
  else if (!compact && !(may_be_fast && (c->cu_hint > 0 || fast_protected(p, c->tile_min))))
    pl = may_be_fast && fast_may_pay(p.n, p.k, p.m, p.batch) ? plan_beside_256(p.n, p.k, p.m, p.batch)
                                                             : plan_tiles(p.dtype, p.n, p.k, p.m, p.batch);
  // (a product on its own stays with the faster kernel)
  c->fast_plain = pl.fast || (may_be_fast && fast_alone(p.n, p.k, p.m, p.batch));
  c->tile_m = c->tile_n = pl.tile;
  c->ksplit = pl.ksplit;
  c->fold = pl.fold;
  c->fast = pl.fast;
  c->ntm = (p.n + pl.tile - 1) / pl.tile;
  c->ntn = (p.m + pl.tile - 1) / pl.tile;
  make_layout(c);
  // (a product that fits the library's static scratch in the compact plan has to fit it in any)
  if (!compact && c->lay.total > (size_t)GECC_STATIC_SCRATCH_BYTES) plan_product(c, true);
}

int check_ws(const gecc_ctx* c) {
  if (!c) return GECC_ERR_ARG;
  if (!c->ws || c->ws_bytes < c->lay.total) return GECC_ERR_WORKSPACE;
  return GECC_OK;
}

int hip_rc(hipError_t e) { return e == hipSuccess ? GECC_OK : GECC_ERR_HIP; }

// The counters at the front of the workspace have to start at zero: done once per attached
// workspace, on the stream of the first call that launches scans.
int prep(gecc_ctx* c, hipStream_t st) {
  if (c->ws_zeroed == c->ws) return GECC_OK;
  if (launch_zero_words(reinterpret_cast<uint32_t*>(c->ws + c->lay.done), SCAN_DONE_WORDS, st) != hipSuccess)
    return GECC_ERR_HIP;
  c->ws_zeroed = c->ws;
  return GECC_OK;
}

// operands need only their natural alignment; 16-byte aligned rows get the vector paths
bool aligned_to(const void* p, size_t a) { return reinterpret_cast<uintptr_t>(p) % a == 0; }

DecodeArgs decode_args(gecc_ctx* c, void* A, const double* A_par, void* B, const double* B_par,
                       float* C, double* C_par, gecc_report* rep) {
  DecodeArgs d;
  d.p = c->p;
  d.tile_m = c->tile_m; d.tile_n = c->tile_n; d.ntm = c->ntm; d.ntn = c->ntn;
  d.rp_ld = c->rp_ld; d.cp_ld = c->cp_ld;
  d.A = A; d.B = B; d.C = C;
  d.A_par = A_par; d.B_par = B_par; d.C_par = C_par;
  d.rowpart = reinterpret_cast<float*>(c->ws + c->lay.rowpart);
  d.colpart = reinterpret_cast<float*>(c->ws + c->lay.colpart);
  d.synd = reinterpret_cast<double*>(c->ws + c->lay.synd);
  d.allow = reinterpret_cast<double*>(c->ws + c->lay.allow);
  d.state = reinterpret_cast<DecodeState*>(c->ws + c->lay.state);
  d.blockmax = reinterpret_cast<double*>(c->ws + c->lay.blockmax);
  d.nblk = (c->p.n + c->p.m + 63) / 64;
  d.audit_a = reinterpret_cast<double*>(c->ws + c->lay.audit_a);
  d.audit_b = reinterpret_cast<double*>(c->ws + c->lay.audit_b);
  d.report = rep;
  d.nbj = 0;
  d.ia_stride = c->p.stride_a; d.jb_stride = c->p.stride_b; d.ic_stride = c->p.stride_c; d.jc_stride = 0;
  d.gate_word = nullptr;
  if (blocked(c)) {
    // the decoder sees every block as an item of its own: n, m are the block sizes
    const gecc_params& p = c->p;
    d.p.n = p.block_n; d.p.m = p.block_m; d.p.batch = c->nbi * c->nbj;
    d.nbj = c->nbj;
    d.ia_stride = p.trans_a ? (int64_t)p.block_n : (int64_t)p.block_n * p.lda;
    d.jb_stride = p.trans_b ? (int64_t)p.block_m * p.ldb : (int64_t)p.block_m;
    d.ic_stride = (int64_t)p.block_n * p.ldc; d.jc_stride = p.block_m;
    d.nblk = 1;
    d.blockmax += (size_t)((p.n + p.m + 63) / 64) * 4;     // the per-block maxima live behind the per-workgroup ones
    d.gate_word = reinterpret_cast<int32_t*>(c->ws + c->lay.gate);
  }
  return d;
}

// Blocked mode: the row blocks of A (column blocks of B) as batch items of the scans -- a copy of
// the context whose n (m) is the block size, whose batch is the number of blocks and whose batch
// stride walks from block to block.  Both views use the tile scan for their operand (encoding and
// audit alike) where it applies.
gecc_ctx view_a(const gecc_ctx* c) {
  gecc_ctx v = *c;
  v.p.n = c->p.block_n; v.p.batch = c->nbi;
  v.p.stride_a = c->p.trans_a ? (int64_t)c->p.block_n : (int64_t)c->p.block_n * c->p.lda;
  v.nbi = v.nbj = 0; v.tile_op = GECC_MAT_A;
  return v;
}
gecc_ctx view_b(const gecc_ctx* c) {
  gecc_ctx v = *c;
  v.p.m = c->p.block_m; v.p.batch = c->nbj;
  v.p.stride_b = c->p.trans_b ? (int64_t)c->p.block_m * c->p.ldb : (int64_t)c->p.block_m;
  v.nbi = v.nbj = 0; v.tile_op = GECC_MAT_B;
  return v;
}

ScanArgs scan_base(const gecc_ctx* c, const void* X, int64_t ld, int64_t xs) {
  ScanArgs s{};
  s.X = X; s.dtype = c->p.dtype; s.ld = ld; s.xs = xs; s.batch = c->p.batch;
  s.gate = nullptr; s.gate_stride = 0; s.gate_value = 0;
  return s;
}

// The four scans of the path.  Each operand is reduced once along its contiguous index (rowdot:
// one launch) and once along the other (coldot: two stages), whichever way it is stored.
struct ScanJob {
  ScanArgs s;
  bool rowdot;
  int kind;   // GECC_K_x, for the timing records
};

// Brackets the launches between its construction and done() with a timing record, when the
// context records launches of that class.  ahead: records that were begun before this one and are not done
// yet (a launch that does the work of several classes leaves a record of each).
struct Timed {
  gecc_ctx* c;
  hipStream_t st;
  int kind, at;
  bool on;
  hipError_t err;
  Timed(gecc_ctx* ctx, int k, hipStream_t s, int ahead = 0) : c(ctx), st(s), kind(k), at(ctx->ev_n + ahead), err(hipSuccess) {
    on = c->ev && ((c->ev_mask >> k) & 1u) && at < c->ev_cap;
    if (on) err = hipEventRecord(c->ev[2 * at], st);
  }
  hipError_t done(hipError_t launch_result) {
    if (launch_result != hipSuccess) return launch_result;
    if (err != hipSuccess) return err;
    if (on) {
      if ((err = hipEventRecord(c->ev[2 * at + 1], st)) != hipSuccess) return err;
      c->ev_kind[at] = kind;
      ++c->ev_n;
    }
    return hipSuccess;
  }
};

// reduce A over its row index i (length n) -> [2][k]; w = null: Section III's index weights
ScanJob scan_a_over_n(gecc_ctx* c, const void* A, const double* w, double* out, const int32_t* gate) {
  const gecc_params& p = c->p;
  ScanJob j{scan_base(c, A, p.lda, p.stride_a), p.trans_a != 0, gate ? GECC_K_AUDIT_A : GECC_K_ENCODE_A};
  ScanArgs& s = j.s;
  s.w = w; s.out = out; s.w_stride = 2 * (int64_t)p.n; s.out_stride = 2 * (int64_t)p.k;
  if (gate) { s.gate = gate; s.gate_stride = sizeof(DecodeState); s.gate_value = PH_AUDIT; }
  if (p.trans_a) { s.R = p.k; s.Cc = p.n; }   // stored k x n
  else { s.R = p.n; s.Cc = p.k; s.scratch = reinterpret_cast<double*>(c->ws + c->lay.scan_a); }
  return j;
}
// reduce A over its column index l (length k) -> [2][n]
ScanJob scan_a_over_k(gecc_ctx* c, const void* A, const double* w, double* out, int64_t out_stride) {
  const gecc_params& p = c->p;
  ScanJob j{scan_base(c, A, p.lda, p.stride_a), p.trans_a == 0, GECC_K_PARITY_R};
  ScanArgs& s = j.s;
  s.w = w; s.out = out; s.w_stride = 2 * (int64_t)p.k; s.out_stride = out_stride;
  if (p.trans_a) { s.R = p.k; s.Cc = p.n; s.scratch = reinterpret_cast<double*>(c->ws + c->lay.scan_a); }
  else { s.R = p.n; s.Cc = p.k; }
  return j;
}
// reduce B over its column index j (length m) -> [2][k]
ScanJob scan_b_over_m(gecc_ctx* c, const void* B, const double* w, double* out, const int32_t* gate) {
  const gecc_params& p = c->p;
  ScanJob j{scan_base(c, B, p.ldb, p.stride_b), p.trans_b == 0, gate ? GECC_K_AUDIT_B : GECC_K_ENCODE_B};
  ScanArgs& s = j.s;
  s.w = w; s.out = out; s.w_stride = 2 * (int64_t)p.m; s.out_stride = 2 * (int64_t)p.k;
  if (gate) { s.gate = gate; s.gate_stride = sizeof(DecodeState); s.gate_value = PH_AUDIT; }
  if (p.trans_b) { s.R = p.m; s.Cc = p.k; s.scratch = reinterpret_cast<double*>(c->ws + c->lay.scan_b); }   // stored m x k
  else { s.R = p.k; s.Cc = p.m; }
  return j;
}
// reduce B over its row index l (length k) -> [2][m]
ScanJob scan_b_over_k(gecc_ctx* c, const void* B, const double* w, double* out, int64_t out_stride) {
  const gecc_params& p = c->p;
  ScanJob j{scan_base(c, B, p.ldb, p.stride_b), p.trans_b != 0, GECC_K_PARITY_C};
  ScanArgs& s = j.s;
  s.w = w; s.out = out; s.w_stride = 2 * (int64_t)p.k; s.out_stride = out_stride;
  if (p.trans_b) { s.R = p.m; s.Cc = p.k; }
  else { s.R = p.k; s.Cc = p.m; s.scratch = reinterpret_cast<double*>(c->ws + c->lay.scan_b); }
  return j;
}

// The tile scan of operand `op` (as stored: rows x contiguous columns).  enc_out: where the
// index-weighted reduction of Section III goes (A_P or B_P, or an audit buffer), or null;
// par_w / par_out: weights and destination of the parity block of C-bar along the other axis
// (P_r = A B_P or P_c = A_P B), or null.
TileScanJob tile_job(gecc_ctx* c, int op, const void* X, double* enc_out, const double* par_w, double* par_out,
                     int64_t par_out_stride, const int32_t* gate) {
  const gecc_params& p = c->p;
  const bool is_a = op == GECC_MAT_A;
  const bool tr = is_a ? p.trans_a != 0 : p.trans_b != 0;
  TileScanJob t{};
  t.X = X; t.dtype = p.dtype; t.batch = p.batch; t.stream = c->stream;
  t.ld = is_a ? p.lda : p.ldb;
  t.xs = is_a ? p.stride_a : p.stride_b;
  const int len = is_a ? p.n : p.m;                 // the axis the encoding sums over
  t.R = is_a ? (tr ? p.k : p.n) : (tr ? p.m : p.k);
  t.Cc = is_a ? (tr ? p.n : p.k) : (tr ? p.k : p.m);
  (void)len;
  // A stored n x k and B stored m x k keep the encoded axis in the rows: column part.  The other
  // two layouts keep it in the columns: row part.
  const bool enc_is_col = is_a ? !tr : tr;
  t.col_scratch = reinterpret_cast<double*>(c->ws + (is_a ? c->lay.scan_a : c->lay.scan_b));
  t.row_scratch = reinterpret_cast<double*>(c->ws + c->lay.scan_row);
  const int64_t k2 = 2 * (int64_t)p.k;
  if (enc_out) {
    if (enc_is_col) { t.col_on = true; t.wr = nullptr; t.col_out = enc_out; t.col_out_stride = k2; }
    else            { t.row_on = true; t.wc = nullptr; t.row_out = enc_out; t.row_out_stride = k2; }
  }
  if (par_w) {
    if (enc_is_col) { t.row_on = true; t.wc = par_w; t.wc_stride = k2; t.row_out = par_out; t.row_out_stride = par_out_stride; }
    else            { t.col_on = true; t.wr = par_w; t.wr_stride = k2; t.col_out = par_out; t.col_out_stride = par_out_stride; }
  }
  if (gate) { t.gate = gate; t.gate_stride = sizeof(DecodeState); t.gate_value = PH_AUDIT; }
  return t;
}

// Whether the tile scan serves this operand: its rows have to allow it, and the operand has to be
// large enough for one pass to beat two (small operands are bound by the number of dependent
// launches, and the two separate scans need one launch less: a row scan carries the second stage
// of a column scan).  From 64 MiB on the one pass wins: fp32 products of 2^24 elements an operand
// 512^3 x 64 NN 160.2 -> 150.5 us, NT 151.9 -> 148.5, 500^3 x 128 314.8 -> 294.8, 640 x 256 x 640
// x 128 272.7 -> 262, while 256 x 512 x 384 x 200 stays; bf16 of as many elements +-1.5 %.  Rows
// below 256 elements leave part of a tile row's 64 x 16 bytes idle and wait for 2^25 elements.  A
// function of shape and alignment alone, so that an encoding and the audit that re-forms it always
// take the same kernel.
bool use_tile(const gecc_ctx* c, const TileScanJob& t) {
  const int64_t n = (int64_t)t.R * t.Cc * t.batch;
  return tile_scan_ok(t) && n >= c->tile_min && (t.Cc >= 256 || n >= std::min<int64_t>(2 * c->tile_min, (int64_t)1 << 25));
}

// Scans in stream order.  The second stage of a coldot is held back: the next rowdot carries it in
// the same launch unless it reads that stage's output (or is gated differently); anything else
// flushes it first.  The caller flushes before the results are needed.
struct ScanQueue {
  gecc_ctx* c;
  hipStream_t st;
  Stage2Job pending{};
  uint32_t* done() const { return reinterpret_cast<uint32_t*>(c->ws + c->lay.done); }
  hipError_t flush() {
    if (!pending.valid) return hipSuccess;
    pending.valid = false;
    Timed t(c, GECC_K_STAGE2, st);
    return t.done(launch_stage2(pending, Stage2Job{}, st));
  }
  hipError_t run(const ScanJob& j) {
    hipError_t e;
    const ScanArgs& s = j.s;
    const bool reads_pending = s.w != nullptr && (s.w == pending.out || s.w == pending.row_out);
    const bool can_carry = j.rowdot && pending.valid && !reads_pending && s.batch == pending.batch &&
                           s.gate == pending.gate && s.gate_stride == pending.gate_stride &&
                           s.gate_value == pending.gate_value;
    if (pending.valid && !can_carry && (e = flush()) != hipSuccess) return e;
    Timed t(c, j.kind, st);
    if (j.rowdot) {
      e = launch_rowdot(s, can_carry ? &pending : nullptr, st);
      pending.valid = false;
      return t.done(e);
    }
    // (a gated column scan finishes by itself where it can: the audits then need no launch for it)
    ScanArgs f = s;
    if (s.gate && coldot_done_words(f) > 0) f.done = done();
    return t.done(launch_coldot_stage1(f, &pending, st));
  }
  // a tile scan: what is left of its second stage becomes the pending one
  hipError_t run_tile(const TileScanJob& tj, int kind) {
    hipError_t e;
    if (pending.valid && (e = flush()) != hipSuccess) return e;
    TileScanJob f = tj;
    if (tj.gate) f.done = done();
    Timed t(c, kind, st);
    return t.done(launch_tile_scan(f, &pending, st));
  }
};

// whether two scans that do not read each other's results may go in one launch
bool may_pair(const ScanJob& x, const ScanJob& y) {
  const ScanArgs s[2] = {x.s, y.s};
  const bool row[2] = {x.rowdot, y.rowdot};
  return scan_pair_fits(s, row);
}

// Sums that a chain of launches leaves to their readers: the operand parities A_P and B_P (read by the scans that use
// them as weights) and the parity blocks P_r and P_c of C-bar (read by the threshold pass).
struct Left { Parts ap, bp, pr, pc; };
bool any(const Parts& p) { return p.nchunk > 0 || p.nseg > 0; }
// what a second stage still has to do, in its column part and in its row part
Parts chunks_of(const Stage2Job& j) { return j.valid && j.Cc > 0 ? Parts{j.scratch, nullptr, j.nchunk, 0} : Parts{}; }
Parts segs_of(const Stage2Job& j) { return j.valid && j.R > 0 ? Parts{nullptr, j.row_scratch, 0, j.nseg} : Parts{}; }
Stage2Job stage2_of(const Parts& p, double* out, int64_t out_stride, int len, int batch) {
  Stage2Job j{};
  j.valid = any(p);
  j.batch = batch;
  if (p.nchunk > 0) { j.scratch = p.chunks; j.nchunk = p.nchunk; j.out = out; j.out_stride = out_stride; j.Cc = len; }
  else if (p.nseg > 0) { j.row_scratch = p.segs; j.nseg = p.nseg; j.row_out = out; j.row_out_stride = out_stride; j.R = len; }
  return j;
}
// adds up now what p0 and p1 (A_P and B_P, or P_r and P_c) have left, in one launch
hipError_t finish_parts(gecc_ctx* c, const Stage2Job& j0, const Stage2Job& j1, hipStream_t st) {
  if (!j0.valid && !j1.valid) return hipSuccess;
  Timed t(c, GECC_K_STAGE2, st);
  return t.done(j0.valid ? launch_stage2(j0, j1, st) : launch_stage2(j1, j0, st));
}

GemmArgs gemm_args(const gecc_ctx* c, const void* A, const void* B, float* C) {
  const gecc_params& p = c->p;
  GemmArgs g{};
  g.A = A; g.B = B; g.C = C;
  g.dtype = p.dtype; g.trans_a = p.trans_a; g.trans_b = p.trans_b;
  g.n = p.n; g.k = p.k; g.m = p.m; g.batch = p.batch;
  g.lda = p.lda; g.ldb = p.ldb; g.ldc = p.ldc;
  g.sa = p.stride_a; g.sb = p.stride_b; g.sc = p.stride_c;
  g.tile_m = c->tile_m; g.tile_n = c->tile_n; g.ntm = c->ntm; g.ntn = c->ntn; g.fast = c->fast; g.fold = c->fold;
  g.cu_hint = c->cu_hint; g.split_first = -1;
  if (c->ksplit > 1 && c->ws && c->ws_bytes >= c->lay.total) {
    g.ksplit = c->ksplit;
    g.split_part = reinterpret_cast<float*>(c->ws + c->lay.ksplit);
    g.split_bytes = c->lay.total - c->lay.ksplit;    // (last in the layout but for blocked mode's, which has no split here)
    g.split_done = reinterpret_cast<uint32_t*>(c->ws + c->lay.done);
  }
  g.rp_ld = c->rp_ld; g.cp_ld = c->cp_ld;
  return g;
}

// the product kernel(s), bracketed by a timing record when timing is enabled
hipError_t timed_gemm(gecc_ctx* c, const GemmArgs& g, const GemmSide* side, hipStream_t st) {
  Timed t(c, GECC_K_PRODUCT, st);
  return t.done(launch_gemm(g, side, st));
}

}  // namespace

extern "C" {

int gecc_create(gecc_ctx** out, const gecc_params* p) {
  if (!out || !p) return GECC_ERR_ARG;
  *out = nullptr;
  if (p->n < 1 || p->k < 1 || p->m < 1 || p->batch < 1) return GECC_ERR_ARG;
  if (p->dtype != GECC_F32 && p->dtype != GECC_BF16) return GECC_ERR_ARG;
  if ((p->trans_a != 0 && p->trans_a != 1) || (p->trans_b != 0 && p->trans_b != 1)) return GECC_ERR_ARG;
  if (p->lda < (p->trans_a ? p->n : p->k)) return GECC_ERR_ARG;
  if (p->ldb < (p->trans_b ? p->k : p->m)) return GECC_ERR_ARG;
  if (p->ldc < p->m) return GECC_ERR_ARG;
  if (p->batch > 1) {
    const int64_t rows_a = p->trans_a ? p->k : p->n, rows_b = p->trans_b ? p->m : p->k;
    if (p->stride_a < rows_a * p->lda || p->stride_b < rows_b * p->ldb ||
        p->stride_c < (int64_t)p->n * p->ldc)
      return GECC_ERR_ARG;
  }
  if (!(p->tau_r1 >= 0) || !(p->tau_r2 >= 0) || !(p->tau_q1 >= 0) || !(p->tau_q2 >= 0) ||
      !(p->tau_op >= 0) || !(p->tau_rep >= 0) || !(p->tau_rel >= 0))
    return GECC_ERR_ARG;
  if (p->weighted != 0 && p->weighted != 1) return GECC_ERR_ARG;
  if ((p->block_n == 0) != (p->block_m == 0) || p->block_n < 0 || p->block_m < 0) return GECC_ERR_ARG;
  if (p->block_n > 0 && (p->block_n % 128 || p->block_m % 128 || p->n % p->block_n || p->m % p->block_m ||
                         p->batch != 1 || p->weighted != 1))
    return GECC_ERR_ARG;
  if ((int64_t)p->n + p->m > (int64_t)1 << 30) return GECC_ERR_ARG;
  gecc_ctx* c = new (std::nothrow) gecc_ctx;
  if (!c) return GECC_ERR_ARG;
  c->p = *p;
  {
    const char* e = getenv("GECC_CU_COUNT");       // test hook: see GemmArgs::cu_hint
    c->cu_hint = e ? atoi(e) : 0;
    if (c->cu_hint < 0) c->cu_hint = 0;
    const char* t = getenv("GECC_TILE_MIN");       // test hook: operands of that many elements or more take the one-pass scan
    c->tile_min = (t && atoll(t) > 0) ? atoll(t) : ((int64_t)64 << 20) / (int64_t)elem_size(p->dtype);    // 64 MiB
  }
  // Operands that fit the 256 MiB memory-side cache, or nearly so, are still there for the product when a scan has
  // read them; loads past the caches pay only beyond (clean passes, ordinary loads -> such loads: both operands
  // 201 MB 4096 x 8192 x 8192 NT 443 -> 508 us, 104 MB 9000 x 4000 x 4000 508 -> 548, 335 MB 4096 x 8192 x 16384 NT
  // 921 -> 956; 402 MB 16384 x 8192 x 8192 1600 -> 1563, 587 MB 4096 x 16384 x 14336 NT 1808 -> 1738).
  c->stream = ((int64_t)p->n + p->m) * p->k * p->batch * (int64_t)elem_size(p->dtype) >= ((int64_t)384 << 20);
  // the larger operand is read once for both of its reductions (tile scan), the other one twice
  c->tile_op = p->n >= p->m ? GECC_MAT_A : GECC_MAT_B;
  c->nbi = p->block_n > 0 ? p->n / p->block_n : 0;
  c->nbj = p->block_n > 0 ? p->m / p->block_m : 0;
  c->pieces = p->dtype == GECC_BF16 ? 3 : 1;
  c->w_cols_a = (2 * c->pieces * c->nbi + 7) / 8 * 8;
  c->w_cols_b = (2 * c->pieces * c->nbj + 7) / 8 * 8;
  // slab strides of the partial sums: a multiple of 2 KiB would put the same line of every slab
  // into the same memory channel
  c->rp_ld = p->n % 256 == 0 ? p->n + 16 : p->n;
  c->cp_ld = p->m % 256 == 0 ? p->m + 16 : p->m;
  c->ws = nullptr;
  c->ws_bytes = 0;
  c->ws_zeroed = nullptr;
  c->panel = nullptr;
  c->n_panel = 0;
  c->fault_bias = 0;
  c->ev = nullptr;
  c->ev_kind = nullptr;
  c->ev_mask = 0;
  c->ev_cap = 0;
  c->ev_n = 0;
  plan_product(c, false);
  *out = c;
  return GECC_OK;
}

namespace {
void drop_panels(gecc_ctx* ctx) {
  for (int g = 0; g < ctx->n_panel; ++g) delete ctx->panel[g];
  delete[] ctx->panel;
  ctx->panel = nullptr;
  ctx->n_panel = 0;
}
}  // namespace

void gecc_destroy(gecc_ctx* ctx) {
  if (!ctx) return;
  drop_panels(ctx);
  gecc_timing_enable(ctx, 0, 0);
  delete ctx;
}

int gecc_timing_enable(gecc_ctx* ctx, int32_t max_records, uint32_t kinds_mask) {
  if (!ctx || max_records < 0) return GECC_ERR_ARG;
  for (int i = 0; i < 2 * ctx->ev_cap; ++i) (void)hipEventDestroy(ctx->ev[i]);
  delete[] ctx->ev;
  delete[] ctx->ev_kind;
  ctx->ev = nullptr;
  ctx->ev_kind = nullptr;
  ctx->ev_cap = 0;
  ctx->ev_n = 0;
  ctx->ev_mask = 0;
  if (max_records == 0) return GECC_OK;
  ctx->ev = new (std::nothrow) hipEvent_t[2 * (size_t)max_records];
  ctx->ev_kind = new (std::nothrow) int32_t[(size_t)max_records];
  if (!ctx->ev || !ctx->ev_kind) {
    delete[] ctx->ev; delete[] ctx->ev_kind;
    ctx->ev = nullptr; ctx->ev_kind = nullptr;
    return GECC_ERR_ARG;
  }
  for (int i = 0; i < 2 * max_records; ++i)
    if (hipEventCreate(&ctx->ev[i]) != hipSuccess) {
      for (int j = 0; j < i; ++j) (void)hipEventDestroy(ctx->ev[j]);
      delete[] ctx->ev; delete[] ctx->ev_kind;
      ctx->ev = nullptr; ctx->ev_kind = nullptr;
      return GECC_ERR_HIP;
    }
  ctx->ev_cap = max_records;
  ctx->ev_mask = kinds_mask;
  return GECC_OK;
}

int gecc_timing_read(gecc_ctx* ctx, float* host_ms, int32_t* host_kind, int32_t cap, int32_t* count) {
  if (!ctx || !host_ms || !count || cap < 0) return GECC_ERR_ARG;
  const int n = ctx->ev_n < cap ? ctx->ev_n : cap;
  for (int i = 0; i < n; ++i) {
    if (hipEventSynchronize(ctx->ev[2 * i + 1]) != hipSuccess) return GECC_ERR_HIP;
    if (hipEventElapsedTime(&host_ms[i], ctx->ev[2 * i], ctx->ev[2 * i + 1]) != hipSuccess) return GECC_ERR_HIP;
    if (host_kind) host_kind[i] = ctx->ev_kind[i];
  }
  *count = n;
  ctx->ev_n = 0;
  return GECC_OK;
}

size_t gecc_workspace_bytes(const gecc_ctx* ctx) { return ctx ? ctx->lay.total : 0; }

int gecc_set_workspace(gecc_ctx* ctx, void* dev_workspace, size_t bytes) {
  if (!ctx || !dev_workspace) return GECC_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(dev_workspace) % 256) return GECC_ERR_ALIGN;
  if (bytes < ctx->lay.total) return GECC_ERR_WORKSPACE;
  ctx->ws = static_cast<char*>(dev_workspace);
  ctx->ws_bytes = bytes;
  ctx->ws_zeroed = nullptr;     // its counters are zeroed by the first call that launches something
  return GECC_OK;
}

size_t gecc_a_par_len(const gecc_ctx* ctx) {
  return ctx ? 2 * (size_t)ctx->p.k * (blocked(ctx) ? ctx->nbi : 1) : 0;
}
size_t gecc_b_par_len(const gecc_ctx* ctx) {
  return ctx ? 2 * (size_t)ctx->p.k * (blocked(ctx) ? ctx->nbj : 1) : 0;
}
size_t gecc_c_par_len(const gecc_ctx* ctx) {
  if (!ctx) return 0;
  if (blocked(ctx)) return (size_t)ctx->nbi * ctx->nbj * (2 * (size_t)ctx->p.block_n + 2 * (size_t)ctx->p.block_m + 4);
  return 2 * (size_t)ctx->p.n + 2 * (size_t)ctx->p.m + 4;
}
int32_t gecc_item_count(const gecc_ctx* ctx) { return ctx ? items_of(ctx) : 0; }

int gecc_encode_a(gecc_ctx* ctx, const void* dev_A, double* dev_A_par, void* stream) {
  int rc = check_ws(ctx);
  if (rc) return rc;
  if (!dev_A || !dev_A_par) return GECC_ERR_ARG;
  if (!aligned_to(dev_A, elem_size(ctx->p.dtype)) || !aligned_to(dev_A_par, 8)) return GECC_ERR_ALIGN;
  if ((rc = prep(ctx, (hipStream_t)stream))) return rc;
  if (blocked(ctx)) {
    gecc_ctx v = view_a(ctx);
    const int rc2 = gecc_encode_a(&v, dev_A, dev_A_par, stream);
    ctx->ev_n = v.ev_n;
    return rc2;
  }
  ScanQueue q{ctx, (hipStream_t)stream};
  const TileScanJob tj = tile_job(ctx, GECC_MAT_A, dev_A, dev_A_par, nullptr, nullptr, 0, nullptr);
  hipError_t e = ctx->tile_op == GECC_MAT_A && use_tile(ctx, tj) ? q.run_tile(tj, GECC_K_ENCODE_A)
                                                                : q.run(scan_a_over_n(ctx, dev_A, nullptr, dev_A_par, nullptr));
  return hip_rc(e != hipSuccess ? e : q.flush());
}

int gecc_encode_b(gecc_ctx* ctx, const void* dev_B, double* dev_B_par, void* stream) {
  int rc = check_ws(ctx);
  if (rc) return rc;
  if (!dev_B || !dev_B_par) return GECC_ERR_ARG;
  if (!aligned_to(dev_B, elem_size(ctx->p.dtype)) || !aligned_to(dev_B_par, 8)) return GECC_ERR_ALIGN;
  if ((rc = prep(ctx, (hipStream_t)stream))) return rc;
  if (blocked(ctx)) {
    gecc_ctx v = view_b(ctx);
    const int rc2 = gecc_encode_b(&v, dev_B, dev_B_par, stream);
    ctx->ev_n = v.ev_n;
    return rc2;
  }
  ScanQueue q{ctx, (hipStream_t)stream};
  const TileScanJob tj = tile_job(ctx, GECC_MAT_B, dev_B, dev_B_par, nullptr, nullptr, 0, nullptr);
  hipError_t e = ctx->tile_op == GECC_MAT_B && use_tile(ctx, tj) ? q.run_tile(tj, GECC_K_ENCODE_B)
                                                                : q.run(scan_b_over_m(ctx, dev_B, nullptr, dev_B_par, nullptr));
  return hip_rc(e != hipSuccess ? e : q.flush());
}

namespace {

int check_multiply_args(gecc_ctx* ctx, const void* dev_A, const double* dev_A_par, const void* dev_B,
                        const double* dev_B_par, float* dev_C, double* dev_C_par, const gecc_fault* dev_faults,
                        int32_t n_faults) {
  int rc = check_ws(ctx);
  if (rc) return rc;
  if (!dev_A || !dev_A_par || !dev_B || !dev_B_par || !dev_C || !dev_C_par) return GECC_ERR_ARG;
  if (n_faults < 0 || n_faults > GECC_MAX_FAULTS || (n_faults > 0 && !dev_faults)) return GECC_ERR_ARG;
  if (!aligned_to(dev_A, elem_size(ctx->p.dtype)) || !aligned_to(dev_B, elem_size(ctx->p.dtype)) ||
      !aligned_to(dev_C, 4) || !aligned_to(dev_C_par, 8) || !aligned_to(dev_A_par, 8) ||
      !aligned_to(dev_B_par, 8))
    return GECC_ERR_ALIGN;
  return GECC_OK;
}

// The scans that ride (side) and those of them that cannot finish by themselves and go first (alone).
struct Riders { bool on; GemmSide side; const ScanJob* alone[2]; };
// left: null, or what the operand parities have left (the riders' own chunks are then left to the threshold pass)
Riders plan_riders(const gecc_ctx* ctx, const GemmArgs& g, uint32_t* done, const ScanJob* pr, const ScanJob* pc, const Left* left) {
  Riders r{};
  if (gemm_takes_256(g)) return r;
  // (the counters behind those of a k-split product)
  const int64_t tiles = (int64_t)ctx->ntm * ctx->ntn * ctx->p.batch;
  int used = ctx->ksplit > 1 && tiles <= SCAN_DONE_WORDS ? (int)tiles : 0;
  int at = 0;
  const ScanJob* jobs[2] = {pc, pr};
  for (int x = 0; x < 2; ++x) {
    if (!jobs[x]) continue;
    int words = 0;
    if (make_side_job(jobs[x]->s, left ? (x ? left->bp : left->ap) : Parts{}, jobs[x]->rowdot, left ? nullptr : done + used,
                      SCAN_DONE_WORDS - used, r.side.j[at], words)) {
      used += words;
      ++at;
    } else {
      r.side.j[at] = SideJob{};
      r.alone[x] = jobs[x];
    }
  }
  // (the rule counts a row scan by fours of rows, which is how it was measured)
  int64_t scans = ctx->p.batch;
  for (const SideJob& j : r.side.j) scans += j.kind == SIDE_ROW ? (int64_t)((j.s.R + 3) / 4) * j.s.batch : j.nblk;
  r.on = scans_ride(ctx->p, ctx->tile_m, ctx->ksplit, scans, pr && pc);
  return r;
}

// Whether an operand parity in `nchunk` parts is left to its readers beside the product: a column scan reads the
// weights of its own rows, and one workgroup adds all of them up for P_g, about 1 us a round of loads.  Up to 8 rounds
// beside any product, 16 beside one of 2^20 symbols.  Whole calls, bf16, us, finished first -> left (with the scans
// before the product's workgroups; behind them 1200 x 3000 x 1500 takes 66.3):
//   left       2880 x 520 x 2504     59.9 -> 53.1      finished   300 x 6000 x 1000   51.3 -> 52.5   (12 rounds)
//              1200 x 3000 x 1500    80.1 -> 76.7                 1000 x 6000 x 300   51.0 -> 55.2
//              500 x 2000 x 4000 TT  69.4 -> 65.5
bool parts_beside(const gecc_ctx* c, int nchunk) {
  const int at_once = nchunk <= 8 ? 4 : nchunk <= 16 ? 2 : 1;
  const int64_t rounds = (2 * (int64_t)c->p.k + 256 * at_once - 1) / (256 * at_once) * (nchunk <= 16 ? 1 : 2);
  return nchunk <= 32 && rounds <= ((int64_t)c->p.n * c->p.m >= (1 << 20) ? 16 : 8);
}

// S3: the parity blocks pr, pc of C-bar (null: formed already), the data block, the fused syndrome partial
// sums, P_g.  The scans of the parity blocks ride in the product's launch (scans_ride) or go first, on q.
// left: null, or what is left of A_P and B_P; what is then left of P_r and P_c is added to it.
hipError_t product(gecc_ctx* ctx, ScanQueue& q, const ScanJob* pr, const ScanJob* pc, Left* left, const void* dev_A, const double* dev_A_par,
                   const void* dev_B, const double* dev_B_par, float* dev_C, double* dev_C_par, const gecc_fault* dev_faults,
                   int32_t n_faults, hipStream_t st) {
  const gecc_params& p = ctx->p;
  GemmArgs g = gemm_args(ctx, dev_A, dev_B, dev_C);
  g.rowpart = reinterpret_cast<float*>(ctx->ws + ctx->lay.rowpart);
  g.colpart = reinterpret_cast<float*>(ctx->ws + ctx->lay.colpart);
  g.faults = dev_faults;
  g.n_faults = n_faults;
  g.fault_bias = ctx->fault_bias;
  // P_g is formed inside the product kernel, which also resets the decoder state for the
  // fused verification that follows
  g.A_par = dev_A_par; g.B_par = dev_B_par;
  g.pg_out = dev_C_par + 2 * (size_t)p.n + 2 * (size_t)p.m;
  g.pg_stride = 2 * (int64_t)p.n + 2 * (int64_t)p.m + 4;
  g.state = reinterpret_cast<DecodeState*>(ctx->ws + ctx->lay.state);
  hipError_t e;
  Riders r = plan_riders(ctx, g, q.done(), pr, pc, left);
  if (left) {
    if ((e = q.flush()) != hipSuccess) return e;
    // (a row scan, and scans in launches of their own, read their weights finished)
    auto as_parts = [&](const Parts& w, const ScanJob* reader) { return r.on && reader && !reader->rowdot && parts_beside(ctx, w.nchunk); };
    const int64_t k2 = 2 * (int64_t)p.k;
    Stage2Job ja{}, jb{};
    if (!as_parts(left->ap, pc)) { ja = stage2_of(left->ap, const_cast<double*>(dev_A_par), k2, p.k, p.batch); left->ap = Parts{}; }
    if (!as_parts(left->bp, pr)) { jb = stage2_of(left->bp, const_cast<double*>(dev_B_par), k2, p.k, p.batch); left->bp = Parts{}; }
    if ((e = finish_parts(ctx, ja, jb, st)) != hipSuccess) return e;
    if (r.on) {
      r = plan_riders(ctx, g, q.done(), pr, pc, left);
      if (any(left->ap)) { r.side.par = left->ap; r.side.par_out = const_cast<double*>(dev_A_par); }
      else if (any(left->bp)) { r.side.par = left->bp; r.side.par_out = const_cast<double*>(dev_B_par); }
      int at = 0;
      for (int x = 0; x < 2; ++x) {          // (the riders' order: P_c, P_r)
        if (!(x ? pr : pc)) continue;
        const SideJob& sj = r.side.j[at++];
        if (sj.kind == SIDE_COL && sj.gy > 1) (x ? left->pr : left->pc) = Parts{sj.s.scratch, nullptr, sj.gy, 0};
      }
      return timed_gemm(ctx, g, &r.side, st);
    }
    if (pr && pc && pr->rowdot == pc->rowdot && may_pair(*pr, *pc)) {
      const ScanArgs s[2] = {pr->s, pc->s};
      const bool row[2] = {pr->rowdot, pc->rowdot};
      Parts out[2] = {};
      Timed t(ctx, GECC_K_PARITY_RC, st);
      if ((e = t.done(launch_scan_pair(s, row, out, st))) != hipSuccess) return e;
      left->pr = out[0];
      left->pc = out[1];
    } else if (pr && pc) {
      // (a column scan, then a row scan that carries its second stage: in one launch they are no faster, bf16 4096^3 20.9 us and 23.8)
      if ((e = q.run(pr->rowdot ? *pc : *pr)) != hipSuccess || (e = q.run(pr->rowdot ? *pr : *pc)) != hipSuccess ||
          (e = q.flush()) != hipSuccess)
        return e;
    } else if (pr || pc) {
      if ((e = q.run(pr ? *pr : *pc)) != hipSuccess) return e;
      (pr ? left->pr : left->pc) = chunks_of(q.pending);
      q.pending = Stage2Job{};
    }
    // (of 64 chunks the threshold pass takes 3 us longer, a launch 5)
    auto late = [&](const Parts& w) { return w.nchunk > 64; };
    const Stage2Job jr = late(left->pr) ? stage2_of(left->pr, dev_C_par, g.pg_stride, p.n, p.batch) : Stage2Job{};
    const Stage2Job jc = late(left->pc) ? stage2_of(left->pc, dev_C_par + 2 * (size_t)p.n, g.pg_stride, p.m, p.batch) : Stage2Job{};
    if ((e = finish_parts(ctx, jr, jc, st)) != hipSuccess) return e;
    if (jr.valid) left->pr = Parts{};
    if (jc.valid) left->pc = Parts{};
    return timed_gemm(ctx, g, nullptr, st);
  }
  if (!r.on) {
    // (a column scan goes before a row scan, which can carry its second stage; two row scans: P_c first, which
    // can carry what the encoding of B left)
    const ScanJob* first = pr && pc && pr->rowdot ? pc : pr;
    const ScanJob* then = first == pc ? pr : pc;
    if (first && (e = q.run(*first)) != hipSuccess) return e;
    if (then && (e = q.run(*then)) != hipSuccess) return e;
    if ((e = q.flush()) != hipSuccess) return e;
    return timed_gemm(ctx, g, nullptr, st);
  }
  for (const ScanJob* j : r.alone)
    if (j && (e = q.run(*j)) != hipSuccess) return e;
  if ((e = q.flush()) != hipSuccess) return e;
  return timed_gemm(ctx, g, &r.side, st);
}

// Blocked mode: the plan of a narrow product (parity columns or rows of all blocks against a whole operand).
// The 256 x 256-tile kernel where it is the faster one and takes these operands, by its launcher's own test; else
// gemm_tile, whose partial tiles go where the main product's partial sums will go afterwards (as many k ranges
// as fit there in the tile that runs).
void narrow_plan(gecc_ctx* ctx, GemmArgs& g) {
  const gecc_params& p = ctx->p;
  g.rowpart = nullptr; g.colpart = nullptr; g.faults = nullptr; g.n_faults = 0;
  ProductPlan pl = {128, 1, p.dtype == GECC_BF16 && fast_may_pay(g.n, g.k, g.m, 1), false};
  auto take = [&] {
    g.tile_m = g.tile_n = pl.tile;
    g.ntm = (g.n + pl.tile - 1) / pl.tile;
    g.ntn = (g.m + pl.tile - 1) / pl.tile;
    g.fast = pl.fast;
    g.fold = pl.fold;
  };
  take();
  if (!gemm_takes_256(g)) {
    pl = plan_tiles(p.dtype, g.n, g.k, g.m, 1, true);
    take();
  }
  g.split_part = reinterpret_cast<float*>(ctx->ws + ctx->lay.rowpart);
  g.split_bytes = ctx->lay.synd - ctx->lay.rowpart;
  g.split_done = reinterpret_cast<uint32_t*>(ctx->ws + ctx->lay.done);
  const size_t one_range = (size_t)g.ntm * g.ntn * pl.tile * pl.tile * sizeof(float);
  while (pl.ksplit > 1 && pl.ksplit * one_range > g.split_bytes) --pl.ksplit;
  g.ksplit = pl.ksplit;
}

// Blocked mode, S3: the parity blocks of every block of C-bar on the matrix units -- the parity
// columns of all column blocks of B-bar, split into operand-type pieces, form one narrow operand
// W_B (and the parity rows of all row blocks of A-bar one flat operand W_A); A W_B^T and W_A B are
// two plain products of the same kernels -- then the data block with the fused partial sums.
hipError_t blocked_multiply(gecc_ctx* ctx, const void* dev_A, const double* dev_A_par, const void* dev_B,
                            const double* dev_B_par, float* dev_C, double* dev_C_par, const gecc_fault* dev_faults,
                            int32_t n_faults, hipStream_t st) {
  const gecc_params& p = ctx->p;
  void* WA = ctx->ws + ctx->lay.w_a;
  void* WB = ctx->ws + ctx->lay.w_b;
  float* side_r = reinterpret_cast<float*>(ctx->ws + ctx->lay.side_r);
  float* side_c = reinterpret_cast<float*>(ctx->ws + ctx->lay.side_c);
  hipError_t e;
  {
    Timed t(ctx, GECC_K_PARITY_R, st);
    if ((e = launch_split_parities(dev_B_par, WB, p.dtype, ctx->nbj, p.k, ctx->pieces, ctx->w_cols_b, st)) != hipSuccess) return e;
    GemmArgs g = gemm_args(ctx, dev_A, WB, side_r);
    g.trans_b = 1; g.m = ctx->w_cols_b; g.ldb = p.k; g.ldc = ctx->w_cols_b;
    narrow_plan(ctx, g);
    if ((e = t.done(launch_gemm(g, nullptr, st))) != hipSuccess) return e;
  }
  {
    Timed t(ctx, GECC_K_PARITY_C, st);
    if ((e = launch_split_parities(dev_A_par, WA, p.dtype, ctx->nbi, p.k, ctx->pieces, ctx->w_cols_a, st)) != hipSuccess) return e;
    GemmArgs g = gemm_args(ctx, WA, dev_B, side_c);
    g.trans_a = 0; g.n = ctx->w_cols_a; g.lda = p.k; g.ldc = p.m;
    narrow_plan(ctx, g);
    if ((e = t.done(launch_gemm(g, nullptr, st))) != hipSuccess) return e;
  }
  {
    BlockedParityArgs b{};
    b.nb = p.block_n; b.mb = p.block_m; b.k = p.k; b.nbi = ctx->nbi; b.nbj = ctx->nbj; b.pieces = ctx->pieces;
    b.side_r = side_r; b.ld_r = ctx->w_cols_b; b.side_c = side_c; b.ld_c = p.m;
    b.A_par = dev_A_par; b.B_par = dev_B_par; b.C_par = dev_C_par;
    b.state = reinterpret_cast<DecodeState*>(ctx->ws + ctx->lay.state);
    b.itemmax = reinterpret_cast<double*>(ctx->ws + ctx->lay.blockmax) + (size_t)((p.n + p.m + 63) / 64) * 4;
    b.gate_word = reinterpret_cast<int32_t*>(ctx->ws + ctx->lay.gate);
    Timed t(ctx, GECC_K_DECODE, st);
    if ((e = t.done(launch_blocked_parities(b, st))) != hipSuccess) return e;
  }
  GemmArgs g = gemm_args(ctx, dev_A, dev_B, dev_C);
  g.rowpart = reinterpret_cast<float*>(ctx->ws + ctx->lay.rowpart);
  g.colpart = reinterpret_cast<float*>(ctx->ws + ctx->lay.colpart);
  g.faults = dev_faults;
  g.n_faults = n_faults;
  g.pg_out = nullptr;      // P_g of every block and the resets are done above
  g.state = nullptr;
  return timed_gemm(ctx, g, nullptr, st);
}

}  // namespace

int gecc_multiply(gecc_ctx* ctx, const void* dev_A, const double* dev_A_par, const void* dev_B,
                  const double* dev_B_par, float* dev_C, double* dev_C_par,
                  const gecc_fault* dev_faults, int32_t n_faults, void* stream) {
  int rc = check_multiply_args(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_faults, n_faults);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  if ((rc = prep(ctx, st))) return rc;
  if (blocked(ctx)) return hip_rc(blocked_multiply(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_faults, n_faults, st));
  ScanQueue q{ctx, st};
  const gecc_params& p = ctx->p;
  const int64_t rec = 2 * (int64_t)p.n + 2 * (int64_t)p.m + 4;
  const ScanJob pr = scan_a_over_k(ctx, dev_A, dev_B_par, dev_C_par, rec);
  const ScanJob pc = scan_b_over_k(ctx, dev_B, dev_A_par, dev_C_par + 2 * (size_t)p.n, rec);
  return hip_rc(product(ctx, q, &pr, &pc, nullptr, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_faults, n_faults, st));
}

namespace {

// S4 + S5.  summary = 0 leaves the first report to the decoder's first pass (saves a launch).  left: what is
// left of P_r and P_c, which dev_C_par then gets here.
int verify_impl(gecc_ctx* ctx, const float* dev_C, const double* dev_C_par, gecc_report* dev_report,
                int32_t fused, int summary, const Left& left, hipStream_t st) {
  DecodeArgs d = decode_args(ctx, nullptr, nullptr, nullptr, nullptr, const_cast<float*>(dev_C),
                             const_cast<double*>(dev_C_par), dev_report);
  hipError_t e;
  if (!fused && blocked(ctx)) return GECC_ERR_ARG;   // (blocked mode verifies from the product's own partial sums)
  if (!fused) {
    // (the fused path had its state reset by gecc_multiply)
    const gecc_params& p = ctx->p;
    PartialArgs pa{};
    pa.C = dev_C; pa.n = p.n; pa.m = p.m; pa.batch = p.batch; pa.ldc = p.ldc; pa.sc = p.stride_c;
    pa.rowpart = const_cast<float*>(d.rowpart); pa.colpart = const_cast<float*>(d.colpart);
    pa.tile_m = ctx->tile_m; pa.tile_n = ctx->tile_n; pa.ntm = ctx->ntm; pa.ntn = ctx->ntn;
    pa.rp_ld = ctx->rp_ld; pa.cp_ld = ctx->cp_ld;
    pa.state = d.state;
    Timed t(ctx, GECC_K_PARTIALS, st);
    if ((e = t.done(launch_partials(pa, st))) != hipSuccess) return hip_rc(e);
  }
  {
    Timed t(ctx, GECC_K_THRESHOLD, st);
    e = blocked(ctx) ? launch_threshold_blocked(d, ctx->p.n, ctx->p.m, st) : launch_threshold(d, left.pr, left.pc, st);
    if ((e = t.done(e)) != hipSuccess) return hip_rc(e);
  }
  if (!summary) return GECC_OK;
  Timed t(ctx, GECC_K_DECODE, st);
  return hip_rc(t.done(launch_summarize(d, st)));
}

// S6 + S7.  with_summary = 1: the first decoder pass also writes the first report.
int correct_impl(gecc_ctx* ctx, void* dev_A, const double* dev_A_par, void* dev_B, const double* dev_B_par,
                 float* dev_C, double* dev_C_par, gecc_report* dev_report, int with_summary, hipStream_t st) {
  DecodeArgs d = decode_args(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_report);
  const int32_t* gate = &d.state->phase;
  // (the repair comes when no scan has anything left in its scratch, 16 bytes a line at the least)
  const RepairScratch scratch{ctx->ws + ctx->lay.scan_a, ctx->lay.ksplit - ctx->lay.scan_a,
                              reinterpret_cast<uint32_t*>(ctx->ws + ctx->lay.done), SCAN_DONE_WORDS};
  hipError_t e;
  // operand audit: re-form the parities of A and B as the product read them
  // (an encoding made by the tile scan is re-formed by the tile scan: same sums, same order)
  ScanQueue q{ctx, st};
  const ScanJob ja = scan_a_over_n(ctx, dev_A, nullptr, const_cast<double*>(d.audit_a), gate);
  const ScanJob jb = scan_b_over_m(ctx, dev_B, nullptr, const_cast<double*>(d.audit_b), gate);
  const bool t_is_a = ctx->tile_op == GECC_MAT_A;
  const TileScanJob tj = tile_job(ctx, ctx->tile_op, t_is_a ? dev_A : dev_B,
                                  const_cast<double*>(t_is_a ? d.audit_a : d.audit_b), nullptr, nullptr, 0, gate);
  const bool tile = use_tile(ctx, tj);
  if (!blocked(ctx)) {
    // both and Section V step 2 in one launch, where every column reduction of the audits can finish by itself
    PairArgs pair;
    int words = 0;
    if (make_audit_pair({tile && t_is_a ? 2 : (ja.rowdot ? 0 : 1), ja.s, tj}, {tile && !t_is_a ? 2 : (jb.rowdot ? 0 : 1), jb.s, tj},
                        q.done(), pair, words) && words + ctx->p.batch <= SCAN_DONE_WORDS) {
      {
        Timed td(ctx, GECC_K_DECODE, st), ta(ctx, GECC_K_AUDIT_AB, st, td.on);
        if ((e = ta.done(td.done(launch_finish(d, pair, q.done() + words, with_summary, st)))) != hipSuccess) return hip_rc(e);
      }
      Timed t(ctx, GECC_K_REPAIR, st);
      return hip_rc(t.done(launch_repair(d, scratch, st)));
    }
  }
  // Section V step 2 on the flagged lines; on failure the phase becomes PH_AUDIT
  {
    Timed t(ctx, GECC_K_DECODE, st);
    if ((e = t.done(launch_decode_c(d, with_summary, st))) != hipSuccess) return hip_rc(e);
  }
  if (blocked(ctx)) {
    // the audits of all row blocks of A and all column blocks of B, gated on one word that the
    // first block in need sets; then the repair in three launches (see launch_repair_blocked)
    gecc_ctx va = view_a(ctx), vb = view_b(ctx);
    const int32_t* gw = d.gate_word;
    auto audit = [&](gecc_ctx& v, int op, const void* X, double* out, const ScanJob& old_job, int kind) -> hipError_t {
      ScanQueue qv{&v, st};
      TileScanJob tj = tile_job(&v, op, X, out, nullptr, nullptr, 0, gw);
      tj.gate_stride = 0;
      hipError_t ee;
      if (use_tile(&v, tj)) ee = qv.run_tile(tj, kind);
      else { ScanJob j = old_job; j.s.gate_stride = 0; ee = qv.run(j); }
      if (ee == hipSuccess) { qv.pending.gate_stride = 0; ee = qv.flush(); }
      ctx->ev_n = v.ev_n;
      return ee;
    };
    va.ev_n = ctx->ev_n;
    if ((e = audit(va, GECC_MAT_A, dev_A, const_cast<double*>(d.audit_a),
                   scan_a_over_n(&va, dev_A, nullptr, const_cast<double*>(d.audit_a), gw), GECC_K_AUDIT_A)) != hipSuccess)
      return hip_rc(e);
    vb.ev_n = ctx->ev_n;
    if ((e = audit(vb, GECC_MAT_B, dev_B, const_cast<double*>(d.audit_b),
                   scan_b_over_m(&vb, dev_B, nullptr, const_cast<double*>(d.audit_b), gw), GECC_K_AUDIT_B)) != hipSuccess)
      return hip_rc(e);
    Timed t(ctx, GECC_K_REPAIR, st);
    return hip_rc(t.done(launch_repair_blocked(d, scratch, ctx->nbi, st)));
  }
  // (the coldot of the two first, so that the rowdot carries its second stage)
  if (tile) {
    if ((e = q.run_tile(tj, t_is_a ? GECC_K_AUDIT_A : GECC_K_AUDIT_B)) != hipSuccess) return hip_rc(e);
    if ((e = q.run(t_is_a ? jb : ja)) != hipSuccess) return hip_rc(e);
  } else {
    const bool b_first = ja.rowdot && !jb.rowdot;
    if ((e = q.run(b_first ? jb : ja)) != hipSuccess) return hip_rc(e);
    if ((e = q.run(b_first ? ja : jb)) != hipSuccess) return hip_rc(e);
  }
  if ((e = q.flush()) != hipSuccess) return hip_rc(e);
  // parity differences, operand patches, rank-one repair of C-bar with the residual syndromes
  // kept up to date, then Section V once more -- all in one workgroup per batch item
  Timed t(ctx, GECC_K_REPAIR, st);
  return hip_rc(t.done(launch_repair(d, scratch, st)));
}

}  // namespace

namespace {

// S1-S3 as one chain of scans.  The order of the four scans depends on how the operands are stored
// (which of them are rowdots) and on what reads what: P_r needs B_P, P_c needs A_P.  left: what the threshold pass
// that follows has to add up of P_r and P_c.
int encode_and_multiply(gecc_ctx* ctx, void* dev_A, void* dev_B, float* dev_C, double* dev_A_par,
                        double* dev_B_par, double* dev_C_par, const gecc_fault* dev_faults, int32_t n_faults, Left& left,
                        hipStream_t st) {
  int rc = check_multiply_args(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_faults, n_faults);
  if (rc) return rc;
  if ((rc = prep(ctx, st))) return rc;
  if (blocked(ctx)) {
    if ((rc = gecc_encode_a(ctx, dev_A, dev_A_par, st)) || (rc = gecc_encode_b(ctx, dev_B, dev_B_par, st))) return rc;
    return hip_rc(blocked_multiply(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_faults, n_faults, st));
  }
  const gecc_params& p = ctx->p;
  const int64_t rec = 2 * (int64_t)p.n + 2 * (int64_t)p.m + 4;
  const ScanJob ea = scan_a_over_n(ctx, dev_A, nullptr, dev_A_par, nullptr);
  const ScanJob eb = scan_b_over_m(ctx, dev_B, nullptr, dev_B_par, nullptr);
  const ScanJob pr = scan_a_over_k(ctx, dev_A, dev_B_par, dev_C_par, rec);
  const ScanJob pc = scan_b_over_k(ctx, dev_B, dev_A_par, dev_C_par + 2 * (size_t)p.n, rec);
  ScanQueue q{ctx, st};
  hipError_t e;
  const bool t_is_a = ctx->tile_op == GECC_MAT_A;
  const TileScanJob tj = t_is_a ? tile_job(ctx, GECC_MAT_A, dev_A, dev_A_par, dev_B_par, dev_C_par, rec, nullptr)
                                : tile_job(ctx, GECC_MAT_B, dev_B, dev_B_par, dev_A_par, dev_C_par + 2 * (size_t)p.n, rec, nullptr);
  if (use_tile(ctx, tj)) {
    // the larger operand in one pass: its encoding and its parity block of C-bar together.  That
    // pass reads the other operand's encoding, and the other operand's parity block reads this one's.
    if ((e = q.run(t_is_a ? eb : ea)) != hipSuccess) return hip_rc(e);
    if ((e = q.run_tile(tj, t_is_a ? GECC_K_TILE_A : GECC_K_TILE_B)) != hipSuccess) return hip_rc(e);
    // the other operand's parity block: a row scan over few, long rows (too few workgroups for the
    // row kernel) goes through the tile scan's row part instead
    const ScanJob& po = t_is_a ? pc : pr;
    const TileScanJob to = t_is_a ? tile_job(ctx, GECC_MAT_B, dev_B, nullptr, dev_A_par, dev_C_par + 2 * (size_t)p.n, rec, nullptr)
                                  : tile_job(ctx, GECC_MAT_A, dev_A, nullptr, dev_B_par, dev_C_par, rec, nullptr);
    const bool long_rows = po.rowdot && to.row_on && !to.col_on && po.s.R < 8192 && po.s.Cc >= 4096 && tile_scan_ok(to);
    if (long_rows && (e = q.run_tile(to, po.kind)) != hipSuccess) return hip_rc(e);
    // (P_c reads A_P, P_r reads B_P: what the tile scan left pending comes first)
    if (long_rows) {
      (t_is_a ? left.pc : left.pr) = segs_of(q.pending);
      q.pending = Stage2Job{};
    }
    return hip_rc(product(ctx, q, long_rows || t_is_a ? nullptr : &pr, long_rows || !t_is_a ? nullptr : &pc, &left, dev_A, dev_A_par,
                          dev_B, dev_B_par, dev_C, dev_C_par, dev_faults, n_faults, st));
  }
  // The two encodings in one launch.  Where the sums of a column scan have to be finished before they are read, it and then
  // a row scan that carries its second stage are no slower (bf16 4096^3 16.6 us, in one launch 14.3 and the second stage 4.8).
  // (a column scan goes before a row scan)
  const ScanJob& first = ea.rowdot && !eb.rowdot ? eb : ea;
  const ScanJob& then = &first == &ea ? eb : ea;
  auto late = [&] {
    return parts_beside(ctx, (first.s.R + SCAN_CHUNK_ROWS - 1) / SCAN_CHUNK_ROWS) &&
           plan_riders(ctx, gemm_args(ctx, dev_A, dev_B, dev_C), q.done(), &pr, &pc, &left).on;
  };
  if (!may_pair(ea, eb) || (ea.rowdot != eb.rowdot && !late())) {
    if ((e = q.run(first)) != hipSuccess || (e = q.run(then)) != hipSuccess) return hip_rc(e);
  } else {
    const ScanArgs s[2] = {ea.s, eb.s};
    const bool row[2] = {ea.rowdot, eb.rowdot};
    Parts out[2] = {};
    Timed t(ctx, GECC_K_ENCODE_AB, st);
    if ((e = t.done(launch_scan_pair(s, row, out, st))) != hipSuccess) return hip_rc(e);
    left.ap = out[0];
    left.bp = out[1];
  }
  return hip_rc(product(ctx, q, &pr, &pc, &left, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_faults, n_faults, st));
}

}  // namespace

int gecc_verify(gecc_ctx* ctx, const float* dev_C, const double* dev_C_par, gecc_report* dev_report,
                int32_t fused, void* stream) {
  int rc = check_ws(ctx);
  if (rc) return rc;
  if (!dev_C_par || !dev_report || (!fused && !dev_C)) return GECC_ERR_ARG;
  return verify_impl(ctx, dev_C, dev_C_par, dev_report, fused, 1, Left{}, (hipStream_t)stream);
}

int gecc_correct(gecc_ctx* ctx, void* dev_A, const double* dev_A_par, void* dev_B,
                 const double* dev_B_par, float* dev_C, double* dev_C_par, gecc_report* dev_report,
                 void* stream) {
  int rc = check_ws(ctx);
  if (rc) return rc;
  if (!dev_A || !dev_A_par || !dev_B || !dev_B_par || !dev_C || !dev_C_par || !dev_report)
    return GECC_ERR_ARG;
  if ((rc = prep(ctx, (hipStream_t)stream))) return rc;
  return correct_impl(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_report, 0,
                      (hipStream_t)stream);
}

int gecc_protected_gemm(gecc_ctx* ctx, void* dev_A, void* dev_B, float* dev_C, double* dev_A_par,
                        double* dev_B_par, double* dev_C_par, gecc_report* dev_report, void* stream) {
  int rc;
  if (!dev_report) return GECC_ERR_ARG;
  Left left{};
  if ((rc = encode_and_multiply(ctx, dev_A, dev_B, dev_C, dev_A_par, dev_B_par, dev_C_par, nullptr, 0, left,
                                (hipStream_t)stream)))
    return rc;
  if ((rc = verify_impl(ctx, dev_C, dev_C_par, dev_report, 1, 0, left, (hipStream_t)stream))) return rc;
  return correct_impl(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_report, 1,
                      (hipStream_t)stream);
}

int gecc_protected_gemm_retry(gecc_ctx* ctx, void* dev_A, void* dev_B, float* dev_C, double* dev_A_par,
                              double* dev_B_par, double* dev_C_par, gecc_report* dev_report,
                              gecc_report* host_report, int32_t max_retries, const gecc_fault* dev_faults,
                              int32_t n_faults, int32_t* attempts, void* stream) {
  int rc;
  if (!dev_report || !host_report || max_retries < 0) return GECC_ERR_ARG;
  if (attempts) *attempts = 0;
  for (int32_t a = 0; a <= max_retries; ++a) {
    // the planted faults are transient: they strike the first product only
    Left left{};
    if (a == 0)
      rc = encode_and_multiply(ctx, dev_A, dev_B, dev_C, dev_A_par, dev_B_par, dev_C_par, dev_faults, n_faults, left,
                               (hipStream_t)stream);
    else
      rc = gecc_multiply(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, nullptr, 0, stream);
    if (rc) return rc;
    if ((rc = verify_impl(ctx, dev_C, dev_C_par, dev_report, 1, 0, left, (hipStream_t)stream))) return rc;
    if ((rc = correct_impl(ctx, dev_A, dev_A_par, dev_B, dev_B_par, dev_C, dev_C_par, dev_report, 1,
                           (hipStream_t)stream)))
      return rc;
    if ((rc = gecc_report_to_host(ctx, dev_report, host_report, items_of(ctx), stream))) return rc;
    if (attempts) *attempts = a + 1;
    bool again = false;
    for (int32_t b = 0; b < items_of(ctx); ++b) again = again || host_report[b].status == GECC_UNCORRECTABLE;
    if (!again) break;
  }
  return GECC_OK;
}

namespace {

// Scratch of gecc_protected_gemm_static: one array per GPU, placed by the code-object loader, held
// until the process ends.  In host code the name is only a handle for hipGetSymbolAddress; the
// device address it yields (one per device) is what kernels and copies get.
static __device__ __align__(256) unsigned char scratch[GECC_STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mutex;
char* scratch_addr[MAX_DEVICES] = {};
bool scratch_cleared[MAX_DEVICES] = {};

// device address of `scratch` on the current device, looked up once per device; *first: nobody has
// used the array on this device yet
int static_scratch(char** out, bool* first, int* device) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return GECC_ERR_HIP;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_addr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GECC_ERR_HIP;
    scratch_addr[dev] = static_cast<char*>(p);
  }
  *out = scratch_addr[dev];
  *first = !scratch_cleared[dev];
  *device = dev;
  return GECC_OK;
}

}  // namespace

int gecc_protected_gemm_static(gecc_ctx* ctx, void* dev_A, void* dev_B, float* dev_C, double* dev_A_par,
                               double* dev_B_par, double* dev_C_par, gecc_report* dev_report,
                               void* stream) {
  if (!ctx || !dev_A || !dev_B || !dev_C || !dev_A_par || !dev_B_par || !dev_C_par || !dev_report)
    return GECC_ERR_ARG;
  if (ctx->lay.total > (size_t)GECC_STATIC_SCRATCH_BYTES) return GECC_ERR_SCRATCH;
  char* ws = nullptr;
  bool first = false;
  int dev = 0;
  int rc = static_scratch(&ws, &first, &dev);
  if (rc) return rc;
  // the context's own workspace (if any) is left alone: this call runs on the static one
  char* const keep_ws = ctx->ws;
  const size_t keep_bytes = ctx->ws_bytes;
  char* const keep_zeroed = ctx->ws_zeroed;
  ctx->ws = ws;
  ctx->ws_bytes = GECC_STATIC_SCRATCH_BYTES;
  // every launch leaves the counters at the front of the array at zero, whichever context used it
  // before; the first call on a device clears them (a kernel launch, not an allocation)
  ctx->ws_zeroed = first ? nullptr : ws;
  rc = gecc_protected_gemm(ctx, dev_A, dev_B, dev_C, dev_A_par, dev_B_par, dev_C_par, dev_report, stream);
  ctx->ws = keep_ws;
  ctx->ws_bytes = keep_bytes;
  ctx->ws_zeroed = keep_zeroed;
  if (rc == GECC_OK && first) {
    std::lock_guard<std::mutex> lock(scratch_mutex);
    scratch_cleared[dev] = true;
  }
  return rc;
}

namespace {
int panel_step(const gecc_ctx* ctx, int panels) {
  const int per = (ctx->p.k + panels - 1) / panels;
  return (per + 63) / 64 * 64;
}
}  // namespace

int32_t gecc_panel_count(const gecc_ctx* ctx, int32_t panels) {
  if (!ctx || panels < 1) return 0;
  const int step = panel_step(ctx, panels);
  return (ctx->p.k + step - 1) / step;
}

int gecc_protected_gemm_panels(gecc_ctx* ctx, void* dev_A, void* dev_B, float* dev_C, float* dev_C_partial,
                               double* dev_A_par, double* dev_B_par, double* dev_C_par,
                               gecc_report* dev_report, int32_t panels, const gecc_fault* dev_faults,
                               int32_t n_faults, void* stream) {
  int rc = check_ws(ctx);
  if (rc) return rc;
  if (panels < 1 || ctx->p.batch != 1 || !dev_report || blocked(ctx)) return GECC_ERR_ARG;
  const int P = gecc_panel_count(ctx, panels), step = panel_step(ctx, panels);
  if (P > 1 && !dev_C_partial) return GECC_ERR_ARG;
  if (dev_C_partial && !aligned_to(dev_C_partial, 4)) return GECC_ERR_ALIGN;
  // one context per panel: the same product with k_g terms (host objects, rebuilt when the panel count changes)
  if (ctx->n_panel != P || !ctx->panel || ctx->panel[0]->p.k != (P == 1 ? ctx->p.k : step)) {
    drop_panels(ctx);
    ctx->panel = new (std::nothrow) gecc_ctx*[P];
    if (!ctx->panel) return GECC_ERR_ARG;
    for (int g = 0; g < P; ++g) {
      gecc_params q = ctx->p;
      const int k0 = g * step;
      q.k = ctx->p.k - k0 < step ? ctx->p.k - k0 : step;
      const double f = (double)q.k / (double)ctx->p.k;
      q.tau_r1 *= f; q.tau_r2 *= f; q.tau_q1 *= f; q.tau_q2 *= f;
      gecc_ctx* child = nullptr;
      rc = gecc_create(&child, &q);
      // (a panel may plan more workgroups per tile than the whole product, or another tile)
      if (!rc && child->lay.total > ctx->lay.total) plan_product(child, true);
      if (!rc && child->lay.total > ctx->lay.total) { child->ksplit = 1; make_layout(child); }
      if (rc || child->lay.total > ctx->lay.total) {
        if (child) gecc_destroy(child);
        ctx->n_panel = g;
        drop_panels(ctx);
        return rc ? rc : GECC_ERR_WORKSPACE;
      }
      child->cu_hint = ctx->cu_hint;
      ctx->panel[g] = child;
      ctx->n_panel = g + 1;
    }
  }
  hipStream_t st = (hipStream_t)stream;
  if ((rc = prep(ctx, st))) return rc;
  const gecc_params& p = ctx->p;
  const size_t esz = elem_size(p.dtype);
  const int64_t rec = 2 * (int64_t)p.n + 2 * (int64_t)p.m + 4;
  for (int g = 0; g < P; ++g) {
    gecc_ctx* c = ctx->panel[g];
    c->ws = ctx->ws; c->ws_bytes = ctx->ws_bytes; c->ws_zeroed = ctx->ws_zeroed;
    c->ev = ctx->ev; c->ev_kind = ctx->ev_kind; c->ev_mask = ctx->ev_mask; c->ev_cap = ctx->ev_cap; c->ev_n = ctx->ev_n;
    const int64_t k0 = (int64_t)g * step;
    char* Ag = static_cast<char*>(dev_A) + (p.trans_a ? k0 * p.lda : k0) * (int64_t)esz;
    char* Bg = static_cast<char*>(dev_B) + (p.trans_b ? k0 : k0 * p.ldb) * (int64_t)esz;
    float* Cg = g == 0 ? dev_C : dev_C_partial;
    double* Apg = dev_A_par + 2 * k0;
    double* Bpg = dev_B_par + 2 * k0;
    double* Cpg = dev_C_par + g * rec;
    c->fault_bias = g;
    Left left{};
    rc = encode_and_multiply(c, Ag, Bg, Cg, Apg, Bpg, Cpg, dev_faults, n_faults, left, st);
    if (!rc) rc = verify_impl(c, Cg, Cpg, dev_report + g, 1, 0, left, st);
    if (!rc) rc = correct_impl(c, Ag, Apg, Bg, Bpg, Cg, Cpg, dev_report + g, 1, st);
    if (!rc && g > 0) rc = hip_rc(launch_accumulate(dev_C, dev_C_partial, p.n, p.m, p.ldc, st));
    ctx->ev_n = c->ev_n;
    c->ev = nullptr; c->ev_kind = nullptr; c->ev_cap = 0; c->ev_n = 0;     // the records stay the parent's
    if (rc) return rc;
  }
  return GECC_OK;
}

int gecc_plain_gemm(gecc_ctx* ctx, const void* dev_A, const void* dev_B, float* dev_C, void* stream) {
  if (!ctx || !dev_A || !dev_B || !dev_C) return GECC_ERR_ARG;
  if (!aligned_to(dev_A, elem_size(ctx->p.dtype)) || !aligned_to(dev_B, elem_size(ctx->p.dtype)) ||
      !aligned_to(dev_C, 4))
    return GECC_ERR_ALIGN;
  GemmArgs g = gemm_args(ctx, dev_A, dev_B, dev_C);
  g.rowpart = nullptr; g.colpart = nullptr; g.faults = nullptr; g.n_faults = 0;
  if (ctx->fast_plain && !ctx->fast) {
    // (there are no partial sums to go by the plan's tiles: the other kernel takes the operands in its own, if it takes them)
    GemmArgs f = g;
    f.fast = true;
    f.tile_m = f.tile_n = 128;
    f.ntm = (g.n + 127) / 128;
    f.ntn = (g.m + 127) / 128;
    f.ksplit = 0;
    if (gemm_takes_256(f)) g = f;
  }
  if (g.ksplit > 1 && !gemm_takes_256(g)) {
    const int rc = prep(ctx, (hipStream_t)stream);
    if (rc) return rc;
  }
  return hip_rc(timed_gemm(ctx, g, nullptr, (hipStream_t)stream));
}

int gecc_report_to_host(gecc_ctx* ctx, const gecc_report* dev_report, gecc_report* host_report,
                        int32_t count, void* stream) {
  if (!ctx || !dev_report || !host_report || count < 1) return GECC_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = hipMemcpyAsync(host_report, dev_report, sizeof(gecc_report) * (size_t)count,
                                hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return GECC_ERR_HIP;
  return hip_rc(hipStreamSynchronize(st));
}

int gecc_syndromes_to_host(gecc_ctx* ctx, double* host_syndromes, void* stream) {
  int rc = check_ws(ctx);
  if (rc) return rc;
  if (!host_syndromes) return GECC_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  const size_t bytes = blocked(ctx) ? ((size_t)ctx->nbj * 2 * ctx->p.n + (size_t)ctx->nbi * 2 * ctx->p.m) * sizeof(double)
                                    : (size_t)ctx->p.batch * (2 * (size_t)ctx->p.n + 2 * (size_t)ctx->p.m) * sizeof(double);
  hipError_t e = hipMemcpyAsync(host_syndromes, ctx->ws + ctx->lay.synd, bytes, hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return GECC_ERR_HIP;
  return hip_rc(hipStreamSynchronize(st));
}

const char* gecc_strerror(int code) {
  switch (code) {
    case GECC_OK: return "ok";
    case GECC_ERR_ARG: return "invalid argument (null pointer, size, enum or leading dimension)";
    case GECC_ERR_WORKSPACE: return "workspace missing or too small";
    case GECC_ERR_HIP: return "HIP runtime error";
    case GECC_ERR_ALIGN: return "pointer or leading dimension breaks the alignment rule";
    case GECC_ERR_SCRATCH: return "problem needs more scratch than the library's static buffer holds "
                                  "(GECC_STATIC_SCRATCH_BYTES); use gecc_set_workspace and gecc_protected_gemm";
    default: return "unknown error code";
  }
}

}  // extern "C"
