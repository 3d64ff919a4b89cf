// Rules of the dispatch that are pure functions of sizes and of the device's compute units.  No HIP in here.
#pragma once
#include <algorithm>
#include <cstddef>

namespace ppll {

struct ProductShape { int M, N, K; };

// ---- A set of weight-gradient products C_j[M,N] = A_j^T B_j, reductions over K (batch x tokens) rows, in one launch
constexpr int WG_EDGE = 128, WG_WIDE = 256, WG_STEP = 64;      // output tiles of 128 x 128 or 128 x 256; k of a step of the former
struct WeightGradPlan {
  bool wide;         // tiles of 128 x 256, every one whole
  // else, with cuts > 1, tiles of 128 x 128, some divided along k: the products with a long reduction come first, their tiles
  // [0, whole_tiles) run whole, [whole_tiles, long_tiles) in `cuts` parts each, the tiles of the others whole at the end
  int cuts, long_tiles, whole_tiles, tiles;
  int long_steps;    // steps from which a reduction counts as long
};

inline int wg_steps(int K) { return (K + WG_STEP - 1) / WG_STEP; }
inline long wg_tiles(const ProductShape& p, int width) { return (long)((p.M + WG_EDGE - 1) / WG_EDGE) * ((p.N + width - 1) / width); }

// Whether a set of products runs on 128 x 256 tiles.  Per k a tile takes 1.58 times as long as one of 128 x 128 (two workgroups
// to a unit either way), so the padded tiles decide: width 768 has none, width 384 (1.5 tiles) loses.  Without a workspace the
// launch runs beside other work, which fills what it leaves idle.  With one, the alternative is the divided launch, whose
// rounds are full.
inline bool wg_on_wide_tiles(const ProductShape* p, int n, bool workspace, int units) {
  double narrow = 0.0, wide = 0.0;
  long tiles = 0;
  for (int j = 0; j < n; ++j) {
    narrow += (double)wg_tiles(p[j], WG_EDGE) * p[j].K;
    wide += 1.58 * wg_tiles(p[j], WG_WIDE) * p[j].K;
    tiles += wg_tiles(p[j], WG_WIDE);
  }
  if (units < 8 || tiles < units / 2) return false;
  if (workspace) {
    const long full = tiles / (2L * units), rest = tiles % (2L * units);
    wide *= (full + (rest == 0 ? 0.0 : rest <= units ? 0.62 : 1.0)) * 2 * units / tiles;
  }
  return wide < 0.95 * narrow;
}

// workspace: there is room for two parts per unit, and the launch is the only one beside which nothing else runs.
// wide_ok: the strides allow the wide tiles
inline WeightGradPlan plan_weight_grads(const ProductShape* p, int n, bool workspace, bool wide_ok, int units) {
  WeightGradPlan w{};
  w.cuts = 1;
  w.wide = wide_ok && wg_on_wide_tiles(p, n, workspace, units);
  int longest = 0;
  for (int j = 0; j < n; ++j) longest = std::max(longest, wg_steps(p[j].K));
  // Long enough to be cut: 8 steps, and a quarter of the longest of the set.  A block of 512 images has reductions over 33280
  // rows and, in the class-token layer, over 512 (8 steps): counted as long, those tiles were cut
  // as well, the long ones into no more parts (width 384, two layers: a step took 1255 us, 1091 with them whole at the end).
  w.long_steps = std::max(8, (longest + 3) / 4);
  int least = 1 << 30;
  for (int j = 0; j < n; ++j) {
    const int t = (int)wg_tiles(p[j], WG_EDGE);
    w.tiles += t;
    if (wg_steps(p[j].K) >= w.long_steps) { w.long_tiles += t; least = std::min(least, wg_steps(p[j].K)); }
  }
  const int rest = units > 0 ? w.long_tiles % units : 0;
  w.whole_tiles = w.long_tiles - rest;
  if (w.wide || !workspace || units < 8 || rest == 0) return w;
  // Parts per left-over tile: 2, more when the left-over tiles are few (measured at 89 left-over tiles on 256 units: 2 parts
  // 124 + 10 us for the two kernels, 3 parts 123 + 13, 4 parts 121 + 16; undivided 160); with no whole tiles beside them, one
  // part per unit, however few the tiles: width 64, one layer, has 7, which in 8 parts each take 18 + 5 us at 8320 rows, 159 + 5
  // at 131072 and 311 + 5 at 262144, in up to 36 parts 14 + 5, 68 + 8 and 133 + 8.  Each of 4 steps or more (beyond 8 parts, whose
  // sums take longer, of 8: with 4 the first of these takes 14 + 8), within the workspace.
  int cuts = w.whole_tiles == 0 ? std::max(2, units / rest) : std::max(2, units / (2 * rest));
  while (cuts > 1 && (least / cuts < (cuts > 8 ? 8 : 4) || (long)rest * cuts > 2L * units)) --cuts;
  w.cuts = cuts;
  return w;
}

// ---- The same on tiles of 384 x 192, one workgroup a unit, in the launch at the end of a backward pass (in a pipeline, other blocks' streams run
// beside it)
constexpr int BIG_EDGE_M = 384, BIG_EDGE = 192, BIG_PRODUCTS = 40;   // products of a launch: their table stays below the 4 KB of a kernel's arguments
struct BigGradPlan { bool take; int cuts, long_tiles, whole_tiles, tiles, long_steps; };   // as WeightGradPlan
inline long big_tiles(const ProductShape& p) { return (long)((p.M + BIG_EDGE_M - 1) / BIG_EDGE_M) * ((p.N + BIG_EDGE - 1) / BIG_EDGE); }

// Whether a set of products goes there, and how it is divided: the tiles beyond the last full round in as many parts each as find
// a unit: of 8 steps of 64 k or more for the longest reduction, of 2 for one that just counts as long.  The rule compares what both kernels take, fits to 25 sets of 1 to 6 layers of width 192 to 768
// with 1040 to 25216 rows on 256 units, in microseconds: here 1.96 a step of a round, 8 for the launch, and for divided tiles 4 and 0.107 a
// part (295 KB written and read again); there 0.74 a step of 128 x 128 tiles and unit, 10, and 12 more where they are fewer than
// 0.6 a unit.  Measured there / here: width 384, 3 + 1 layers, 4160 rows 72 / 80, 8320 rows 132 / 123, 9280 rows 148 / 132; 3 + 2 layers,
// 5200 rows 125 / 105; width 768, 2 + 1 layers, 1040 rows 66 / 45.  Shorter reductions were not ahead (640 rows of width 768: 52 / 57).
inline BigGradPlan big_grad_tiles(const ProductShape* p, int n, int units) {
  BigGradPlan b{};
  b.cuts = 1;
  if (units < 8 || n < 1 || n > BIG_PRODUCTS) return b;
  int longest = 0, narrow = 0;
  for (int j = 0; j < n; ++j) longest = std::max(longest, wg_steps(p[j].K));
  b.long_steps = std::max(8, (longest + 3) / 4);
  double there = 0.0;
  for (int j = 0; j < n; ++j) {
    b.tiles += (int)big_tiles(p[j]);
    if (wg_steps(p[j].K) < b.long_steps) continue;
    b.long_tiles += (int)big_tiles(p[j]);
    narrow += (int)wg_tiles(p[j], WG_EDGE);
    there += 0.74 * wg_tiles(p[j], WG_EDGE) * wg_steps(p[j].K) / units;
  }
  there += 10.0 + (narrow < 0.6 * units ? 12.0 : 0.0);
  const int rest = b.long_tiles % units;
  if (rest) b.cuts = std::max(1, std::min(units / rest, longest / 8));
  b.whole_tiles = b.cuts > 1 ? b.long_tiles - rest : b.long_tiles;
  const double rounds = b.long_tiles / units + (rest ? 1.0 / b.cuts : 0.0);
  const double here = 1.96 * rounds * longest + 8.0 + (b.cuts > 1 ? 4.0 + 0.107 * rest * b.cuts : 0.0);
  b.take = longest >= 16 && here < there;
  return b;
}

// ---- A product with few output tiles, on the kernel whose waves split k: 32 x 32 tiles, one per compute unit at most, else 32 x
// 64 ones, one per unit at most; up to 256 rows always, beyond that only where the width or the reduction is at most 384.  The
// alternative is the kernel with copying waves (split_tiles, next), below 128 of K the tiled one.  Microseconds alone on 256 units,
// this kernel / that one, with B [K][N]; B [N][K] as well where that changes the picture:
//   128 x 768 x 768   4.7 / 4.8      256 x 768 x 3072    8.0 / 9.3     300 x 768 x 192     4.9 / 4.4
//   128 x 1536 x 768  4.7 / 4.7      128 x 3072 x 768    5.2 / 4.7     600 x 768 x 384     4.9 / 4.6
//   64 x 2304 x 768   4.7 / 4.6      256 x 2304 x 768    7.6 / 4.9     2600 x 192 x 192    4.9 / 4.5
//   455 x 384 x 384   4.8 / 4.4      257 x 384 x 1536    5.1 / 6.0     1000 x 384 x 1536   6.8 / 6.3
//   B [N][K]:                        256 x 768 x 3072    6.8 / 10.3                        6.3 / 6.8
// (4.5 is what launches one behind the other take).  Ahead where the reduction is long, level or behind where it is short and the tiles are
// many.  The line lies further out because it was drawn against the tiled kernel (256 x 2304 x 768 8.6, 640 x 384 x 384 6.3, 1000 x 384 x
// 1536 12.9); it stays, because the sums of this kernel run in another order.  Beyond width 384 every tile reading its own operand rows
// cost pipelined blocks, whose streams share the chip, more than it gained: against the tiled kernel four blocks of 39 images of 17
// tokens at width 768 took 2180 us a batch on this kernel and 1770 on that one.
//  32 x 64 wherever 32 x 32 would be more than one a unit and these are not: 128 x 3072 x 768 with GELU 8.2 in tiles of 32 x 32, 6.4 in
// these, 200 x 2304 x 768 7.7 and 6.7, 256 x 1536 x 384 6.0 and 5.4; but 256 x 3072 x 768, 768 tiles and 384, 11.0 and 11.9.
constexpr int FEW_ROWS = 256, FEW_WIDTH = 384;
inline bool few_tiles_wide(int M, int N, int units) {
  const long rows = (M + 31) / 32;
  return rows * ((N + 31) / 32) > units && rows * ((N + 63) / 64) <= units;
}
inline bool few_tiles(int M, int N, int K, int units) {
  if (M <= FEW_ROWS) return true;
  return (N <= FEW_WIDTH || K <= FEW_WIDTH) && (long)((M + 31) / 32) * ((N + 63) / 64) <= units;
}

// ---- A product whose 64 x 64 tiles find a compute unit each goes to the kernel with waves that do nothing but copy (640 x 768 x 768,
// 120 tiles: 5.8 us, 8.6 on the tiled kernel).  Beyond that tiles share units: alone on the chip it is ahead a little further (2700 x
// 384 x 384, 258 tiles: 5.2 and 6.3), level or behind from some 320 tiles on (520 x 2304 x 768, 324: 9.1 and 8.9; 640 x 3072 x 768,
// 480: 10.0 and 9.0).  It starts where the kernel does, at 128 of K (1500 x 384 x 136: 3.7 and 4.8).  Tiles of 128 x 128 on the same
// scheme take over further on: copy_wave_tiles().
constexpr int SPLIT_MIN_K = 128;
inline bool split_tiles(int M, int N, int K, int units) {
  return K >= SPLIT_MIN_K && units >= 8 && (long)((M + 63) / 64) * ((N + 63) / 64) <= units;
}

// ---- A bf16 Linear product with k contiguous in A: tiles of 128 x 128 (the tiled kernel), 128 x 256 or 160 x 256
enum ProductEnd { END_PLAIN, END_BIAS, END_RESIDUAL, END_GELU, END_DGELU };   // what its epilogue adds
constexpr int PIPE_MIN_K = 128;
// Time of a launch in rounds of workgroup places (two per compute unit): `last` for a last round of at most one workgroup per
// unit, in which they share none.
inline double tile_rounds(int M, int N, int bm, int bn, int units, double last) {
  const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn), places = 2L * units, full = tiles / places, rest = tiles % places;
  return full + (rest == 0 ? 0.0 : 2 * rest <= places ? last : 1.0);
}
// Rows / 32 of the 256-wide tiles that are expected to beat the tiled kernel, 0 if none.
//
// Above width 512 (the shorter of N and K) the loop is long beside everything else and the rounds decide: one of 128 x 256 tiles
// takes 1.58 times, of 160 x 256 tiles 1.74 times as long as one of 128 x 128 (25216 rows of width 768: 30, 33 and 19 us).  25216 x
// 768 is 2.3 rounds of 128 x 128, 1.15 of 128 x 256, 0.93 of 160 x 256 (K = 3072: 145, 142, 115 us).  Even cases stay on the tiled
// kernel.
//
// Up to there, the epilogue and the change of kernels count as well.  Microseconds of a round (per k, and for the epilogue), a
// least-squares fit to 4059 timings of the products of training steps (within 12 % rms):
//   128 x 128   0.0161 K + 4.1 plain, 4.5 bias, 4.9 residual, 8.1 GELU (two tensors out), 5.2 its derivative (one more in)
//   128 x 256   0.0280 K + 6.0        6.8       6.9           13.5                        10.3
//   160 x 256   0.0316 K + 7.2        8.6       8.1           17.5                        14.1
// and each product that runs on other tiles than its neighbours cost them about 3 us (the code of both kernels was fetched again, 4 us
// more for a tiled product behind one on wide tiles; now that they bring it into L2 themselves it is less, and 3 us keep these three
// kinds of tiles apart more than they need be).  By rounds alone, some products ran longer than on the
// tiled kernel (33280 x 576 x 192 with a bias 24 -> 32 us), and so did steps of width 384 (25216 rows, two layers: products on the
// tiled kernel 690 us, 730 by rounds).  Steps of two layers, 12 to 14 row counts from 2080 to 50432 in all, ms, by rounds / with
// epilogue and change: width 128 4.78 / 4.52, 192 6.91 / 6.81, 256 8.76 / 8.63, 384 13.87 / 13.67, 512 19.44 / 19.44, 576 and 640
// 42.2 / 42.6.  One column of wide tiles reads each row of A once and waits for memory where K is long (33280 x 256 x 768: 28 ->
// 32 us).
inline int wide_tile_rows(int M, int N, int K, ProductEnd end, int units) {
  if (K < PIPE_MIN_K || units < 8) return 0;
  double tiled, c4, c5;
  if (std::min(N, K) > 512) {
    tiled = 0.95 * tile_rounds(M, N, 128, 128, units, 0.62);
    c4 = 1.58 * tile_rounds(M, N, 128, 256, units, 0.62);
    c5 = 1.74 * tile_rounds(M, N, 160, 256, units, 0.62);
  } else {
    if (N <= 256 && K > N) return 0;
    static const double e128[] = {4.1, 4.5, 4.9, 8.1, 5.2}, e4[] = {6.0, 6.8, 6.9, 13.5, 10.3}, e5[] = {7.2, 8.6, 8.1, 17.5, 14.1};
    tiled = 0.97 * tile_rounds(M, N, 128, 128, units, 0.6) * (0.0161 * K + e128[end]) - 3.0;
    c4 = tile_rounds(M, N, 128, 256, units, 0.65) * (0.0280 * K + e4[end]);
    c5 = tile_rounds(M, N, 160, 256, units, 0.65) * (0.0316 * K + e5[end]);
  }
  if (std::min(c4, c5) >= tiled) return 0;
  return c4 <= c5 ? 4 : 5;
}

// ---- Which tiles of a launch of one round go to which XCD (workgroup id % 8).  What an XCD's tiles read passes into its L2 from beyond,
// so the fewer rows of A and columns of B they share among them, the better.
constexpr int HELPERS_LEAST = 4, HELPERS_MOST = 8;   // of an XCD, see helper_workgroups()
struct TileMap {
  int tiles_m, tiles_n, per_xcd;   // workgroups an XCD: tiles, or places of which some have none
  int rows, cols, across;          // blocks of rows x cols tiles, `across` of them side by side; rows = 0: a contiguous stretch, row by row
  bool columns;                    // (of a stretch) column by column
};
// Stretches where they do: they are even, and leave each XCD as many units over.  Blocks where they read a fifth less: 640 x 768 in tiles of
// 64 x 64 is 15 tiles an XCD, in stretches all columns and a row or two of rows, 960 rows and columns, in blocks 5 x 3, 512.
inline TileMap tile_map(int M, int N, int bm, int bn, int units) {
  TileMap t{(M + bm - 1) / bm, (N + bn - 1) / bn, 0, 0, 0, 0, false};
  t.per_xcd = (int)(((long)t.tiles_m * t.tiles_n + 7) / 8);
  t.columns = t.tiles_m < t.tiles_n;
  const int shorter = std::min(t.tiles_m, t.tiles_n), longer = std::max(t.tiles_m, t.tiles_n);
  const int places = units / 8 - t.per_xcd >= HELPERS_LEAST ? units / 8 - HELPERS_LEAST : units / 8;   // units an XCD that may have a tile
  double least = 0.8 * (shorter + std::min(longer, (t.per_xcd + shorter - 1) / shorter + 1));
  for (int across = 1; across <= 8; across *= 2) {
    const int rows = (t.tiles_m * across + 7) / 8, cols = (t.tiles_n + across - 1) / across;
    if ((long)rows * cols > places || rows + cols >= least) continue;
    least = rows + cols;
    t.rows = rows; t.cols = cols; t.across = across;
  }
  if (t.rows) t.per_xcd = t.rows * t.cols;
  return t;
}

// The tile of place `slot` of an XCD; false: none.  (Both this and the next are called by kernels; constexpr makes them callable there.)
constexpr bool tile_at(const TileMap& t, int xcd, int slot, int& tm, int& tn) {
  if (slot >= t.per_xcd) return false;
  if (t.rows) {
    tm = xcd / t.across * t.rows + slot / t.cols;
    tn = xcd % t.across * t.cols + slot % t.cols;
    return tm < t.tiles_m && tn < t.tiles_n;
  }
  const int i = xcd * t.per_xcd + slot;
  tm = t.columns ? i % t.tiles_m : i / t.tiles_n;
  tn = t.columns ? i / t.tiles_m : i % t.tiles_n;
  return i < t.tiles_m * t.tiles_n;
}

// Rows m0 .. m1 and columns n0 .. n1 of tiles that hold all tiles of an XCD, what its helpers bring; may be empty
struct TileRange { int m0, m1, n0, n1; };
constexpr TileRange tiles_of(const TileMap& t, int xcd) {
  if (t.rows) {
    const int m = xcd / t.across * t.rows, n = xcd % t.across * t.cols;
    return {m, std::min(m + t.rows, t.tiles_m), n, std::min(n + t.cols, t.tiles_n)};
  }
  const int i0 = xcd * t.per_xcd, i1 = std::min(i0 + t.per_xcd, t.tiles_m * t.tiles_n);
  if (i0 >= i1) return {0, 0, 0, 0};
  if (t.columns) return {0, t.tiles_m, i0 / t.tiles_m, (i1 - 1) / t.tiles_m + 1};
  return {i0 / t.tiles_n, (i1 - 1) / t.tiles_n + 1, 0, t.tiles_n};
}

// Workgroups per XCD that have no tile and bring operands into L2 (Bring, in gemm_pipe.h): one to a unit left over, up to 8 (640 x 768 x 3072 in
// tiles of 64 x 64, microseconds: none 19.2, four 15.7, eight 11.9, twelve 11.3, sixteen 12.0); fewer than 4 cannot keep ahead of the
// tiles (9280 x 384 x 1536 from memory, no residual: none 19.3, two 20.5, four 19.0; 8320 rows: none 19.5, three 19.3, seven 17.0)
inline int helper_workgroups(int per_xcd, int units) {
  const int left = std::min(HELPERS_MOST, units / 8 - per_xcd);
  return left >= HELPERS_LEAST ? left : 0;
}

// Tiles of 128 x 128 with copying waves, a unit each: wherever no unit gets two, unless they are few and the reduction is short, where the
// tiled kernel's tiles of 64 rows find twice the units.  Microseconds, tiled kernel / this one, operands from beyond L2, by tiles:
//   K = 384:   66 6.4 / 7.3    99 6.6 / 7.5   123 8.6 / 8.4   150 10.2 / 8.9   195 10.6 / 9.8   255 13.5 / 10.8
//   K = 768:   72 8.7 / 9.2   102 9.2 / 9.5   144 13.5 / 10.8   198 14.2 / 12.1   252 19.2 / 14.3
//   K = 1152:  66 11.1 / 10.5   99 13.0 / 11.9   123 15.8 / 11.9   195 17.2 / 13.0   255 22.9 / 15.9
//   K = 3072:  72 25.6 / 23.4   102 26.7 / 23.5   144 34.0 / 24.0   198 36.5 / 26.9   252 49.5 / 34.6
// (products whose 64 x 64 tiles find a unit each are on the kernel above).  Not for a block of a pipeline, beside whose launches others want
// units (four blocks of width 384, 8320 rows: 2566 us a batch on the tiled kernel, 2600 here).  Nor where too few units are left over to bring
// operands, as long as the tiled kernel's grid of whole rows of tiles per XCD needs no second round (9850 rows of width 384, 231 tiles, a
// step of 2 + 1 layers 751 and 756 us; 10500 rows, 249 tiles, x 384 x 1536 30.4 and 22.2).
inline bool copy_wave_tiles(int M, int N, int K, int units) {
  const long rows = (M + 127) / 128, columns = (N + 127) / 128, tiles = rows * columns;
  if (K < PIPE_MIN_K || units < 8 || tiles > units) return false;
  if (helper_workgroups((int)(tiles + 7) / 8, units) == 0 && (rows + 7) / 8 * 8 * columns <= units) return false;
  return K >= 1024 || 2 * tiles >= units;
}

// Rows / 32 of tiles that have a unit to themselves (256 x 256 or 320 x 256, eight waves), where they are expected to beat what
// wide_tile_rows() says (`wide`), else 0.  Microseconds of a round of such a launch: per k, and with the epilogue; fits to 182
// products of widths 192 to 1024 with 1800 to 50000 rows (within 5 % rms; the other tiles 8 to 11 %):
//   128 x 128   0.0150 K + 4.7 plain or bias, 5.8 residual, 9.0 GELU, 6.9 its derivative, and 1.5 a launch
//   128 x 256   0.0260 K + 8.7       11.4     16.4                   13.9
//   160 x 256   0.0311 K + 9.7       12.8     20.3                   16.0
//   256 x 256   0.0237 K + 9.1       11.8     17.7                   13.5
//   320 x 256   0.0287 K + 10.5      13.6     21.2                   15.9
// where the first three count a last round of at most one workgroup a unit as 0.55, 0.65 and 0.60 of one, the others one that fills the
// share f of the units as 0.7 + 0.3 f.  The choice has to be 3 % ahead; over those products it is never behind, and 5 % ahead in
// sum.  (Beside a tiled product the change of kernels costs less than it did: see CodeToL2.  With a microsecond for it, evaluation
// forwards of width 384, 8320 rows, took 342 us, without 338.)  These are launches alone, of one session; the figures of wide_tile_rows() are
// fits to products inside steps, from before the kernels brought their code into L2 and stored through it.  They decide among the
// first three kinds of tiles, these whether the fourth or fifth is ahead of that.
inline int unit_tile_rows(int M, int N, int K, ProductEnd end, int wide, int units) {
  if (K < PIPE_MIN_K || units < 8) return 0;
  struct Cost { int rows, cols; double last, k, end[5], launch; };
  static const Cost tiled = {128, 128, 0.55, 0.0150, {4.7, 4.7, 5.8, 9.0, 6.9}, 1.5}, c4 = {128, 256, 0.65, 0.0260, {8.7, 8.7, 11.4, 16.4, 13.9}, 0.0},
                    c5 = {160, 256, 0.60, 0.0311, {9.7, 9.7, 12.8, 20.3, 16.0}, 0.0}, c8 = {256, 256, 0.7, 0.0237, {9.1, 9.1, 11.8, 17.7, 13.5}, 0.0},
                    c10 = {320, 256, 0.7, 0.0287, {10.5, 10.5, 13.6, 21.2, 15.9}, 0.0};
  const Cost& now = wide == 4 ? c4 : wide == 5 ? c5 : tiled;
  const double other = tile_rounds(M, N, now.rows, now.cols, units, now.last) * (now.k * K + now.end[end]) + now.launch;
  auto cost = [&](const Cost& c) {
    const long tiles = (long)((M + c.rows - 1) / c.rows) * ((N + c.cols - 1) / c.cols), rest = tiles % units;
    return (tiles / units + (rest ? c.last + (1.0 - c.last) * rest / units : 0.0)) * (c.k * K + c.end[end]);
  };
  const double t8 = cost(c8), t10 = cost(c10);
  if (std::min(t8, t10) >= 0.97 * other) return 0;
  return t8 <= t10 ? 8 : 10;
}

// ---- A product of width 192 or 384 and the LayerNorm behind it in one launch, on whole rows: 64 of them a workgroup, two workgroups a unit
// at width 192, one at 384.  Never where the product alone would be on the kernel that splits k (few_tiles): its sums are others.
// Microseconds alone, two launches / one; K = N forward, 4 N forward, 4 N backward, 3 N backward:
//   192:   4160 rows   9.8 / 7.3   12.2 / 11.9   16.2 / 16.4   15.2 / 14.6      384:   4160 rows  11.0 / 11.9   17.5 / 26.0   23.3 / 31.7   20.6 / 26.3
//          8320       11.4 / 7.5   16.1 / 12.1   20.9 / 18.0   19.0 / 16.0             5200       12.5 / 12.0   22.8 / 26.2   29.0 / 32.5   25.4 / 27.3
//         16640       14.1 / 10.4  23.6 / 21.5   34.0 / 27.6   29.3 / 23.0             8320       14.0 / 12.1   25.1 / 31.4   36.6 / 38.8   31.4 / 29.9
//         25216       16.1 / 10.8  29.3 / 25.0   38.9 / 35.1   35.4 / 30.8            16640       24.0 / 26.2   42.9 / 62.6   57.8 / 77.9   51.0 / 65.6
// Width 192: where the product alone is not on the kernel with copying waves (two blocks of 4160 rows with it on both sides of that line:
// 405 us a step in two launches, 412 in one).  Width 384: one workgroup a unit waits for its own operands (0.78 us per 64 k), so only a
// short reduction and one round (25216 rows: a step of 2 + 1 layers 0.3 % behind), not too small a part of one (5200 rows, 82 tiles: 0.4 %
// behind).
inline bool norm_tiles(int M, int N, int K, int units) {
  if (units < 8 || few_tiles(M, N, K, units) || split_tiles(M, N, K, units)) return false;
  const long tiles = (M + 63) / 64;
  return N <= 192 || (K <= N && tiles <= units && 10 * tiles >= 4 * units);
}
// Of these, at width 384, not where the product alone would be on 128 x 128 tiles with copying waves: alone on the device, 3 + 1 layers,
// us a step (an evaluation) in two launches and in one, with them 8320 rows 867 and 872 (339 and 343), 9280 976 and 979 (361 and 365),
// 10465 985 and 986 (377 and 378), 10790 997 and 1001 (380 and 383); without them 9815 959 and 959 (361 and 360), 11050 1092 and 1085
// (405 and 398), 12325 1195 and 1187 (435 and 426), 15950 rows, 2 + 2 layers, 1408 and 1399 (514 and 502).  At width 192 one launch is
// ahead of those tiles too: 8320 rows 519 and 507 (217 and 212), 12480 rows 644 and 609 (268 and 253).  Beside other streams they are not taken,
// and one launch is level or ahead: pipelines of four and three blocks of width 384, 8320 rows, 2560 and 2558 us a batch, 2573 and 2566; of
// four of width 192, 8320 rows, 1222 and 1172.
inline bool norm_with_product(int M, int N, int K, bool shared, int units) {
  return norm_tiles(M, N, K, units) && (N <= 192 || shared || !copy_wave_tiles(M, N, K, units));
}

// ---- Pieces of 8 channels a thread of a BatchNorm's apply pass: four share the loads of their channels' parameters, one where four would
// occupy too few units.  Microseconds of a launch on 256 units, one / four pieces (with a residual), by workgroups of four:
//   16 2.1 / 2.6 (2.1 / 2.7)   96 2.5 / 2.7 (2.7 / 2.8)   128 2.6 / 2.8 (2.7 / 2.9)   176 2.9 / 2.9 (3.1 / 2.9)   224 3.1 / 2.9 (3.4 / 3.0)
//   288 3.5 / 3.4 (3.7 / 3.6)   512 4.8 / 3.9 (5.1 / 4.0)   1024 7.8 / 6.3 (9.1 / 7.2)   2048 13.4 / 11.5 (18.0 / 15.6)
constexpr int AP_PIECES = 4;
inline int bn_apply_pieces(size_t chunks, int units) {
  return 8 * ((chunks + 256 * AP_PIECES - 1) / (256 * AP_PIECES)) <= 5 * (size_t)units ? 1 : AP_PIECES;
}

// ---- The matrix-core attention addresses the keys, queries and values of an image with 32-bit byte offsets
inline bool att_offsets_fit(int T, int H) { return (long)T * H * (3 * 64 * 2) <= 0x7fffffffL; }

// ---- Attention of shapes that the matrix-core kernel does not take: one workgroup per (image, head), or one per 16 rows of one
constexpr size_t UNIT_LDS = 160 * 1024;
constexpr int ATT_ROWS = 16;
// Rows kernel: quads of a head row, floats between rows in LDS, floats of a row of scores
struct AttShape { int T, H, dh, q4, pitch, tp; };
#ifdef __HIPCC__
__host__ __device__
#endif
inline AttShape att_shape(int T, int H, int dh) {
  const int q4 = (dh + 3) / 4;
  return {T, H, dh, q4, 4 * q4 + 4, ((T + 3) / 4) * 4 + 4};
}
inline size_t att_rows_lds(const AttShape& a, bool bwd) {
  return ((size_t)2 * a.T * a.pitch + (bwd ? 2 : 1) * ATT_ROWS * a.pitch + (bwd ? 2 : 1) * ATT_ROWS * a.tp + (bwd ? 2 * a.T + 8 : 0)) * sizeof(float);
}
inline size_t att_heads_lds(int T, int dh, bool bwd) {
  return ((size_t)2 * T * (dh + 1) + (bwd ? 8 : 4) * (dh + T) + (bwd ? 2 * T : 0)) * sizeof(float);
}
// Whether the rows kernel takes it.  It has many times the workgroups, and each of them reads all keys and values of its head
// again: ahead while there are few heads (2.2 to 30 times at 128 of them), and with many as long as two of its workgroups share
// a unit.  Where one alone fits and two of the other kernel do, its time grows with the heads while the other's does not up to
// two a unit, and they cross at about 1.5 heads a unit.  Microseconds on 256 units, heads kernel / rows kernel, 128 heads and 512:
//   197 tokens, head size 32, backward   1458 / 429   1510 / 1876      65 tokens, 128, backward   621 / 225   647 / 896
//   256 tokens, head size 32, forward     738 / 182    763 / 805       256 tokens, 32, backward  2176 / 623  2235 / 2731
inline bool att_by_rows(int T, int H, int dh, bool bwd, long heads, int units) {
  const size_t rows = att_rows_lds(att_shape(T, H, dh), bwd);
  if (rows > UNIT_LDS) return false;
  return 2 * rows <= UNIT_LDS || 2 * att_heads_lds(T, dh, bwd) > UNIT_LDS || heads <= units + units / 4;
}

}  // namespace ppll
