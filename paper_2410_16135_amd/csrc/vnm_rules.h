// Rules that choose between kernels or launch shapes by sizes alone.  Plain C++ without HIP, so that they can be
// compiled and checked on any host.
#pragma once
#include <stdint.h>
#include <initializer_list>

namespace vnm {

// ---- RIA scores (vnm_score.hip)
// Column sums: waves per workgroup and rows in flight per thread.  One pass of a workgroup covers
// 8 * waves * flight rows; on short matrices the rows that a wide pass would repeat at the end cost more than the
// bandwidth it gains on tall ones.  Device time of the whole vnm_ria_scores with (waves, flight) =
// (4, 4) / (4, 8) / (8, 8) / (16, 8), us: 96 x 1000 9.6 / 10.1 / 11.4 / 12.8, 500 x 1000 12.0 / 11.8 / 11.6 / 14.4,
// 768 x 1000 13.8 / 13.3 / 14.7 / 14.7, 2048 x 1000 24.1 / 22.4 / 21.7 / 21.8, 4096 x 4096 64.0 / 58.3 / 55.2 / 54.2,
// 11008 x 4096 151 / 136 / 130 / 126.
// Rows without 16-byte alignment are read element by element, and only waves hide that: 1000 x 1031
// 42.6 / 42.5 / 31.5 / 25.5, 16 x 1031 12.5 / 12.6 / 12.5 / 12.5.
struct ColsumShape { int waves, flight; };
inline ColsumShape colsum_shape(int64_t out, bool aligned) {
  if (!aligned || out >= 3072) return {16, 8};
  if (out >= 1536) return {8, 8};
  if (out > 384) return {4, 8};
  return {4, out > 32 ? 4 : 1};                       // 16 x 1000: 7.8 us with one row in flight, 8.6 with four
}
// Scores: rows per workgroup, from the number of (1024 columns, row) units.  More rows share the column reciprocals;
// fewer give a small matrix workgroups for every compute unit.  Whole call with 1 / 4 / 8 / 16 rows, us:
// 96 x 1000 8.8 / 9.6 / 10.3 / 11.6, 1000 x 1000 16.5 / 15.7 / 16.3 / 17.7, 1000 x 4096 28.2 / 23.8 / 23.8 / 24.4,
// 2048 x 4096 47.1 / 38.4 / 36.8 / 36.9, 4096 x 4096 80.7 / 64.1 / 62.9 / 61.0, 11008 x 64 85.6 / 78.4 / 77.4 / 76.9.
inline int score_rows(int64_t out, int64_t in) {
  const int64_t units = (in + 1023) / 1024 * out;
  return units <= 1024 ? 1 : units <= 4096 ? 4 : units <= 12288 ? 8 : 16;
}

// ---- products on the canonical triple (vnm_spmm_plain.hip, scalar kernel in vnm_aux.hip)
constexpr int kPlainTok = 128;                // tokens of a workgroup of the many-token kernel, lane = two tokens
constexpr int kPlainCols = 256;               // columns of X it holds in LDS at most
constexpr int64_t kPlainManyTokens = 32;      // from here on it is used: a quarter of its tokens.  Below, the other
                                              // kernel's work grows with the tokens, in groups of 4

// Many tokens: column blocks per chunk of K (at most one per lane and kPlainCols columns; an even number, so that every
// chunk starts at an even column), and rows per wave: as many as still give every compute unit two workgroups (a chunk
// of X is turned around once per 16 rows_per_wave rows).
struct PlainPlan { int blocks, rows_per_wave; int64_t groups; };
inline PlainPlan plain_plan(int64_t T, int64_t out, int M) {
  int nb = kPlainCols / M;
  nb = nb > 64 ? 64 : (nb < 1 ? 1 : nb);
  if (nb > 1) nb &= ~1;
  const int64_t tiles = (T + kPlainTok - 1) / kPlainTok;
  int rw = 4;
  while (rw > 1 && tiles * ((out + 16 * rw - 1) / (16 * rw)) < 512) rw >>= 1;
  return {nb, rw, tiles * ((out + 16 * rw - 1) / (16 * rw))};
}

// Sizes both kernels can index: row groups on grid.y for many tokens (on grid.x for few), token tiles on grid.x, 32-bit
// byte offsets into a row of X.
inline bool plain_sizes_fit(int64_t T, int64_t out, int64_t in, int M) {
  if (in >= (1 << 30)) return false;
  if (T < kPlainManyTokens) return out <= 32ll * 0x7FFFFFFF;
  const int64_t tiles = (T + kPlainTok - 1) / kPlainTok;
  return tiles <= 0x7FFFFFFF && plain_plan(T, out, M).groups / tiles <= 65535;
}

// Whether the scalar kernel, one thread per output that walks all B column blocks, is the faster one: it is where
// there are few blocks, because the others pay for a lane per block, or for moving all of X through LDS, whatever
// their number (M = 255: 128 columns of X for each one that is used).  Estimates in us, from device times over 1283
// layers (8 to 40000 x 8 to 9000, M 4 to 255, 1 to 8192 tokens): with the scalar kernel alone 20.3 us in the geometric
// mean, without it 12.6, by this rule 9.99, with the better of both every time 9.97.
//   scalar       0.45 us per block (two dependent loads) and its loads, 2.6 ps per output and block: the larger of the
//                two and 0.6 of the smaller
//   few tokens   3.7 us for one token, else 6.3, or 2.9 ns per wave of 8 rows x 4 tokens
//   many tokens  per workgroup 2.8 us + 1.7 per chunk + 0.09 per block and row of a wave, 256 workgroups at once
inline bool plain_scalar_faster(int64_t T, int64_t out, int64_t B, int M) {
  const double by_latency = 1.6 + 0.45 * (double)B, by_loads = 2.6e-6 * (double)out * (double)T * (double)B;
  const double scalar = by_latency > by_loads ? by_latency + 0.6 * by_loads : by_loads + 0.6 * by_latency;
  if (T < kPlainManyTokens) {
    const int64_t per = T < 3 ? T : 4;
    const double waves = 2.9e-3 * (double)((out + 7) / 8) * (double)((T + per - 1) / per), least = T == 1 ? 3.7 : 6.3;
    return scalar < (waves > least ? waves : least);
  }
  const PlainPlan p = plain_plan(T, out, M);
  const int64_t chunks = (B + p.blocks - 1) / p.blocks, rounds = (p.groups + 255) / 256;
  const double blocks = (double)(B < p.blocks ? B : p.blocks);
  return scalar < (2.8 + (double)chunks * (1.7 + 0.09 * blocks * p.rows_per_wave)) * (double)rounds;
}

// ---- pieces of K of the staged product, for T <= 2048 tokens and `pairs` (token tile, 256 channels) pairs, before the
// limits that scratch and 4 steps per piece set.
// Up to 256 tokens about 200 workgroups measured best.  Beyond that the partial products (pieces x T x out floats
// written, then read by the reduction) weigh in: 256 workgroups while that fills the compute units in one generation, and two
// pieces up to 128 pairs.  Either way only where K is long enough to pay for the reduction: by the columns of X (8 * M *
// steps) and the results (T * out, in units of 2^15, a pair of 128 tokens).  Staged product with these pieces against
// one, which is the kernel with two wave groups where that one runs (1030 random layers, 64 to 12000 x 500 to 14000, M 4
// to 16, 65 to 2048 tokens, weights from HBM; geometric mean and range) above the line and below it:
//   results up to 7    0.55 (0.15-1.30)                          22 to 78    0.68 (0.32-1.18)   1.30 (0.80-1.88)
//              7 to 14 0.67 (0.20-1.25)   1.14 (0.88-1.32)       78 to 128   0.83 (0.57-1.32)   1.14 (0.86-1.62)
//             14 to 22 0.72 (0.28-1.36)   1.21 (0.79-1.54)
// Beyond 128 pairs two pieces take a second generation, 0.94 to 1.28 at 200 to 280 steps; M > 10 keeps the line it had
// (129 pairs: 1.02 at 103 steps, 0.66 at 205; 160 pairs 1.08 and 0.96).
// M > 10: one piece has one wave group there, from 8 row blocks on on half of the compute units, and pieces pay earlier: 1205
// x 1688 at M = 16 and 504 tokens (14 steps) 43 us in one piece, 34 in three; 705 wide at M = 12 and 354 tokens (9
// steps) 1.33.
// 198 random layers that the other line would not split (M 11 to 16, 8 to 102 units of results), all in pieces as before this
// line 1, none 1.009 (weights from the last-level cache) and 1.027 (from HBM), up to 1.34; by this line 0.969 and 0.974,
// up to 1.13, with the better of both every time 0.965.
inline int64_t split_pieces(int64_t T, int64_t out, int64_t pairs, int64_t steps, int M) {
  const int64_t results = (T * out + 32767) / 32768, length = steps * M;
  if (pairs > 128) return M > 10 && T > 256 && steps >= 192 ? 2 : 1;
  const int64_t least = results <= 7 ? 0 : results <= 14 ? 128 : results <= 22 ? 240
                      : results <= 78 ? (T <= 256 ? 300 : 380) : T <= 600 ? 420 : T <= 1500 ? 500 : 660;
  const int64_t least_one_group = out <= 448 ? (results <= 14 ? 128 : 240) : results <= 34 ? 0 : results <= 50 ? 220 : 320;
  if (length < (M > 10 && results <= 78 ? least_one_group : least)) return 1;
  return T <= 256 ? (200 + pairs / 2) / pairs : pairs <= 85 ? 256 / pairs : 2;
}

// ---- reduction of a product whose K dimension is split (vnm_spmm_smfmac.hip, vnm_spmm_skinny.hip)
// Whether the partial products are still in the L2 of the XCD that wrote them when the reduction reads them.  Workgroup
// n runs on XCD n mod 8.  With one token tile (or the few-token kernels) and a multiple of 1024 channels the workgroups
// that write 256 channels, and the workgroups of 256 results that reduce them, have the same n mod 8 (for a multiple of
// 2048 every time, for 1024 every other token), and the eight L2s of 4 MiB hold the weight and the parts.  Measured up
// to 34 MiB; beyond that the order makes no difference.
inline bool parts_stay_in_l2(int64_t T, int64_t out, int pieces, int64_t weight_bytes, bool one_tile) {
  return pieces > 1 && one_tile && out % 1024 == 0 && weight_bytes + pieces * T * out * 4 < (34ll << 20);
}
// The reduction with 16-byte loads and 1024 results per workgroup, rather than one result per thread.  Below 2^19
// results the launch is what counts, and one per thread spreads it wider: a 4096 / 11008 block at 24 tokens (three
// reductions) 73.7 us against 74.2.  And not where that kernel meets its parts in its own L2: whole call, M = 12,
// 8192 x 2048 at 100 tokens 23.5 us against 28.4, 4096 x 4096 at 256 tokens 16.5 against 18.5; elsewhere the wide one:
// 11008 x 4096 at 200 tokens 43.2 -> 40.7, 4096 x 4096 at 700 tokens 43.4 -> 40.7, 8192 x 8192 at 100 tokens 33.8 -> 33.3.
inline bool reduce_wide(int64_t T, int64_t out, bool in_l2) { return T * out >= (1 << 19) && !in_l2; }

// ---- numbering of the staged product's workgroups over the XCDs (vnm_spmm_smfmac.hip)
// Workgroup n runs on XCD n mod 8, each with an L2 of its own.  What each of them fetches of the weight and of the staged
// X, as shares of the whole, where n counts token tiles first, then groups of 256 channels, then pieces of K:
//   grid order   X: the tiles of one residue modulo gcd(tiles, 8) -- all of them where the number of tiles is odd;
//                the weight: min(1, tiles / 8); with one tile the groups of one residue modulo gcd(groups, 8)
//   XCD order    (an XCD takes consecutive n) an eighth of the weight; X of one piece, an eighth at least
// The XCD order is taken where it saves each L2 4 MiB, in a split product with pieces of 10 steps or more, or 8 MiB
// unsplit, and where the reduction does not need grid order to meet its parts in its own L2.  Time against grid order
// by MiB saved, 1500 random sizes (600 to 16384 x 600 to 12000, 65 to 4000 tokens): split 0-2 1.008, 2-4 1.001, 4-6 0.979,
// 6-8 0.950, 10-12 0.897, 20 and more 0.862; unsplit 0-2 1.019, 4-6 1.006, 6-8 0.991, 8-10 0.986, 12-14 0.978, 20 and more
// 0.975.  4096 x 11008 at M = 5: 320 tokens 52.1 -> 41.3 us, 1124 tokens (9 tiles) 146 -> 106; 2048 x 11008 at M = 8 and 868
// tokens 67 -> 44; 4096 x 4096 unsplit at 4096 tokens saves nothing and would lose 64.9 -> 71.7.
inline bool tiles_by_xcd(int64_t tiles, int64_t groups, int64_t steps, int pieces, int64_t weight_bytes, int64_t staged_bytes,
                         bool in_l2) {
  auto residues = [](int64_t n) { return n % 8 == 0 ? 8 : n % 4 == 0 ? 4 : n % 2 == 0 ? 2 : 1; };
  double x_grid = 1.0, w_grid = tiles < 8 ? (double)tiles / 8 : 1.0;
  if (tiles > 1) x_grid = 1.0 / residues(tiles);
  else {
    const double spread = pieces < 8 ? (double)pieces / 8 : 1.0, met = 1.0 / residues(groups);
    w_grid = spread < met ? (spread > 0.125 ? spread : 0.125) : met;
  }
  const double x_xcd = pieces > 8 ? 0.125 : 1.0 / pieces;
  const double saved = (w_grid - 0.125) * (double)weight_bytes + (x_grid - x_xcd) * (double)staged_bytes;
  if (in_l2) return false;
  return pieces > 1 ? saved >= (4 << 20) && steps / pieces >= 10 : saved >= (8 << 20);
}

// The numberings: grid order, runs (the XCD order above), boxes: the XCDs form a grid of 2^log_t parts of the token
// tiles x 8 / 2^log_t parts of the groups, each takes one box, token tiles fastest; boxes differ by at most one in each
// direction, the launch is 8 of the largest; and columns: runs with the groups fastest, every XCD then has a share of
// the tiles.
struct XcdOrder {
  enum Kind { kGrid, kRuns, kBoxes, kColumns } kind;
  unsigned log_t;
};
inline unsigned xcd_box_most(int64_t tiles, int64_t groups, unsigned log_t) {
  const int64_t xt = 1 << log_t, xg = 8 / xt;
  return (unsigned)(((tiles + xt - 1) / xt) * ((groups + xg - 1) / xg));
}
// Boxes for two kinds of unsplit launches.
// A single generation (two wave groups, below): the grid that makes an XCD fetch least without a second one.  4096 x 4096 at
// M = 5, 16 tiles x 16 groups 45.4 -> 44.4 us against runs, 12 x 16 42.9 -> 42.7; M = 8 32.4 -> 30.9.  Where no grid of boxes
// does without a second one, columns if they fetch less than grid order: 660 x 2968 at V = 128, M = 8 and 10442 tokens
// (82 tiles x 3 groups) 45.8 us in grid order, 27.6 in columns, 34.2 with one wave group; 90 random launches of that
// kind against one wave group 0.907 (0.74-1.34) in grid order, 0.827 (0.68-1.03) by this rule.
// Otherwise 8 parts of the tiles (8 row blocks per workgroup only: the others carry no code for it), where runs and grid
// order make every XCD fetch most of X (the number of tiles not a multiple of 8) and the weight is the smaller part.  Not
// where the largest box, of one more tile than the others, takes a generation (32 workgroups per XCD) more than an even share
// of the launch: 5832 x 3032 at M = 8 and 2324 tokens (19 tiles x 12 groups, 36 workgroups instead of 28.5) 43.8 us in
// runs, 61.1 in boxes; and only where an XCD fetches 1 MiB less, and 1 MiB more than that for every percent by which
// that box exceeds the even share: 3702 x 792 at M = 5 and 2198 tokens (24 instead of 18 workgroups, 0.9 MiB) 40.1 and
// 46.4.  262 random launches with 17 tiles or more, where a box saves 1 MiB at least: boxes everywhere 0.986 of the time
// without, up to 1.46; by this rule 112 of them, 0.941, none above 1.02.  vnm_spmm_staged: 3072 x 768 at M = 8 and 12608
// tokens (99 tiles) 48 -> 40 us (vnm_spmm runs the resident kernel there), 2304 x 1536 at 6000 (47) 26.0 -> 20.3.  Boxes
// in other shapes lose on more than one generation: 11008 x 4096 at V = 32, M = 5 and 2048 tokens in 2 x 4 boxes 46.0 ->
// 49.1.
inline XcdOrder xcd_order(int64_t tiles, int64_t groups, int64_t steps, int pieces, int64_t weight_bytes, int64_t staged_bytes,
                          bool one_generation, bool wide, bool in_l2) {
  XcdOrder o{XcdOrder::kGrid, 0};
  if (in_l2) return o;
  const double w = (double)weight_bytes, x = (double)staged_bytes;
  if (one_generation) {
    const int64_t share = (tiles * groups + 7) / 8;
    double best = 1e300;
    for (unsigned l = 0; l <= 3; ++l) {
      const int64_t xt = 1 << l, xg = 8 / xt;
      if (tiles < xt || groups < xg || (xcd_box_most(tiles, groups, l) > 32 && share <= 32)) continue;
      const double bytes = w * (double)((groups + xg - 1) / xg) / (double)groups + x * (double)((tiles + xt - 1) / xt) / (double)tiles;
      if (bytes < best) { best = bytes; o = {XcdOrder::kBoxes, l}; }
    }
    if (o.kind == XcdOrder::kGrid && share >= groups) {
      const int64_t residues = tiles % 8 == 0 ? 8 : tiles % 4 == 0 ? 4 : tiles % 2 == 0 ? 2 : 1;
      const double columns = w + x * (double)(share / groups + 2) / (double)tiles;
      if (columns < (tiles < 8 ? (double)tiles / 8 : 1.0) * w + x / (double)residues) o.kind = XcdOrder::kColumns;
    }
    return o;
  }
  if (tiles_by_xcd(tiles, groups, steps, pieces, weight_bytes, staged_bytes, in_l2)) o.kind = XcdOrder::kRuns;
  if (pieces == 1 && tiles >= 16 && wide) {
    const int64_t residues = tiles % 8 == 0 ? 8 : tiles % 4 == 0 ? 4 : tiles % 2 == 0 ? 2 : 1;
    const double now = o.kind == XcdOrder::kRuns ? w / 8 + x : w + x / (double)residues;
    const double saved = (now - (w + x / 8)) / 1048576.0;
    const int64_t most = xcd_box_most(tiles, groups, 3), even = (tiles * groups + 7) / 8;
    const double excess = (double)most * 8.0 / (double)(tiles * groups) - 1.0;
    if ((most + 31) / 32 <= (even + 31) / 32 && saved >= 1.0 + 100.0 * excess) o = {XcdOrder::kBoxes, 3};
  }
  return o;
}

// ---- the staged product's deep K loop: six operand sets and images in flight instead of three or four
// For pieces of a split K on a launch that leaves compute units without a workgroup: a step then waits for its operands
// rather than for the matrix cores.  Most where the other loop has a ring of three images only (M >= 8): 4096 x 11008 at
// M = 8 and 700 tokens 75.0 -> 63.2 us, 8192 x 8192 at 320 tokens 60.1 -> 51.0, 232 sizes with M = 8 and 9 and 8 steps or
// more per piece 5.5 % less time, none 1 % slower.  For M <= 7, with a ring of four, filling the longer ring costs more
// than it gives below 48 steps (272 sizes 0.6 % slower, up to 3.9) and pays from there on (151 sizes, 1.2 % less).  Not
// unsplit: 644 sizes 1.3 % slower, 16384 x 1024 at M = 4 and 700 tokens 31.7 -> 34.1.
// It looks five steps ahead: at least 8 steps in every piece (its first ring of images), and 64 steps in all (its last
// loads of the weight end inside the sections behind it).  Instantiated for one column table and up to six copies of
// the image per wave, which is M = 9.
inline bool deep_loop(int pieces, int64_t workgroups, int64_t last_piece, int64_t row_blocks, int64_t steps, int M, int tables) {
  return pieces > 1 && workgroups < 256 && last_piece >= (M >= 8 ? 8 : 48) && row_blocks * steps >= 64 && M <= 9 && tables == 1;
}

// ---- one to four tokens on the vector ALUs (vnm_spmm_gemv.hip)
// A ring of 2 steps per wave is enough: the stream is kept going by the 16 to 32 waves of a unit, and deeper rings
// measured slower (ring 2 / 4 / 8, 4096 x 4096, 64:2:5, one token: 7.0 / 7.2 / 8.1 us).
constexpr int kGemvRing = 2;
constexpr int64_t kGemvLds = 150 * 1024;
// LDS: the rows of X, per wave a ring of strips of 32 halfwords per token (half tiles: 64, for pairs of steps), the
// waves' sums.
inline int64_t gemv_lds(int tokens, int64_t in, int waves, bool half) {
  return tokens * (in * 2 + 128) + (int64_t)waves * kGemvRing * tokens * (half ? 128 : 64) + (int64_t)waves * tokens * 64 * 4;
}
// Half tiles (16 rows per workgroup) while they are at most one workgroup per compute unit.  Whole / half tiles at 1 and
// at 4 tokens, us: weights from HBM 4096 x 4096, M = 5 7.3 / 6.2 and 8.9 / 7.4, M = 8 5.6 / 4.9 and 6.5 / 5.7; 4096 x
// 11008, M = 8 11.8 / 8.4 and 13.5 / 10.7; 1024 x 8192, M = 5 10.2 / 7.2 and 11.9 / 9.2; 128 x 128 2.5 / 2.3 and 3.1 /
// 2.7; 64 x 11008, M = 8 6.9 / 5.4 and 9.7 / 7.8; from the last-level cache 4096 x 4096, M = 5 6.6 / 6.1 and 8.3 / 7.4,
// 4096 x 11008, M = 8 9.4 / 8.6 and 12.5 / 10.9.  23 layers at 1, 2 and 4 tokens: 0.82, 0.84 and 0.86 of the time from
// HBM, 0.89, 0.89 and 0.88 from that cache.
// 4100 x 4096 (65 row blocks) keeps whole tiles.  Rows of X too long for half tiles but not for whole ones: whole tiles
// beyond 32 row blocks, below that the few-token kernel (64 x 73600, M = 16, one token 17.3 us on whole tiles, 8.8
// there; 4096 x 73600, V = 32 30.6 and 50.2).
inline bool gemv_half(int tokens, int64_t row_blocks, int64_t in) {
  return row_blocks <= 64 && (row_blocks <= 32 || gemv_lds(tokens, in, 16, true) <= kGemvLds);
}
// Waves per workgroup.  Whole tiles: 8 where they are more than compute units, so that several workgroups share a unit
// and one's start-up (X, the first weights) overlaps the others' streaming, otherwise 16.  Half tiles: 8 where a pass of
// them holds a row of X and K is short, else 16.  With 16 / 8, one token, us (halves of a tile in grid order): 4096 x
// 4096, M = 5 (103 steps) 6.3 / 6.5, M = 8 (64) 5.1 / 4.6; 4096 x 11008, M = 5 11.9 / 12.4; 1024 x 8192, M = 5 5.9 /
// 6.9; 2048 x 5504, M = 12 (58 steps) 3.9 / 4.2; 2048 x 2048, M = 5 3.9 / 3.7; 128 x 128 2.9 / 2.3.
inline int gemv_waves(int tokens, int64_t row_blocks, int64_t in, int64_t steps) {
  if (gemv_half(tokens, row_blocks, in)) return in <= 8 * 64 * 8 && steps <= 80 ? 8 : 16;
  return 2 * row_blocks > 256 ? 8 : 16;
}
// Which layers it takes.  Three and four tokens: only where the tiles leave compute units idle and K is short.  Otherwise the
// vector ALUs become the limit and the matrix-core few-token kernel is faster: 11008 x 4096 at 64:2:5 (344 tiles) and
// four tokens 13.2 us against 12.7.  This kernel's time over that one's at 3 and 4 tokens (halves of a tile in grid order,
// up to 11 % slower than they run), 160 random layers of up to 128 row blocks by K steps: up to 80 0.32 to 0.81, 81 to
// 130 0.40 to 0.9 (1.02 at M = 16), 131 to 180 0.78 to 1.02, 181 to 224 0.90 to 1.11, 225 to 290 0.51 to 1.24, more 0.97
// to 1.43.
inline bool gemv_takes(int tokens, int64_t row_blocks, int64_t in, int64_t steps) {
  if (tokens > 2 && (2 * row_blocks > 256 || steps > 224)) return false;
  return gemv_lds(tokens, in, gemv_waves(tokens, row_blocks, in, steps), gemv_half(tokens, row_blocks, in)) <= kGemvLds;
}

// ---- the staged product with two groups of waves per workgroup, each on half of the steps
// For unsplit launches of at most one workgroup of 4 row blocks per compute unit: with 8 row blocks they would leave half
// of the units idle, with one wave per SIMD every step waits for its operands.  Weights from HBM, before / with two groups:
// 4096 x 4096 at 2048 tokens (256 workgroups) M = 5 61.6 / 44.4 us, M = 8 41.5 / 30.9, V = 32 and M = 8 46.8 / 33.4; at 1500
// (192) 60.9 / 42.7; 8192 x 4096 at 1024 63.4 / 46.0; 11008 x 4096 at 300 63.0 / 43.9; 5504 x 2048 at 1000 33.4 / 25.0.
// Pieces of a split K keep the deep loop (4096 x 4096 at 700 tokens 33.0 against 34.3 with two groups; two groups instead of
// the split 42).  LDS holds two rings up to M = 10.
// Below 8 row blocks one group is a workgroup of 4 waves on as many compute units, and two take steps to make up for the
// exchange at the end: 256 x 600 at 7455 tokens and M = 5 (15 steps) 9.5 us with one, 11.2 with two.  Two groups against one,
// geometric mean and range over 350 random launches of that kind: 8-16 steps 1.08 (0.88-1.25), 17-31 1.00 (0.85-1.13), 32-55
// 0.95 (0.85-1.06), more 0.88 (0.75-1.09); but at M = 8, where one group has a ring of three images and two have four
// each, 8-13 1.07 (0.89-1.17), 14-23 0.92 (0.79-1.10), 24-55 0.82 (0.65-1.01), more 0.67.  340 launches of 8 row blocks
// and more: 8-16 steps 0.84, more 0.79.
inline bool kgroups(int pieces, int64_t workgroups, int64_t row_blocks, int64_t steps, int M) {
  const int least = row_blocks >= 8 ? 8 : M == 8 ? 24 : 56;
  return pieces == 1 && workgroups <= 256 && steps >= least && M <= 10;
}

// ---- pruning (vnm_prune_fast.hip): K steps of 8 column blocks that a workgroup takes at a time
// Its LDS: weight tile u16 [V][NC + 4], column sums f64 [NC], kept columns u32 [blocks], with scores f32 [V][NC + 4]
inline int64_t prune_fast_lds(int V, int M, int steps, bool scored) {
  const int64_t NC = (int64_t)steps * 8 * M, blocks = (int64_t)steps * 8;
  return V * (NC + 4) * 2 + NC * 8 + blocks * 4 + (scored ? V * (NC + 4) * 4 : 0);
}
// Rows of W a thread requests at a time, where `groups` threads share a column of V rows: the fewest that need no more trips
// than 12, which used to be taken everywhere.  Requests beyond the last row are made all the same, and from |w| alone
// (62, 67, 80 and 109 registers at 4, 6, 8 and 12) the registers are workgroups less; with scores (95 and, computed on
// the fly, 143 at any number: another phase needs them) it is the requests only.  From HBM, us, with 12 / with this:
// from |w| 4096 x 4096 at 64:2:5 (6 rows) 25.5 / 22.3, V = 64, M = 12 (7) 21.0 / 18.0, 11008 x 4096 at V = 32, M = 4 (4)
// 59.1 / 50.7, 1000 x 1000 at V = 64, M = 8 (4) 7.1 / 6.6, and always 8 would lose where 11 rows then take two trips:
// 11008 x 4096 at 64:2:5 48.9 / 51.1; from scores 120 sizes 1.04 times this with 12 (up to 1.10), 1.01 with 6; a refresh
// 1.016 and 1.003 (215 sizes).
inline int prune_batch(int V, int groups) {
  const int rows = (V + groups - 1) / groups, trips = (rows + 11) / 12;
  for (const int b : {4, 6, 8}) if ((rows + b - 1) / b == trips) return b;
  return 12;
}
// Pruning from scores.  As wide as three workgroups per compute unit allow: a wider span reads longer runs of a row,
// another workgroup hides more of the dependent phases.  11008 x 4096 with at most 40 / 52 / 64 KiB of LDS, us:
// V = 64, M = 8 101.6 / 86.5 / 86.5; V = 32, M = 8 91.9 / 77.4 / 77.4; V = 32, M = 9 90.8 / 90.8 / 105.3;
// V = 128, M = 4 133 / 114 / 114; V = 64, M = 5 112 / 112 / 106; V = 32, M = 5 102 / 102 / 111.
// Narrower while there are too few workgroups for that to matter: 1024 x 1024 at V = 32, M = 4 with 128 / 256
// workgroups 10.5 / 8.8, at M = 8 9.1 / 8.6; with 160 at M = 7 9.7 against 10.3 with 320; 8 steps with 256 workgroups
// (500 x 4096, V = 32, M = 4) 11.7 against 10.8 for 4 steps.  Over 324 sizes and patterns 0.3 % from the best choice.
inline int prune_scored_steps(int V, int M, int64_t row_blocks, int64_t steps) {
  int k = 8;
  while (k > 1 && (prune_fast_lds(V, M, k, true) > 52 * 1024 || (steps + k - 1) / k * row_blocks < (k > 4 ? 512 : 160))) k >>= 1;
  return k;
}

// Pruning from RIA scores computed on the fly (mask refresh): weight tile u16 [V][NC + 4], column sums f64 [NC], kept columns
// u32 [blocks], f64 [3][NC] of the columns and [2][V] of the rows, four flags
inline int64_t prune_ria_lds(int V, int M, int steps) {
  const int64_t NC = (int64_t)steps * 8 * M, blocks = (int64_t)steps * 8;
  return V * (NC + 4) * 2 + NC * 8 + blocks * 4 + 3 * NC * 8 + 2 * V * 8 + 16;
}
// Whole refresh of 4096 x 4096, us, with 2 / 4 / 8 steps: V = 64, M = 5 98 / 82 / 91; V = 64, M = 8 75 / 69 / 85; V = 128,
// M = 5 95 / 87 / 117; V = 64, M = 12 (80 KiB at 4) 72 / 80 / 102; V = 32, M = 8 (49 KiB at 8) 82 / 69 / 70 and on 2000
// x 3000 43 / 37 / 41; V = 32, M = 4 120 / 90 / 79.  Fewer where that leaves too few workgroups: 200 x 304 at V = 128, M
// = 8 with 1 / 2 / 4 / 8 steps 32 / 34 / 36 / 55; 1000 x 1000 at V = 32, M = 8 25.0 / 24.3 / 24.4 / 30.2.
inline int prune_ria_steps(int V, int M, int64_t row_blocks, int64_t steps) {
  int k = 8;
  while (k > 1 && (prune_ria_lds(V, M, k) > (k > 4 ? 40 : 50) * 1024 || (steps + k - 1) / k * row_blocks < (k > 4 ? 512 : 160))) k >>= 1;
  return k;
}

}  // namespace vnm
