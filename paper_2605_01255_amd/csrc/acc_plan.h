// Host-side choices by size: which tile a product takes, how a float32 sketch is formed, and the table of raised LDS limits.
// Plain C++ with no HIP in it, so that the choices can be checked without a GPU.
#pragma once
#include <stdint.h>

#include <mutex>

namespace acc {

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

// Which kernel and tile a product takes: the least of six estimates, launch + rounds x (cost of a tile + K tiles x time of
// a K tile), in nanoseconds, with rounds = tiles over 256 compute units.  A larger tile needs fewer bytes from L2 per
// multiply-add (a 128 x 128 K tile multiplies for 0.2 us and takes 0.36 to move, however many stages are in flight), a
// smaller one leaves fewer compute units idle.  From two rounds on, two work-groups of two stages per compute unit cover
// each other's waits better than one of four (4096 x 2048 x 2048 on 128 x 128: 34 against 41 us).  The constants are fits
// to 45 shapes from 256 x 512 x 512 to 16384 x 3072 x 8192, good to about 15 %.  256 x 192 is there for the shapes that it
// makes one full round of: 4096 x 3072 x 3072 62 us (192 tiles of 256 x 256: 72), 8192 x 1032 x 4096 68 (73); where both fill
// the chip the persistent 256 x 256 kernel is ahead (16384 x 3072 x 3072: 255).  Measured us on 256 x 256 / 192 x 128 /
// 128 x 128 / 128 x 64 / 64 x 64, with what the kernels this replaced took (256 x 256 from 192 tiles on, else a two-stage
// 128 x 128) in brackets:
//   16384 x 3072 x 3072 228 / 293 / 286 /  - /  - [228]    16384 x 1152 x 3072 139 / 116 / 129 / 166 / 222 [139]
//   6000 x 4096 x 4096  188 / 168 / 180 /  - /  - [188]    4096 x 2048 x 2048   53 /  38 /  34 /  41 /   - [35]
//   4096 x 1024 x 3072   71 /  30 /  29 / 30 / 39 [36-41]  1053 x 3048 x 1600   35 /  18 /  15 /  17 /  22
//   384 x 3072 x 3072    57 /  28 /  23 / 17 / 16 [34]     2048 x 1024 x 1024   27 /  14 /  12 / 9.0 / 9.4
// In one round three stages in flight are as good as four or better, the LDS they leave free included (2049 x 1544 x 1032 on
// 128 x 128: 13.7 us against 14.2; 2049 x 1032 x 1544 17.3 and 17.8; 192 x 128 2 to 3 % likewise).
enum class GemmTile { k256, k256x192, k192x128, k128, k128x64, k64 };
struct GemmChoice {
  GemmTile tile;
  bool one_round;
};
static inline GemmChoice pick_gemm_tile(int64_t M, int64_t N, int64_t K, bool persist_ok) {
  struct Cost { GemmTile tile; int bm, bn, launch, per_tile, per_k, alone_per_tile, alone_per_k; };  // alone: one round
  static const Cost costs[] = {{GemmTile::k256, 256, 256, 5000, 2000, 1330, 2000, 1330},
                               {GemmTile::k256x192, 256, 192, 3000, 3500, 1180, 5000, 1120},
                               {GemmTile::k192x128, 192, 128, 3000, 1700, 580, 3500, 500},
                               {GemmTile::k128, 128, 128, 3000, 2000, 460, 3000, 370},
                               {GemmTile::k128x64, 128, 64, 3000, 1500, 280, 1500, 260},
                               {GemmTile::k64, 64, 64, 3000, 500, 200, 500, 230}};
  const int64_t kt = ceil_div(K, 64);
  GemmChoice best{GemmTile::k128, true};
  int64_t best_ns = INT64_MAX;
  for (const Cost& c : costs) {
    if (c.tile == GemmTile::k256 && !persist_ok) continue;
    const int64_t rounds = ceil_div(ceil_div(M, c.bm) * ceil_div(N, c.bn), 256);
    int64_t per_k = rounds == 1 ? c.alone_per_k : rounds * c.per_k;
    if (c.tile == GemmTile::k64 && rounds == 2) per_k = 300;  // the second tile hides in the first one's waits
    const int64_t ns = c.launch + rounds * (rounds == 1 ? c.alone_per_tile : c.per_tile) + kt * per_k;
    if (ns < best_ns) { best_ns = ns; best = GemmChoice{c.tile, rounds == 1}; }
  }
  return best;
}

// Which kernel the product of two gradient factors takes, whose contraction is their rank.  Up to 256 elements there are four K
// tiles at most and no pipeline to fill: a tile costs its latency, its write and, where it is added to C, its read, and work-groups
// that share a compute unit cover each other's.  So the ring kernel with two stages and as many work-groups as LDS holds (128 x 64
// three, 64 x 64 added to C five; written 64 x 64 tiles have three stages, three work-groups), larger tiles where the output gives
// every compute unit several; one work-group per compute unit with everything requested at once, the three-stage kernel of 192 x 192
// tiles, lost by 41 % on average over 84 outputs of at most one round of it (512 x 512 at rank 256 8.6 us against 3.8, 1032 x 1544
// at rank 128 7.1 against 4.4, 3072 x 1024 at rank 256 9.1 against 5.7, 3072 x 3072 at 256 11.3 against 10.9, behind the exact products
// of a pass 11.4 to 14.2 against 10.8 to 13.4).
//   written        the least of base + (tiles of the fullest compute unit) x (tile + K tiles x time of one), in nanoseconds,
//                  and from three K tiles on the persistent kernel's: 1.3 % behind the best of nine candidates on average over
//                  138 outputs (13 % at most), 3 % where C is float.  A fourth 128 x 64 tile on a compute unit, which holds three, is
//                  priced as the second batch it is; a fourth 64 x 64, of which it holds three too, by less, its time a tile being
//                  fitted to many batches (8192 x 8192 at rank 256, 64 to a compute unit: 77.9 us; 4672 x 1792 at rank 32, eight: 8.3
//                  us, 192 x 128 7.2)
//   added to C     by size: the read of C counts more than the products.  The three-stage kernel requests C with its operands
//                  and stays where its one round is nearly full (3072 x 3072 at rank 64: 10.6 us, 128 x 64 10.9) and at short ranks
//                  of outputs beyond 1024 of its tiles (8192 x 8192 at rank 64: 67 us, 128 x 64 88).  2.2 % behind the best on
//                  average (14 % at most), 1 % where C is float
// Above 256 the estimates of the exact products (pick_gemm_tile) hold; but a bfloat16 C that is added to keeps the three-stage kernel
// where that makes one full round (3072 x 3072 at r = 512 19.0 us, 128 x 64 tiles 20.0; at 1024 27.0 and 29.8).
enum class FactorTile { k64, k128x64, k128, k192x128, kThreeStage, kPersist, kAsExact };
constexpr int64_t kFactorMaxK = 256;
static inline FactorTile pick_factor_tile(int64_t M, int64_t N, int64_t K, bool bf16_c, bool sum) {
  auto tiles = [&](int64_t bm, int64_t bn) { return ceil_div(M, bm) * ceil_div(N, bn); };
  const int64_t t192 = tiles(192, 192);
  const bool full_round = bf16_c && sum && t192 <= 256 && tiles(128, 64) > 768;   // of the three-stage kernel
  if (K > kFactorMaxK) return full_round && K <= 1024 ? FactorTile::kThreeStage : FactorTile::kAsExact;
  if (sum) {
    if (K > 192 && tiles(192, 128) >= 2048) return FactorTile::k192x128;
    if (!bf16_c || tiles(64, 64) <= 768) return FactorTile::k64;
    return full_round || (t192 > 1024 && K <= 128) ? FactorTile::kThreeStage : FactorTile::k128x64;
  }
  struct Cost { FactorTile tile; int bm, bn, base, per_tile, per_k; };
  static const Cost costs[] = {{FactorTile::k64, 64, 64, 3000, 450, 180},
                               {FactorTile::k128x64, 128, 64, 3000, 600, 270},
                               {FactorTile::k128, 128, 128, 3200, 1300, 430},
                               {FactorTile::k192x128, 192, 128, 3600, 1700, 580},
                               {FactorTile::kPersist, 256, 256, 3500, 3500, 1400}};
  const int64_t kt = ceil_div(K, 64);
  FactorTile best = FactorTile::k64;
  int64_t best_ns = INT64_MAX;
  for (const Cost& c : costs) {
    if (c.tile == FactorTile::kPersist && !(bf16_c && K > 128)) continue;
    const int64_t per_cu = ceil_div(tiles(c.bm, c.bn), 256);
    int64_t ns = c.base + per_cu * (c.per_tile + kt * c.per_k);
    if (per_cu > 3) ns += c.tile == FactorTile::k128x64 ? 900 : c.tile == FactorTile::k64 ? 200 : 0;   // three are resident
    if (ns < best_ns) { best_ns = ns; best = c.tile; }
  }
  return best;
}

// Token splits of the sketch contraction: enough work-groups to fill 256 CUs, at most 32 partials.
static inline int generic_sketch_splits(int64_t n, int64_t c, int64_t r) {
  const int64_t tiles = ceil_div(c, 64) * ceil_div(r, 64);
  int64_t g = ceil_div(1024, tiles);
  const int64_t max_by_k = ceil_div(n, 256);
  if (g > max_by_k) g = max_by_k;
  if (g > 32) g = 32;
  if (g < 1) g = 1;
  return (int)g;
}

constexpr int64_t kMaxOperandBytes = 0xFFFFFFFFll;  // buffer resources address 4 GiB

// Slabs and token splits of the bfloat16 sketch with 64 sketch columns, one work-group per compute unit at most.  `most`: the splits
// that slabs of 512 channels make; never more, the workspace holds those.
struct SketchSplit {
  int ch;          // channels of a slab
  int64_t splits;
  bool two_sums;   // fewer splits than `most`: even and odd stages are summed apart, so that no running sum gets longer
};

// Work-groups on the fullest of the eight dies: a die takes whole pairs of slab and split with all their column slices, and has 32
// compute units.
static inline int64_t sketch_groups_of_a_die(int64_t slabs, int64_t columns, int64_t splits) {
  return ceil_div(slabs * splits, 8) * columns;
}

// The splits of 512 channels, on slabs narrowed as far as that makes one work-group per compute unit at most (two of them on one
// get in each other's way: 4096 x 1024 at rank 256, 128 / 256 / 512 work-groups of 512 / 256 / 128 channels 12.2 / 10.6 / 11.5 us;
// 1622 x 1408 at rank 384, 36 work-groups of 256 channels on two dies 29.1 us of a pass, 18 of 512 27.0).
static inline SketchSplit narrow_sketch_slabs(int64_t n, int64_t channels, int64_t r, int64_t most) {
  const int64_t made = ceil_div(n, round_up(ceil_div(n, most), 32)), columns = ceil_div(r, 64);
  int ch = 512;
  while (ch > 128 && sketch_groups_of_a_die(ceil_div(channels, ch / 2), columns, made) <= 32) ch /= 2;
  return SketchSplit{ch, most, false};
}

// Or fewer splits on narrower slabs, where that is the less by an estimate,  start + iterations of 32 tokens x one + partial tiles
// written and read back,  in nanoseconds: narrow slabs generate S more often, but half as many splits of twice the tokens write
// half as many partials, which is what a sketch of a few thousand tokens spends a third of its time on.  Three quarters of the
// splits at most (8 splits for 10 lose, 2500 x 2048 at rank 256 37.1 us against 34.4) and 0.23 us ahead; at most twice the stages, so
// that neither of the two sums has more of them than a split had; and no die with more work-groups than compute units (21418 x 448
// at rank 384, 36 on two of them: 43.6 us of a pass against 38.6).
// Fitted to 278 forward passes (256 to 32768 tokens, 256 to 8192 channels, rank 16 to 512, 64 to 3072 outputs), of which it
// takes fewer splits in 51: 8.9 % ahead of the splits of 512 channels there on average, behind in none.  us, the splits of 512
// channels / chosen: 4096 x 4096 at rank 128 56.1 / 52.3, 2048 x 4096 at 256 46.8 / 41.8, 600 x 8192 at 256 53.0 / 49.6, 1500 x
// 5120 at 256 52.1 / 46.0, 4096 x 1024 at 256 27.1 / 26.0; 4096, 6000 and 16384 x 3072 at 256 stay, and 15018 x 2208 at 128
// (75.0, 77.0 with 14 splits for 25).
static inline SketchSplit pick_sketch_split(int64_t n, int64_t channels, int64_t r, int64_t most) {
  struct Cost { int ch, start, per_iteration; };
  static const Cost costs[] = {{512, 1450, 477}, {256, 700, 372}, {128, 0, 264}};
  const int64_t stages = ceil_div(ceil_div(n, most), 32), made = ceil_div(n, stages * 32);
  auto estimate = [&](const Cost& c, int64_t iterations, int64_t splits) {
    return c.start + iterations * c.per_iteration + splits * channels * r * 4 / 1000 * 172 / 1000;
  };
  SketchSplit best = narrow_sketch_slabs(n, channels, r, most);
  int64_t best_ns = INT64_MAX;
  for (const Cost& c : costs)
    if (c.ch == best.ch) best_ns = estimate(c, stages, made) - 230;
  for (const Cost& c : costs) {
    int64_t full = 256 / (ceil_div(channels, c.ch) * ceil_div(r, 64));
    if (full > most) full = most;
    for (int64_t splits : {full, full / 2}) {
      if (splits < 1) continue;
      const int64_t iterations = ceil_div(ceil_div(n, splits), 32), fewer = ceil_div(n, iterations * 32);
      if (iterations > 2 * stages || 4 * fewer > 3 * made) continue;
      if (sketch_groups_of_a_die(ceil_div(channels, c.ch), ceil_div(r, 64), fewer) > 32) continue;
      const int64_t ns = estimate(c, iterations, fewer);
      if (ns < best_ns) { best_ns = ns; best = SketchSplit{c.ch, splits, true}; }
    }
  }
  return best;
}

// Plan of the sketch of `channels` columns of an [n, ld] matrix.
struct SketchPlan {
  bool fast;             // the tuned kernel
  int ch, rc;            // its tile: channels x sketch columns
  int n_cslab, n_js, G;  // channel slabs, column slices, token splits
  int tokens_per_split;
  bool two_sums;
  int room;              // partial tiles that the workspace holds, at least G
};
static inline SketchPlan plan_sketch(int64_t n, int64_t channels, int64_t r, int64_t ld, bool bf16_io, bool bf16_factor, bool one_launch) {
  SketchPlan sp{};
  sp.fast = bf16_io && n * ld * 2 <= kMaxOperandBytes && channels * r * 4 <= kMaxOperandBytes / 2;
  if (!sp.fast) {
    sp.G = sp.room = generic_sketch_splits(n, channels, r);
    return sp;
  }
  auto operand_fits = [&](int64_t tokens) { return tokens * ld * 2 + 64 * ld * 2 <= kMaxOperandBytes; };
  // 8-wave tiles of 512 channels as a rule, one work-group per compute unit.  64 sketch columns (64 accumulators per
  // lane) by default: half the partial bytes of the 128-column tile for the same generator and matrix work.
  // The 128-column tile stays where eight or more column slices would re-read a long token range from L2
  // (measured: r = 512 at 65536 tokens), and in the one-launch kernel, which interleaves it with GEMM tiles;
  // the choice must be the same in every call that sees this descriptor (workspace size, forward, backward).
  sp.ch = 512;
  const bool wide = r % 128 == 0 && (one_launch || (r > 256 && n > 32768));
  sp.rc = wide ? 128 : 64;
  sp.n_cslab = (int)ceil_div(channels, sp.ch);
  sp.n_js = (int)ceil_div(r, sp.rc);  // the last column slice may be partly empty (rank % 64 != 0)
  int64_t G = 256 / ((int64_t)sp.n_cslab * sp.n_js);  // never more work-groups than compute units
  const int64_t max_by_tokens = ceil_div(n, 256);
  if (G > max_by_tokens) G = max_by_tokens;
  if (G > 64) G = 64;
  if (G < 1) G = 1;
  auto tokens = [&](int64_t splits) { return round_up(ceil_div(n, splits), 32); };
  sp.room = (int)ceil_div(n, tokens(G));
  if (!wide) {
    // a float factor shows the order of its sums and keeps that of the splits of 512 channels
    SketchSplit c = bf16_factor ? pick_sketch_split(n, channels, r, G) : narrow_sketch_slabs(n, channels, r, G);
    if (c.two_sums && !operand_fits(tokens(c.splits))) c = narrow_sketch_slabs(n, channels, r, G);
    sp.ch = c.ch;
    sp.two_sums = c.two_sums;
    G = c.splits;
  }
  sp.tokens_per_split = (int)tokens(G);
  sp.G = (int)ceil_div(n, sp.tokens_per_split);
  sp.n_cslab = (int)ceil_div(channels, sp.ch);
  if (!operand_fits(sp.tokens_per_split)) {
    sp.fast = false;
    sp.G = sp.room = generic_sketch_splits(n, channels, r);
  }
  return sp;
}

// Which tile a float32 product takes: the least time of a K tile of 32, fixed + tiles per compute unit x per_tile nanoseconds.
// The matrix pipe bounds all of them, so the estimates follow the area, and a small tile only loses by its operands' latency;
// what decides is how many tiles the fullest compute unit gets.  Two stages and as many work-groups as LDS holds (64 x 64 five,
// 64 x 32 six, 32 x 32 eight): they start, wait and store at different times, which is worth more than transfers further ahead
// (2048 x 2048 x 1024 66.5 us against 70.7 on 128 x 64 with three stages, two work-groups; 2504 x 1000 x 3000 128 against 160
// on 64 x 32 with four).  Only where 32 x 32 tiles are 2.5 or fewer to a compute unit, or 64 x 32 one, there is nobody to cover
// a wait: four stages; so too up to four 32 x 32 to a compute unit where the contraction is long (1 to 4 % over seven products
// of 1472 to 3392 elements: 405 x 1728 x 3392 58.2 us against 60.3; six shorter ones are 1 to 2 % ahead with two).  128 x 64
// where it is two or three to a compute unit, all of them resident: as fast as four of 64 x 64, with a quarter less to move,
// and ahead of six, of which five are (2337 x 2496 x 1472 138 us and 158, 2500 x 2304 x 1024 96 and 111).  Constants fitted to
// 150 measurements (50 shapes from 128 x 128 x 4096 to 4096 x 4096 x 1024 in three orders of the operands): the chosen form is
// 2.9 % behind the best of eleven on average, 13 % at most (three and four stages everywhere and their own fit: 5.4 and 29 %).
// Measured us, 64 x 64 / 64 x 32 / 32 x 32, the chosen one marked [before]:
//   2048 x 2048 x 1024  68 / 79  / 85 (67* on 128 x 64) [69-71]     2048 x 1024 x 2048  71* / 73 / 89 [72]
//   300 x 4096 x 2048   70  / 56* / 58 [57]                         2504 x 1000 x 3000  143 / 129* / 166 [159]
//   4096 x 4096 x 1024  255* / 288 / 346 [264]                      3072 x 1024 x 3072  148* / 152 / 196 [163]
//   256 x 512 x 256     8.0 / 10.3 / 6.1* [6.1]                     3000 x 3000 x 1000  147* / 159 / 191 [162]
enum class F32TileShape { k64, k32, k128x64, k64x32 };
struct F32Choice {
  F32TileShape tile;
  int ns_per_k;   // estimate of a K tile
  bool deep;      // 32 x 32 and 64 x 32: four stages
};
// k: elements of a split's contraction.
static inline F32Choice pick_f32_tile(int64_t M, int64_t N, int64_t k, int64_t splits, bool all_tiles) {
  struct Cost { F32TileShape tile; int bm, bn, per_tile, fixed, resident, more_per_tile, more_fixed; };  // more: above `resident`
  static const Cost costs[] = {{F32TileShape::k64, 64, 64, 460, 100, 5, 460, 100}, {F32TileShape::k32, 32, 32, 145, 100, 8, 145, 100},
                               {F32TileShape::k64x32, 64, 32, 227, 115, 6, 225, 370}, {F32TileShape::k128x64, 128, 64, 950, 0, 3, 950, 0}};
  F32Choice best{F32TileShape::k64, 0, false};
  int64_t best_ns = INT64_MAX;
  for (int i = 0; i < (all_tiles ? 4 : 2); ++i) {
    const int64_t tiles = ceil_div(M, costs[i].bm) * ceil_div(N, costs[i].bn) * splits, per_cu = ceil_div(tiles, 256);
    if (costs[i].tile == F32TileShape::k128x64 && (per_cu < 2 || per_cu > 3)) continue;
    const Cost& c = costs[i];
    const int64_t ns = per_cu <= c.resident ? c.fixed + per_cu * c.per_tile : c.more_fixed + per_cu * c.more_per_tile;
    if (ns < best_ns) {
      best_ns = ns;
      best = F32Choice{c.tile, (int)(ns < INT32_MAX ? ns : INT32_MAX), tiles <= (c.tile != F32TileShape::k32 ? 256 : k < 1280 ? 640 : 1024)};
    }
  }
  return best;
}

// Whether a float32 layer's sketch (an M x N product in `splits` token splits) and its exact product (n x out_n) share a launch,
// which has one tile for both: where each would take 32 x 32 by itself.  Always with four stages, also where one of them alone
// has enough work-groups for two (`deep` is false): the other one's are there beside them, and a launch less is worth more than
// either.  us of a forward pass, two launches / shared with two stages / with four, 108 measured, shared with four never behind
// the two launches and at most 3 % behind two stages (d_in x d_out, tokens; the sketch's work-groups first, where the other order
// is ahead by up to 13 %, see gemm_f32_pair_kernel):
//   1 product of the two not deep: 256 x 512, 2624 19.1 / 14.6 / 14.9     384 x 768, 1024 23.5 / 18.5 / 17.9   3072 x 384, 256 40.2 / 45.8 / 36.7
//   both deep:                     256 x 512, 256  11.8 / 7.5 / 7.4       1544 x 512, 512 26.5 / 25.7 / 21.6   3072 x 768, 300 38.6 / 43.0 / 34.5
static inline bool f32_pair(int64_t M, int64_t N, int64_t splits, int64_t n, int64_t out_n) {
  return pick_f32_tile(M, N, 0, splits, true).tile == F32TileShape::k32 && pick_f32_tile(n, out_n, 0, 1, true).tile == F32TileShape::k32;
}

// How the sketch of a float32 layer is formed.  Stored: S is written once, into the part of the workspace that the partial
// products leave free (the libm-grade generator then runs once per entry of S instead of once per entry and 64 channels),
// with token splits enough to fill the chip as far as that room goes; one split writes a float32 factor directly.  Generic:
// S is generated inside the product, all splits that there is room for.  When S takes nearly all the room, one or two
// splits are left, K tiles in series that few work-groups share, and the generic form is ahead.  The lesser of
//   stored    4.6 us + 4 per million entries of S + K tiles of a split x a K tile's time (1.15 of pick_f32_tile's: both
//             operands have their rows contiguous) + 5 us where partial products are added up
//   generic   5 us + 256 tokens of a split x (20 us + 8 per work-group of 64 x 64 on a compute unit)
// Measured us, tokens x channels at rank: stored / generic
//   8192 x 256 r = 64    80 / 34     16384 x 512 r = 16  150 / 71     32768 x 1024 r = 64  300 / 153   (one split)
//   4096 x 256 r = 64    42 / 29     3000 x 256 r = 256   35 / 28     65536 x 2048 r = 32  586 / 449
//   2048 x 256 r = 64    24 / 27     14000 x 512 r = 64   40 / 62     24000 x 1024 r = 64   63 / 118   (four)
//   60000 x 2048 r = 32  263 / 402   8192 x 512 r = 64    20 / 41     4096 x 4096 r = 256   93 / 194
struct F32SketchPlan {
  bool stored;
  int64_t splits, k_per_split;
};
static inline F32SketchPlan plan_f32_sketch(int64_t n, int64_t channels, int64_t r, bool f32_factor) {
  const int64_t count = channels * r, s_size = n * r, generic_splits = generic_sketch_splits(n, channels, r);
  const int64_t room = generic_splits * count;
  F32SketchPlan plan{false, 0, 0};
  if (s_size > room) return plan;
  int64_t G = ceil_div(256, ceil_div(channels, 32) * ceil_div(r, 32));
  if (G > ceil_div(n, 256)) G = ceil_div(n, 256);
  if (G > (room - s_size) / count) G = (room - s_size) / count;
  if (G < 1) {
    if (!f32_factor) return plan;
    G = 1;
  }
  plan.k_per_split = round_up(ceil_div(n, G), 32);
  plan.splits = ceil_div(n, plan.k_per_split);
  const double k_tile = 1.15 * pick_f32_tile(channels, r, plan.k_per_split, plan.splits, true).ns_per_k;
  const double stored = 4600 + 0.004 * s_size + plan.k_per_split / 32 * k_tile + (plan.splits > 1 || !f32_factor ? 5000 : 0);
  const int64_t groups = ceil_div(generic_splits * ceil_div(channels, 64) * ceil_div(r, 64), 256);
  const double generic = 5000 + ceil_div(n, generic_splits) / 256.0 * (20000 + 8000 * groups);
  plan.stored = stored < generic;
  return plan;
}

// Kernels whose dynamic-LDS limit has been raised, and on which devices (the attribute sticks to the function, so it is set
// once per kernel and device, not per launch).  Shared by all host threads; holds every kernel of the library.
class RaisedLimits {
 public:
  static constexpr int kKernels = 512, kDevices = 64;
  bool has(const void* kernel, int device) {
    std::lock_guard<std::mutex> lock(mutex_);
    for (int i = 0; i < count_; ++i)
      if (entries_[i].kernel == kernel) return device >= 0 && device < kDevices && (entries_[i].devices >> device & 1);
    return false;
  }
  void add(const void* kernel, int device) {
    if (device < 0 || device >= kDevices) return;
    std::lock_guard<std::mutex> lock(mutex_);
    int i = 0;
    while (i < count_ && entries_[i].kernel != kernel) ++i;
    if (i == kKernels) return;
    if (i == count_) entries_[count_++] = Entry{kernel, 0};
    entries_[i].devices |= (uint64_t)1 << device;
  }

 private:
  struct Entry { const void* kernel; uint64_t devices; };
  Entry entries_[kKernels];
  int count_ = 0;
  std::mutex mutex_;
};

}  // namespace acc
