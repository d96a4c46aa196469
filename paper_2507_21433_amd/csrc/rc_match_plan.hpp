// Plans of the tile searches: which tiles, how many shares of each, how large a workspace.  Plain C++, so that the arithmetic can
// be checked where there is no GPU.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "rc.h"

namespace rc {

constexpr int kStepElements = 64;                      // of the reduction, per pipeline step
constexpr int kMaxGrid = 512;                          // workgroups of a tile-kernel launch, at most
constexpr int kScheduleHeader = (8 + kMaxGrid) * 32;   // ints ahead of the claim words of a dynamic tile schedule
// Partial selection result of one pool tile for one query.
struct Part {
  float best;
  int idx;
  float second;
  int pad;
};

// rows of the pool per selection workgroup: about 2048 workgroups, at least 32 rows each
inline int select_rows(int64_t P, int64_t Q) {
  const int64_t qtiles = (Q + 63) / 64;
  int64_t chunks = 2048 / (qtiles > 0 ? qtiles : 1);
  if (chunks < 1) chunks = 1;
  int64_t rows = (P + chunks - 1) / chunks;
  rows = (rows + 31) / 32 * 32;
  return (int)(rows < 32 ? 32 : rows);
}

// Layer-mean mode: how the L layers are split into groups.  A workgroup walks the layers of one
// group, so large problems (many tiles) use one group and write every sum once; small ones split
// the layers until there are enough workgroups to fill the chip.
struct LayerSplit {
  int G, groups;
};
inline LayerSplit layer_split(int L, int64_t tiles) {
  int64_t want = (1024 + tiles - 1) / (tiles > 0 ? tiles : 1);
  if (want < 1) want = 1;
  if (want > L) want = L;
  LayerSplit r;
  r.G = (int)((L + want - 1) / want);
  r.groups = (L + r.G - 1) / r.G;
  return r;
}

// What a launch of more than one round keeps behind the rest of the workspace: the header (counters and progress
// words, 128 bytes each) and one claim word per slot of every workgroup's walk.
constexpr int kChunk = 32;
constexpr int kStealMin = 64;
constexpr int kTailShare = 10;   // the last tenth of every list can be taken from its back
constexpr int kDynamicRounds = 16;  // launches of fewer rounds keep the fixed schedule: nothing to gain there
inline int64_t virtual_grid(int64_t total) { return (total + 8 * kChunk - 1) / (8 * kChunk) * (8 * kChunk); }
inline size_t schedule_bytes(int64_t total) {
  // the walks of a launch with fewer workgroups than kMaxGrid are longer; together they never hold more than
  // one slot per virtual workgroup plus one per workgroup
  return (size_t)(kScheduleHeader + virtual_grid(total > 0 ? total : 1) + kMaxGrid) * sizeof(int);
}
// Tile shape: with many queries a 128x128 accumulator tile per wave (all 256 accumulation registers
// of a lane) in every mode.  What is carried across phases is kept out of the fp32 register budget: the
// per-head mode packs its running minimum into 16-bit fixed point, the layer-mean mode keeps
// its running sum in the workspace (up to 128 columns in registers).
struct TileShape {
  int bp, bq;
};
constexpr TileShape kBlockTile = {256, 256};
// Few query blocks (a decoding step of a handful of requests): a 64-column tile does a quarter of
// the matrix work per pool slice and leaves the kernel to the speed of the pool stream.
constexpr TileShape kNarrowTile = {256, 64};
constexpr TileShape kMidTile = {256, 128};

// Query counts that a 256-column grid pads badly (160 queries are 1.6 times their work, 300 are 1.7 times):
// a 192-column tile, and one of 192 pool rows x 320 columns with as many accumulators as fit beside it.
constexpr TileShape kWideTile = {256, 192};
constexpr TileShape kLowTile = {192, 320};

// Tile of a search in whole tiles.  Up to 128 queries the narrow ones.  Beyond, the shape with the lowest estimate
//   rounds(shape) * (us per pipeline step of a full round, by the number of query tiles: 1, 2, more)
// where a last round of which a part r of the compute units has work takes 0.55 + 0.45 r of a full one; another
// shape than 256 x 256 is taken when it is at least 4 % below.  The constants are measured (48 layers x 4096 blocks,
// 16 layers x 4100 blocks of 32 tokens per head); where the lines lie, in us per launch, 256 / 192 / 320 columns:
//   block     Q = 160 2802 / 2487 / 3427   256 3074 / 4038 / 3903   320 4950 / 4363 / 3987   384 5072 / 4490 / 7117
//             Q = 512 5475 / 6188 / 7469   640 7470 / 7835 / 7124   960 10230 / 10388 / 10239
//   per head  Q = 160 3239 / 2647 / 2900   300 5281 / 4007 / 3519   384 4914 / 4098 / 4998   640 7213 / 7005 / 5026
constexpr TileShape kShapes[3] = {kBlockTile, kWideTile, kLowTile};
constexpr double kStepUs[2][3][3] = {{{2.0, 1.75, 1.65}, {1.67, 1.42, 1.31}, {1.69, 1.6, 1.57}},
                                     {{2.0, 2.0, 1.9}, {1.65, 1.5, 1.45}, {2.0, 1.7, 1.65}}};
// rounds of one workgroup per compute unit (an MI355X has 256), in full ones
inline double rounds_of(double wgs) {
  const double part = wgs / 256.0, full = (double)(int64_t)part;
  return part > full ? full + 0.55 + 0.45 * (part - full) : full;
}
struct TileChoice {
  TileShape ts;
  double step_us;  // estimate of the launch, in us per pipeline step of a tile (more than 128 queries)
};
inline TileChoice tile_choice(int mode, int64_t L, int64_t P, int64_t Q) {
  if (Q <= kNarrowTile.bq) return {kNarrowTile, 0.0};
  if (Q <= kMidTile.bq) return {kMidTile, 0.0};
  int best = 0;
  double best_cost = 0.0;
  for (int i = 0; i < 3; ++i) {
    const int64_t nqt = (Q + kShapes[i].bq - 1) / kShapes[i].bq;
    const double tiles = (double)(L * ((P + kShapes[i].bp - 1) / kShapes[i].bp)) * (double)nqt;
    const double cost = rounds_of(tiles) * kStepUs[mode == RC_SCORE_PER_HEAD_ALL][i][nqt < 3 ? nqt - 1 : 2];
    if (i == 0 || cost < (best == 0 ? 0.96 : 1.0) * best_cost) {
      best = i;
      best_cost = cost;
    }
  }
  return {kShapes[best], best_cost};
}
inline TileShape tile_for(int mode, int64_t L, int64_t P, int64_t Q) { return tile_choice(mode, L, P, Q).ts; }
// Columns of a tile whose reduction is shared by several workgroups: 192 where 256 pad badly.  256 -> 192 columns, us per
// launch: block, 2 layers x 4096, Q = 300 274 -> 231; per head, 3 x 11147, Q = 133 769 -> 707, 42 x 844, Q = 192 430 -> 354,
// 4 x 4096, Q = 384 579 -> 491.
inline int share_columns(int64_t Q) {
  if (Q <= kMidTile.bq) return Q <= kNarrowTile.bq ? kNarrowTile.bq : kMidTile.bq;
  return Q <= kWideTile.bq || (Q > kBlockTile.bq && Q <= 2 * kWideTile.bq) ? kWideTile.bq : kBlockTile.bq;
}

// Layer-mean search in whole tiles of 256 rows: the columns of a tile.  As in tile_for, by the cost of a step; the
// launch has rounds enough (layer_split) for their number not to matter.  64 layers x 2048 blocks, Q = 128:
// 256 columns 1962 us, 128 columns and the sums in registers 1756, its pool loads
// non-temporal 1577.
inline int mean_columns(int64_t Q) {
  if (Q <= kMidTile.bq) return share_columns(Q);
  constexpr double step_us[2][3] = {{2.0, 1.75, 1.65}, {1.67, 1.42, 1.31}};
  const int64_t n256 = (Q + 255) / 256, n192 = (Q + 191) / 192;
  return n192 * step_us[1][n192 < 3 ? n192 - 1 : 2] < 0.96 * n256 * step_us[0][n256 < 3 ? n256 - 1 : 2] ? kWideTile.bq : kBlockTile.bq;
}
// What its launch takes in us where every workgroup walks one layer (up to 1024 tiles): rounds, of a last round of which a part r of
// the compute units has work idle + (1 - idle) r, times the steps of both tensors.  More than 128 queries: the steps of the block
// score's kernels, which are shorter where query tiles share the pool slices; one step for all counts took 7 x 2094 x 534 (16 heads)
// in 4 shares, 1379 us, not whole, 1184.  Fitted to 230 timed calls of up to 256 tiles, 0.8 to 1.25 of it each.
inline double mean_tiles_us(int64_t L, int64_t P, int64_t Q, int64_t steps) {
  const int bq = mean_columns(Q);
  const int64_t nqt = (Q + bq - 1) / bq, tiles = L * ((P + 255) / 256) * nqt;
  const double step_us = bq == kNarrowTile.bq ? 1.24 : bq == kMidTile.bq ? 1.40 : kStepUs[0][bq == kWideTile.bq][nqt < 3 ? nqt - 1 : 2];
  const double idle = bq <= kMidTile.bq ? 0.55 : 0.62, part = (double)(tiles % 256) / 256.0;
  return ((double)(tiles / 256) + (part > 0.0 ? idle + (1.0 - idle) * part : 0.0)) * 2.0 * (double)steps * step_us + 8.0;
}
// byte offset of the selection partials inside the layer-mean workspace (after the sums: one
// tile of 256 x bq floats per (group, pool tile, query tile))
inline size_t layer_mean_part_offset(int groups, int64_t npt, int64_t nqt, int bq) {
  return (size_t)groups * (size_t)npt * (size_t)nqt * 256 * (size_t)bq * sizeof(float);
}

// A tile kernel launch runs in rounds of one workgroup per compute unit, and a problem with few
// tiles (a call for one layer, a small pool) leaves most of the chip idle or pays a whole round
// for a few left-over tiles.  Such problems split the reduction of every tile over S workgroups
// (S even: half of them on the K tensor, half on V).  In per-head mode the shares are the H heads (the
// score is a minimum over heads, not a sum over the reduction).
// More than 128 queries (192 or 256 columns): S is the power of two with the lowest estimated time, in units of
// one pipeline step:
//   rounds(S) * (steps of a share + 6 for filling the pipeline and storing the share)
//   + 0.03 per tile share for the pass that adds the shares + 5 for its launch,
// and the split is used when that is at least 10 % below the estimate for whole tiles.  The
// constants come from measurements of 1 to 144 tiles of the 256 x 256 shape (within 10 % from 64
// tiles up; a single layer of 16 tiles takes 116 us against 112 estimated).  A share has at least
// 8 steps; the shares of all tiles take at most 512 MB; problems of more than one round are left
// alone, but for their last layers (tail_layers).  Block mode only.
// At most 128 queries (64 and 128 columns, bound by the pool stream): a share is cheap to store, so the
// split also evens out the last round of launches of several rounds.  Estimated in us: a step of a full round
// takes 1.3 (64 columns) or 1.5 us; a round of which a part r of the compute units has work takes 0.55 + 0.45 r
// of it (a compute unit alone is not much faster than 256 together: 0.86 us per step measured at r = 1/4, 1.2 at
// r = 1/2); 5 us to fill the pipeline and store; the shares written and read at 4 TB/s and 6 us for the pass over
// them; used when that is at least 10 % below whole tiles.  S / 2 is any divisor of the steps, the head count in
// per-head mode; at most 2048 shares, 4096 for launches of more than one round (512 MB either way).
// Measured, whole tiles -> shares: per-head, 32 layers x 2531 blocks of 32 tokens, Q = 24 (320 tiles) 2120 -> 1850 us;
// 256-column shares -> these: one layer of 4096 blocks, Q = 16 (256 shares) 82 -> 53 us, one tile, Q = 32 33 -> 19 us;
// powers of two only -> any divisor: one layer of 6000 blocks of 10 heads, Q = 40 105 -> 90 us (S = 10).
// The layer-mean search goes by the block score's estimate; its selection walks all layers in one pass, which that
// does not count.  Above 256 tiles, whole tiles (a small workspace) -> shares, us: 64 layers of 8 heads, 1100 x 16 931 -> 883,
// 1280 x 64 1096 -> 1099, 1280 x 128 1243 -> 1267, 1400 x 128 1312 -> 1192; 52 x 1264 x 1, blocks of 128 KB 3545 -> 2735; 25 x
// 5134 x 1, blocks of 16 KB 746 -> 781 (the worst of 60 shapes).
// The decision depends on the shape alone (an MI355X has 256 compute units), so that the workspace
// size does not depend on the device that happens to be current.
constexpr int kSplitComputeUnits = 256;
inline int narrow_split_count(int mode, int64_t L, int64_t P, int64_t Q, int T, int H) {
  const int bq = share_columns(Q);
  const int64_t tiles = L * ((P + 255) / 256);
  const int steps = T * H * 128 / kStepElements;  // per tensor
  const double step_us = bq == kNarrowTile.bq ? 1.3 : 1.5;
  auto estimate = [&](int S) {
    const int64_t wgs = tiles * S;
    double rounds = (double)(wgs / kSplitComputeUnits);
    const double rest = (double)(wgs % kSplitComputeUnits) / kSplitComputeUnits;
    if (rest > 0.0) rounds += 0.55 + 0.45 * rest;
    const double shares = S > 1 ? (double)wgs * 256.0 * (double)Q * 8.0 / 4e6 + 6.0 : 0.0;  // written, read: 4 TB/s; a launch
    return rounds * (2.0 * steps / S * step_us + 5.0) + shares;
  };
  int best = 1;
  double best_cost = 0.9 * estimate(1);
  auto consider = [&](int S) {
    if (tiles * S > (tiles > kSplitComputeUnits ? 4096 : 2048) || estimate(S) >= best_cost) return;
    best_cost = estimate(S);
    best = S;
  };
  if (mode == RC_SCORE_PER_HEAD_ALL) {
    if (H > 1) consider(H);
  } else {
    for (int half = 1; steps / half >= 8; ++half)
      if (steps % half == 0) consider(2 * half);
  }
  return best;
}
// The rule for 256-column tiles at every query count; block mode leaves at most 128 queries alone from half a round on.
inline int wide_split_count(int mode, int64_t L, int64_t P, int64_t Q, int T, int H) {
  if (P <= 0 || Q <= 0 || L <= 0) return 1;
  const int64_t tiles = L * ((P + 255) / 256) * ((Q + 255) / 256);
  if (tiles > kSplitComputeUnits) return 1;  // more than one round: measured gains of 0-6 % only (workgroups of
                                             // later rounds start as earlier ones end, the rounds are not that rigid)
  if (mode == RC_SCORE_PER_HEAD_ALL) {
    if (H < 2 || tiles * H > 2048) return 1;
    auto rounds = [&](int64_t wgs) { return (double)((wgs + kSplitComputeUnits - 1) / kSplitComputeUnits); };
    const double whole = rounds(tiles) * (4.0 * T * H + 6.0);
    const double heads = rounds(tiles * H) * (4.0 * T + 6.0) + 0.03 * (double)(tiles * H) + 5.0;
    return heads < 0.9 * whole ? H : 1;
  }
  if (Q <= kMidTile.bq && tiles * 2 > kSplitComputeUnits) return 1;
  const int steps = T * H * 128 / kStepElements;  // per tensor
  auto estimate = [&](int S) {
    const double rounds = (double)((tiles * S + kSplitComputeUnits - 1) / kSplitComputeUnits);
    return rounds * (2.0 * steps / S + 6.0) + (S > 1 ? 0.03 * (double)(tiles * S) + 5.0 : 0.0);
  };
  int best = 1;
  double best_cost = 0.9 * estimate(1);
  for (int S = 2; tiles * S <= 2048 && 2 * steps / S >= 8 && steps % (S / 2) == 0; S *= 2) {
    const double c = estimate(S);
    if (c < best_cost) {
      best_cost = c;
      best = S;
    }
  }
  return best;
}
// The two rules above give a number of shares that divides the work evenly.  Block score and layer mean, up to a round of tiles, take
// any even number instead (the shares of a tensor are a step longer or shorter) where the estimate below is 4 to 7 % less than for
// theirs, by the width of the tiles: a round of workgroups is filled better, and shares whose first slices are a power of two of KB
// apart crowd the same memory channels.  What a launch of S shares per tile takes, in us: its rounds (of a last round of which a part r
// of the compute units has work, idle + (1 - idle) r; 256 columns: 0.75 to 0.8 of a full one from a fifth of the units to two thirds,
// and without that floor few tiles got too few shares, 2 x 512 x 209 28 of them and not 64, 63 and 61 us, the layer mean 1 x 427 x 208 53
// and 48) times the steps of a share and what it takes to fill its pipeline and store, a time per workgroup for the pass that adds it, one per layer and share for the layer mean's (a thread of it walks the shares of all
// layers: with a time per workgroup in its place 2 x 5750 x 16 153 -> 182 us, 1 x 11475 x 20 156 -> 170), and the launches behind.
// One set of constants per width of the tiles.  Fitted to 819 drawn shapes (1 to 64 layers, 64 to 16 384 blocks, 1 to 1024 queries) of
// which every number of shares was timed: with this choice a shape takes 0.4 to 2.2 % longer than with its best number, and is 1.02 to
// 1.08 times as fast as with the rules above.  None of the block score's is more than 3 % slower than by those, three of the layer
// mean's are: 1 x 699 x 220 52 -> 55 us, 1 x 1013 x 252, 32 tokens 88 -> 92, 5 x 3295 x 237, 4 heads 221 -> 231; of 140 others whose
// number changed since, the worst are 15 x 3361 x 89, 10 heads 812 -> 865 and 1 x 721 x 212 50 -> 54.  64 columns with a step of 1.14 us and 9 to fill took 2 x 8278 x 42 in 6 shares, 246 us, not the rules' 16, 236, nor 10,
// 235.  Us per call, the rules above -> this:
//   1 x 3273 x 667 269 -> 175 (6 shares)   6 x 1347 x 456, 16 heads 793 -> 604 (6)   18 x 248 x 54, blocks of 32 tokens, 10 heads 189 -> 146
//   (14)   9 x 405 x 134, 16 heads 203 -> 140 (14)   1 x 5942 x 139, 32 tokens 245 -> 181 (10)   2 x 9667 x 268, 16 heads 1036 -> 883 (8)
//   layer mean 4 x 1273 x 261, 32 tokens, 16 heads 722 -> 555 (6)   whole tiles again: 2 x 4737 x 992 664 -> 596, 1 x 12000 x 800 721 -> 618
struct ShareCost {
  double step_us, fill_us, idle, flat, wg_us, mean_share_us, launch_us;
  double margin;  // another number than the rules' is taken where its estimate is below this part of theirs
};
// `layers`: of a layer mean, 0 for the block score
inline double shares_us(const ShareCost& c, int64_t layers, int64_t wgs, int64_t steps, int S) {
  const double part = (double)(wgs % kSplitComputeUnits) / kSplitComputeUnits;
  const double last = part > 0.0 ? std::max(c.idle + (1.0 - c.idle) * part, c.flat + 0.12 * part) : 0.0;
  const double rounds = (double)(wgs / kSplitComputeUnits) + last;
  return rounds * (2.0 * (double)steps / S * c.step_us + c.fill_us) + (double)wgs * c.wg_us + (double)(layers * S) * c.mean_share_us + c.launch_us;
}
// The number of the two rules above.  192 and 256 columns cut every query count the 192 are used for into the same number of tiles.
inline int alike_split_count(int mode, int64_t L, int64_t P, int64_t Q, int T, int H) {
  if (P <= 0 || Q <= 0 || L <= 0) return 1;
  return Q <= kMidTile.bq ? narrow_split_count(mode, L, P, Q, T, H) : wide_split_count(mode, L, P, Q, T, H);
}
inline int block_split_count(bool mean, int64_t L, int64_t P, int64_t Q, int T, int H) {
  if (P <= 0 || Q <= 0 || L <= 0) return 1;
  const bool narrow = Q <= kMidTile.bq;
  const int alike = alike_split_count(RC_SCORE_BLOCK, L, P, Q, T, H);
  const int bq = share_columns(Q);
  const int64_t tiles = L * ((P + 255) / 256) * ((Q + bq - 1) / bq), steps = (int64_t)T * H * 128 / kStepElements;  // of a tensor
  if (tiles > kSplitComputeUnits) return alike;
  constexpr ShareCost costs[4] = {{1.21, 6.8, 0.58, 0.0, 0.010, 0.064, 12.0, 0.96},
                                  {1.30, 16.0, 0.54, 0.0, 0.006, 0.060, 12.0, 0.95},
                                  {1.45, 22.3, 0.56, 0.0, 0.009, 0.070, 15.0, 0.93},
                                  {1.785, 17.3, 0.45, 0.72, 0.097, 0.100, 11.0, 0.93}};
  const ShareCost& cost = costs[bq / 64 - 1];
  const int64_t layers = mean ? L : 0;
  const double whole = mean ? mean_tiles_us(L, P, Q, steps)
                       : narrow ? shares_us(cost, 0, tiles, steps, 1) - cost.launch_us + 6.0  // one share, neither added nor another launch
                                : 2.0 * (double)steps * tile_choice(RC_SCORE_BLOCK, L, P, Q).step_us + 8.0;
  int best = alike;
  double best_us = cost.margin * (alike > 1 ? shares_us(cost, layers, tiles * alike, steps, alike) : whole);
  // 8 steps of a share at least, 9 of 256 columns, whose store takes as long (1 x 516 x 256, 3 heads: 46.6 us in 24 shares of 8, 46.5 in
  // the rules' 16 of 12); 512 MB for all of them
  for (int half = 1; steps / half >= (bq == kBlockTile.bq ? 9 : 8) && tiles * 2 * half <= 2048; ++half) {
    const double us = shares_us(cost, layers, tiles * 2 * half, steps, 2 * half);
    if (us < best_us) {
      best = 2 * half;
      best_us = us;
    }
  }
  return whole < best_us ? 1 : best;
}
inline int split_count(int mode, int64_t L, int64_t P, int64_t Q, int T, int H) {
  return mode == RC_SCORE_BLOCK ? block_split_count(false, L, P, Q, T, H) : alike_split_count(mode, L, P, Q, T, H);
}

struct SplitLayout {
  int S, bq;
  int64_t npt, nqt;
  int sel_rows;
  int64_t nchunks;
  size_t part_offset, bytes;
};
inline SplitLayout split_layout(int S, int64_t L, int64_t P, int64_t Q) {
  SplitLayout r;
  r.S = S;
  r.bq = share_columns(Q);
  r.npt = (P + 255) / 256;
  r.nqt = (Q + r.bq - 1) / r.bq;
  r.sel_rows = select_rows(P, Q);
  r.nchunks = (P + r.sel_rows - 1) / r.sel_rows;
  r.part_offset = (size_t)L * (size_t)S * (size_t)r.npt * (size_t)r.nqt * 256 * (size_t)r.bq * sizeof(float);
  r.bytes = r.part_offset + (size_t)L * (size_t)r.nchunks * (size_t)Q * sizeof(Part);
  return r;
}

// ---- What a call computes depends on the workspace it is given as well: the plan of the rules above needs from tens of
// KB (whole tiles) to 512 MB (shares), up and down with Q and P, and an engine that keeps one workspace for all its calls
// must not be refused for a small step.  So every call takes a workspace of `floor` bytes, the need of the plan with
// 256-column shares by wide_split_count or else with pool tiles of 256 rows, and uses the faster plan where it fits, the plan with
// shares that are all alike where only that does.
struct MatchPlan {
  int S;         // shares per tile, 1 = whole tiles of shape ts
  TileShape ts;
};
inline size_t whole_tiles_bytes(TileShape ts, int64_t L, int64_t P, int64_t Q) {
  const int64_t npt = (P + ts.bp - 1) / ts.bp, nqt = (Q + ts.bq - 1) / ts.bq;
  const int64_t n = L * (npt > 0 ? npt : 1) * Q;
  return (size_t)(n > 0 ? n : 1) * sizeof(Part) + schedule_bytes(L * npt * nqt);
}
inline TileShape floor_tile(int64_t Q) {
  return Q <= kNarrowTile.bq ? kNarrowTile : Q <= kMidTile.bq ? kMidTile : kBlockTile;
}
// shares of 256 columns (256 KB each) and the partials of the pool chunks
inline size_t wide_shares_bytes(int S, int64_t L, int64_t P, int64_t Q) {
  const SplitLayout sl = split_layout(S, L, P, Q);
  return sl.bytes - sl.part_offset + (size_t)L * (size_t)S * (size_t)sl.npt * (size_t)((Q + 255) / 256) * 65536 * sizeof(float);
}
inline size_t match_floor_bytes(int mode, int64_t L, int64_t P, int64_t Q, int T, int H) {
  const int S = wide_split_count(mode, L, P, Q, T, H);
  return S > 1 ? wide_shares_bytes(S, L, P, Q) : whole_tiles_bytes(floor_tile(Q), L, P, Q);
}
inline size_t plan_bytes(const MatchPlan& p, int64_t L, int64_t P, int64_t Q) {
  return p.S > 1 ? split_layout(p.S, L, P, Q).bytes : whole_tiles_bytes(p.ts, L, P, Q);
}
// The plan of a call with `avail` bytes, at least match_floor_bytes().
inline MatchPlan match_plan(int mode, int64_t L, int64_t P, int64_t Q, int T, int H, size_t avail) {
  MatchPlan p = {split_count(mode, L, P, Q, T, H), tile_for(mode, L, P, Q)};
  if (plan_bytes(p, L, P, Q) > avail) p.S = alike_split_count(mode, L, P, Q, T, H);
  if (plan_bytes(p, L, P, Q) > avail) p = {wide_split_count(mode, L, P, Q, T, H), floor_tile(Q)};
  return p;
}

// A launch of whole tiles whose last round leaves most compute units idle gives its last layers to a launch of shares, which
// runs first: the number of layers with the lowest estimate in us, 0 = none.  Whole tiles by tile_choice; shares by rounds of
// them, with 6 steps to fill the pipeline and store each, 0.06 us for the pass that adds one, 20 us for the four further
// launches and the drain between.  Used where that is 4 % below whole tiles alone, 2 % per head (there whole tiles take 10 %
// longer than estimated, shares as long).  For blocks of 32 KB of K and V and larger (smaller ones, whose round is short beside
// what the launches cost, were not measured).  Of 150 drawn shapes that get a tail the median is 1.11 times as fast and one is more
// than 0.5 % slower; whole tiles -> these, us:
//   block     40 x 6209 x 300, 10 heads 6288 -> 5961 (2 layers)   3 x 15320 x 412, 16 heads 2865 -> 2448 (1)   14 x 4673 x 382, 10 heads
//             2431 -> 2091 (1)   45 x 6258 x 187 3919 -> 3714 (5)   8 x 8530 x 139, 4 heads 682 -> 558 (1)   38 x 2867 x 338,
//             blocks of 32 tokens 5496 -> 5481 (6)   the least: 9 x 2100 x 982, 10 heads 1559 -> 1580, 3 x 9666 x 592 1160 -> 1176 (in two runs)
//             left alone: 7 x 4960 x 883, 16 heads 3630, 3728 with a tail of 1
//   per head  11 x 6340 x 216, 32 tokens 3692 -> 2400 (1)   39 x 2005 x 195 2028 -> 1528 (7)   5 x 6409 x 415, 10 heads 2040 -> 1596 (1)
//             left alone: 38 x 2048 x 890, 10 heads 6234, 6431 with a tail of 1
// Layers are searched in one way each, so identical pool blocks of a layer still see the same instructions.
inline int tail_layers(int mode, int64_t L, int64_t P, int64_t Q, int T, int H) {
  if (Q <= kMidTile.bq || P <= 0 || L < 2 || T * H < 64) return 0;
  const double steps = 4.0 * T * H;
  const int64_t tiles = L * ((P + 255) / 256) * ((Q + 255) / 256);
  if (tiles <= kSplitComputeUnits || tiles >= kDynamicRounds * kSplitComputeUnits) return 0;
  const int bq = share_columns(Q), shape = bq == kWideTile.bq ? 1 : 0;
  const int64_t nqt = (Q + bq - 1) / bq, per_layer = (P + 255) / 256 * nqt;
  const double step_us = kStepUs[mode == RC_SCORE_PER_HEAD_ALL][shape][nqt < 3 ? nqt - 1 : 2];
  const double margin = mode == RC_SCORE_PER_HEAD_ALL ? 0.98 : 0.96;
  int best = 0;
  double best_us = margin * steps * tile_choice(mode, L, P, Q).step_us;
  for (int n = 1; n < L && n * per_layer <= kSplitComputeUnits; ++n) {
    const int S = wide_split_count(mode, n, P, Q, T, H);
    if (S < 2) continue;
    const double wgs = (double)(n * per_layer * S);
    const double us = steps * tile_choice(mode, L - n, P, Q).step_us + rounds_of(wgs) * (steps / S + 6.0) * step_us + 0.06 * wgs + 20.0;
    if (us < best_us) {
      best = n;
      best_us = us;
    }
  }
  return best;
}
// bytes for both launches, which take the workspace in turn
inline size_t tail_bytes(int n, int mode, int64_t L, int64_t P, int64_t Q, int T, int H) {
  const MatchPlan head = {1, tile_for(mode, L - n, P, Q)}, tail = {wide_split_count(mode, n, P, Q, T, H), kBlockTile};
  return std::max(plan_bytes(head, L - n, P, Q), plan_bytes(tail, n, P, Q));
}

// The layer-mean search, in the same way: whole tiles of mean_columns() columns, or shares by the block score's rule.
inline size_t mean_tiles_bytes(int L, int64_t P, int64_t Q) {
  const int bq = mean_columns(Q);
  const int64_t npt = (P + 255) / 256, nqt = (Q + bq - 1) / bq;
  const int sel_rows = select_rows(P, Q);
  const int64_t nchunks = (P + sel_rows - 1) / sel_rows;
  return layer_mean_part_offset(layer_split(L, npt * nqt).groups, npt, nqt, bq) +
         (size_t)(nchunks > 0 ? nchunks : 1) * (size_t)(Q > 0 ? Q : 1) * sizeof(Part);
}
inline size_t mean_plan_bytes(int S, int L, int64_t P, int64_t Q) {
  return S > 1 ? split_layout(S, L, P, Q).bytes : mean_tiles_bytes(L, P, Q);
}
inline size_t mean_floor_bytes(int L, int64_t P, int64_t Q, int T, int H) {
  const int S = wide_split_count(RC_SCORE_BLOCK, L, P, Q, T, H);
  return S > 1 ? wide_shares_bytes(S, L, P, Q) : mean_tiles_bytes(L, P, Q);
}
// Shares per tile of a call with `avail` bytes, at least mean_floor_bytes(); 1 = whole tiles.
inline int mean_split_count(int L, int64_t P, int64_t Q, int T, int H, size_t avail) {
  for (const int S : {block_split_count(true, L, P, Q, T, H), alike_split_count(RC_SCORE_BLOCK, L, P, Q, T, H)})
    if (mean_plan_bytes(S, L, P, Q) <= avail) return S;
  return wide_split_count(RC_SCORE_BLOCK, L, P, Q, T, H);
}

}  // namespace rc
