// Listed candidates with a wave per list: which calls, and how their lists are dealt to waves and workgroups.  Plain C++, so
// that the arithmetic can be checked where there is no GPU.
#pragma once
#include <cstdint>

namespace rc {

constexpr int kCandPerWg = 16;  // candidates of a workgroup, or of a wave
constexpr int kWideWaves = 8;   // waves of a workgroup, at most
constexpr int64_t kWideMostWaves = 1 << 25;

// Slots (pairs of candidates) of a wave for lists of C: two waves share a list of 17 to 32, and so on.
struct WideLists {
  int parts, per, slots;
};
inline WideLists wide_lists(int64_t C) {
  WideLists w;
  w.parts = (int)((C + kCandPerWg - 1) / kCandPerWg);
  w.per = (int)((C + w.parts - 1) / w.parts);
  w.slots = w.per <= 4 ? 2 : w.per <= 8 ? 4 : w.per <= 12 ? 6 : 8;
  return w;
}
// Calls for candidates_wide_kernel: at least half as many pairs as there are pool blocks (per layer, or in all for the
// distances), so that lists share blocks, or lists of 17 to 24 (33 to 40, ...), of which workgroups of 16 leave half a
// workgroup idle; and slots enough to keep the chip's memory pipeline full, which a workgroup per list does with fewer.
// Measured, workgroup per list -> wave per list, us (layers x pool x queries x C):
//   32 x 4096 x 256 x 16 1304 -> 1209   45 x 533 x 88 x 24 2005 -> 1245   11 x 194 x 66 x 14 102 -> 44   37 x 1823 x 795 x 19 6710 -> 4898
//   4 x 2343 x 91 x 13 (2912 slots) 118 -> 123   3 x 231 x 60 x 14 (1440) 65 -> 114   13 x 1216 x 29 x 19 (a third of the blocks) 123 -> 95
//   fewer pairs, full workgroups: 64 x 4096 x 32 x 16 340 -> 366   25 x 2810 x 48 x 9 234 -> 252   48 x 3100 x 96 x 12 (distances) 766 -> 798
// A launch has fewer than 2^32 threads along its grid, which a wave per list reaches with 2^26 waves; a workgroup per 16
// candidates of a list, three-dimensional, does not.
inline bool wide_wins(int64_t lists, int64_t Q, int64_t C, int64_t P, int block_bytes) {
  if (C < 1 || P < 1 || P > 0x7fffffffLL / block_bytes || lists > kWideMostWaves || C > (1 << 20)) return false;
  const WideLists w = wide_lists(C);
  const int64_t slots = lists * w.parts * w.slots;
  if (lists * w.parts > kWideMostWaves) return false;
  return (2 * Q * C >= P && slots >= 3000) || (C > 16 && (C - 1) % 16 < 8 && slots >= 4000);
}

// Eight waves to a workgroup, kept together by a barrier per two windows, or one: eight where they fill the rounds of 256
// workgroups (0.87 of them) and there are 3000 waves; below that compute units idle beside others with a workgroup more.
// Neighbouring lists go to one XCD while the waves of a layer are about as many as an XCD works on at once, and up to 1700
// of them (with eight to a workgroup) where a block is listed more than twice in a layer; with fewer blocks in common, all
// XCDs do better on the same part of the layer.
// One wave -> eight, us (layers x pool x queries x C): 64 x 4096 x 256 x 16 2431 -> 2120 (17.2 -> 14.7 GB from memory; the
// blocks and queries once are 11.9)   44 x 257 x 110 x 19, blocks of 128 KB 1106 -> 907   distances 58 x 988 x 125 x 22 2789 -> 2399
//   rounds filled to 0.78 to 0.85: 48 x 700 x 100 x 16 508 -> 590   64 x 500 x 130 x 6 420 -> 459;  few waves: 33 x 103 x 28 x 21 94 -> 115
// Dealt out -> by XCD, both of eight: 37 x 788 x 304 x 20 737 -> 590   29 x 1892 x 579 x 23 3040 -> 2621   4 x 1730 x 235 x 23 96 -> 72
//   17 x 4697 x 226 x 24 (a block listed 1.2 times) 853 -> 864   11 x 6837 x 609 x 17 (1.5) 2171 -> 2354   distances, 2000 waves of a
//   group, 16 x 2000 x 1000 x 20 2003 -> 2261, groups not alike, 37 x 1985 x 543 x 6 1524 -> 1911
struct WidePlan {
  WideLists lists;
  int waves;        // of a workgroup
  int64_t wgs_z;    // workgroups of a layer, or of a group of layers
  int64_t items;    // workgroups
  int64_t per_xcd;  // workgroups of an XCD's run; 0: they are dealt out one after the other
};
inline WidePlan wide_plan(int64_t Q, int64_t C, int64_t P, int64_t z, bool alike) {
  WidePlan p;
  p.lists = wide_lists(C);
  const int64_t waves = Q * p.lists.parts, wgs = z * ((waves + kWideWaves - 1) / kWideWaves);
  const int64_t rounds = (wgs + 255) / 256;  // of the 256 compute units of an MI355X
  const bool shared = waves > 448 && waves <= 1700 && alike && Q * C > 2 * P && z * waves >= 1800;
  const bool full = z * waves >= 3000 && 100 * z * waves >= 87 * rounds * 256 * kWideWaves;
  p.waves = shared || full ? kWideWaves : 1;
  p.wgs_z = (waves + p.waves - 1) / p.waves;
  p.items = z * p.wgs_z;
  p.per_xcd = waves <= 448 || shared ? (p.items + 7) / 8 : 0;
  return p;
}
inline int64_t wide_grid(int64_t items, int64_t per_xcd) { return per_xcd ? per_xcd * 8 : items; }

}  // namespace rc
