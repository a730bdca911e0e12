// The launch plan of the interleaved attention kernels: units, classes, shares.  Plain arithmetic, for the kernels and for host
// code that replays it.
#ifndef SMART_TVA_PLAN_H_
#define SMART_TVA_PLAN_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smart_tree.h"

namespace smart {
namespace tva {

constexpr int kBlock = 16;            // tokens per cache block
constexpr int kTile = 32;             // keys per tile = two cache blocks
constexpr int kClasses = 3;           // sequences are classed by rows = nodes x group heads per kv head
constexpr int kSmallRows = 32;        // class 0: all rows fit one 32-row MFMA tile
constexpr int kMediumRows = 64;       // class 1: all rows fit two 32-row MFMA tiles
constexpr int kLargeRows = 256;       // class 2: row groups of 256 = one workgroup of eight wavefronts x 32 rows
constexpr int kMinTilesPerWorker[kClasses] = {16, 16, 8};  // workers are 8-wave workgroups

// ---------------------------------------------------------------------------
// A "unit" is one 32-key tile of one (sequence, kv head, row group) segment.
// Sequences fall in three classes with separate unit spaces:
//   class 0  n * G <= 32 rows: one row group, eight wavefronts share a worker's tiles
//   class 1  33 .. 64 rows: one row group, tiles staged in LDS, two key groups of wavefronts
//   class 2  more rows: row groups of 256 rows, eight wavefronts x 32 rows per worker
// ---------------------------------------------------------------------------
struct SeqInfo {
  int32_t len;    // prefix length, clamped
  int32_t n;      // tree nodes, clamped to [0, SMART_MAX_NODES]
  int32_t tiles;  // ceil(len / 32)
  int32_t rg;     // row groups (1 for class 1)
};

// Class 2 shares its workers by time rather than by tiles.  The eight wavefronts of a workgroup take one 32-row
// tile each (two per SIMD), so a 32-key tile of a segment with up to four row tiles takes what one wavefront
// takes (measured: 0.68 .. 0.76 us), and with five or more what two on one SIMD take (0.9 .. 1.07 us).  In units
// of 0.06 us: kLargeTileCost[row tiles] per tile.  (What a segment costs beside its tiles: TreeCost.)
constexpr int kLargeTileCost[kLargeRows / 32 + 1] = {11, 11, 11, 12, 12, 16, 16, 17, 17};
// (the same currency for a tile of classes 0 and 1, for dealing the workgroups to the classes.  A class 0 tile takes 10 where
// all workgroups stream and 6 .. 7 among many of class 2, so no one number fits all.  Over 19 calls with class 0 trees among
// others 9 takes 0.1 % longer than 8 and 10 takes 1.1 %; 8 / 9 / 10 us: 60 sequences of 500 .. 4000 tokens, 1 .. 24 nodes 113.3 /
// 118.0 / 119.4, 64 of 16384, 1 .. 48 nodes 1231 / 1245 / 1239, 32 of 3072 .. 4096, 1 .. 14 nodes 92.4 / 92.2 / 94.6, 64 of 4096,
// 4 .. 10 nodes 184.0 / 178.9 / 182.9, 48 of 100 .. 8000, 1 .. 48 nodes, 2 kv heads 54.6 / 54.6 / 56.4, 48 of 200 .. 3000, 1 .. 64
// nodes 98.8 / 97.3 / 97.7.)
constexpr int kClassTileCost[kClasses] = {8, 10, 1};
constexpr int kFp8StreamTileCost = 5;
// What a segment costs beside its prefix tiles where the prefix kernel finishes the rows itself (kFinish): its tree part,
// and where workers hold several segments its start and end, in units of classes 0 and 1 (a tile) and of class 2: see
// tree_cost.
struct TreeCost {
  int32_t small, large;
};

// What the unit space of class 2 holds of one sequence: per kv head its row groups in order, all but the last
// with eight row tiles.
struct LargeSpans {
  int32_t cost_last;   // cost of a tile of the last row group
  int64_t span_full;   // units of a row group with eight row tiles
  int64_t span_last;   // units of the last row group
  int64_t span_head;   // units of one kv head: (rg - 1) span_full + span_last
};
template <bool kFinish>
__host__ __device__ inline LargeSpans large_spans(const SeqInfo& si, int G, TreeCost tc) {
  LargeSpans ls;
  const int rows_last = si.n * G - (si.rg - 1) * kLargeRows;
  ls.cost_last = kLargeTileCost[rows_last > 0 ? (rows_last + 31) / 32 : 0];
  const bool any = (kFinish || si.tiles > 0) && si.rg > 0;
  const int tree = kFinish ? tc.large : 0;
  ls.span_full = any ? (int64_t)si.tiles * kLargeTileCost[kLargeRows / 32] + tree : 0;
  ls.span_last = any ? (int64_t)si.tiles * ls.cost_last + tree : 0;
  ls.span_head = any ? (si.rg - 1) * ls.span_full + ls.span_last : 0;
  return ls;
}
// Units of a segment of class 0 or 1.
template <bool kFinish>
__host__ __device__ inline int segment_units(const SeqInfo& si, TreeCost tc) {
  return si.tiles + (kFinish ? tc.small : 0);
}
// Units of the whole sequence (classes 0 and 1: its tiles per kv head; class 2: in the cost currency).
template <bool kFinish>
__host__ __device__ inline int64_t sequence_units(const SeqInfo& si, int cls, int G, int Hkv, TreeCost tc) {
  if (cls < 2) return (int64_t)segment_units<kFinish>(si, tc) * Hkv * si.rg;
  return large_spans<kFinish>(si, G, tc).span_head * Hkv;
}
// Tile of a class-2 segment at which a share that begins `off` units into the segment begins (a share boundary
// inside a tile goes down to the tile's beginning).
__host__ __device__ inline int large_tile_at(int64_t off, int cost, int tiles) {
  const int64_t t = off / cost;
  return t > tiles ? tiles : (int)t;
}
// First unit of worker w of W over U units (w = W: U).  Every piece of code that cuts the unit space of class 2
// calls this one function, so that workers and the combine step agree on the pieces.
__host__ __device__ inline int64_t share_begin(int64_t w, int64_t U, int64_t W) { return (w * U) / W; }

__host__ __device__ inline int seq_class(int rows) { return rows <= kSmallRows ? 0 : (rows <= kMediumRows ? 1 : 2); }
// With an fp8 cache there is no class 0: trees of up to 64 rows are class 1 (streamed into registers, one or two row
// tiles), larger ones class 2 (tiles staged in LDS as for bf16, after conversion).
template <bool kFp8>
__host__ __device__ inline int plan_class(int rows) {
  return kFp8 ? (rows <= kMediumRows ? 1 : 2) : seq_class(rows);
}

// What the plan records of one sequence: lengths and sizes clamped to what the arrays hold.  The
// offsets themselves are checked by offsets_malformed for the whole batch: only a running sum
// guarantees that the sizes add up to at most total_nodes, which is what the host sized the
// partial-result slots and the combine grid for.
// (The row groups are the same with an fp8 cache: one up to 64 rows, else groups of 256.)
template <bool kAllMedium = false>
__host__ __device__ inline SeqInfo sequence_info(int len, int base, int next, int total_nodes, int G, int max_blocks) {
  const int cap = max_blocks * kBlock;
  len = len < 0 ? 0 : (len > cap ? cap : len);
  int n = next - base;
  if (base < 0 || n < 0 || base + n > total_nodes) n = 0;
  n = n > SMART_MAX_NODES ? SMART_MAX_NODES : n;
  const int rows = n * G;
  SeqInfo si;
  si.len = len;
  si.n = n;
  si.tiles = (len + kTile - 1) / kTile;
  si.rg = rows == 0 ? 0 : (rows <= kMediumRows ? 1 : (rows + kLargeRows - 1) / kLargeRows);
  return si;
}

// The prefix kernel is ONE launch of max(workgroups, kClasses) workgroups; the classes share
// them in proportion to their cost (kClassTileCost per tile of classes 0 and 1; the units of class 2
// are costs already), so that all of them finish together.  Every class with work gets at least one
// workgroup, the shares are rounded down, and what is left over goes to the classes whose workgroups
// are loaded most, so the classes never need more workgroups than were launched.  Returns the workers
// per class and the first workgroup of each class (entry kClasses: one past the last).
// kOnlySmall: the plan of the fp8-cache kernel, which has no class 0 (plan_class).
template <bool kOnlySmall, bool kFinish>
__host__ __device__ inline void apportion(const int64_t (&all_u)[kClasses], const int64_t (&all_s)[kClasses], TreeCost tc,
                                          int workgroups, int64_t (&workers)[kClasses], int64_t (&first_wg)[kClasses + 1]) {
  const int64_t tot_u[kClasses] = {kOnlySmall ? 0 : all_u[0], all_u[1], all_u[2]};
  // (fp8 cache: class 1 is the register stream of half as many bytes per tile; measured 4 .. 8 units per tile
  // against class 2's 11 .. 17, the higher figure where the whole launch is bound by memory)
  const int64_t weight[kClasses] = {kClassTileCost[0], kOnlySmall ? kFp8StreamTileCost : kClassTileCost[1],
                                    kClassTileCost[2]};
  const int64_t launched = workgroups > kClasses ? workgroups : kClasses;
  int64_t cost[kClasses], total = 0;
#pragma unroll
  for (int c = 0; c < kClasses; ++c) {
    cost[c] = tot_u[c] * weight[c];
    total += cost[c];
  }
  int64_t wg[kClasses], used = 0;
  int biggest = 0;
#pragma unroll
  for (int c = 0; c < kClasses; ++c) {
    // (binary64 division: exact enough for a share of a few hundred workgroups, far cheaper than
    // a 64-bit integer division, and every wavefront that plans runs this same code)
    wg[c] = tot_u[c] > 0 ? (int64_t)((double)cost[c] * (double)launched / (double)(total > 0 ? total : 1)) : 0;
    if (tot_u[c] > 0 && wg[c] < 1) wg[c] = 1;
    used += wg[c];
    if (cost[c] > cost[biggest]) biggest = c;
  }
  // What the rounding left over (fewer than kClasses workgroups) goes one by one to the class whose workgroups carry
  // the most cost each: the kernel ends with its slowest class, and a class of four workgroups that is owed 4.5 runs
  // 12 % longer than the rest.  At most kClasses - 1 shares were raised to one, which the biggest class gives back.
  int64_t rest = launched - used;
  for (int k = 0; k < kClasses && rest > 0; ++k) {
    int worst = -1;
#pragma unroll
    for (int c = 0; c < kClasses; ++c)
      if (tot_u[c] > 0 && (worst < 0 || (double)cost[c] * (double)wg[worst] > (double)cost[worst] * (double)wg[c])) worst = c;
    if (worst < 0) break;
    wg[worst] += 1;
    rest -= 1;
  }
#pragma unroll
  for (int c = 0; c < kClasses; ++c)
    if (c == biggest && wg[c] + rest >= 1) wg[c] += rest;
  int64_t first = 0;
#pragma unroll
  for (int c = 0; c < kClasses; ++c) {
    // A worker is a workgroup in every class, as many as pay by the prefix tiles alone (so that segments of 64 tiles go to four
    // workers each, tree parts or not), but one for every segment: one sequence of 200 tokens, 8 kv heads, on three workers
    // 26.7 us, on eight 10.4.  Never more workers than units: where partials are merged by another kernel (not kFinish) a segment
    // without prefix has no unit, and a worker without one would leave no partial between those of its neighbours, which are
    // merged without a gap.  (With kFinish every segment has the units of its tree part.  Few 64-bit comparisons: all
    // wavefronts of a workgroup wait for this.)
    const int64_t pay = (tot_u[c] - (kFinish ? all_s[c] * (c == 2 ? tc.large : tc.small) : 0)) /
                        (kMinTilesPerWorker[c] * (c == 2 ? kLargeTileCost[0] : 1));
    const int32_t dealt = (int32_t)wg[c], segs = (int32_t)all_s[c];
    int32_t w = pay < dealt ? (int32_t)pay : dealt;
    if (w < segs) w = segs < dealt ? segs : dealt;
    if (!kFinish && w > tot_u[c]) w = (int32_t)tot_u[c];
    workers[c] = w;
    first_wg[c] = first;
    first += w;
  }
  first_wg[kClasses] = first;
}

// Workers w_first .. w_last whose shares touch units [ub, ub + span): all of them, because no share is empty (W <= U, see
// apportion).
__host__ __device__ inline void segment_workers(int64_t ub, int64_t span, int64_t U, int64_t W, int64_t& w_first,
                                                int64_t& w_last) {
  w_first = ((ub + 1) * W - 1) / U;
  w_last = ((ub + span) * W - 1) / U;
}

}  // namespace tva
}  // namespace smart
#endif
