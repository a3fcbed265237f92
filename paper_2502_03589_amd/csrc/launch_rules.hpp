// Host arithmetic behind the prefill and projection launches: which kernel shape a call takes
// and the extents of its grid.  Plain C++, so that it can be checked without a GPU.
#pragma once
#include <cstdint>

namespace hack {

constexpr int64_t kMaxLaunchThreads = 0xFFFFFFFF;  // of one grid dimension

// ---------------------------------------------------------------------------
// Projection: tile shapes, and what w rounds of one workgroup per compute unit of them take in
// microseconds at hidden 4096 (all of it scales with hidden): offset + per_round * w.  Measured
// with 48 output heads:
//   tokens      16/64   250    512   1024   1500   2048   3000   4096   8192
//   32 x 128     20.6   30.8   49.4   93
//   64 x 128     27.5   28.3   39.3   77    112    131    193    253    497
//   128 x 128   36     37.5   38.0   86    123    132    202    252    487
//   256 x 128   54     58.7   58.4   62.4  123    127    187    212    409
//   256 x 256   91    103    102    104    106    117    222    228    380
// Small tiles put a short prompt on more compute units (its weights are a latency-bound stream
// of three to four steps in flight per workgroup); large ones fetch E and W fewer times
// (the stream from L2 bounds a full chip).  A V block lies in one tile, so partitions of 64
// and 128 start at tiles of as many tokens.
// ---------------------------------------------------------------------------
struct ProjectTile {
  int bm, bn;  // tokens x output channels
  int threads;
  float offset, per_round;
};
constexpr ProjectTile kProjectTiles[] = {{32, 128, 256, 6.0f, 14.5f}, {64, 128, 256, 6.0f, 22.0f},
                                         {128, 128, 512, 0.0f, 40.0f}, {256, 128, 512, 0.0f, 65.0f},
                                         {256, 256, 512, 0.0f, 115.0f}};
constexpr int kProjectTileCount = sizeof(kProjectTiles) / sizeof(kProjectTiles[0]);
constexpr int kChipUnits = 256;

inline int64_t project_workgroups(const ProjectTile& t, int batch, int len, int heads) {
  return (int64_t)batch * ((len + (int64_t)t.bm - 1) / t.bm) * (((int64_t)heads * 128 + t.bn - 1) / t.bn);
}

// Index of the tile shape of a call with `heads` output heads (query, key and value); the last
// one where no shape's launch fits a grid.
inline int choose_project_tile(int batch, int len, int heads, int partition) {
  int best = kProjectTileCount - 1;
  float least = 0.0f;
  for (int i = kProjectTileCount - 1; i >= 0 && kProjectTiles[i].bm >= partition; --i) {
    const ProjectTile& t = kProjectTiles[i];
    const int64_t n = project_workgroups(t, batch, len, heads);
    if (n * t.threads > kMaxLaunchThreads) continue;
    const float us = t.offset + t.per_round * (float)((n + kChipUnits - 1) / kChipUnits);
    if (least == 0.0f || us < least) {
      best = i;
      least = us;
    }
  }
  return best;
}

// ---------------------------------------------------------------------------
// Prefill attention
// ---------------------------------------------------------------------------
constexpr int kPrefillSlots = 512;         // four-wave workgroups resident at two waves per SIMD
constexpr int64_t kPrefillGridX = 1 << 22; // workgroups in the grid's x extent, at most

struct PrefillGrid {
  int64_t workgroups;
  int64_t x, y;   // workgroup w is at (w % x, w / x); the last row's rest is empty
  int groups;     // key groups of four waves in a workgroup
};

// `rows` row blocks of `heads` head groups (all kv heads) of `batch` sequences.
// A grid runs at the pace of its longest chain of blocks where that is longer than a
// workgroup slot's even share of all blocks; two key groups halve it.  Measured (32/8 heads,
// chain over share, one group -> two): 1500 tokens causal 2.6, 75.8 -> 63.0 us; 4 x 1000 at
// partition 128 1.8, 68.8 -> 63.2; 512 tokens 7.1, 25.3 -> 22.9; but 3000 tokens 1.3, 136 ->
// 158, and chains of two or three blocks lose more to the merge than they gain (63 tokens,
// 14.1 -> 16.1).  With stochastic rounding each group also draws the thresholds of Q, 64 a
// lane: chains below ten blocks lose (100 tokens at partition 32, 20.7 -> 24.6 us; 300 at 64,
// 34.4 -> 36.9; 640 at 128, 47.3 -> 49.8), longer ones gain (640 at 32, 65.2 -> 59.5).
inline PrefillGrid prefill_grid(int rows, int heads, int batch, int len, int partition, bool causal, bool stochastic) {
  PrefillGrid g;
  g.workgroups = (int64_t)rows * heads * batch;
  const int64_t blocks = ((int64_t)len + partition - 1) / partition;
  const int64_t share = (g.workgroups * (causal ? blocks + 1 : 2 * blocks) / 2 + kPrefillSlots - 1) / kPrefillSlots;
  g.groups = blocks >= (stochastic ? 10 : 4) && 5 * blocks > 8 * share ? 2 : 1;
  // One dimension of a grid holds 2^32 - 1 threads: 16.7 million workgroups, which a batch of
  // short prompts with many heads exceeds.
  g.x = g.workgroups < kPrefillGridX ? g.workgroups : kPrefillGridX;
  g.y = (g.workgroups + kPrefillGridX - 1) / kPrefillGridX;
  return g;
}

}  // namespace hack
