// Host arithmetic behind the prefill and projection launches: which kernel shape a call takes
// and the extents of its grid.  Plain C++, so that it can be checked without a GPU.
#pragma once
#include <cstdint>

namespace hack {

constexpr int64_t kMaxLaunchThreads = 0xFFFFFFFF;  // of one grid dimension

// ---------------------------------------------------------------------------
// Projection: tile shapes, and what a launch of n workgroups of them takes in microseconds at
// h = hidden / 4096.  `slots` workgroups of a shape are resident on the chip's 256 compute units
// (two a unit where LDS allows it); each round of that many takes full_a + full_b h, a last round
// of at most one a unit part_a + part_b h, and a last round between the two most_a + most_b h.
// The constants are fitted to these launches (us; 4096 hidden, 48 output heads, partition 32; at
// 1024 in brackets; at partition 64 a round of 64 x 128 tiles takes 2 to 3 us more):
//   tokens         64          350          512          1000         1500         3000
//   32 x 128    22.5 [9.9]  51.3 [21.3]  53.7 [21.1]  95.2 [34.0]   134 [46.2]   268 [85.9]
//   64 x 128    28.8 [11.8] 36.4 [15.6]  40.8 [16.1]  75.2 [27.2]   110 [37.6]   195 [61.9]
//   128 x 128   37.6 [14.5] 40.1 [16.3]  43.7 [16.1]  86.4 [30.4]   122 [42.1]   216 [68.6]
//   256 x 128   55.3 [19.3] 60.3 [23.9]  63.3 [24.1]  65.3 [25.6]   123 [44.2]   194 [63.6]
//   256 x 256   91.5 [32.5]  101 [41.4]   102 [41.7]   104 [42.7]   116 [45.9]   224 [76.5]
// Over 84 shapes (20, 36 and 48 heads) the choice takes 0.9% more than the fastest tile (3.0%
// with one workgroup a unit assumed and everything proportional to hidden).
// Small tiles put a short prompt on more compute units (its weights are a latency-bound stream
// of three to four steps in flight per workgroup); large ones fetch E and W fewer times
// (the stream from L2 bounds a full chip).  A V block lies in one tile, so partitions of 64
// and 128 start at tiles of as many tokens.
// ---------------------------------------------------------------------------
struct ProjectTile {
  int bm, bn;          // tokens x output channels
  int threads, slots;
  float part_a, part_b, most_a, most_b, full_a, full_b;
};
constexpr ProjectTile kProjectTiles[] = {{32, 128, 256, 512, 2.2f, 16.8f, 2.8f, 27.0f, 2.8f, 27.0f},
                                         {64, 128, 256, 512, 2.5f, 24.3f, 4.0f, 34.0f, 5.0f, 39.0f},
                                         {128, 128, 512, 256, 5.5f, 37.0f, 5.5f, 37.0f, 5.5f, 37.0f},
                                         {256, 128, 512, 256, 6.0f, 58.0f, 6.0f, 58.0f, 6.0f, 58.0f},
                                         {256, 256, 512, 256, 19.0f, 89.0f, 19.0f, 89.0f, 15.0f, 95.0f}};
constexpr int kProjectTileCount = sizeof(kProjectTiles) / sizeof(kProjectTiles[0]);

inline int64_t project_workgroups(const ProjectTile& t, int batch, int len, int heads) {
  return (int64_t)batch * ((len + (int64_t)t.bm - 1) / t.bm) * (((int64_t)heads * 128 + t.bn - 1) / t.bn);
}

// Index of the tile shape of a call with `heads` output heads (query, key and value); the last
// one where no shape's launch fits a grid.
inline int choose_project_tile(int batch, int len, int heads, int hidden, int partition) {
  const float h = (float)hidden / 4096.0f;
  int best = kProjectTileCount - 1;
  float least = 0.0f;
  for (int i = kProjectTileCount - 1; i >= 0 && kProjectTiles[i].bm >= partition; --i) {
    const ProjectTile& t = kProjectTiles[i];
    const int64_t n = project_workgroups(t, batch, len, heads);
    if (n * t.threads > kMaxLaunchThreads) continue;
    const int64_t rest = n % t.slots;
    const float full = t.full_a + t.full_b * h;
    const float last = rest == 0 ? 0.0f : (rest <= 256 ? t.part_a + t.part_b * h : t.most_a + t.most_b * h);
    const float us = (float)(n / t.slots) * full + last;
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
