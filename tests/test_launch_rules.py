"""Host rules of the prefill and projection launches (launch_rules.hpp), compiled for the CPU:
grids stay within a launch's limits, and the projection's tile is the fastest one measured."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_03589_amd", "csrc")
CXX = shutil.which("g++") or shutil.which("c++")
MAX_THREADS = 2 ** 32 - 1  # of one grid dimension

DRIVER = r"""
#include <cstdio>
#include "launch_rules.hpp"
// p <batch> <len> <heads> <hidden> <partition>                         -> bm bn threads workgroups
// a <rows> <heads> <batch> <len> <partition> <causal> <stochastic>    -> workgroups x y groups
int main() {
  char kind;
  while (std::scanf(" %c", &kind) == 1) {
    if (kind == 'p') {
      int b, l, h, hid, p;
      if (std::scanf("%d %d %d %d %d", &b, &l, &h, &hid, &p) != 5) return 1;
      const hack::ProjectTile& t = hack::kProjectTiles[hack::choose_project_tile(b, l, h, hid, p)];
      std::printf("%d %d %d %lld\n", t.bm, t.bn, t.threads, (long long)hack::project_workgroups(t, b, l, h));
    } else {
      int r, h, b, l, p, c, s;
      if (std::scanf("%d %d %d %d %d %d %d", &r, &h, &b, &l, &p, &c, &s) != 7) return 1;
      const hack::PrefillGrid g = hack::prefill_grid(r, h, b, l, p, c != 0, s != 0);
      std::printf("%lld %lld %lld %d\n", (long long)g.workgroups, (long long)g.x, (long long)g.y, g.groups);
    }
  }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if CXX is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("rules")
    src, exe = str(d / "rules.cpp"), str(d / "rules")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.run([CXX, "-std=c++17", "-O1", "-I", CSRC, "-o", exe, src], check=True)

    def ask(kind, *args):
        out = subprocess.run([exe], input=" ".join(map(str, (kind, *args))), capture_output=True, text=True, check=True)
        return tuple(int(x) for x in out.stdout.split())
    return ask


def attention_rows(q_heads, kv_heads, length):
    """Row blocks and head groups of a prefill: four waves take HW heads by 4 / HW blocks of 32 rows."""
    group = q_heads // kv_heads
    hw = 4 if group >= 3 else group
    rows = 32 * (4 // hw)
    return -(-length // rows), kv_heads * -(-group // hw)


@pytest.mark.parametrize("q_heads,kv_heads,batch,length", [
    (32, 8, 1, 1), (32, 8, 1, 8192), (64, 64, 65535, 1), (65, 65, 65535, 20), (300, 300, 65535, 1),
    (512, 128, 65535, 40), (8, 8, 65535, 2000), (256, 256, 40000, 100), (1, 1, 1, 2 ** 21),
])
def test_prefill_grid_covers_every_workgroup_within_the_limits(rules, q_heads, kv_heads, batch, length):
    """The largest batches with many heads are more workgroups than the 2^32 - 1 threads of one
    grid dimension hold (16.7 million of 256 threads)."""
    rows, heads = attention_rows(q_heads, kv_heads, length)
    n, x, y, groups = rules("a", rows, heads, batch, length, 32, 1, 0)
    assert n == rows * heads * batch
    assert x * groups * 256 <= MAX_THREADS and 1 <= y <= 65535
    assert x * y >= n > x * (y - 1)


@pytest.mark.parametrize("heads,batch,length,partition", [
    (48, 1, 1, 32), (48, 1, 8192, 64), (129, 65535, 1, 128), (129, 65535, 1, 32), (200, 65535, 1, 128),
    (200, 65535, 100, 64), (48, 65535, 300, 32), (250, 65535, 1, 16),
])
def test_projection_tile_fits_the_grid_wherever_the_largest_does(rules, heads, batch, length, partition):
    """A small tile is not taken where its workgroups times threads exceed 2^32 - 1 and a larger
    tile's do not."""
    bm, bn, threads, n = rules("p", batch, length, heads, 4096, partition)
    largest = batch * -(-length // 256) * -(-heads // 2) * 512
    assert bm >= partition and bm % 32 == 0
    if largest <= MAX_THREADS:
        assert n * threads <= MAX_THREADS


TILES = [(32, 128), (64, 128), (128, 128), (256, 128), (256, 256)]
# tokens -> us of 32 x 128, 64 x 128, 128 x 128, 256 x 128, 256 x 256 tiles (partition 32)
MEASURED = {  # (batch, output heads, hidden)
    (1, 20, 1024): {
        64: (9.6, 11.6, 14.2, 18.8, 32.1),
        250: (10.5, 12.3, 15.2, 23.3, 41.5),
        350: (10.9, 12.7, 15.6, 23.3, 41.1),
        512: (12.2, 12.3, 15.0, 23.3, 41.1),
        1000: (19.2, 15.3, 15.7, 23.6, 41.2),
        1500: (21.8, 17.2, 17.7, 25.4, 42.8),
        3000: (38.4, 28.3, 29.7, 28.5, 45.8),
    },
    (1, 48, 1024): {
        64: (9.9, 11.8, 14.5, 19.3, 32.5),
        250: (13.0, 13.0, 15.8, 23.8, 42.0),
        350: (21.3, 15.6, 16.3, 23.9, 41.4),
        512: (21.1, 16.1, 16.1, 24.1, 41.7),
        1000: (34.0, 27.2, 30.4, 25.6, 42.7),
        1500: (46.2, 37.6, 42.1, 44.2, 45.9),
        3000: (85.9, 61.9, 68.6, 63.6, 76.5),
    },
    (2, 36, 1024): {
        64: (9.9, 11.8, 14.5, 19.4, 32.6),
        250: (19.9, 15.4, 16.2, 24.0, 42.0),
        350: (23.2, 16.8, 16.9, 24.6, 42.0),
        512: (28.6, 24.7, 28.0, 24.5, 41.8),
        1000: (43.8, 35.7, 39.3, 42.1, 45.3),
        1500: (63.2, 46.4, 52.1, 44.2, 50.2),
        3000: (117.1, 83.4, 89.3, 81.4, 83.9),
    },
    (1, 20, 4096): {
        64: (21.6, 28.0, 36.7, 53.7, 90.8),
        250: (22.9, 29.3, 38.2, 59.0, 101.0),
        350: (23.8, 29.9, 38.9, 59.4, 100.6),
        512: (30.9, 30.1, 38.5, 59.5, 101.7),
        1000: (50.2, 37.5, 41.5, 60.0, 101.5),
        1500: (65.6, 45.9, 50.2, 70.2, 107.7),
        3000: (118.5, 81.9, 89.8, 75.3, 115.3),
    },
    (1, 48, 4096): {
        64: (22.5, 28.8, 37.6, 55.3, 91.5),
        250: (32.7, 31.0, 39.5, 59.8, 102.8),
        350: (51.3, 36.4, 40.1, 60.3, 100.9),
        512: (53.7, 40.8, 43.7, 63.3, 102.2),
        1000: (95.2, 75.2, 86.4, 65.2, 104.4),
        1500: (134.3, 110.4, 121.8, 123.2, 115.9),
        3000: (268.4, 195.0, 216.4, 194.0, 224.2),
    },
    (2, 36, 4096): {
        64: (22.3, 28.6, 37.8, 55.4, 91.5),
        250: (50.6, 37.6, 40.8, 60.5, 102.3),
        350: (61.9, 42.4, 44.6, 65.8, 103.0),
        512: (78.9, 70.3, 79.8, 62.6, 103.1),
        1000: (136.4, 111.4, 121.7, 123.3, 111.2),
        1500: (202.8, 148.8, 162.5, 132.4, 127.0),
        3000: (392.4, 277.3, 300.0, 260.0, 241.4),
    },
}


@pytest.mark.parametrize("key", sorted(MEASURED))
def test_projection_tile_is_the_fastest_measured(rules, key):
    """Within 6% of the fastest shape (5% is what one shape's time moves between runs)."""
    batch, heads, hidden = key
    for length, times in MEASURED[key].items():
        tile = rules("p", batch, length, heads, hidden, 32)[:2]
        assert times[TILES.index(tile)] <= 1.06 * min(times), (length, tile)


def test_gpu_tests_reach_the_tiles_they_name(rules):
    from tests import test_gpu_project_tiles as gpu
    seen = set()
    for (bits, pi, B, Hq, H, lengths, page, rounding), tile in zip(gpu.CASES, gpu.TILES):
        for length in lengths:
            assert rules("p", B, length, Hq + 2 * H, 192, pi)[:2] == tile, (Hq, H, length)
    for bits, pi, B, Hq, H, length, page, rounding, tile in gpu.DEEP:
        assert rules("p", B, length, Hq + 2 * H, 4096, pi)[:2] == tile, (Hq, H, length)
        seen.add(tile)
    assert seen == set(TILES)


def test_gpu_tests_reach_both_key_group_counts(rules):
    from tests import test_gpu_prefill_tiles as gpu
    for bits, pi, hq, hkv, B, length, causal, rounding, page, groups in gpu.SAMPLED:
        rows, heads = attention_rows(hq, hkv, length)
        assert rules("a", rows, heads, B, length, pi, int(causal), rounding)[3] == groups, (hq, hkv, B, length)
        assert -(-length // pi) >= 4
