"""Host rules of the prefill and projection launches (launch_rules.hpp), compiled for the CPU:
grids stay within a launch's limits."""
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
      const hack::ProjectTile& t = hack::kProjectTiles[hack::choose_project_tile(b, l, h, p)];
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
