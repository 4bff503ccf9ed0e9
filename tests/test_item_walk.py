"""How the workgroups of a grid share a list of items (csrc/item_walk.hpp), compiled for the host and walked in full:
every item belongs to exactly one workgroup, whatever the grid, the list and the workgroups that other work holds."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#define __device__
#define __forceinline__ inline
using std::min;
#include "item_walk.hpp"
using namespace semmoe;

static int bad = 0;

// the workgroups that keep to a first list are those that have its items
static void first_list(int grid, int items) {
  const int skip = side_workgroups(items, grid);
  for (int b = 0; b < grid && skip > 0; ++b)
    if (b / 8 >= skip && share_of(items, grid, b, true, 0).count != 0) bad = 1, std::printf("grid %d: %d items reach workgroup %d\n", grid, items, b);
}

static void walk(int grid, int total, bool spread, int items_before) {
  const int skip = items_before < 0 ? 0 : side_workgroups(items_before, grid);
  std::vector<int> seen(total, 0);
  for (int b = 0; b < grid; ++b) {
    // a workgroup of every XCD has to be left; share_of would divide by zero otherwise
    if (grid % 8 == 0 && skip >= grid / 8) { bad = 1; std::printf("grid %d before %d: nobody left\n", grid, items_before); return; }
    const ItemWalk w = share_of(total, grid, b, spread, skip);
    if (skip > 0 && b / 8 < skip && w.count != 0) bad = 1;  // it has other work
    for (int r = 0; r < w.count; ++r) {
      const int i = w.item(r);
      if (i < 0 || i >= total || seen[i]++) { bad = 1; std::printf("grid %d total %d before %d: item %d of workgroup %d\n", grid, total, items_before, i, b); return; }
    }
  }
  for (int i = 0; i < total; ++i)
    if (!seen[i]) { bad = 1; std::printf("grid %d total %d before %d: item %d left out\n", grid, total, items_before, i); return; }
}

int main() {
  const int grids[] = {1, 3, 5, 7, 8, 12, 13, 16, 24, 32, 40, 100, 128, 256, 504, 512};
  for (int grid : grids) {
    for (int items = 0; items <= grid; ++items) first_list(grid, items);
    std::vector<int> totals;
    for (int t = 0; t <= 40; ++t) totals.push_back(t);
    for (int m = 1; m <= 3; ++m)
      for (int off = -9; off <= 9; ++off)
        if (m * grid + off > 40) totals.push_back(m * grid + off);
    for (int total : totals) {
      walk(grid, total, true, -1);
      walk(grid, total, false, -1);
      for (int before = 0; before <= grid + 9; before += before < 40 ? 1 : 7) walk(grid, total, true, before);
    }
  }
  return bad;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("item_walk")
    (d / "walk.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2503_04398_amd", "csrc"),
                    str(d / "walk.cpp"), "-o", str(d / "walk")], check=True)
    return str(d / "walk")


def test_every_item_has_one_workgroup(driver):
    r = subprocess.run([driver], stdout=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[:2000]
