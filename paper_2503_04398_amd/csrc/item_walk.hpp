// How the workgroups of a grid share a list of items: integer arithmetic alone, without the runtime's headers, so that it
// can be compiled and walked on the host as well.
#pragma once

namespace semmoe {

// A workgroup's share of a list of `total` items: item(0), item(1), ... item(count - 1).  Workgroups are handed to the 8
// XCDs round-robin by workgroup id, and each XCD has its own L2 and its own path to memory.  In every full round of the
// grid an XCD's workgroups take a contiguous run of the list (neighbouring items share weight or token panels, which
// its L2 then holds) and all XCDs together one run as well, whose panels meet in the memory-side cache: with an eighth
// of the whole list per XCD instead, 8 experts of d = F = 2880 took 511 us against 484.  The last, partly filled round
// is dealt out evenly over the XCDs: left to the first ones alone, 384 weight tiles on 512 workgroups ran on six XCDs
// and at six eighths of the memory rate.
struct ItemWalk {
  int count, first, step, last;  // last: the item of the partly filled round (-1: none)
  __device__ __forceinline__ int item(int r) const { return r + 1 == count && last >= 0 ? last : first + r * step; }
};

// Share of workgroup `b` of a grid of `grid`.
// spread = false: the partly filled round goes to the first XCDs after all.  Better where the items are few, share their
// panels and wait for L2 rather than memory (192 pieces of one set of weights, d 4096, F 1536: 46 us against 50).
// skip: so many workgroups of every XCD have other work and take no part.  Fewer than an XCD has (side_workgroups), and
// 0 unless the grid is whole eights.
__device__ __forceinline__ ItemWalk share_of(int total, int grid, int b, bool spread, int skip) {
  ItemWalk w;
  if (grid % 8 != 0) {
    const int full = total / grid;
    w.step = grid;
    w.first = b;
    w.last = b < total - full * grid ? full * grid + b : -1;
    w.count = full + (w.last >= 0 ? 1 : 0);
    return w;
  }
  const int per = (grid >> 3) - skip, g = 8 * per;
  const int full = total / g, rem = total - full * g;
  const int x = b & 7, l = (b >> 3) - skip;
  const int lo = spread ? rem * x / 8 : min(rem, x * per), hi = spread ? rem * (x + 1) / 8 : min(rem, (x + 1) * per);
  w.step = g;
  w.first = x * per + l;
  w.last = lo + l < hi ? full * g + lo + l : -1;
  w.count = l < 0 ? 0 : full + (w.last >= 0 ? 1 : 0);
  return w;
}

// Workgroups of every XCD that keep to a first list of `items` and take no part in the list that follows it (the `skip`
// above).  None where the first list fills more than half of the grid, and none where no workgroup of an XCD would be
// left for the second list: on a grid of 8 every workgroup takes its share of both.
__device__ __forceinline__ int side_workgroups(int items, int grid) {
  if (grid % 8 != 0 || items * 2 > grid) return 0;
  const int skip = (items + 7) / 8;
  return skip < grid / 8 ? skip : 0;
}

}  // namespace semmoe
