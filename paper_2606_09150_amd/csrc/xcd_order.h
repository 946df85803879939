// Order in which workgroups take the items of a launch (plain C++: the kernels
// and a host test share it).
#pragma once

namespace uf {

// Workgroups are dealt to the 8 XCDs in turn.  Where those resident at once span
// several heads (NT rows each), item i of n becomes one of a contiguous range of
// items per XCD (equal ranges up to one item), so that an XCD's workgroups stream
// the same head's tiles through its L2.  With a head's rows more than a quarter
// of the resident workgroups the order stays: every XCD streams one or two heads
// anyway.  12 heads, against the order of the grid: 73 tiles of 64 tokens 484 -> 462
// us, 37 tiles of 128 503 -> 496 us, backward of the latter 1685 -> 1672 us, of 12 x 2
// heads and 24 tiles of 64 183 -> 177.5 us; at 192 tiles of 128 the forward was 0 to
// 2 % slower, depending on the card.  The items must be of one kind: an XCD whose
// range holds the longer ones runs on alone.
constexpr int xcd_item(int i, int n, int NT, int resident) {
  if (NT * 4 > resident) return i;
  const int x = i & 7, k = i >> 3, q = n >> 3, r = n & 7;
  return x * q + (x < r ? x : r) + k;
}

// The same for a split launch: items 0 .. whole-1 are whole rows, the n - whole
// others slices of a row.  Each kind is dealt by itself, so that every XCD gets
// its share of both, and whole rows still start first.
constexpr int xcd_split_item(int i, int n, int whole, int NT, int resident) {
  return i < whole ? xcd_item(i, whole, NT, resident) : whole + xcd_item(i - whole, n - whole, NT, resident);
}

}  // namespace uf
