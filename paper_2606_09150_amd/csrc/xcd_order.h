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

// Whether the ranges of n rows with these list lengths hold about as many entries
// each: the largest at most 1/8 over the mean, by four rows of each range.  Heads
// with lists of their own lengths would otherwise leave some XCDs with the long
// ones: 16 heads of 33 tiles of 128, the first four with ten times the entries of the
// others, forward 365 us in the order of the grid and 1,190 in ranges, backward 1,470
// and 3,830; 16 heads of 64 tiles of 64 alike 405 and 1,070, 1,320 and 3,450.  (Runs of
// 4, 8, 16 or 32 rows per XCD instead of one range kept only part of what ranges
// gain with even lists and were up to twice as slow as the grid's order with every
// second or fourth head long.)  With even lists the check costs 0.2 to 0.7 % of a launch
// (480p forward 472.6 -> 475.0 us, backward 1,619 -> 1,627; in the order of the grid 480.7
// and 1,631), backwards of few rows 2 %, and forwards of 257 to 768 64-token rows 2 to 5 %
// (292 rows of 292 tiles 247 -> 259 us, in the order of the grid 290).
template <class Counts>
constexpr bool xcd_even(Counts counts, int n) {
  int c[32] = {}, total = 0, most = 0;
#pragma unroll
  for (int k = 0; k < 32; ++k) c[k] = counts[unsigned(k) * unsigned(n) >> 5];
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int load = (c[4 * x] + c[4 * x + 1]) + (c[4 * x + 2] + c[4 * x + 3]);
    total += load;
    most = most > load ? most : load;
  }
  return 64 * most <= 9 * total;
}

}  // namespace uf
