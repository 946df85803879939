// Which split of the work a list builder takes (plain C++: the launch and a
// host test share it).
#pragma once

namespace uf {

// A wave per row of nk_cap key tiles (four rows to a workgroup, no barrier) against a
// workgroup per row.  A row takes a wave four times as long, so there have to be
// enough rows to fill the chip with waves: more of them the longer the rows are, up
// to 18 a CU.  Bernoulli lists, wave / workgroup, us: 444 rows of 148 tiles 5.1 / 5.1,
// 777 of 148 5.2 / 5.6, 768 of 512 6.2 / 6.0, 1,152 of 512 6.9 / 7.0, 1,050 of 700 8.2 /
// 7.8, 1,575 of 700 8.5 / 9.2, 2,304 of 960 10.9 / 10.9 and of 1,024 12.4 / 11.8, 3,042 of
// 1,352 15.2 / 17.0, 64 of 4,096 25.6 / 13, 195 of 12,480 73 / 31, 2,340 of 12,480 106 / 87,
// 4,680 of 12,480 152 / 149, 8,970 of 12,480 246 / 263.
constexpr bool lists_wave_per_row(int rows, int nk_cap) {
  return rows >= 4608 || (rows >= 768 && 5LL * rows >= 8LL * nk_cap);
}

}  // namespace uf
