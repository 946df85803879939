// Which split of the work a list builder takes (plain C++: the launches and a
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

// Whether the top-k selection scores each row in a workgroup of its own, one wave per 64
// candidates (three take four), at most one wave per SIMD of 256 CUs.  That form /
// the better of four rows to a workgroup and of a launch for the scores, us: 4 rows of
// 62 candidates 10.0 / 12.4, 8 of 124 14.5 / 18.5, 592 of 37 12.1 / 12.7, 732 of 61 12.3 / 13.4,
// 1,024 of 64 15.4 / 15.3, 2,560 of 64 29.9 / 28.5; 512 of 96 13.5 / 14.9, 640 of 120 15.8 / 16.6,
// 800 of 100 19.7 / 17.7, 960 of 120 20.6 / 18.5; 12 of 186 15.3 / 16.2, 250 of 250 15.7 / 17.5,
// 256 of 160 12.9 / 15.5, 320 of 240 22.4 / 18.3, 384 of 192 16.5 / 16.2.
constexpr bool topk_row_alone(int rows, int nc) {
  const int waves = nc <= 64 ? 1 : nc <= 128 ? 2 : 4;
  return nc <= 256 && rows <= 1024 / waves;
}

}  // namespace uf
