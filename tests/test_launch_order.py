"""Rules of the launches, compiled for the host and read back: the order in which
an attention launch's workgroups take rows and slices (csrc/xcd_order.h), and how
many lanes a list row gets (csrc/list_rule.h)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_09150_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "list_rule.h"
#include "xcd_order.h"
int main(int c, char** v) {
  if (c == 2) {                             // list lengths on standard input
    static int counts[1 << 16];
    for (int i = 0; i < atoi(v[1]); ++i)
      if (scanf("%d", counts + i) != 1) return 1;
    return printf("%d\n", int(uf::xcd_even(counts, atoi(v[1])))) < 0;
  }
  if (c == 4) return printf("%d\n", int(uf::topk_row_alone(atoi(v[2]), atoi(v[3])))) < 0;
  if (c == 3) return printf("%d\n", int(uf::lists_wave_per_row(atoi(v[1]), atoi(v[2])))) < 0;
  const int n = atoi(v[1]), whole = atoi(v[2]), nt = atoi(v[3]), resident = atoi(v[4]);
  for (int i = 0; i < n; ++i) printf("%d\n", uf::xcd_split_item(i, n, whole, nt, resident));
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(PROGRAM)
    exe = str(d / "order")
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(d / "order.cpp"), "-o", exe], check=True)
    return lambda *args, stdin="": [int(x) for x in subprocess.check_output([exe, *map(str, args)],
                                                                             input=stdin.encode()).split()]


# (rows, rows kept whole, slices of each other row, rows of a head, resident workgroups)
@pytest.mark.parametrize("rows,whole,split,nt,resident", [
    (444, 256, 4, 37, 256), (304, 256, 5, 19, 256), (456, 256, 5, 19, 256), (36, 20, 3, 6, 256), (36, 13, 7, 6, 768),
    (444, 0, 4, 37, 256), (444, 444, 1, 37, 256), (5, 0, 51, 5, 256), (2304, 2048, 2, 192, 256), (300, 299, 64, 25, 768)])
def test_whole_rows_and_slices_are_dealt_alike_to_every_xcd(rules, rows, whole, split, nt, resident):
    n = whole + (rows - whole) * split
    items = rules(n, whole, nt, resident)
    assert sorted(items) == list(range(n))
    assert all(x < whole for x in items[:whole])                 # whole rows start first
    on_xcd = [items[x::8] for x in range(8)]                     # workgroup i runs on XCD i % 8
    for kind in (lambda it: it < whole, lambda it: it >= whole):
        share = [sum(map(kind, it)) for it in on_xcd]
        assert max(share) - min(share) <= 1
    # the XCDs' loads, in row-times, differ by at most a row and a slice
    load = [sum(1.0 if i < whole else 1.0 / split for i in it) for it in on_xcd]
    assert max(load) - min(load) <= 1.0 + 1.0 / split
    if nt * 4 <= resident:                                       # and its items of a kind are neighbours
        for it in on_xcd:
            for kind in ([i for i in it if i < whole], [i for i in it if i >= whole]):
                assert not kind or kind == list(range(kind[0], kind[0] + len(kind)))


def _lengths(heads, nt, long, every, few, full=400):
    """List lengths of `heads` heads of nt rows; `long` of them (each `every`-th head) are full."""
    return [full if h % every == 0 and h // every < long else few for h in range(heads) for _ in range(nt)]


# A contiguous range of rows per XCD is taken only where it gives no XCD much more to do.
@pytest.mark.parametrize("counts,even", [
    (_lengths(12, 37, 12, 1, 0), 1), (_lengths(1, 257, 1, 1, 0), 1), ([0] * 300, 1), ([400, 399, 401] * 100, 1),
    ([90 + (7 * i * i) % 11 for i in range(888)], 1), (_lengths(80, 16, 40, 2, 40), 1),
    (_lengths(16, 19, 2, 1, 40), 0), (_lengths(16, 33, 4, 1, 40), 0), (_lengths(16, 33, 4, 4, 40), 0),
    (_lengths(16, 64, 4, 1, 40), 0), (_lengths(12, 73, 3, 1, 120), 0), ([0] * 280 + [400] * 20, 0),
    ([400] * 300 + [200] * 300, 0)])
def test_rows_go_to_xcds_in_ranges_only_with_even_lists(rules, counts, even):
    assert rules(len(counts), stdin=" ".join(map(str, counts))) == [even]


# (rows, key tiles of a row, a wave per row): where one side was at least 4 % faster
@pytest.mark.parametrize("rows,nk,wave", [
    (52, 156, 0), (64, 512, 0), (64, 4096, 0), (195, 12480, 0), (338, 1352, 0), (768, 1024, 0), (768, 4096, 0),
    (1014, 1352, 0), (2304, 2048, 0), (2340, 12480, 0), (777, 148, 1), (1752, 292, 1), (1575, 700, 1), (2400, 960, 1),
    (4056, 1352, 1), (7680, 960, 1), (8970, 12480, 1)])
def test_few_or_long_list_rows_get_a_workgroup(rules, rows, nk, wave):
    assert rules(rows, nk) == [wave]


# (rows, ranked candidates, a workgroup per row): where one side was at least 4 % faster
@pytest.mark.parametrize("rows,nc,alone", [
    (4, 62, 1), (8, 124, 1), (592, 37, 1), (732, 61, 1), (512, 96, 1), (12, 186, 1), (250, 250, 1), (256, 160, 1),
    (2560, 64, 0), (800, 100, 0), (960, 120, 0), (320, 240, 0), (444, 148, 0), (480, 240, 0), (1, 257, 0)])
def test_few_topk_rows_get_a_workgroup(rules, rows, nc, alone):
    assert rules("topk", rows, nc) == [alone]
