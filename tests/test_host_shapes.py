"""Rules that share work out over the chip, on the CPU: pure functions of the sizes."""
import itertools

from tests._native import run_host

SCORES = r"""
#include <cstdio>
#include <cstdlib>
#include "internal.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 5 <= argc; i += 5) {
    const aiwc::ScoreShape s = aiwc::score_shape(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2]),
                                                 std::atoi(argv[i + 3]), std::atoi(argv[i + 4]), 256, 163840);
    std::printf("%d %d %d %d %zu\n", s.rows, s.row_blocks, s.chunks, s.split, s.lds);
  }
}
"""


def test_score_shapes(tmp_path):
    cases = [(oob, f, n, t, C) for oob, f, n, t, C in itertools.product(
        (0, 1), (1, 2, 100, 1700), (1, 63, 64, 65, 1110, 10000, 262144), (1, 2, 3, 4, 5, 7, 8, 9, 100, 16384), (2, 21, 255))]
    out = run_host(tmp_path, SCORES, [str(v) for c in cases for v in c]).splitlines()
    assert len(out) == len(cases)
    for (oob, f, n, t, C), line in zip(cases, out):
        rows, blocks, chunks, split, lds = map(int, line.split())
        case = (oob, f, n, t, C, rows, blocks, chunks, split)
        assert rows % 64 == 0 and 64 <= rows <= 512 and (blocks - 1) * rows < n <= blocks * rows, case
        assert lds <= 163840 // 3 and 1 <= chunks <= -(-t // 8), case
        # a tree's waves are a power of two, and all of them have one
        assert split in (1, 2, 4, 8) and split * min(t, 8) <= 8, case
        # a wave walks at most 128 held-out rows at a time: no second round of them
        # while there are idle waves or workgroups
        if not oob:
            assert rows <= 128 * split, case
    # few trees over rows that fill the chip
    few = dict(zip(cases, out))
    for oob, n, t in itertools.product((0, 1), (10000, 262144), (1, 2, 4)):
        rows, blocks, chunks, split, _ = map(int, few[(oob, 1, n, t, 21)].split())
        assert blocks * t * split >= min(8 * 256, n // 64 * t), (oob, n, t, rows, blocks, split)
