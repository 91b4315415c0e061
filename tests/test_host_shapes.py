"""Rules that share work out over the chip, on the CPU: pure functions of the sizes."""
import itertools

import pytest

from tests._native import build_host, run_exe, run_host

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


# the default launch shape of a fit (256 CUs of 160 KB LDS, the program's own device
# queries), and the autotuner's candidates
TUNER = r"""
#include <cstdio>
#include <cstdlib>
#include "internal.h"
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
  return hipSuccess;
}
}
int main(int argc, char** argv) {
  const int n = std::atoi(argv[1]), items = std::atoi(argv[2]), bins = std::atoi(argv[3]);
  const aiwc::GrowConfig base = aiwc::grow_config(n, items, std::vector<int32_t>(35, bins), 12, n, false);
  std::vector<aiwc::GrowConfig> all = aiwc::tune_candidates(base);
  all.insert(all.begin(), base);
  for (const auto& c : all) std::printf("%d %d %d %d\n", c.block, c.huge_min, c.occupancy, c.big_cols);
}
"""


@pytest.mark.parametrize("n", [60, 700, 1024, 2220, 4097, 6000, 16384, 16385, 40000, 200000])
def test_tuner_times_the_default_shape(tmp_path, n):
    exe = build_host(tmp_path, TUNER)
    for items in (1, 300, 900, 2000, 20000):
        shapes = [tuple(map(int, v.split())) for v in run_exe(exe, [n, items, 64]).splitlines()]
        base, shapes = shapes[0], shapes[1:]
        form = [(b, h if n > h else None, occ, bc) for b, h, occ, bc in shapes]
        assert (base[0], base[1] if n > base[1] else None, *base[2:]) == form[0], (items, base, shapes[0])
        assert len(set(form)) == len(form)
        for b, h, occ, bc in shapes:
            # a limit without wide nodes holds for every training set that shares the
            # choice (up to the next power of two), as one- and two-wave workgroups need
            if n <= h:
                assert h >= 1 << (n - 1).bit_length(), (items, b, h)
            else:
                assert b >= 192
        # no wide nodes up to 16384 rows: every workgroup size at every occupancy
        narrow = {(b, occ) for b, h, occ, _ in form if h is None}
        every = {(b, occ) for b in (64, 128, 192, 256, 512, 1024) for occ in (4, 5, 6)}
        assert narrow == (every if n <= 16384 else set())
        limits = {h for _, h, _, _ in form if h is not None}
        assert limits >= {h for h in (64, 512, 1024, 4096) if h < n}


@pytest.mark.parametrize("items", [1, 300, 900, 2000, 20000])
def test_wide_limit_alone_finds_a_shape(tmp_path, monkeypatch, items):
    monkeypatch.setenv("AIWC_RF_HUGE_MIN", "1000")
    exe = build_host(tmp_path, TUNER)
    for n in (1001, 2220, 9000, 100000):
        block, limit = map(int, run_exe(exe, [n, items, 64]).split()[:2])
        assert limit == 1000 and block >= 192
    assert int(run_exe(exe, [1000, 20000, 64]).split()[0]) == 64


ROUTES = r"""
#include <cstdio>
#include <cstdlib>
#include "internal.h"
int main(int argc, char** argv) {
  for (int i = 2; i + 5 <= argc; i += 5) {
    aiwc_rf_forest f;
    f.params.push_back({1, 1, std::atoi(argv[i + 1]), 1, 1});
    f.n_train.push_back(std::atoi(argv[i]));
    const aiwc::TreesView t = aiwc::trees_of(&f, 0);
    std::printf("%d\n", (int)aiwc::predict_route(t, std::atoi(argv[i + 2]), std::atoi(argv[i + 3]), std::atoi(argv[i + 4]),
                                                       std::atoi(argv[1]) != 0));
  }
}
"""
ROW, LANES, PARTS, DIRECT, STAGED = range(5)


def test_prediction_routes(tmp_path):
    exe = build_host(tmp_path, ROUTES)

    def routes(cases, sums=0):
        return [int(v) for v in run_exe(exe, [sums] + [v for c in cases for v in c]).split()]

    # (training rows, min.node.size, rows, trees, columns): fastest in measurements
    want = {
        (2220, 9, 1, 505, 35): ROW, (2220, 9, 60, 505, 35): ROW, (300, 5, 700, 300, 20): ROW,
        (400, 30, 1500, 400, 35): ROW, (300, 5, 3000, 200, 20): LANES, (300, 5, 8000, 60, 20): LANES,
        (20000, 5, 3000, 60, 20): LANES, (2220, 5, 20, 2000, 20): PARTS, (2220, 5, 100, 1100, 20): PARTS,
        (40, 30, 700, 1100, 20): DIRECT, (300, 30, 700, 1100, 20): DIRECT, (300, 5, 8000, 122, 20): DIRECT,
        (300, 5, 900, 513, 20): DIRECT, (30, 50, 100000, 500, 70): DIRECT, (200000, 5, 4096, 500, 65): STAGED,
        (200000, 5, 200000, 500, 65): STAGED, (2220, 5, 60000, 500, 35): STAGED, (40, 9, 40000, 500, 75): STAGED,
    }
    assert dict(zip(want, routes(list(want)))) == want
    # sums alone are a launch less by the other routes
    assert routes([(3158, 5, 18858, 22, 28), (300, 5, 750, 300, 20), (300, 5, 900, 300, 20)]) == [LANES, ROW, ROW]
    assert routes([(3158, 5, 18858, 22, 28), (300, 5, 750, 300, 20), (300, 5, 900, 300, 20)], 1) == [DIRECT, ROW, LANES]
    # each route takes the fewest rows of what it is for, and none comes back
    for n_train, k, trees, C in itertools.product((30, 300, 2220, 30000, 200000), (1, 9), (1, 40, 500, 600, 1100), (5, 66)):
        seen = routes([(n_train, k, n, trees, C) for n in (1, 10, 100, 300, 1000, 2000, 4096, 5000, 20000, 100000, 10 ** 6)])
        assert seen[0] in (ROW, PARTS)
        firsts = [r for i, r in enumerate(seen) if i == 0 or r != seen[i - 1]]
        assert STAGED not in firsts[:-1] and (PARTS not in seen or trees > 512) and (LANES not in seen or trees <= 512)
