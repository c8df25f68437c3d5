"""The autotuner's choice (csrc/mhd_tune.hpp) on tables of made-up times: the
kept launch is the smallest entry of the times that the caller gets, it is the
best of what was timed up to the 1 % that pass F's own shape has to gain, and
the search takes no more timings than one sweep of pass F did (36 uniform, 36
for one shape in both modes)."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NT = 6
MAIN = r"""
#include <cstdio>
#include "mhd_tune.hpp"
int main() {
  double u[6][2], f[6][2][6];
  int built[6], n = 0;
  while (scanf("%d", &built[0]) == 1) {
    for (int t = 1; t < 6; ++t) scanf("%d", &built[t]);
    for (auto& t : f) for (auto& m : t) for (double& v : m) scanf("%lf", &v);
    double ms[6][2] = {};
    smhd::TuneChoice c{-1, -1, -1};
    n = 0;
    int switches = 0, last = -1;
    const int rc = smhd::tune_march<6>([&](int t) { return built[t] != 0; },
        [&](int t, int m, int ft, double& v) {
          v = f[t][m][ft];
          ++n;
          switches += t != last;
          last = t;
          return built[t] && built[ft] ? 0 : 7;
        }, ms, c);
    printf("%d %d %d %d %d %d", rc, c.tile, c.mode, c.ftile, n, switches);
    for (auto& t : ms) for (double v : t) printf(" %.17g", v);
    printf("\n");
  }
}
"""


def _run(tmp_path, tables):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "tune.cpp", tmp_path / "tune"
    src.write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2405_02483_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True, capture_output=True)
    text = "\n".join(" ".join(map(str, b)) + " " + " ".join("%.17g" % v for t in f for m in t for v in m)
                     for b, f in tables)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
    return [line.split() for line in out.splitlines()]


def _table(rng, spread, gain):
    f = [[[0.0] * NT for _ in range(2)] for _ in range(NT)]
    for t in range(NT):
        for m in range(2):
            uni = 10.0 * (1.0 + spread * rng.random())
            for ft in range(NT):
                f[t][m][ft] = uni if ft == t else uni * (1.0 - gain + 2.0 * gain * rng.random())
    return f


def test_choice(tmp_path):
    rng = random.Random(1)
    tables = []
    for n in range(300):
        built = [1] * NT if n % 3 else [int(rng.random() < 0.7) for _ in range(NT)]
        if not any(built):
            built[2] = 1
        tables.append((built, _table(rng, rng.choice((0.0, 0.005, 0.05, 0.5)), rng.choice((0.0, 0.005, 0.03, 0.2)))))
    for (built, f), r in zip(tables, _run(tmp_path, tables)):
        rc, tile, mode, ftile, n, switches = map(int, r[:6])
        ms = [float(v) for v in r[6:]]
        assert rc == 0 and n <= 72
        assert switches <= 3 * NT * 2 + 15          # (tables are made again for a new shape only)
        timed = {q: ms[q] for q in range(2 * NT) if built[q // 2]}
        assert all(ms[q] == 0.0 for q in range(2 * NT) if not built[q // 2])
        assert (tile, mode) == divmod(min(timed, key=timed.get), 2)
        uni = {(t, m): f[t][m][t] for t in range(NT) for m in range(2) if built[t]}
        top = min(uni.values())
        assert f[tile][mode][ftile] == ms[2 * tile + mode]
        if ftile == tile:
            assert uni[tile, mode] == top
        else:
            assert f[tile][mode][ftile] < 0.99 * top
        # nothing within reach was left: the fastest launch, with each shape
        t, m = min(uni, key=uni.get)
        reach = min(f[t][m][ft] for ft in range(NT) if built[ft])
        assert ms[2 * tile + mode] <= (reach if reach < 0.99 * top else top)


def test_close_launches_and_the_final_pass(tmp_path):
    """64x8 (4) and 16x16 (2) within a percent throughout, where only 16x16
    gains from pass F in 64x8."""
    f = [[[60.0] * NT for _ in range(2)] for _ in range(NT)]
    for m in range(2):
        f[4][m] = [39.5, 39.6, 39.7, 39.8, 39.12 + m, 39.9]
        f[2][m] = [39.5, 39.6, 39.31 + m, 39.8, 34.7 + m, 39.9]
    r = _run(tmp_path, [([1] * NT, f)])[0]
    assert [int(v) for v in r[:4]] == [0, 2, 0, 4]
    ms = [float(v) for v in r[6:]]
    assert ms[2 * 2] == 34.7 == min(ms) and ms[2 * 4] == 39.12
