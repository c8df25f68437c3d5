// The autotuner's choice of a launch (host code, independent of the device):
// which shapes and modes are timed, how often, and which is kept.
#pragma once

#include <algorithm>

namespace smhd {

struct TuneChoice {
  int tile, mode, ftile;   // shape of the passes, launch mode, shape of pass F
};

// timed(tile, mode, ftile, ms): milliseconds of one stage in that launch;
// nonzero stops the search and is returned.  ok(tile): the shape is built.
//
// Every candidate keeps the fastest of its rounds: a launch's time varies from
// call to call by several percent (the memory system's state), more than some
// candidates differ, so the rounds go over all candidates in turn.  First
// the uniform launches (ms[tile][mode]; untouched where not ok).  Then pass F in
// every other shape, for the uniform launches within kNear of the fastest
// (kPairs at most): a uniform launch can owe its place to pass F alone (512^3
// float64, ms per stage: 64x8 39.12 and 16x16 39.31 throughout, but 34.7 with
// 16x16 and pass F in 64x8, while 64x8 has no better shape for F).  The first
// round goes over all of them, the others over those close to the fastest.
// At most 36 + 35 timings; pass F swept for both modes of every shape near the
// fastest took up to 252, the sweep of the fastest shape alone 72.
//
// Pass F's own shape is kept if it beats every uniform launch by more than the
// timing noise (kGain; the fastest of three rounds varies by about 0.1 %), and
// then ms[tile][mode] is the time with it: the kept launch is the smallest
// entry either way.
template <int NT, class Ok, class Timed>
int tune_march(const Ok& ok, const Timed& timed, double (&ms)[NT][2], TuneChoice& best) {
  constexpr int kRounds = 3, kPairs = 5;
  constexpr double kNear = 1.02, kClose = 1.03, kGain = 0.99;
  bool seen[NT][2] = {};
  for (int round = 0; round < kRounds; ++round)
    for (int t = 0; t < NT; ++t)
      for (int m = 0; m < 2 && ok(t); ++m) {
        double v = 0.0;
        if (const int rc = timed(t, m, t, v)) return rc;
        ms[t][m] = seen[t][m] ? std::min(ms[t][m], v) : v;
        seen[t][m] = true;
      }
  struct Cand { int tile, mode, ftile; double ms; };
  auto faster = [](const Cand& a, const Cand& b) { return a.ms < b.ms; };
  Cand uni[2 * NT], fin[kPairs * NT];
  int nu = 0, nf = 0;
  for (int t = 0; t < NT; ++t)
    for (int m = 0; m < 2; ++m)
      if (seen[t][m]) uni[nu++] = {t, m, t, ms[t][m]};
  std::sort(uni, uni + nu, faster);
  const Cand top = uni[0];
  best = {top.tile, top.mode, top.tile};
  for (int q = 0; q < std::min(nu, kPairs) && uni[q].ms < kNear * top.ms; ++q)
    for (int f = 0; f < NT; ++f)
      if (ok(f) && f != uni[q].tile) fin[nf++] = {uni[q].tile, uni[q].mode, f, 0.0};
  // (by shapes, so that each table is made once a round)
  std::sort(fin, fin + nf, [](const Cand& a, const Cand& b) {
    return a.tile != b.tile ? a.tile < b.tile : (a.ftile != b.ftile ? a.ftile < b.ftile : a.mode < b.mode);
  });
  for (int round = 0; round < kRounds; ++round) {
    for (int q = 0; q < nf; ++q) {
      double v = 0.0;
      if (const int rc = timed(fin[q].tile, fin[q].mode, fin[q].ftile, v)) return rc;
      fin[q].ms = round ? std::min(fin[q].ms, v) : v;
    }
    if (round == 0 && nf > 1) {
      std::sort(fin, fin + nf, faster);
      int n = 1;
      while (n < std::min(nf, kPairs) && fin[n].ms < kClose * fin[0].ms) ++n;
      nf = n;
    }
  }
  if (nf) {
    const Cand f = *std::min_element(fin, fin + nf, faster);
    if (f.ms < kGain * top.ms) {
      best = {f.tile, f.mode, f.ftile};
      ms[f.tile][f.mode] = f.ms;
    }
  }
  return 0;
}

}  // namespace smhd
