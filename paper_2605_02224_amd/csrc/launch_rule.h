// Which query kernel answers a launch and how it is laid out.  Plain host code, so that the
// rules can be checked without a GPU.  All of them only choose between kernels that give the
// same rows.
#pragma once
#include <cstdint>

namespace mknn {

enum class Walk { kRows = 0, kWaves = 1, kScan = 2 };

struct LaunchSize {
  int64_t nq = 0;
  int32_t kmax = 0;         // neighbours walked for, the largest of the launch
  bool per_query = false;   // a k and a prefix per query
  int64_t m = 0, n = 0;     // the launch's prefix; points of the cloud
  int64_t longest = 0;      // entries of the cloud's longest list
};

// Launches by rows are bucketed from here on.
constexpr int64_t kSortMinQueries = 8192;
// Sizes between which walk_for() chooses.
constexpr int64_t kSmallQueries = 16384, kLargeQueries = 65536;
// The wave kernel gains less from neighbours in a wavefront than the bucketing costs (five
// launches, 20 us and up) until launches are larger: 1M-point torus, k = 16, 65536 queries 176
// us as they come, 200 us bucketed; 262144 queries 608 and 604; 1000000 queries 2100 and 1943.
// With long rows, or the plane fit's gather of their points, it is ahead from about 150k on, by
// a few per cent, and costs nothing from half kWaveSortQueries on: 200k points, 131072 queries
// k = 64 718 and 716 us, k = 20 with planes 412 and 415; 160000 876 and 863, 494 and 489; 262144
// 1360 and 1317, 776 and 758.
constexpr int64_t kWaveSortQueries = 262144;

// ---- Clouds with long lists.  Most clouds' longest lists grow slowly (torus, sphere, solid: 140
// entries at 3k points, 500 at 1M); sheets, whose hull meets their rim, have some of 1000 to
// 12000 (height fields of 100k to 1M points, up to n / 32), and a point far from the others, or
// inside a closed surface, is adjacent to a large part of the cloud (20 outliers of 200k points:
// 53551).  Queries that come to such a list read it to its end, which a wavefront's other
// queries wait for.
constexpr int64_t kLongList = 1024;
inline bool long_lists(const LaunchSize &l) { return l.longest > kLongList; }
// Some list is a good part of the cloud: many queries meet it, and the row kernel's four
// queries side by side read it together.
inline bool hub_lists(const LaunchSize &l) {
  return l.longest > 4096 && l.longest > l.n / 16;
}

// Rows or wavefronts.  The wave kernel's steps are short (a query's critical path is half the
// row kernel's), the row kernel's lanes are fuller for short rows of many queries.  us per
// launch over a 1M-point torus, rows (bucketed; k = 16 gathering from 196608 on) / wave (bucketed
// from kWaveSortQueries on, k = 64 from half):
//   queries      k=1         k=8          k=16         k=20         k=32         k=64
//   10000       47 / 27     74 / 43      95 / 55     117 / 60     147 / 72     258 / 111
//   32768       50 / 33     88 / 73     118 / 98     148 / 110    192 / 147    396 / 258
//   65536       81 / 51    144 / 137    199 / 175    250 / 196    338 / 260    678 / 444
//   98304      107 / 86    199 / 202    272 / 249    342 / 279    469 / 370    950 / 626
//   262144     221 / 176   422 / 448    541 / 611    781 / 708   1042 / 948   2129 / 1526
//   1000000    739 / 541  1412 / 1431  1746 / 1959  2518 / 2232  3387 / 3015  7240 / 5171
// (Between kLargeQueries and 196608 the two are within 10% for k of 8 to 16, either way by cloud.)
// Prefixes cut lists short, which leaves the wave kernel's batches half empty; the scan kernel
// drops a list where the prefix ends, and the rows lose least.  Over 400k points, rows / wave /
// scan, prefix of 100k: 65536 queries k=8 115 / 147 / 133, k=32 270 / 320 / 296, k=64 603 / 613 /
// 574; 500k queries k=16 694 / 1167 / 865, k=20 1078 / 1359 / 1031, k=64 3635 / 3655 / 2558; 20000
// queries k=32 130 / 141 / 142; 4096 queries k=16 51 / 37 / 50.  A k and prefix per query
// (prefixes of 400 to 400k; all 400k): 20000 queries k <= 32 229 / 209 / 201 (238 / 184 / 234);
// 70000 k <= 32 404 / 348 / 321 (415 / 300 / 350), k <= 64 764 / 554 / 488 (786 / 409 / 518);
// 131072 k <= 16 369 / 363 / 345 (395 / 340 / 383), k <= 32 538 / 496 / 448 (550 / 427 / 491);
// 200000 k <= 4 331 / 322 / 317 (367 / 343 / 367), k <= 16 464 / 476 / 444 (503 / 453 / 514);
// 262144 k <= 4, bucketed 379 / 428 / 417 (417 / 434 / 454); 500k queries k <= 16 856 / 973 / 883
// (927 / 870 / 957), k <= 32 1399 / 1434 / 1153 (1449 / 1150 / 1231).
// Few queries in a prefix, time of waves over rows, mean of 16 or 24 draws (prefixes of a half, a
// quarter, a twentieth and a hundredth; torus, solid, sphere and height field of 400k points; in
// the box and near): k=2 4200 queries 0.90-0.99, 5000 0.95-1.04, 6500 1.04-1.18, 8191 1.04-1.30;
// k=4 0.89-0.96, 0.95-0.99, 0.95-1.11, 0.95-1.23; k=8 a twentieth and up 0.75-0.97, a hundredth 0.87,
// 0.90, 1.01, 1.10; 8192 and up (rows bucketed) 0.40-0.92.  k=32 and 64 2048 queries 0.52-0.55, 8192
// 0.60-0.66, 14000 0.81-0.85, 16384 0.86-0.93: single draws reach 1.3 there (a few slow queries hold
// the waves up, which bucketed rows share).
// Long lists: 200k queries with a k and prefix each over a height field (longest list 2755), all
// 400k points: k <= 32 rows 1094, waves 912, scan 1073; k <= 4 563 / 526 / 695.  With a hub, larger
// launches go by rows but for k = 1, and for k <= 16 up to kLargeQueries: a sphere and its centre
// (60k points, longest list 17096), 65536 queries k=8 rows 815, waves 762; k=32 1002 / 1354; 200k
// queries k=32 1725 / 3080; 70000 queries k <= 32 each 1162 / 1383, scan 2190.
inline Walk walk_for(const LaunchSize &l) {
  if (hub_lists(l) && l.nq > 8192) {
    if (l.per_query) return Walk::kRows;
    if (l.kmax == 1) return Walk::kWaves;
    return l.kmax <= 16 && l.m >= l.n && l.nq <= kLargeQueries ? Walk::kWaves : Walk::kRows;
  }
  const bool uniform = !l.per_query, prefix = uniform && l.m < l.n;
  // as many wavefronts as are resident at once, each on one short query: rows, four to a
  // wavefront and not bucketed either, issue less
  if (prefix && l.kmax > 1 && l.nq < kSortMinQueries &&
      (l.kmax <= 4 ? l.nq > 5000 : l.kmax <= 8 && l.nq > 6500 && l.m < l.n / 32))
    return Walk::kRows;
  if (l.nq <= kSmallQueries || (uniform && l.kmax == 1)) return Walk::kWaves;
  if (!uniform) {
    if (l.nq <= kLargeQueries || (long_lists(l) && l.nq < kWaveSortQueries)) return Walk::kWaves;
    if (l.kmax > 16) return l.kmax <= 32 && l.nq <= 98304 ? Walk::kWaves : Walk::kScan;
    // (bucketing costs what the waves gain from it)
    return l.nq < (l.kmax <= 4 ? kWaveSortQueries : 131073) ? Walk::kWaves : Walk::kRows;
  }
  if (prefix) {
    const int64_t scan_min = l.kmax > 32 ? kLargeQueries : kWaveSortQueries;
    return l.kmax > 16 && l.nq >= scan_min ? Walk::kScan : Walk::kRows;
  }
  return l.nq <= kLargeQueries || l.kmax > 16 ? Walk::kWaves : Walk::kRows;
}

// Queries from which a launch of the wave or scan kernel is bucketed.  Single neighbours with a
// hub earlier: the descents that end in its list then share their wavefronts (sphere and centre,
// 200k queries 1270 us as they come, 552 bucketed).
inline int64_t wave_sort_min(const LaunchSize &l, bool planes) {
  if (l.kmax == 1 && hub_lists(l)) return 32768;
  return l.kmax > 32 || planes ? kWaveSortQueries / 2 : kWaveSortQueries;
}

// Whether the rows of a launch (a batch's class) of nq queries gather candidates: it takes a third
// fewer instructions, but rows wait for each other's merges, which only other wavefronts' work
// hides, and short rows have few lists to take meanwhile.  ms per launch over a 1M-point torus,
// step by step / gathered: k=16 1M queries 1.99 / 1.75, 262144 0.599 / 0.541, 131072 0.316 / 0.337;
// k=8 1M queries 1.39 / 1.40.  Such rows know no merge threshold.
constexpr bool gather_rows(int32_t k, int64_t nq) { return k > 8 && nq >= 196608; }

// How the wave kernel lays the queries out: lanes per query in the descent, and queries per
// wavefront (at most 64 / lanes; a second one only once every resident wavefront has one).
// Eight queries a wavefront pay for short rows, and for bucketed launches over clouds past the
// caches, 8 lanes / 16, us: 65536 queries over a 400k-point torus k=1 43 / 56, k=4 98 / 101, k=20
// 193 / 180, k=32 259 / 241 (with a k and prefix each k <= 4 212 / 198); 300k of k=20 over 400k
// points 706 / 671, 500k over a solid of 5M 1240 / 1290; and not where lists are long (height
// field, 65536 queries k=1 219 / 149, 300k of k=20 1410 / 1140).
struct WaveShape {
  int32_t lanes, per_wave;
};
inline WaveShape wave_shape(const LaunchSize &l, int64_t resident) {
  WaveShape w;
  const bool eight =
      l.kmax <= (l.per_query ? 1 : 8) || (l.kmax <= 32 && l.nq >= kWaveSortQueries);
  w.lanes = eight && !long_lists(l) && l.nq >= 8 * resident ? 8 : 16;
  w.per_wave = 1;
  // a single neighbour has no expansion to wait for: four descents side by side as soon as they
  // leave wavefronts enough (8191 queries over 400k points 21.1 us, one each 23.8; in a prefix of
  // 20k 11.2 and 15.5)
  if (l.kmax == 1 && l.nq > 3 * resident / 8) w.per_wave = 4;
  while (w.per_wave * 2 <= 64 / w.lanes && l.nq > w.per_wave * resident) w.per_wave *= 2;
  return w;
}

}  // namespace mknn
