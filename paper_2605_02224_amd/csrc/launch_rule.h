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
// launches, 20 us and up) until launches are larger: 1M-point torus, k = 16, 65536 queries 182
// us as they come, 215 us bucketed; 262144 queries 594 and 590; 1000000 queries 2081 and 1928.
// With long rows, or the plane fit's gather of their points, it pays from half as many: 200k
// queries over 200k points, k = 64 1.42 and 1.33 ms, k = 20 with planes 714 and 692 us.
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
// launch over a 1M-point torus, rows (bucketed) / wave (bucketed from kWaveSortQueries on):
//   queries      k=1         k=8          k=16         k=20         k=32         k=64
//   10000       51 / 26     69 / 43      89 / 52     111 / 58     140 / 72     248 / 168
//   32768       51 / 34     90 / 77     122 / 102    152 / 114    195 / 152    375 / 327
//   65536       76 / 50    136 / 134    188 / 182    241 / 207    312 / 277    633 / 525
//   98304      101 / 81    182 / 200    255 / 268    328 / 305    433 / 407    899 / 708
//   262144     213 / 172   397 / 430    567 / 590    730 / 676    990 / 917   2071 / 1591
//   1000000    695 / 534  1388 / 1433  1947 / 1928  2507 / 2199  3373 / 2974  7195 / 5374
// Prefixes cut lists short, which leaves the wave kernel's batches half empty; the scan kernel
// drops a list where the prefix ends, and the rows lose least.  Over 400k points, rows / wave /
// scan, prefix of 100k: 65536 queries k=8 114 / 145 / 133, k=32 268 / 352 / 297, k=64 579 / 720 /
// 576; 500k queries k=16 680 / 1139 / 866, k=20 1067 / 1337 / 986, k=64 3622 / 3724 / 2447; 20000
// queries k=32 131 / 148 / 206; 4096 queries k=16 50 / 39 / 52.  A k and prefix per query
// (prefixes of 400 to 400k; all 400k): 20000 queries k <= 32 236 / 207 / 207 (250 / 184 / 218);
// 70000 k <= 32 402 / 364 / 367 (414 / 309 / 399), k <= 64 scan 474, waves 528; 131072 k <= 16 375 / 375 / 354 (395 / 350 / 399),
// k <= 32 533 / 513 / 462 (568 / 439 / 512); 200000 k <= 4 333 / 333 / 326 (358 / 362 / 373), k <= 16
// 458 / 487 / 454 (498 / 457 / 524); 262144 k <= 4, bucketed 370 / 417 / 411 (408 / 422 / 447); 500k
// queries k <= 16 878 / 983 / 890 (944 / 871 / 965), k <= 32 1414 / 1418 / 1147 (1464 / 1145 / 1243).
// Few queries in a prefix, rows / waves, over 400k points on a torus and in a solid: 6500 queries
// k=2, m=100k 17.9 / 21.3 and 18.5 / 20.8, k=4, m=24k 19.5 / 21.6 and 20.7 / 23.6; 8191 queries
// k=8, m=4k 24 / 26 and 25 / 29; 16384 queries k=32, m=100k 124 / 106 and 123 / 138, k=64 246 / 195
// and 240 / 267 (13000 queries: waves are ahead in both).
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
  if (prefix && l.kmax > 1) {
    // as many wavefronts as are resident at once, each on one short query: rows, four to a
    // wavefront and not bucketed either, issue less
    if (l.nq > 4096 && l.nq < kSortMinQueries && (l.kmax <= 4 || (l.kmax <= 16 && l.m < l.n / 32)))
      return Walk::kRows;
    if (l.nq > 15360 && l.kmax > 16 && l.nq <= kSmallQueries) return Walk::kRows;
  }
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
// step by step / gathered: k=16 1M queries 1.95 / 1.79, 262144 0.567 / 0.538, 131072 0.316 / 0.337;
// k=8 1M queries 1.39 / 1.40.  Such rows know no merge threshold.
constexpr bool gather_rows(int32_t k, int64_t nq) { return k > 8 && nq >= 196608; }

// How the wave kernel lays the queries out: lanes per query in the descent, and queries per
// wavefront (at most 64 / lanes; a second one only once every resident wavefront has one).
// Eight queries a wavefront pay for short rows and for bucketed launches, 8 lanes / 16, us: 65536
// queries over a 400k-point torus k=1 45 / 54, k=4 97 / 101, k=20 187 / 181, k=32 255 / 243 (with a
// k and prefix each k <= 4 212 / 198); 500k over a solid of 5M k=20 1240 / 1290; and not where lists are long (height field, 65536 queries
// k=1 219 / 149, 300k of k=20 1410 / 1140).
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
