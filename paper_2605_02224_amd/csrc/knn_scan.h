// The wave kernel's walk (knn_wave.h) with another expansion, for launches with a k and prefix
// per query: most lists end early in their prefix there, and batches laid out by the lists'
// lengths stay half empty.
//
// Four rows of 16 lanes scan a list of the query's each, taken in turn from a queue of N's
// nearest unexpanded sites, and drop it where the prefix ends.  A step appends the entries that
// may rank (not farther than the k-th site, not nearer than the list's owner) to a buffer in
// LDS; once it holds 32, or no list is left, one sorting network merges it into N.
//
// N is one 32-bit key per lane, ascending, as in knn_wave.h, but position p's exact key lies at
// place p in LDS; the low bits number the sites during a merge only.  A site offered twice meets
// its own copy next to it in the merged order and is dropped there.  What equal upper bits can
// hide -- a site dropped while it agrees with the k-th, a copy kept apart from its own by a
// third site -- is noticed, and such a query answered again by answer_exact().  An entry nearer
// than its list's owner is a transition site or in the list of a nearer one, expanded as well.
//
// What bounds it is instruction issue (1.34e9 in 1.31 ms for 500k queries of k = 32 in a prefix
// of 100k of 400k points): 500k queries of k <= 32 with a prefix each 1.15 ms, by rows 1.40.
#pragma once
#include "knn_wave.h"

namespace mknn {

constexpr uint32_t kScanPad = 0xffffff00u;   // empty position of N

// R: positions of N (16, 32 or 64), at least the launch's largest k.
template <int DW, int R>
struct ScanLds {
  static constexpr int C = R <= 32 ? 64 - R : 64;   // candidates a merge takes
  static constexpr int Full = 32;                   // candidates that start one
  static constexpr int Q = 16;                      // lists queued at a time
  struct __align__(16) Site {
    double d;
    int32_t r;
    uint32_t key;   // in the buffer: all bits of the float
  };
  struct __align__(16) List {
    uint32_t st, len, own, pad;   // own: the owner's key
  };
  Site site[R + (R <= 32 ? Full + 64 : 2 * C)];   // N, then the buffer
  List next[Q];
  uint32_t ring[64 / DW][R];

  // the site a key names (bits 1 .. 7: a position of N, or R and up the buffer's from b on)
  __device__ __forceinline__ const Site &of(uint32_t key, int b) const {
    const uint32_t at = (key & 0xfeu) << 3;
    return *reinterpret_cast<const Site *>(reinterpret_cast<const char *>(site) + at +
                                           (at < 16u * R ? 0 : 16 * b));
  }
};

// rows of 16 ascending -> halves of 32 ascending
__device__ __forceinline__ uint32_t scan_row_pairs(uint32_t x, int lane) {
  x = exchange<31, 16>(x, lane);
  x = exchange<8, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  return exchange<1, 1>(x, lane);
}
// halves of 32 ascending -> the wavefront ascending
__device__ __forceinline__ uint32_t scan_halves(uint32_t x, int lane) {
  x = exchange<63, 32>(x, lane);
  x = exchange<16, 16>(x, lane);
  x = exchange<8, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  return exchange<1, 1>(x, lane);
}

// N while a query is expanded.  Uniform but for `key`.
template <int DW, int R>
struct ScanMerger {
  using Lds = ScanLds<DW, R>;
  using Site = typename Lds::Site;
  uint32_t key;        // lane p: position p of N (lanes R and up: empty)
  uint32_t thr;        // key of the k-th position
  uint64_t again;      // not 0: the query is to be answered again with exact keys

  __device__ __forceinline__ void set_threshold(int k) {
    thr = min(readlane_u32(key, k - 1) | kTieBits, kMaxKey);
  }
  // Merges the buffer's candidates b .. b + n - 1, n <= C, into N.
  __device__ __forceinline__ void merge(Lds &w, int k, int lane, int b, int n) {
    if constexpr (R <= 32) {
      // N and the candidates side by side in the lanes
      uint32_t x = w.site[(lane < R ? 0 : b) + lane].key & ~kTieBits;
      x = lane < R ? key : x;
      x = (lane < R + n ? x : kScanPad) | (uint32_t)(lane << 1);
      x = scan_row_pairs(sort_rows(x, lane), lane);
      if (R == 32 || n > 16) x = scan_halves(x, lane);
      const Site v = w.of(x, b);
      const uint64_t copy = lanes_where(v.r == (int32_t)wave_shr1((uint32_t)v.r)) &
                            lanes_where(x < kScanPad) & ~1ull;
      const int to = lane - lanes_below(copy);
      const uint64_t in = lanes_where(to < R) & ~copy;
      place(w, v, x, to, in, lane);
      set_threshold(k);
      again |= ~(in | copy) & lanes_where((x & ~0xfeu) <= thr);
      if (__popcll(copy) > n) again = 1;
    } else {
      uint32_t y = w.site[R + b + lane].key & ~kTieBits;
      y = (lane < n ? y : kScanPad) | (uint32_t)((R + lane) << 1);
      y = sort_rows(y, lane);
      if (n > 16) y = scan_halves(scan_row_pairs(y, lane), lane);
      // against the descending candidates: the 64 smaller keys of both and the 64 larger
      y = lane_value(y, 63 - lane);
      const uint32_t o = key | (uint32_t)(lane << 1);
      const uint32_t x = merge_bitonic(min(o, y), lane);
      y = merge_bitonic(max(o, y), lane);
      const Site v = w.of(x, b), z = w.of(y, b);
      const uint64_t copy = lanes_where(v.r == (int32_t)wave_shr1((uint32_t)v.r)) &
                            lanes_where(x < kScanPad) & ~1ull;
      const int32_t last = __builtin_amdgcn_readlane(v.r, 63);
      const int32_t before = __builtin_amdgcn_update_dpp(last, z.r, 0x138, 0xf, 0xf, false);
      const uint64_t copy2 = lanes_where(z.r == before) & lanes_where(y < kScanPad);
      const int gone = __popcll(copy);
      const int to = lane - lanes_below(copy);
      const int to2 = R + lane - gone - lanes_below(copy2);
      const uint64_t in2 = lanes_where(to2 < R) & ~copy2;
      wave_lds_sync();
      if (in_mask(in2)) w.site[to2] = Site{z.d, z.r, y & ~0xfeu};
      place(w, v, x, to, ~copy, lane);
      set_threshold(k);
      again |= ~(in2 | copy2) & lanes_where((y & ~0xfeu) <= thr);
      if (gone + __popcll(copy2) > n) again = 1;
    }
  }
  // The sites v of the lanes in `in` go to the positions `to`; then every lane its position's.
  __device__ __forceinline__ void place(Lds &w, const Site &v, uint32_t x, int to, uint64_t in,
                                        int lane) {
    wave_lds_sync();
    if (in_mask(in)) w.site[to] = Site{v.d, v.r, x & ~0xfeu};
    wave_lds_sync();
    key = w.site[lane].key;
    if (R < 64) key = lane < R ? key : kScanPad;
  }
};

// Alg. 2 for query t of the wavefront.  The control flow is uniform.  False: to be answered by
// answer_exact() (kept out of this loop, whose registers it would take).
template <int DW, int R>
__device__ __forceinline__ bool scan_expand(const QueryArgs &a, ScanLds<DW, R> &w, const WaveQuery &q,
                                       int t, int lane) {
  using Lds = ScanLds<DW, R>;
  double d = INFINITY;
  int32_t r = kEmpty;
  const int seeds = min(q.nt, q.k);   // the last transition sites, nearest first
  if (lane < seeds) {
    const float4 c = ring_site(a, w.ring[t][(uint32_t)(q.nt - 1 - lane) & (R - 1u)]);
    d = sq_dist(q.qx, q.qy, q.qz, c);
    r = __float_as_int(c.w);
  }
  if (seeds == 0) {
    write_row(a, q, d, r, lane);
    return true;
  }
  const double d1 = readlane_f64(d, 0);
  if (!(d1 < INFINITY)) return false;
  // D -> the key's order bits: the float32 of (D - D_1) s, s a power of two that puts the
  // cloud's extent near 1; both roundings are monotone
  const double s = a.key_scale, off = -(d1 * s);
  auto order_bits = [&](double v) { return __float_as_uint((float)__builtin_fma(v, s, off)); };
  ScanMerger<DW, R> N;
  N.key = lane < seeds ? order_bits(d) & ~kTieBits : kScanPad;
  N.again = 0;
  if (R == 64 || lane < R) w.site[lane] = typename Lds::Site{d, r, N.key};
  N.set_threshold(q.k);
  wave_lds_sync();

  const int l = lane & 15;
  const bool prefix = q.m < a.n;
  uint32_t pos = (uint32_t)l, rem = 0, own = 0;   // the row's list: the lane's entry, entries left
  uint64_t busy = 0;                              // rows with a list
  uint32_t lists = 0;
  for (;;) {
    // ---- queue the lists of the nearest unexpanded sites
    const uint32_t lim = min(readlane_u32(N.key, q.k - 2) | kTieBits, kMaxKey);
    const uint64_t open = lanes_where(N.key <= lim) & lanes_where((N.key & 1u) == 0);
    if (!(open | busy)) break;
    uint32_t turn = (uint32_t)lanes_below(open);
    turn = in_mask(open) ? turn : ~0u;
    if (turn < (uint32_t)Lds::Q) {
      const uint64_t dsc = a.lst[(uint32_t)w.site[lane].r];
      w.next[turn] = typename Lds::List{(uint32_t)dsc, (uint32_t)(dsc >> 32), N.key, 0u};
    }
    const uint32_t queued = min((uint32_t)__popcll(open), (uint32_t)Lds::Q);
    uint32_t taken = 0;
    int count = 0;
    wave_lds_sync();
    // ---- scan them, until a merge is due
    do {
      if (taken < queued) {
        // the rows without a list take the next ones
        const uint64_t rows = ~busy & 0x8000800080008000ull;
        const uint32_t at = taken + (uint32_t)lanes_below(rows);
        if (in_mask(~busy & lanes_where(at < queued))) {
          const typename Lds::List e = w.next[at];
          pos = e.st + (uint32_t)l;
          rem = e.len;
          own = e.own;
        }
        taken = min(taken + (uint32_t)__popcll(rows), queued);
      }
      // every lane loads: a chunk reaches at most 15 records past the end of its list, which
      // the arena's padding covers, and a row without a list stays where it is
      const float4 c = a.ent[pos];
      const int32_t cr = __float_as_int(c.w);
      const double cd = sq_dist(q.qx, q.qy, q.qz, c);
      const uint32_t u = order_bits(cd);
      uint64_t cand = lanes_where((uint32_t)l < rem) & lanes_where(u <= N.thr) &
                      lanes_where(u >= own);
      rem = __builtin_elementwise_sub_sat(rem, 16u);
      if (prefix) {
        // ascending ranks: the list ends where the prefix does
        cand &= lanes_where(cr < q.m);
        rem = dpp_i32<kDppRowBcast15>(0, cr) < q.m ? rem : 0u;
      }
      busy = lanes_where(rem != 0);
      pos += in_mask(busy) ? 16u : 0u;
      if (cand) {
        const int at = count + lanes_below(cand);
        if (in_mask(cand)) w.site[R + at] = typename Lds::Site{cd, cr, u};
        count += __popcll(cand);
      }
    } while ((busy != 0 || taken < queued) && count < Lds::Full);
    // ---- the sites whose lists were taken are expanded; merge the candidates
    N.key |= turn < taken ? 1u : 0u;
    wave_lds_sync();
    for (int b = 0; b < count; b += Lds::C) N.merge(w, q.k, lane, b, min(count - b, Lds::C));
    // copies that equal keys keep apart are expanded once more each: not without end
    lists += taken;
    if (N.again != 0 || lists > 4u * R) return false;
  }
  // ---- the exact keys, and the order of those whose upper bits agree
  d = INFINITY;
  r = kEmpty;
  const uint64_t real = lanes_where(N.key < kScanPad);
  if (in_mask(real)) {
    d = w.site[lane].d;
    r = w.site[lane].r;
  }
  const uint64_t tie = lanes_where((N.key ^ wave_shr1(N.key)) <= kTieBits) & real &
                       lanes_where(lane <= q.k) & ~1ull;
  if (tie) {
    order_lanes(d, r, lane);
    if (lanes_where(r == (int32_t)wave_shr1((uint32_t)r)) & real & lanes_where(lane < q.k) & ~1ull)
      return false;
  }
  write_row(a, q, d, r, lane);
  return true;
}


// Plain launch: per_wave consecutive sorted queries per wavefront (1 .. 64 / DW).
template <int DW, int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8)))
void knn_scan_kernel(QueryArgs a, int32_t per_wave) {
  __shared__ ScanLds<DW, R> lds[4];
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t begin = ((int64_t)xcd_tile(blockIdx.x, gridDim.x) * 4 + wid) * per_wave;
  if (begin >= a.nq) return;   // whole wavefronts leave
  const int cnt = (int)(a.nq - begin < per_wave ? a.nq - begin : per_wave);
  const int lane = threadIdx.x & 63;
  ScanLds<DW, R> &w = lds[wid];
  Descent<DW, R> q;
  q.run(a, w.ring, begin, cnt);
  uint64_t todo = lanes_where((lane & (DW - 1)) == 0) & lanes_where(q.k > 0), again = 0;
  while (todo) {
    const int t = pop_lane(todo) / DW;
    wave_lds_sync();   // the sites of the query before
    if (!scan_expand(a, w, q.query(t), t, lane)) again |= 1ull << t;
  }
  while (again) answer_exact(a, q.query(pop_lane(again)), lane);
}

}  // namespace mknn
