// The query kernels' walk: descents side by side, expansions one query per wavefront.
//
// What bounds the expansions is the issue of instructions, vector and scalar alike (1M queries
// of k=64: 5.93e9 in 5.15 ms; the lists sit in the caches), so the split follows where each part
// keeps the 64 lanes busy.  Descents alone wait for their chains of loads (k=1: 0.30e9 in 0.48
// ms, wavefronts waiting for 70% of it).
//
//   descent (Alg. 1): DW lanes per query, 64 / DW queries of a wavefront side by side.  A
//     step reads DW consecutive entries of a row's current list; the first strictly closer
//     one is the next transition site, whose record index goes to the row's ring in LDS.
//     The rows branch on their own chunks, but every step is the same instructions.
//   expansion (Alg. 2): the queries of the wavefront one after the other, 64 lanes each.
//     Everything that steers it (list descriptors, candidate masks, the threshold) is then
//     uniform: scalar registers, ballots and lane reads instead of per-row shuffles.  A
//     batch lays the next unexpanded neighbours' lists end to end over the 64 lanes (4-5
//     lists of about 14 entries), so a k=16 query takes about 4.5 batches where one list at
//     a time took 23 chunks of 16 lanes, 62% filled.
//
// Expanding a neighbour before it is known to be final is harmless: the lists of some sites
// that are displaced later are scanned as well.  The query ends when the first k - 1 sites of
// N are expanded.  N is then exact: N[1] is the end of the descent, and by Theorem 1 the
// (i+1)-th neighbour is a transition site or in the list of one of the first i, all of them
// expanded, so it has been offered and the first i + 1 of N are the true ones.
//
// N is one 32-bit key per lane, ascending: a lane holds the float32 of D - D_1 (a monotone
// map of D), its low 7 bits replaced by the number of the LDS slot that holds the site's
// exact key (D in float64, rank) and an "expanded" flag.  Inserting a candidate is a lane
// read, a wave-wide shift by one lane and a median of three, whatever k is.  Keys that agree
// in the upper 24 bits are not ordered by the map; nothing depends on their order until
//   - the end, where neighbours in the row that agree are ordered by their exact keys,
//   - a key that is dropped past lane 63 while it agrees with the k-th: keep_nearest() then
//     decides by the exact keys, which are still in their slots, which of them stay.
// Sites already offered are recognised by rank in an open-addressed table in LDS.
//
// Measured, against the row kernel: 2000 queries of k=20 over 1M points 30 us for 77; 200k of
// k=64 over 200k points 1.05 ms for 1.55; 500k of k=1 0.245 ms for 0.31; 131k of k=32 with pending
// deletions 0.60 ms for 0.86; 1M queries of k=16 over 1M points 1.96 ms for 1.75 (the row kernel
// gathers candidates there).
#pragma once
#include "knn_group.h"

namespace mknn {

constexpr int kWaveSlots = 128;          // LDS slots of exact keys, per wavefront
constexpr int kWaveSeen = 512;           // table of offered ranks, per wavefront
constexpr uint32_t kHeadRecord = 0xffffffffu;   // ring entry of the head, which has no record
constexpr uint32_t kPadKey = 0xffffffffu;       // empty position of N
constexpr uint32_t kMaxKey = 0x7f8000ffu;       // largest key of a number (D - D_1 = +inf)
constexpr uint32_t kTieBits = 0xffu;            // slot and flag: no part of the order
constexpr int kWaveInsert = 5;           // new keys up to which they are inserted one by one

// R: entries per row of the ring, a power of two >= the launch's largest k.
template <int DW, int R>
struct WaveLds {
  double d[kWaveSlots];        // slots: the exact key (D, rank) of a site
  int32_t r[kWaveSlots];
  int32_t seen[kWaveSeen];
  uint32_t ring[64 / DW][R];

  // the slot a key names (bits 1 .. 7)
  __device__ __forceinline__ double &d_of(uint32_t key) {
    return *reinterpret_cast<double *>(reinterpret_cast<char *>(d) + ((key & 0xfeu) << 2));
  }
  __device__ __forceinline__ int32_t &r_of(uint32_t key) {
    return *reinterpret_cast<int32_t *>(reinterpret_cast<char *>(r) + ((key & 0xfeu) << 1));
  }
};

// the lanes where p holds (the builtin takes the comparison's mask as it is)
__device__ __forceinline__ uint64_t lanes_where(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(b >> 32), lane);
  return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ float readlane_f32(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ uint32_t readlane_u32(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int32_t)v, lane);
}
// Takes the lowest set bit out of a uniform mask and returns its number; sets bit i.  (One
// scalar instruction each, where the compiler takes two and three for the 64-bit forms.)
__device__ __forceinline__ int pop_lane(uint64_t &mask) {
  const int j = __builtin_ctzll(mask);
  asm("s_bitset0_b64 %0, %1" : "+s"(mask) : "s"(j) : );
  return j;
}
__device__ __forceinline__ void set_bit(uint64_t &mask, uint32_t i) {
  asm("s_bitset1_b64 %0, %1" : "+s"(mask) : "s"(i) : );
}
// the value of x in lane `from`
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int from) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int32_t)x);
}
// x with lane `lane` (uniform) set to the uniform v (the compiler's intrinsic, for which it
// has no builtin)
__device__ uint32_t writelane_u32(uint32_t v, int lane, uint32_t x) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ int lanes_below(uint64_t mask) {   // set bits below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
__device__ __forceinline__ bool in_mask(uint64_t mask) {   // this lane's bit
  return __builtin_amdgcn_inverse_ballot_w64(mask);
}
__device__ __forceinline__ uint32_t median(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));
}
// lane l reads lane l - 1; lane 0 reads 0
__device__ __forceinline__ uint32_t wave_shr1(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)x, 0x138, 0xf, 0xf, true);
}

// Marks the ranks r of the lanes in `want` as offered; the lanes whose rank had not been (one
// of several lanes with the same rank).  At most kWaveSeen - 64 ranks are in the table, so
// every probe ends at the rank or at a free entry.
__device__ __forceinline__ uint64_t mark_seen(int32_t *seen, int32_t r, uint64_t want) {
  uint64_t fresh = 0;
  uint32_t h = (uint32_t)r;
  while (want) {
    h &= kWaveSeen - 1;
    int32_t old = __builtin_nondeterministic_value(old);   // outside `want`: not looked at
    if (in_mask(want)) {
      old = kEmpty;
      __hip_atomic_compare_exchange_strong(&seen[h], &old, r, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    const uint64_t free = want & lanes_where(old == kEmpty);
    fresh |= free;
    want &= ~(free | lanes_where(old == r));
    ++h;
  }
  return fresh;
}
__device__ __forceinline__ void clear_seen(int32_t *seen, int lane) {
  const int4 e = make_int4(kEmpty, kEmpty, kEmpty, kEmpty);
  int4 *p = reinterpret_cast<int4 *>(seen);
#pragma unroll
  for (int i = 0; i < kWaveSeen / 256; ++i) p[64 * i + lane] = e;
}

// ---- networks over 32-bit keys.  A compare-exchange of lanes l and l ^ X is the median of
// the key, the partner's and a bound that is 0 in the lanes that keep the smaller one (bit
// BIT clear) and all ones in the others: one lane move and one instruction.
template <int BIT>
__device__ __forceinline__ uint32_t keep_bound(int lane) { return (lane & BIT) ? ~0u : 0u; }
template <int X, int BIT>
__device__ __forceinline__ uint32_t exchange(uint32_t x, int lane) {
  uint32_t p;
  if constexpr (X == 16) p = (uint32_t)__builtin_amdgcn_ds_swizzle((int32_t)x, 0x401F);
  else if constexpr (X == 31) p = (uint32_t)__builtin_amdgcn_ds_swizzle((int32_t)x, 0x7C1F);
  else if constexpr (X == 63) p = lane_value(x, 63 - lane);
  else if constexpr (X == 32) {
    // both halves of x, each in all lanes of a register: the exchange needs no selection
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    x = h[0];
    p = h[1];
  } else p = (uint32_t)xor_lane<X>((int32_t)x);
  return median(x, p, keep_bound<BIT>(lane));
}
// every row of 16 lanes ascending
__device__ __forceinline__ uint32_t sort_rows(uint32_t x, int lane) {
  x = exchange<1, 1>(x, lane);
  x = exchange<3, 2>(x, lane);
  x = exchange<1, 1>(x, lane);
  x = exchange<7, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  x = exchange<1, 1>(x, lane);
  x = exchange<15, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  return exchange<1, 1>(x, lane);
}
// rows of 16 ascending -> the wavefront ascending
__device__ __forceinline__ uint32_t merge_rows(uint32_t x, int lane) {
  x = exchange<31, 16>(x, lane);
  x = exchange<8, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  x = exchange<1, 1>(x, lane);
  x = exchange<63, 32>(x, lane);
  x = exchange<16, 16>(x, lane);
  x = exchange<8, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  return exchange<1, 1>(x, lane);
}
// a bitonic wavefront -> ascending
__device__ __forceinline__ uint32_t merge_bitonic(uint32_t x, int lane) {
  x = exchange<32, 32>(x, lane);
  x = exchange<16, 16>(x, lane);
  x = exchange<8, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  return exchange<1, 1>(x, lane);
}

// Sorts the lanes by (d, r) by exchanges of neighbours, for the few queries that need it.
__device__ __forceinline__ void order_lanes(double &d, int32_t &r, int lane) {
  bool moved;
  do {
    moved = false;
#pragma unroll
    for (int odd = 0; odd < 2; ++odd) {
      int p = odd ? ((lane + 1) ^ 1) - 1 : lane ^ 1;
      p = p < 0 || p > 63 ? lane : p;
      const double pd = __shfl(d, p);
      const int32_t pr = __shfl(r, p);
      const bool take = p > lane ? key_less(pd, pr, d, r) : key_less(d, r, pd, pr);
      d = take ? pd : d;
      r = take ? pr : r;
      moved |= take;
    }
  } while (lanes_where(moved) != 0);
}

// the bits of a row's DW lanes, in every lane of the row
template <int DW>
__device__ __forceinline__ uint32_t row_or(uint32_t x) {
  x |= (uint32_t)xor_lane<1>((int32_t)x);
  x |= (uint32_t)xor_lane<2>((int32_t)x);
  x |= (uint32_t)xor_lane<7>((int32_t)x);
  if constexpr (DW == 16) x |= (uint32_t)xor_lane<15>((int32_t)x);
  return x;
}

// One query of the wavefront, in uniform registers.
struct WaveQuery {
  double qx, qy, qz;
  int32_t qi;      // caller index
  int32_t k, m;    // neighbours walked for; prefix
  int32_t nt;      // transition sites (0: the prefix holds no live site)
};

// The row of a finished query: position `lane` holds (d, r), r == kEmpty past the end.
// Pending deletions (a.dead): the first kout unmarked positions are kept, in order; they are
// the kout nearest remaining sites whenever the walk's positions hold that many.  A row with
// fewer is exact only if the walk did not fill its k positions, and is counted otherwise.
__device__ __forceinline__ void write_row(const QueryArgs &a, const WaveQuery &q, double d,
                                          int32_t r, int lane) {
  const int32_t ko = !a.dead ? q.k : a.kq ? a.kq[q.qi] : a.kout;
  const int64_t row = a.row_off ? a.row_off[q.qi] : q.qi * (int64_t)ko;
  if (!a.dead) {
    if (lane < ko) {
      a.out_idx[row + lane] = r == kEmpty ? -1 : r;
      a.out_dist[row + lane] = r == kEmpty ? INFINITY : (float)sqrt(d);
    }
    return;
  }
  const bool listed = lane < q.k && r != kEmpty;
  uint32_t e = 0;
  if (listed) e = a.dead[r];
  const bool live = listed && (e == 0 || e > a.epoch);
  const uint64_t lm = lanes_where(live);
  const int before = lanes_below(lm), kept = __popcll(lm);
  if (live && before < ko) {
    a.out_idx[row + before] = r;
    a.out_dist[row + before] = (float)sqrt(d);
  }
  if (lane >= kept && lane < ko) {
    a.out_idx[row + lane] = -1;
    a.out_dist[row + lane] = INFINITY;
  }
  if (kept < ko && __popcll(lanes_where(listed)) == q.k && lane == 0) atomicAdd(a.overflow, 1u);
}

// Alg. 1 and Alg. 2 as written, one list after the other, the whole wavefront on one query,
// with the exact keys (D, rank) of N in the lanes.  For queries whose first distance is not
// finite (and, in the scan kernel, those with sites tied in their keys that it cannot order).
__device__ __forceinline__ void answer_exact(const QueryArgs &a, const WaveQuery &q, int lane) {
  double d = INFINITY;
  int32_t r = kEmpty;
  if (a.head < q.m) {
    int32_t cur = a.head;
    double dcur = sq_dist(q.qx, q.qy, q.qz, make_float4(a.hx, a.hy, a.hz, 0.f));
    if (lane == 0) {
      d = dcur;
      r = cur;
    }
    const float4 none = make_float4(0.f, 0.f, 0.f, __int_as_float(kEmpty));
    for (bool jumped = true; jumped;) {
      jumped = false;
      const uint64_t dsc = a.lst[cur];
      const uint32_t st = (uint32_t)dsc, len = (uint32_t)(dsc >> 32);
      for (uint32_t b = 0; b < len && !jumped; b += 64) {
        const float4 c = b + lane < len ? a.ent[st + b + lane] : none;
        const bool in = __float_as_int(c.w) < q.m;
        const double cd = sq_dist(q.qx, q.qy, q.qz, c);
        const uint64_t closer = lanes_where(in) & lanes_where(cd < dcur);
        if (closer) {
          // the transition sites get closer one by one: the newest goes first
          const int j = __builtin_ctzll(closer);
          dcur = readlane_f64(cd, j);
          cur = __builtin_amdgcn_readlane(__float_as_int(c.w), j);
          const double pd = __shfl_up(d, 1);
          const int32_t pr = __shfl_up(r, 1);
          d = lane ? pd : dcur;
          r = lane ? pr : cur;
          jumped = true;
        }
        if (lanes_where(in) != ~0ull) break;   // the end of the list or of the prefix
      }
    }
    for (int it = 0; it < q.k - 1; ++it) {
      const int32_t own = __builtin_amdgcn_readlane(r, it);
      if (own == kEmpty) break;
      const double od = readlane_f64(d, it);
      const uint64_t dsc = a.lst[own];
      const uint32_t st = (uint32_t)dsc, len = (uint32_t)(dsc >> 32);
      for (uint32_t b = 0; b < len; b += 64) {
        const float4 c = b + lane < len ? a.ent[st + b + lane] : none;
        const int32_t cr = __float_as_int(c.w);
        const bool in = cr < q.m;
        const double cd = sq_dist(q.qx, q.qy, q.qz, c);
        const double kd = readlane_f64(d, q.k - 1);
        uint64_t cand = lanes_where(in) & lanes_where(cd >= od) & lanes_where(cd <= kd);
        while (cand) {
          const int j = pop_lane(cand);
          const double nd = readlane_f64(cd, j);
          const int32_t nr = __builtin_amdgcn_readlane(cr, j);
          if (lanes_where(r == nr)) continue;
          const bool keep = key_less(d, r, nd, nr);
          const double pd = __shfl_up(d, 1);
          const int32_t pr = __shfl_up(r, 1);
          const bool first = lane == 0 || key_less(pd, pr, nd, nr);
          d = keep ? d : first ? nd : pd;
          r = keep ? r : first ? nr : pr;
        }
        if (lanes_where(in) != ~0ull) break;
      }
    }
  }
  write_row(a, q, lane < q.k ? d : INFINITY, lane < q.k ? r : kEmpty, lane);
}

// The record of a ring entry.
__device__ __forceinline__ float4 ring_site(const QueryArgs &a, uint32_t e) {
  return e == kHeadRecord ? make_float4(a.hx, a.hy, a.hz, __int_as_float(a.head)) : a.ent[e];
}

// Some of the keys `lost`, which fell out of the full N, agree with the k-th in their upper bits
// (they are <= thr): N with the nearest of those that agree, by their exact keys.  At k = 64 every
// key that falls out next to one like it comes here, a few in a hundred queries of most clouds
// and several in each where a query is far from all points or amid a shell; answering those
// again with exact keys throughout took as long as the rest (4096 queries of k=64 over 400k
// points 129 us, settled here 60).
template <int DW, int R>
__device__ __forceinline__ uint32_t keep_nearest(WaveLds<DW, R> &w, uint32_t N, uint32_t lost,
                                                 uint32_t thr, int lane) {
  uint64_t out = lanes_where(lost <= thr);
  while (out) {
    const uint32_t o = readlane_u32(lost, pop_lane(out));
    const double d = w.d_of(N);
    const int32_t r = w.r_of(N);
    uint64_t agree = lanes_where((N ^ o) <= kTieBits);   // the k-th is among them
    int far = pop_lane(agree);
    double fd = readlane_f64(d, far);
    int32_t fr = __builtin_amdgcn_readlane(r, far);
    while (agree) {
      const int j = pop_lane(agree);
      const double jd = readlane_f64(d, j);
      const int32_t jr = __builtin_amdgcn_readlane(r, j);
      const bool farther = key_less(fd, fr, jd, jr);
      far = farther ? j : far;
      fd = farther ? jd : fd;
      fr = farther ? jr : fr;
    }
    if (key_less(w.d_of(o), w.r_of(o), fd, fr)) N = writelane_u32(o, far, N);
  }
  return merge_rows(sort_rows(N, lane), lane);
}

// Alg. 2 for query t of the wavefront.  All control flow is uniform.  False: to be answered
// by answer_exact() (kept out of this loop, whose registers it would take).
template <int DW, int R>
__device__ __forceinline__ bool expand(const QueryArgs &a, WaveLds<DW, R> &w, const WaveQuery &q,
                                       int t, int lane) {
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
  uint32_t N = kPadKey;
  clear_seen(w.seen, lane);
  if (lane < seeds) {
    N = (order_bits(d) & ~kTieBits) | (uint32_t)(lane << 1);
    w.d[lane] = d;
    w.r[lane] = r;
  }
  wave_lds_sync();
  mark_seen(w.seen, r, ~0ull >> (64 - seeds));
  int nreal = seeds, nslot = seeds, nseen = seeds;   // keys in N, slots used, ranks marked
  uint32_t thr = min(readlane_u32(N, q.k - 1) | kTieBits, kMaxKey);
  // Lists are laid over the lanes whole, the last one cut where the lanes end; within a
  // prefix most of a list may lie past it, so a list gets at most 24 lanes at a time there.
  // The rest of a cut list goes first in the next batch: lane i of `pend` holds the rest of
  // the list that ended at lane i (at most 3, which fit one batch).
  const uint32_t cap = q.m < a.n ? 24u : 64u;
  uint64_t pend = 0;
  uint32_t pst = 0, plen = 0;
  for (;;) {
    const uint32_t lim = min(readlane_u32(N, q.k - 2) | kTieBits, kMaxKey);
    const uint64_t open = lanes_where(N <= lim) & ~lanes_where((N & 1u) != 0);
    if (!(open | pend)) break;
    uint32_t u;
    uint64_t cand;
    // (a prefix, cap = 24, ends most lists soon)
    const uint64_t runs = pend & lanes_where(plen >= (cap == 64u ? 64u : 256u));
    if (runs) {
      // what is left of a long list is read on by itself, 64 entries a step: neither the
      // descriptors of the sites behind it are loaded nor a layout made (200k points with 20
      // far outliers, 53551 entries in the longest list: 300 queries of k=8 1.26 ms, now 0.96;
      // 65536 of k=20 10.97 ms, now 4.9)
      const int j = __builtin_ctzll(runs);
      uint32_t st = readlane_u32(pst, j), len = readlane_u32(plen, j);
      do {
        const float4 c = a.ent[st + (uint32_t)lane];
        r = __float_as_int(c.w);
        d = sq_dist(q.qx, q.qy, q.qz, c);
        u = order_bits(d);
        const uint64_t in = lanes_where(r < q.m);
        cand = in & lanes_where(u <= thr);
        st += 64;
        len = in == ~0ull ? len - 64 : 0;
      } while (!cand && len >= 64);
      pst = writelane_u32(st, j, pst);
      plen = writelane_u32(len, j, plen);
      if (len == 0) pend &= ~(1ull << j);
    } else {
      // descriptors of the next unexpanded sites (about 4 fit a batch)
      uint64_t dsc = __builtin_nondeterministic_value(dsc), win = 0;
      if (open) {
        win = open & (0xffull << __builtin_ctzll(open));
        if (in_mask(win)) dsc = a.lst[(uint32_t)w.r_of(N)];
      }
      const uint32_t dst = (uint32_t)dsc, dlen = (uint32_t)(dsc >> 32);
      // ---- lay the lists over the lanes.  The i-th list starts at the i-th set bit of
      //      `starts`; lane i of `at` holds its first entry's index less that lane
      uint32_t at = __builtin_nondeterministic_value(at), rest = __builtin_nondeterministic_value(rest);
      uint32_t total = 0;
      uint64_t starts = 0, cut = 0;
      int lists = 0;
      auto lay = [&](uint32_t st, uint32_t len) {
        at = writelane_u32(st - total, lists, at);
        ++lists;
        set_bit(starts, total);
        const uint32_t room = min(cap, 64u - total);
        total += min(len, room);
        if (len > room) {
          set_bit(cut, total - 1);
          rest = writelane_u32(len - room, (int)total - 1, rest);
        }
      };
      while (pend) {
        const int j = pop_lane(pend);
        lay(readlane_u32(pst, j), readlane_u32(plen, j));
      }
      uint64_t left = win & lanes_where(dlen != 0);
      while (left) {
        if (total >= 64) break;
        const int j = pop_lane(left);
        lay(readlane_u32(dst, j), readlane_u32(dlen, j));
      }
      N |= in_mask(win & ~left) ? 1u : 0u;   // an empty list is expanded already
      if (total == 0) continue;
      // ---- the batch's entries.  Lanes past the last list read on behind it (the arena is
      //      padded for that) and are left out
      const uint32_t base = lane_value(at, lanes_below(starts >> 1));
      const float4 c = a.ent[base + (uint32_t)lane];
      r = __float_as_int(c.w);
      const uint64_t in = lanes_where(r < q.m) & (~0ull >> (64 - total));
      d = sq_dist(q.qx, q.qy, q.qz, c);
      u = order_bits(d);
      if (cut) {   // ascending ranks: a list goes on if its last entry here is in the prefix
        pend = cut & in;
        pst = base + (uint32_t)lane + 1u;
        plen = rest;
      }
      cand = in & lanes_where(u <= thr);
    }
    if (!cand) continue;
    if (nseen > kWaveSeen - 128) {   // keep the table sparse: only N's ranks still matter
      clear_seen(w.seen, lane);
      const bool real = lane < nreal;
      const int32_t mine = real ? w.r_of(N) : kEmpty;
      wave_lds_sync();
      mark_seen(w.seen, mine, lanes_where(real));
      nseen = nreal;
    }
    uint64_t fresh = mark_seen(w.seen, r, cand);
    if (!fresh) continue;
    const int nc = __popcll(fresh);
    nseen += nc;
    if (nslot + nc > kWaveSlots) {   // renumber the slots that N still uses
      const bool real = lane < nreal;
      double md = 0;
      int32_t mr = 0;
      if (real) {
        md = w.d_of(N);
        mr = w.r_of(N);
      }
      wave_lds_sync();
      if (real) {
        w.d[lane] = md;
        w.r[lane] = mr;
        N = (N & ~(kTieBits & ~1u)) | (uint32_t)(lane << 1);
      }
      nslot = nreal;
    }
    const int below = lanes_below(fresh);
    const uint32_t key = (u & ~kTieBits) | (uint32_t)((nslot + below) << 1);
    if (in_mask(fresh)) {
      w.d_of(key) = d;
      w.r_of(key) = r;
    }
    nslot += nc;
    wave_lds_sync();
    // ---- insert
    uint32_t lost = kPadKey;   // the keys that fall out of N, in any lane
    if (nc <= kWaveInsert) {
      // one by one: every position keeps the middle of its key, the one before and the new.
      // Once the last lane is full, within these keys or before, each pushes one out (an empty
      // lane's key is above every threshold)
      int left = nc;
      do {
        const uint32_t nk = readlane_u32(key, pop_lane(fresh));
        --left;
        if (nreal + nc > 64) lost = writelane_u32(max(readlane_u32(N, 63), nk), left, lost);
        N = median(wave_shr1(N), nk, N);
      } while (fresh);
    } else {
      // at once: sort the new keys, reversed against N the smaller of each pair are the 64
      // smallest of both, bitonic
      uint32_t x;
      if (nc <= 16) {
        const int to = in_mask(fresh) ? 48 + below : 0;
        x = (uint32_t)__builtin_amdgcn_ds_permute(4 * to, (int32_t)key);
        x = in_mask((0xffffull >> (16 - nc)) << 48) ? x : kPadKey;
        x = (uint32_t)xor_lane<15>((int32_t)sort_rows(x, lane));
      } else {
        x = in_mask(fresh) ? key : kPadKey;
        x = merge_rows(sort_rows(x, lane), lane);
        x = lane_value(x, 63 - lane);
      }
      lost = max(N, x);
      N = merge_bitonic(min(N, x), lane);
    }
    nreal = min(64, nreal + nc);
    thr = min(readlane_u32(N, q.k - 1) | kTieBits, kMaxKey);
    if (__builtin_expect(nreal == 64 && lanes_where(lost <= thr) != 0, 0)) {   // agrees with the k-th
      N = keep_nearest(w, N, lost, thr, lane);
      thr = min(readlane_u32(N, q.k - 1) | kTieBits, kMaxKey);
    }
  }
  // ---- the exact keys, and the order of those whose upper bits agree
  d = INFINITY;
  r = kEmpty;
  if (lane < nreal) {
    d = w.d_of(N);
    r = w.r_of(N);
  }
  const uint64_t tie = lanes_where((N ^ wave_shr1(N)) <= kTieBits) & lanes_where(lane < nreal) &
                       lanes_where(lane <= q.k) & ~1ull;
  if (tie) order_lanes(d, r, lane);
  write_row(a, q, d, r, lane);
  return true;
}

// The queries begin .. begin + cnt - 1 (sorted positions) of request a on one wavefront, cnt
// <= 64 / DW, DW lanes each, taken through Alg. 1.
template <int DW, int R>
struct Descent {
  float qx = 0.f, qy = 0.f, qz = 0.f;
  int32_t qi = 0;        // caller index
  int32_t k = 0, m = 0;  // neighbours to walk for (0: nothing left to do); prefix
  int32_t nt = 0;        // transition sites; the last R are in the row's ring

  __device__ __forceinline__ void run(const QueryArgs &a, uint32_t (&ring)[64 / DW][R],
                                      int64_t begin, int cnt) {
    const int lane = threadIdx.x & 63;
    const int l = lane & (DW - 1), g = lane / DW;
    if (g < cnt) {
      const int64_t s = begin + g;
      if (a.qs) {
        const float4 v = a.qs[s];
        qx = v.x;
        qy = v.y;
        qz = v.z;
        qi = __float_as_int(v.w);
      } else {
        qi = (int32_t)s;
        qx = a.q[3 * s];
        qy = a.q[3 * s + 1];
        qz = a.q[3 * s + 2];
      }
      k = a.kq ? a.kq[qi] : a.k;
      // pending deletions: walk for more neighbours than the row keeps
      if (a.kq && a.dead) k = min(k + kLazyMargin, R);
      const int64_t mm = a.mq ? (int64_t)a.mq[qi] : (int64_t)a.m;
      m = (int32_t)(mm < a.n ? mm : a.n);
      if (k < 1 || k > R || m < 1) k = 0;
    }
    // pos is the lane's entry of the row's chunk, rem the entries left in the row's list (0:
    // the descent has ended)
    const double x = qx, y = qy, z = qz;
    double dcur = 0;
    int32_t cur = a.head;
    uint32_t pos = (uint32_t)l, rem = 0;
    if (k > 0 && a.head < m) {
      dcur = sq_dist(x, y, z, make_float4(a.hx, a.hy, a.hz, 0.f));
      if (l == 0) ring[g][0] = kHeadRecord;
      nt = 1;
      const uint64_t dsc = a.lst[a.head];
      pos = (uint32_t)dsc + (uint32_t)l;
      rem = (uint32_t)(dsc >> 32);
    }
    const uint32_t mine = 1u << l;
    if (lanes_where(rem != 0)) do {
      // every lane loads, without a branch: a chunk reaches at most DW - 1 <= 15 records past
      // the end of its list, which the arena's padding covers
      const float4 c = a.ent[pos];
      const int32_t r = __float_as_int(c.w);
      const bool in = (uint32_t)l < rem && r < m;
      const double dv = sq_dist(x, y, z, c);
      // per row: the closer entries (bits 0 .. DW - 1), and bit DW if the list or the prefix ends
      const uint32_t hit = row_or<DW>(in ? (dv < dcur ? mine : 0u) : 1u << DW);
      const bool more = hit == 0 && rem > (uint32_t)DW;
      // a row that has ended stays where it is
      rem = more ? rem - DW : 0u;
      pos += more ? (uint32_t)DW : 0u;
      const uint32_t j = (uint32_t)__builtin_ctz(hit | 1u << DW);
      if (j < (uint32_t)DW) {
        // the first strictly closer entry is the next transition site
        const int src = (lane & ~(DW - 1)) + (int)j;
        dcur = __shfl(dv, src);
        cur = (int32_t)lane_value((uint32_t)r, src);
        if (l == 0) ring[g][(uint32_t)nt & (R - 1u)] = pos + j;
        ++nt;
        const uint64_t dsc = a.lst[(uint32_t)cur];
        pos = (uint32_t)dsc + (uint32_t)l;
        rem = (uint32_t)(dsc >> 32);
      }
    } while (lanes_where(rem != 0));
    // k == 1: the end of the descent is the answer
    if (k == 1 && nt > 0 && !a.dead) {
      if (l == 0) {
        const int64_t row = a.row_off ? a.row_off[qi] : (int64_t)qi;
        a.out_idx[row] = cur;
        a.out_dist[row] = (float)sqrt(dcur);
      }
      k = 0;
    }
    wave_lds_sync();   // the ring is read by other lanes
  }
  // query t of the wavefront, in uniform registers
  __device__ __forceinline__ WaveQuery query(int t) const {
    const int src = t * DW;
    WaveQuery q;
    q.qx = readlane_f32(qx, src);
    q.qy = readlane_f32(qy, src);
    q.qz = readlane_f32(qz, src);
    q.qi = __builtin_amdgcn_readlane(qi, src);
    q.k = __builtin_amdgcn_readlane(k, src);
    q.m = __builtin_amdgcn_readlane(m, src);
    q.nt = __builtin_amdgcn_readlane(nt, src);
    return q;
  }
};

// Queries begin .. begin + cnt - 1 of request a on one wavefront.  begin and cnt are uniform;
// every lane of the wavefront calls.
template <int DW, int R>
__device__ __forceinline__ void wave_walk(const QueryArgs &a, WaveLds<DW, R> &w, int64_t begin,
                                          int cnt) {
  const int lane = threadIdx.x & 63;
  Descent<DW, R> q;
  q.run(a, w.ring, begin, cnt);
  uint64_t todo = lanes_where((lane & (DW - 1)) == 0) & lanes_where(q.k > 0), again = 0;
  while (todo) {
    const int t = pop_lane(todo) / DW;
    wave_lds_sync();   // the slots of the query before
    if (!expand(a, w, q.query(t), t, lane)) again |= 1ull << t;
  }
  while (again) answer_exact(a, q.query(pop_lane(again)), lane);
}

// Plain launch: per_wave consecutive sorted queries per wavefront (1 .. 64 / DW).
template <int DW, int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8)))
void knn_wave_kernel(QueryArgs a, int32_t per_wave) {
  __shared__ WaveLds<DW, R> lds[4];
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t begin = ((int64_t)xcd_tile(blockIdx.x, gridDim.x) * 4 + wid) * per_wave;
  if (begin >= a.nq) return;   // whole wavefronts leave
  const int cnt = (int)(a.nq - begin < per_wave ? a.nq - begin : per_wave);
  wave_walk<DW, R>(a, lds[wid], begin, cnt);
}

}  // namespace mknn
