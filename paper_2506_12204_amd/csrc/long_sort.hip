// The long queues of a batch (more than kSegLargeCap requests each), all
// together: the two-pass LSD radix sort of tile_sort.hip over tiles of 8192
// requests, a tile never spanning two queues and its digit offsets taken over
// its own queue's tiles. Every queue is scheduled as the drained min-heap of
// Algorithm 1 (ids ascending by (priority, length, id)) with the waits of
// Eq. 1 and exact class totals.
//
// The planner of the batched call (b_plan) has filed the queues and b_medium
// laid them out (long_layout); the number of tiles is known on the device
// only, so the grids are the workgroups that fit and each takes a run of
// consecutive tiles, loading the next tile's input while it works on one.
//   l_count   descriptors, ranges and first-digit counts of every tile
//   l_scan    the counts' prefix over each queue's tiles; one more workgroup
//             makes the plan from the ranges
//   l_first   first scatter
//   l_mid_count, l_scan, l_mid_scatter   per middle pass of wide keys (they
//             return at once for two-digit keys)
//   l_histF   final-digit counts and length sums of every tile
//   l_scan    their prefixes
//   l_final   order, waits, class totals
// Small batches leave out the l_scan launches after the first (kFoldTiles).
// Launches instead of one cooperative kernel with grid syncs: 16 queues of
// 2^20 requests took 760 us there (its launch alone 24 us), 317 us here; 1000 of
// 20,000 923 us, 462 us here.
#include <algorithm>
#include <type_traits>

#include "tile_common.h"

namespace semsched {

namespace {

constexpr int LR = kLongTile / TT;  // rounds per thread
static_assert(LR * TT == kLongTile, "a tile is whole rounds of the workgroup");
constexpr int kFirstBits = 10;
// Room for at most kFoldTiles tiles, and kFoldRows for each queue if all were
// long: the middle and final passes sum their queue's count rows themselves
// instead of reading l_scan's prefixes, which saves three of the twelve
// launches (each about 4 us, also when it returns at once). 4 queues of 20,665:
// 77 us with l_scan, 63 so; 70 of 20,000: 88, 73; one of 2^19: 83, 74; two: 91,
// 83 (wide keys). From 128 rows on the sums cost what the launches did: one
// queue of 2^20 90, 87, with wide keys 102, 106.
constexpr uint32_t kFoldTiles = 256, kFoldRows = 96;

// Runs f with the element form of the plan's keys.
template <typename F>
__device__ __forceinline__ void with_codec(const Plan* pl, F&& f) {
  if (pl->W == 32) {
    KeyCodec32 kc;
    kc.init(kFirstBits, pl);
    f(kc);
  } else if (pl->packed) {
    KeyCodec64 kc;
    kc.init(kFirstBits, pl);
    f(kc);
  } else {
    KeyCodecGather kc;
    kc.init(kFirstBits, pl);
    f(kc);
  }
}
template <typename Codec>
__device__ __forceinline__ void set_queue(Codec&, const BArgs&, const LongTileDesc&) {}
__device__ __forceinline__ void set_queue(KeyCodecGather& kc, const BArgs& a,
                                          const LongTileDesc& x) {
  kc.lengths = a.length + (x.first - x.lo);
}

// Tiles of the batch's long queues, or 0 when there is nothing to do here: no
// such queues, or an error ends the call (the planner raises one for long
// queues that do not fit the workspace and then leaves their places
// unwritten). Only l_count asks: no kernel that runs beside it writes the
// error bits, so all its waves see the same. The passes after it take its
// answer (BCtl::long_run), not the bits: l_scan's first pass raises one itself
// while it runs, and waves of a workgroup that read the word before and after
// would part ahead of a barrier. From then on Plan::ok says whether to go on.
__device__ __forceinline__ uint32_t long_tiles(const BArgs& a) {
  if (a.ctl->count[kListLong] == 0 || a.ctl->long_elems > a.long_cap || load_agent(a.flags) != 0)
    return 0;
  return a.ctl->long_tiles;
}

// This workgroup's run of tiles [lo, hi).
__device__ __forceinline__ void tile_run(uint32_t tiles, uint32_t& lo, uint32_t& hi) {
  const uint32_t per = (tiles + gridDim.x - 1) / gridDim.x;
  lo = min(tiles, blockIdx.x * per);
  hi = min(tiles, lo + per);
}

__global__ __launch_bounds__(TT) void l_count(BArgs a) {
  __shared__ uint32_t s_cnt[kMaxBins * kCountCopies];
  __shared__ uint32_t s_red[4][TWV];
  const uint32_t tiles = long_tiles(a);
  uint32_t lo, hi;
  tile_run(tiles, lo, hi);
  const int t = threadIdx.x;
  if (blockIdx.x == 0 && t == 0) a.ctl->long_run = tiles;
  const uint32_t copy = (uint32_t)lane_id() & (kCountCopies - 1);
  if (lo >= hi) return;  // (uniform)
  // the queue of the first tile by a search, of the others by walking on
  uint32_t k = 0;
  for (uint32_t end = a.ctl->count[kListLong]; end - k > 1;) {
    const uint32_t mid = (k + end) / 2;
    if (a.tstart[mid] <= lo) k = mid;
    else end = mid;
  }
  for (uint32_t tt = lo; tt < hi; ++tt) {
    if (a.tstart[k + 1] <= tt) ++k;  // (every long queue has a tile)
    LongTileDesc x;
    x.item0 = a.tstart[k];
    x.rows = a.tstart[k + 1] - x.item0;
    x.s = a.lists[2 * kSubLists * a.seg_cap + k];
    const int64_t base = a.offsets[x.s];
    x.lo = (tt - x.item0) * (uint32_t)kLongTile;
    x.cnt = (int32_t)min((int64_t)kLongTile, a.offsets[x.s + 1] - base - (int64_t)x.lo);
    x.first = base + x.lo;
    x.at = a.lbase[k] + x.lo;
    if (t == 0) a.tdesc[tt] = x;
    if (x.lo == 0) {  // (uniform) the queue's first tile: its scan items, its totals
      const uint32_t parts = x.rows <= kLongRowsFew ? 1u : (uint32_t)kLongScanParts;
      if ((uint32_t)t < parts) a.imap[a.istart[k] + t] = k * kLongScanParts + t;
      const int64_t C2 = 2 * (1 + (int64_t)a.num_classes);
      for (int64_t i = t; i < C2; i += TT) a.totals[x.s * C2 + i] = 0;
    }
    uint32_t pv[LR];
    int32_t lv[LR];
#pragma unroll
    for (int r = 0; r < LR; ++r) {
      const int i = min(r * TT + t, x.cnt - 1);
      pv[r] = a.priority[x.first + i];
      lv[r] = a.length[x.first + i];
    }
    clear_counts(s_cnt);
    block_sync();
    TileRanges rg;
#pragma unroll
    for (int r = 0; r < LR; ++r) {
      const bool in = r * TT + t < x.cnt;
      rg.add(in, pv[r], lv[r], a.num_classes);
      atomicAdd(&s_cnt[((uint32_t)lv[r] & ((1u << kFirstBits) - 1)) * kCountCopies + copy],
                in ? 1u : 0u);
    }
    rg.write(s_red, a.lranges + 4 * (size_t)tt);  // (holds a barrier)
    write_counts(s_cnt, a.lcount + (size_t)tt * kMaxBins);
    block_sync();  // the counts are read before they are cleared
  }
}

// The plan of all long queues together, from the tiles' ranges (one workgroup).
__device__ void long_plan(const BArgs& a, uint32_t tiles, uint32_t (*red)[TWV]) {
  const int t = threadIdx.x;
  uint4 v = make_uint4(0xffu, 0u, 0xffffffffu, 0u);
  uint32_t bad = 0, longest = 0;
  for (uint32_t i = t; i < tiles; i += TT) {
    const uint4 x = reinterpret_cast<const uint4*>(a.lranges)[i];
    v.x = min(v.x, x.x);
    v.y = max(v.y, x.y & 0xffu);
    bad |= x.y & 0x80000000u;
    v.z = min(v.z, x.z);
    v.w = max(v.w, x.w);
    longest = max(longest, a.tdesc[i].lo + (uint32_t)a.tdesc[i].cnt);
  }
  v.y |= bad;
  stage_ranges(v, red);
  longest = wave_max_u32(longest);
  __shared__ uint32_t s_longest[TWV];
  if (lane_id() == 0) s_longest[wave_no()] = longest;
  block_sync();
  if (t != 0) return;
  const uint4 all = collect_ranges(red, TWV);
  for (int i = 0; i < TWV; ++i) longest = max(longest, s_longest[i]);
  Plan p = {};
  if (all.y >> 31) {
    atomicOr(a.flags, kFlagRange);
  } else {
    make_plan(kFirstBits, longest - 1, false, false, all.x, all.y, all.z, all.w, &p);
    p.ok = 1;
    // a wave's 512 waits, each below longest * 2^bits, in 64 bits
    p.sum64 = bit_width32(longest) + bit_width32(all.w) + 9 <= 64 ? 1u : 0u;
  }
  *a.plan = p;
}

// Prefixes of the count rows over each queue's tiles, per digit: pass s's
// counts, or (FINAL) the final digit's counts and length sums. A queue of at
// most kLongRowsFew tiles is one item, a wave per 64 digits running down the
// rows; a longer one is an item per PD digits (64 or 128 bytes of a row), its
// rows split over the workgroup's lanes in NC runs, each read twice: once for
// the runs' sums, once to write the prefixes.
template <bool FINAL>
__global__ __launch_bounds__(TT) void l_scan(BArgs a, int s) {
  constexpr int PD = FINAL ? 16 : 32;
  constexpr int RL = kWave / PD;   // runs of a wave
  static_assert(kMaxBins / PD <= kLongScanParts, "an item per part");
  __shared__ uint32_t s_c[TWV][PD];
  __shared__ uint64_t s_w[FINAL ? TWV : 1][PD];
  __shared__ uint32_t s_red[4][TWV];
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0) return;
  const bool planner = !FINAL && s == 0;  // workgroup 0 makes the plan instead
  if (planner && blockIdx.x == 0) {
    long_plan(a, tiles, s_red);
    return;
  }
  if (FINAL && !a.plan->ok) return;
  if (!FINAL && s > 0 && (!a.plan->ok || s >= (int)a.plan->nscatter - 1)) return;
  const uint32_t items = a.ctl->long_items;
  const uint32_t workers = gridDim.x - (planner ? 1u : 0u);
  const int w = wave_no();
  const int lane = lane_id();
  const uint32_t nb = FINAL ? a.plan->nbins[a.plan->nscatter - 1] : (uint32_t)kMaxBins;
  constexpr int U = FINAL ? 8 : 16;  // rows in flight
  // Adds rows [r0, r1) of digit d, and with WRITE stores every row's prefix.
  auto run_rows = [&](auto write, uint32_t r0, uint32_t r1, uint32_t d, uint32_t& c,
                      uint64_t& l) {
    for (uint32_t r = r0; r < r1; r += U) {
      typename std::conditional<FINAL, uint64_t, uint32_t>::type x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const size_t at = (size_t)min(r + u, r1 - 1) * kMaxBins + d;
        if constexpr (FINAL) x[u] = a.lfinal[at];
        else x[u] = a.lcount[at];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (r + u < r1) {
          const size_t at = (size_t)(r + u) * kMaxBins + d;
          if constexpr (decltype(write)::value) {
            a.hist[at] = c;
            if constexpr (FINAL) a.lwait[at] = l;
          }
          if constexpr (FINAL) {
            c += (uint32_t)(x[u] >> kSumBits);
            l += x[u] & kSumMask;
          } else {
            c += x[u];
          }
        }
      }
    }
  };
  for (uint32_t it = blockIdx.x - (planner ? 1u : 0u); it < items; it += workers) {
    const uint32_t im = a.imap[it];
    const uint32_t k = im / kLongScanParts, part = im % kLongScanParts;
    const uint32_t row0 = a.tstart[k], rows = a.tstart[k + 1] - row0;
    if (rows <= kLongRowsFew) {  // (uniform)
      const uint32_t d = (uint32_t)(w * kWave + lane);
      uint32_t c = 0;
      uint64_t l = 0;
      if (d < nb) run_rows(std::true_type{}, row0, row0 + rows, d, c, l);
      continue;
    }
    if (part * PD >= nb) continue;  // (uniform)
    const uint32_t dl = lane % PD, d = part * PD + dl;
    const uint32_t per = (rows + TWV * RL - 1) / (TWV * RL);
    const uint32_t r0 = row0 + min(rows, (uint32_t)(w * RL + lane / PD) * per);
    const uint32_t r1 = min(row0 + rows, r0 + per);
    uint32_t c = 0;
    uint64_t l = 0;
    if (d < nb) run_rows(std::false_type{}, r0, r1, d, c, l);
    // exclusive prefix over the runs: within the wave, then over the waves
    uint32_t ic = c;
    uint64_t il = l;
#pragma unroll
    for (int off = PD; off < kWave; off <<= 1) {
      const uint32_t oc = __shfl_up(ic, off, kWave);
      const uint64_t ol = FINAL ? __shfl_up((unsigned long long)il, off, kWave) : 0ull;
      if (lane >= off) {
        ic += oc;
        il += ol;
      }
    }
    if (lane >= kWave - PD) {
      s_c[w][dl] = ic;
      if constexpr (FINAL) s_w[w][dl] = il;
    }
    block_sync();
    c = ic - c;
    l = il - l;
    for (int v = 0; v < w; ++v) {  // (w is uniform)
      c += s_c[v][dl];
      if constexpr (FINAL) l += s_w[v][dl];
    }
    block_sync();  // the sums are read before the next item writes them
    if (d < nb) run_rows(std::true_type{}, r0, r1, d, c, l);
  }
}

// The digit's start in the queue of tile x (every thread its digit), from the
// prefix and count of the queue's last tile. Holds barriers.
__device__ __forceinline__ uint32_t queue_digit_start(const BArgs& a, const LongTileDesc& x,
                                                      uint32_t* scan32) {
  const size_t last = (size_t)(x.item0 + x.rows - 1) * kMaxBins + threadIdx.x;
  uint32_t sum;
  return block_excl_scan_u32<TT>(a.hist[last] + a.lcount[last], scan32, sum);
}

// Small batches: what l_scan would have left for tile `tt`, summed here from
// the queue's own count rows (every thread its digit): the counts and length
// sums of the tiles before it, and of all of them.
struct Folded {
  uint32_t before, all;
  uint64_t wbefore, wall;
};
template <bool FINAL>
__device__ __forceinline__ Folded fold_rows(const BArgs& a, const LongTileDesc& x, uint32_t tt) {
  constexpr uint32_t U = FINAL ? 8 : 16;  // rows in flight
  const uint32_t r1 = x.item0 + x.rows;
  Folded f = {0, 0, 0, 0};
  for (uint32_t r = x.item0; r < r1; r += U) {
    typename std::conditional<FINAL, uint64_t, uint32_t>::type v[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const size_t at = (size_t)min(r + u, r1 - 1) * kMaxBins + threadIdx.x;
      if constexpr (FINAL) v[u] = a.lfinal[at];
      else v[u] = a.lcount[at];
    }
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      if (r + u >= r1) continue;  // (uniform)
      const uint32_t c = FINAL ? (uint32_t)(v[u] >> (FINAL ? kSumBits : 0)) : (uint32_t)v[u];
      const uint64_t l = FINAL ? (uint64_t)v[u] & kSumMask : 0ull;
      f.all += c;
      f.wall += l;
      if (r + u < tt) {
        f.before += c;
        f.wbefore += l;
      }
    }
  }
  return f;
}

struct LongFirstLds {
  uint64_t stage[kLongTile];
  uint16_t cnt[TWV][kMaxBins];
  uint32_t base[kMaxBins];
  uint32_t scan32[TWV + 1];
};

// Scatter of this workgroup's tiles by a 10-bit digit: the first pass (FIRST:
// from the requests, by the low length bits) or a middle pass. FOLD: no l_scan
// ran after the counts.
template <bool FIRST, bool FOLD, typename Codec>
__device__ void long_scatter(const BArgs& a, Codec kc, int s, uint32_t lo, uint32_t hi,
                             LongFirstLds& sh) {
  const int t = threadIdx.x;
  const int w = wave_no();
  const int j0 = w * kWave * LR + lane_id();
  constexpr uint32_t M0 = kMaxBins - 1;
  const uint32_t dshift = a.plan->shift[s];
  const uint64_t* in = FIRST ? nullptr : a.keys[(s - 1) & 1];
  uint32_t pv[LR], lv[LR];  // the requests, or the elements' halves
  auto load = [&](const LongTileDesc& x) {
#pragma unroll
    for (int r = 0; r < LR; ++r) {
      const int i = min(j0 + r * kWave, x.cnt - 1);
      if constexpr (FIRST) {
        pv[r] = a.priority[x.first + i];
        lv[r] = (uint32_t)a.length[x.first + i];
      } else {
        const uint64_t v = in[x.at + i];
        pv[r] = (uint32_t)(v >> 32);
        lv[r] = (uint32_t)v;
      }
    }
  };
  auto digit = [&](uint64_t e) {
    return FIRST ? kc.lo_of(e) : (kc.u2_of(e) >> dshift) & M0;
  };
  if (lo >= hi) return;  // (uniform)
  LongTileDesc x = a.tdesc[lo];
  load(x);
  uint32_t off = FOLD ? 0u : a.hist[(size_t)lo * kMaxBins + t];
  uint32_t queue0 = 0;  // start of the thread's digit in the queue
  int64_t in_queue = -1;
  for (uint32_t tt = lo; tt < hi; ++tt) {
    set_queue(kc, a, x);
    if (x.s != in_queue) {  // (uniform) another queue: its digit totals
      in_queue = x.s;
      if constexpr (FOLD) {
        const Folded f = fold_rows<false>(a, x, tt);
        uint32_t sum;
        off = f.before;
        queue0 = block_excl_scan_u32<TT>(f.all, sh.scan32, sum);
      } else {
        queue0 = queue_digit_start(a, x, sh.scan32);
      }
    }
    uint64_t e[LR];
    uint32_t dg[LR], rk[LR];
    clear_row(sh.cnt[w]);
#pragma unroll
    for (int r = 0; r < LR; ++r) {
      const int i = j0 + r * kWave;
      e[r] = FIRST ? kc.make(pv[r], lv[r], x.lo + (uint32_t)i)
                   : ((uint64_t)pv[r] << 32) | lv[r];
      // items past the end take the last digit
      dg[r] = i >= x.cnt ? M0 : FIRST ? lv[r] & M0 : digit(e[r]);
      rk[r] = rank_round_c<kFirstBits>(dg[r], sh.cnt[w]);
    }
    const LongTileDesc cur = x;
    const uint32_t mine = queue0 + off;
    if (tt + 1 < hi) {  // the next tile's input loads while this one is written
      x = a.tdesc[tt + 1];
      load(x);
      if constexpr (FOLD) off += a.lcount[(size_t)tt * kMaxBins + t];
      else off = a.hist[(size_t)(tt + 1) * kMaxBins + t];
    }
    block_sync();
    const uint32_t ex = tile_positions(sh.cnt, sh.scan32);
    sh.base[t] = mine - ex;
    block_sync();
#pragma unroll
    for (int r = 0; r < LR; ++r) sh.stage[rk[r] + sh.cnt[w][dg[r]]] = e[r];
    block_sync();
    uint64_t* out = a.keys[s & 1] + (cur.at - cur.lo);  // the queue's elements
    const uint64_t room = a.long_cap - (cur.at - cur.lo);
#pragma unroll
    for (int r = 0; r < LR; ++r) {
      const int j = j0 + r * kWave;
      if (j < cur.cnt) {
        const uint64_t v = sh.stage[j];
        const uint32_t pos = sh.base[digit(v)] + (uint32_t)j;
        if (pos < room) out[pos] = v;  // (always, for consistent counts)
      }
    }
  }
}

__global__ __launch_bounds__(TT) void l_first(BArgs a) {
  __shared__ LongFirstLds sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok) return;
  uint32_t lo, hi;
  tile_run(tiles, lo, hi);
  with_codec(a.plan, [&](auto kc) { long_scatter<true, false>(a, kc, 0, lo, hi, sh); });
}

template <bool FOLD>
__global__ __launch_bounds__(TT) void l_mid_scatter(BArgs a, int s) {
  __shared__ LongFirstLds sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok || s >= (int)a.plan->nscatter - 1) return;
  uint32_t lo, hi;
  tile_run(tiles, lo, hi);
  with_codec(a.plan, [&](auto kc) { long_scatter<false, FOLD>(a, kc, s, lo, hi, sh); });
}

// Digit counts of this workgroup's tiles in middle pass s.
__global__ __launch_bounds__(TT) void l_mid_count(BArgs a, int s) {
  __shared__ uint32_t s_cnt[kMaxBins * kCountCopies];
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok || s >= (int)a.plan->nscatter - 1) return;
  uint32_t lo, hi;
  tile_run(tiles, lo, hi);
  const int t = threadIdx.x;
  const uint32_t copy = (uint32_t)lane_id() & (kCountCopies - 1);
  const uint32_t dshift = a.plan->shift[s];
  with_codec(a.plan, [&](auto kc) {
    for (uint32_t tt = lo; tt < hi; ++tt) {
      const LongTileDesc x = a.tdesc[tt];
      uint64_t e[LR];
#pragma unroll
      for (int r = 0; r < LR; ++r) e[r] = a.keys[(s - 1) & 1][x.at + min(r * TT + t, x.cnt - 1)];
      clear_counts(s_cnt);
      block_sync();
#pragma unroll
      for (int r = 0; r < LR; ++r)
        atomicAdd(&s_cnt[((kc.u2_of(e[r]) >> dshift) & (kMaxBins - 1)) * kCountCopies + copy],
                  r * TT + t < x.cnt ? 1u : 0u);
      block_sync();
      write_counts(s_cnt, a.lcount + (size_t)tt * kMaxBins);
      block_sync();  // the counts are read before they are cleared
    }
  });
}

__global__ __launch_bounds__(TT) void l_histF(BArgs a) {
  __shared__ uint64_t s_bin[kFinalSlots];
  const uint32_t tiles = a.ctl->long_run;
  const Plan* pl = a.plan;
  if (tiles == 0 || !pl->ok) return;
  uint32_t lo, hi;
  tile_run(tiles, lo, hi);
  const int s = (int)pl->nscatter - 1;
  const TileDigit dig = {pl->shift[s], pl->nbits[s]};
  with_codec(pl, [&](auto kc) {
    for (uint32_t tt = lo; tt < hi; ++tt) {
      const LongTileDesc x = a.tdesc[tt];
      set_queue(kc, a, x);
      uint64_t e[LR];
#pragma unroll
      for (int r = 0; r < LR; ++r)
        e[r] = a.keys[(s - 1) & 1][x.at + min(r * TT + (int)threadIdx.x, x.cnt - 1)];
      count_final(kc, dig, (int)pl->nbins[s], e, x.cnt, s_bin, a.lfinal + (size_t)tt * kMaxBins);
      block_sync();  // the bins are read before they are cleared
    }
  });
}

struct LongFinalLds : PlaceLds {
  struct {
    uint64_t stage[kLongTile];
  } u;
};

// Adds v to a 128-bit total. The high word is left alone when nothing goes
// there (nearly always): the workgroups' additions to one line queue.
__device__ __forceinline__ void add_total(uint64_t* o, const U128& v) {
  if ((v.lo | v.hi) == 0) return;
  const uint64_t old = atomicAdd(reinterpret_cast<unsigned long long*>(o), (unsigned long long)v.lo);
  const uint64_t hi = v.hi + (old + v.lo < old ? 1u : 0u);
  if (hi) atomicAdd(reinterpret_cast<unsigned long long*>(o + 1), (unsigned long long)hi);
}

// Order, waits and class totals of this workgroup's tiles. The class sums stay
// in LDS over consecutive tiles of one queue, then go to its totals.
template <bool WIDE_SUMS, bool FOLD, typename Codec>
__device__ void long_final(const BArgs& a, Codec kc, uint32_t lo, uint32_t hi,
                           LongFinalLds& sh) {
  const int t = threadIdx.x;
  const int w = wave_no();
  const int j0 = w * kWave * LR + lane_id();
  const Plan* pl = a.plan;
  const int s = (int)pl->nscatter - 1;
  const TileDigit dig = {pl->shift[s], pl->nbits[s]};
  const uint32_t nb = pl->nbins[s], P = pl->P;
  const bool small = pl->small != 0;
  const uint64_t* in = a.keys[(s - 1) & 1];
  uint64_t e[LR];
  auto load = [&](const LongTileDesc& x, uint64_t (&v)[LR]) {
#pragma unroll
    for (int r = 0; r < LR; ++r) v[r] = in[x.at + min(j0 + r * kWave, x.cnt - 1)];
  };
  auto flush = [&](int64_t q) {  // the class sums to queue q's totals
    uint64_t* tot = a.totals + 2 * q * (1 + a.num_classes);
    if (t == 0) {  // (one addition per workgroup to the queue's total)
      U128 sum = {0, 0};
      for (uint32_t c = 0; c < P; ++c) add128(sum, U128{sh.clo[c], sh.chi[c]});
      add_total(tot, sum);
    }
    block_sync();
    for (uint32_t c = t; c < P; c += TT) {
      add_total(tot + 2 * (1 + pl->pmin + c), U128{sh.clo[c], sh.chi[c]});
      sh.clo[c] = 0;
      sh.chi[c] = 0;
    }
  };
  if (lo >= hi) return;  // (uniform)
  const bool own = (uint32_t)t < nb;  // (rows hold nb digits)
  LongTileDesc x = a.tdesc[lo];
  load(x, e);
  uint32_t off = own && !FOLD ? a.hist[(size_t)lo * kMaxBins + t] : 0u;
  uint64_t woff = own && !FOLD ? a.lwait[(size_t)lo * kMaxBins + t] : 0ull;
  for (uint32_t c = t; c < P; c += TT) {
    sh.clo[c] = 0;
    sh.chi[c] = 0;
  }
  uint32_t queue0 = 0;
  uint64_t wait0 = 0, limit = 0;  // (limit: the queue's size)
  int64_t in_queue = -1;
  for (uint32_t tt = lo; tt < hi; ++tt) {
    block_sync();  // the last tile's class sums are in
    if (x.s != in_queue) {  // (uniform) another queue
      if (in_queue >= 0) flush(in_queue);
      in_queue = x.s;
      limit = (uint64_t)(a.offsets[x.s + 1] - a.offsets[x.s]);
      Folded f = {0, 0, 0, 0};
      if constexpr (FOLD) {
        if (own) f = fold_rows<true>(a, x, tt);
        off = f.before;
        woff = f.wbefore;
      } else if (own) {
        const size_t last = (size_t)(x.item0 + x.rows - 1) * kMaxBins + t;
        const uint64_t v = a.lfinal[last];
        f.all = a.hist[last] + (uint32_t)(v >> kSumBits);
        f.wall = a.lwait[last] + (v & kSumMask);
      }
      uint32_t sum;
      uint64_t wsum;
      queue0 = block_excl_scan_u32<TT>(f.all, sh.scan32, sum);
      wait0 = block_excl_scan_u64<TT>(f.wall, sh.scan64, wsum);
    }
    const LongTileDesc cur = x;
    const uint32_t pos0 = queue0 + off;
    const uint64_t w0 = wait0 + woff;
    // the next tile's elements load while this one is placed
    auto next = [&] {
      if (tt + 1 < hi) {
        x = a.tdesc[tt + 1];
        load(x, e);
        if constexpr (FOLD) {
          const uint64_t v = own ? a.lfinal[(size_t)tt * kMaxBins + t] : 0ull;
          off += (uint32_t)(v >> kSumBits);
          woff += v & kSumMask;
        } else {
          off = own ? a.hist[(size_t)(tt + 1) * kMaxBins + t] : 0u;
          woff = own ? a.lwait[(size_t)(tt + 1) * kMaxBins + t] : 0ull;
        }
      }
    };
    const int64_t qfirst = cur.first - cur.lo;  // the queue's first request
    set_queue(kc, a, cur);
    place_tile<WIDE_SUMS, false>(kc, dig, small, e, cur.cnt, pos0, w0, a.order + qfirst,
                          a.wait + qfirst, limit, sh, next);
  }
  block_sync();
  flush(in_queue);
}

template <bool FOLD>
__global__ __launch_bounds__(TT) void l_final(BArgs a) {
  __shared__ LongFinalLds sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok) return;
  uint32_t lo, hi;
  tile_run(tiles, lo, hi);
  if (a.plan->W == 32 && a.plan->sum64) {
    KeyCodec32 kc;
    kc.init(kFirstBits, a.plan);
    long_final<false, FOLD>(a, kc, lo, hi, sh);
  } else {
    with_codec(a.plan, [&](auto kc) { long_final<true, FOLD>(a, kc, lo, hi, sh); });
  }
}

// The middle passes, final counts and final pass; FOLD: without l_scan launches.
template <bool FOLD, typename Grid>
void launch_passes(const BArgs& a, unsigned scan, Grid&& grid, hipStream_t st) {
  static const int r_count = resident_groups(l_count), r_histF = resident_groups(l_histF),
                   r_mid = resident_groups(l_mid_scatter<FOLD>),
                   r_final = resident_groups(l_final<FOLD>);
  for (int s = 1; s <= max_mid_passes(kFirstBits); ++s) {
    hipLaunchKernelGGL(l_mid_count, grid(r_count), dim3(TT), 0, st, a, s);
    if (!FOLD) hipLaunchKernelGGL(l_scan<false>, dim3(scan), dim3(TT), 0, st, a, s);
    hipLaunchKernelGGL(l_mid_scatter<FOLD>, grid(r_mid), dim3(TT), 0, st, a, s);
  }
  hipLaunchKernelGGL(l_histF, grid(r_histF), dim3(TT), 0, st, a);
  if (!FOLD) hipLaunchKernelGGL(l_scan<true>, dim3(scan), dim3(TT), 0, st, a, 0);
  hipLaunchKernelGGL(l_final<FOLD>, grid(r_final), dim3(TT), 0, st, a);
}

}  // namespace

hipError_t launch_long_queues(const BArgs& a, hipStream_t st) {
  static const int r_count = resident_groups(l_count), r_first = resident_groups(l_first);
  auto grid = [&](int resident) {
    return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(resident, a.max_tiles)));
  };
  const int64_t queues =
      std::min<int64_t>(a.num_segments, (int64_t)(a.long_cap / (kSegLargeCap + 1)));
  const unsigned scan = (unsigned)std::min<uint64_t>(1024, long_items_max(a.long_cap, queues));
  hipLaunchKernelGGL(l_count, grid(r_count), dim3(TT), 0, st, a);
  hipLaunchKernelGGL(l_scan<false>, dim3(scan + 1), dim3(TT), 0, st, a, 0);
  hipLaunchKernelGGL(l_first, grid(r_first), dim3(TT), 0, st, a);
  if (a.max_tiles <= kFoldTiles && a.max_tiles <= kFoldRows * (uint64_t)a.num_segments)
    launch_passes<true>(a, scan, grid, st);
  else
    launch_passes<false>(a, scan, grid, st);
  return hipGetLastError();
}

}  // namespace semsched
