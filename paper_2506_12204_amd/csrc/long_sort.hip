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
//   l_count   descriptors, ranges and first-digit counts of every tile; then the
//             counts' prefix over each queue's tiles, and the plan from the ranges
//   l_first   first scatter
//   l_mid_rows, l_mid_scatter   per middle pass of wide keys (they return at
//             once for two-digit keys): the digit counts and their prefixes,
//             the scatter
//   l_histF   final-digit counts and length sums of every tile
//   l_scanF   their prefixes
//   l_final   order, waits, class totals
// Small batches take all middle passes in one launch, l_mid, and do without the
// prefixes after the first (kFoldTiles).
//
// A batch that turns out to have no long queue, in a workspace with room for
// some, pays for these launches all the same, 3 to 4 us each on the host and 2
// to 3 on the device. Hence kernels of several phases (next_work): 512 queues
// of 256 with room for long ones take 35 us with five launches here, 49 with
// nine; 4096 of 1024 take 80 us with nine, 91 with twelve.
// Launches instead of one cooperative kernel with grid syncs: 16 queues of
// 2^20 requests took 764 us there (its launch alone 24 us), 319 us here; 1000 of
// 20,000 923 us, 435 us here.
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
// instead of reading prefixes that other launches leave. With such launches 4
// queues of 20,665 took 77 us, 63 so; 70 of 20,000: 88, 73; one of 2^19: 83, 74;
// two: 91, 83 (wide keys). From 128 rows on the sums cost what the launches did:
// one queue of 2^20 90, 87, with wide keys 102, 106.
constexpr uint32_t kFoldTiles = 256, kFoldRows = 96;

// Runs f with the element form of the plan's keys. SMALL: the batch's queues have
// at most kFoldTiles tiles, so that their ids (21 bits) always fit above a key.
template <bool SMALL = false, typename F>
__device__ __forceinline__ void with_codec(const Plan* pl, F&& f) {
  static_assert((uint64_t)kFoldTiles * kLongTile <= 1ull << (64 - 39), "39 bits of key at most");
  if (pl->W == 32) {
    KeyCodec32 kc;
    kc.init(kFirstBits, pl);
    f(kc);
  } else if (SMALL || pl->packed) {
    KeyCodec64 kc;
    kc.init(kFirstBits, pl);
    f(kc);
  } else if constexpr (!SMALL) {
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

// The run of tiles [lo, hi) of workgroup `me`.
__device__ __forceinline__ void tile_run(uint32_t tiles, uint32_t me, uint32_t& lo,
                                         uint32_t& hi) {
  const uint32_t per = (tiles + gridDim.x - 1) / gridDim.x;
  lo = min(tiles, me * per);
  hi = min(tiles, lo + per);
}

// A kernel of several phases, each of which needs all of the one before. Each
// is cut into gridDim.x shares; a workgroup takes one share of the first phase
// as it starts and has the same share of the later ones. It does not rely on
// all workgroups being resident: one that has waited for the end of the first
// phase while shares are left (some workgroup has not started) takes a further
// one, and a workgroup that starts and finds none left ends. So every share
// belongs to a workgroup that runs, waits only for such, and every wait ends.
// What a later phase reads is written by agent-scope stores, complete (vmcnt 0)
// before the share is counted as done, and read by agent-scope loads: no fence,
// which would write back or invalidate the L2 in every workgroup (10 to 15 us
// a phase).
constexpr uint32_t kMaxShares = 512;
struct WorkLds {
  uint32_t phase, me;   // the share to work on now
  uint32_t at, owned;   // its place among the workgroup's shares, their number
  uint32_t mine[kMaxShares];
};
// Counts the share just worked on and finds the next one to do (w.phase, w.me);
// false when none is left. Every thread of the workgroup calls it; `begin`: the
// first time. One branch takes all of thread 0's steps, with a barrier on
// either side: were a share counted at the end of the caller's loop body,
// nothing convergent would lie between that branch and this one, and the
// compiler threads them into each other, which sends the other lanes of
// thread 0's wave around the loop ahead of it.
__device__ __forceinline__ bool next_work(const BArgs& a, PhaseKernel kernel, uint32_t phases,
                                          bool begin, WorkLds& w) {
  wait_stores();
  block_sync();
  if (threadIdx.x == 0) {
    const uint32_t shares = gridDim.x;
    constexpr uint32_t kDone = kPhaseLines - 1;
    uint32_t* next = &phase_line(a.grab, kernel, 0)->next;
    uint32_t* done = &phase_line(a.grab, kernel, 0)->count;
    uint32_t phase = begin ? 0u : w.phase;
    uint32_t got = shares;  // a share taken now
    if (begin) {
      w.owned = 0;
      got = atomicAdd(next, 1u);
      if (got >= shares) phase = phases;
    } else {
      if (phase + 1 < phases) {  // the last of a quarter counts it, the last of those the phase
        const uint32_t k = w.me % kDone, due = (shares + kDone - 1 - k) / kDone;
        if (atomicAdd(&phase_line(a.grab, kernel, 1 + (int)k)->count, 1u) + 1 == (phase + 1) * due &&
            atomicAdd(&phase_line(a.grab, kernel, 1)->next, 1u) + 1 ==
                (phase + 1) * min(shares, (uint32_t)kDone))
          store_agent(done, phase + 1);
      }
      if (phase > 0 && w.at + 1 < w.owned) {
        w.at += 1;
      } else if (phase + 1 == phases) {
        phase = phases;
      } else {
        for (uint32_t polls = 1; load_agent(done) <= phase; ++polls) {
          if (phase == 0 && polls % a.claim_polls == 0 && load_agent(next) < shares) {
            got = atomicAdd(next, 1u);
            if (got < shares) break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
        if (got >= shares) {
          phase += 1;
          w.at = 0;
        }
      }
    }
    if (got < shares) {  // (at most `shares` in all, which the list holds)
      w.at = w.owned;
      w.mine[w.owned] = got;
      w.owned += 1;
    }
    w.phase = phase;
    w.me = phase < phases ? w.mine[w.at] : 0u;
  }
  block_sync();
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)w.phase) < phases;
}

struct CountLds {
  uint32_t cnt[kMaxBins * kCountCopies];
  uint32_t red[4][TWV];
};

// Descriptors, ranges and first-digit counts of the tiles [lo, hi).
__device__ void count_tiles(const BArgs& a, uint32_t lo, uint32_t hi, CountLds& sh) {
  uint32_t* s_cnt = sh.cnt;
  const int t = threadIdx.x;
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
      if ((uint32_t)t < parts) store_agent(a.imap + a.istart[k] + t, k * (uint32_t)kLongScanParts + t);
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
    rg.write<true>(sh.red, a.lranges + 4 * (size_t)tt);  // (holds a barrier)
    write_counts<true>(s_cnt, a.lcount + (size_t)tt * kMaxBins);
    block_sync();  // the counts are read before they are cleared
  }
}

// The plan of all long queues together, from the tiles' ranges (one workgroup).
__device__ void long_plan(const BArgs& a, uint32_t tiles, uint32_t (*red)[TWV]) {
  const int t = threadIdx.x;
  uint4 v = make_uint4(0xffu, 0u, 0xffffffffu, 0u);
  uint32_t bad = 0, longest = 0;
  for (uint32_t i = t; i < tiles; i += TT) {
    const uint32_t* r4 = a.lranges + 4 * (size_t)i;
    const uint4 x = make_uint4(load_agent(r4), load_agent(r4 + 1), load_agent(r4 + 2),
                               load_agent(r4 + 3));
    v.x = min(v.x, x.x);
    v.y = max(v.y, x.y & 0xffu);
    bad |= x.y & 0x80000000u;
    v.z = min(v.z, x.z);
    v.w = max(v.w, x.w);
  }
  for (uint32_t k = t; k < a.ctl->count[kListLong]; k += TT) {
    const int64_t s = a.lists[2 * kSubLists * a.seg_cap + k];
    longest = max(longest, (uint32_t)(a.offsets[s + 1] - a.offsets[s]));
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
  __shared__ Plan p;  // (its arrays are indexed: scratch memory otherwise)
  p.ok = 0;
  p.nscatter = 0;
  if (all.y >> 31) {
    atomicOr(a.flags, kFlagRange);
  } else {
    make_plan(kFirstBits, longest - 1, a.force_wide != 0, false, all.x, all.y, all.z, all.w, &p);
    p.ok = 1;
    // a wave's 512 waits, each below longest * 2^bits, in 64 bits
    p.sum64 = bit_width32(longest) + bit_width32(all.w) + 9 <= 64 ? 1u : 0u;
  }
  *a.plan = p;
}

// Prefixes of the count rows over each queue's tiles, per digit: a scatter pass's
// counts, or (FINAL) the final digit's counts and length sums. A queue of at
// most kLongRowsFew tiles is one item, a wave per 64 digits running down the
// rows; a longer one is an item per PD digits (64 or 128 bytes of a row), its
// rows split over the workgroup's lanes in NC runs, each read twice: once for
// the runs' sums, once to write the prefixes.
template <bool FINAL>
struct ScanLds {
  static constexpr int PD = FINAL ? 16 : 32;
  uint32_t c[TWV][PD];
  uint64_t w[FINAL ? TWV : 1][PD];
};
// Worker `me` of `workers`, a workgroup each.
template <bool FINAL>
__device__ void scan_rows(const BArgs& a, uint32_t me, uint32_t workers, ScanLds<FINAL>& sh) {
  constexpr int PD = ScanLds<FINAL>::PD;
  constexpr int RL = kWave / PD;   // runs of a wave
  static_assert(kMaxBins / PD <= kLongScanParts, "an item per part");
  const uint32_t items = a.ctl->long_items;
  const int w = wave_no();
  const int lane = lane_id();
  const uint32_t nb = FINAL ? a.plan->nbins[a.plan->nscatter - 1] : (uint32_t)kMaxBins;
  constexpr int U = 8;  // rows in flight
  // Adds rows [r0, r1) of digit d, and with WRITE stores every row's prefix.
  auto run_rows = [&](auto write, uint32_t r0, uint32_t r1, uint32_t d, uint32_t& c,
                      uint64_t& l) {
    for (uint32_t r = r0; r < r1; r += U) {
      typename std::conditional<FINAL, uint64_t, uint32_t>::type x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const size_t at = (size_t)min(r + u, r1 - 1) * kMaxBins + d;
        if constexpr (FINAL) x[u] = a.lfinal[at];
        else x[u] = load_agent(a.lcount + at);
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
  for (uint32_t it = me; it < items; it += workers) {
    const uint32_t im = load_agent(a.imap + it);
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
      sh.c[w][dl] = ic;
      if constexpr (FINAL) sh.w[w][dl] = il;
    }
    block_sync();
    c = ic - c;
    l = il - l;
    for (int v = 0; v < w; ++v) {  // (w is uniform)
      c += sh.c[v][dl];
      if constexpr (FINAL) l += sh.w[v][dl];
    }
    block_sync();  // the sums are read before the next item writes them
    if (d < nb) run_rows(std::true_type{}, r0, r1, d, c, l);
  }
}

__global__ __launch_bounds__(TT) void l_count(BArgs a) {
  __shared__ WorkLds work;
  __shared__ union {
    CountLds count;
    ScanLds<false> scan;
  } sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0) return;
  for (bool begin = true; next_work(a, kRunCount, 2, begin, work); begin = false) {
    const uint32_t me = (uint32_t)__builtin_amdgcn_readfirstlane((int)work.me);
    if (work.phase == 0) {  // (uniform)
      uint32_t lo, hi;
      tile_run(tiles, me, lo, hi);
      count_tiles(a, lo, hi, sh.count);
      continue;
    }
    // the first share makes the plan, the others scan (it too, if alone)
    const uint32_t planner = gridDim.x > 1 ? 1 : 0;
    if (me == 0) {
      long_plan(a, tiles, sh.count.red);
      block_sync();
    }
    if (me >= planner) scan_rows<false>(a, me - planner, gridDim.x - planner, sh.scan);
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

// Small batches: what a scan would have left for tile `tt`, summed here from
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
      else v[u] = load_agent(a.lcount + at);  // (counted in this launch)
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
// from the requests, by the low length bits) or a middle pass. FOLD: the
// counts were not scanned, and are of this launch (as the elements are).
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
        const uint64_t v = FOLD ? load_agent(in + x.at + i) : in[x.at + i];
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
      if constexpr (FOLD) off += load_agent(a.lcount + (size_t)tt * kMaxBins + t);
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
        if (pos < room) {  // (always, for consistent counts)
          if constexpr (FOLD) store_agent(out + pos, v);  // (read in this launch)
          else out[pos] = v;
        }
      }
    }
  }
}

__global__ __launch_bounds__(TT) void l_first(BArgs a) {
  __shared__ LongFirstLds sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok) return;
  uint32_t lo, hi;
  tile_run(tiles, blockIdx.x, lo, hi);
  with_codec(a.plan, [&](auto kc) { long_scatter<true, false>(a, kc, 0, lo, hi, sh); });
}

// Digit counts of the tiles [lo, hi) in middle pass s.
template <bool FOLD>
__device__ void mid_count(const BArgs& a, int s, uint32_t lo, uint32_t hi, uint32_t* s_cnt) {
  const int t = threadIdx.x;
  const uint32_t copy = (uint32_t)lane_id() & (kCountCopies - 1);
  const uint32_t dshift = a.plan->shift[s];
  with_codec<FOLD>(a.plan, [&](auto kc) {
    for (uint32_t tt = lo; tt < hi; ++tt) {
      const LongTileDesc x = a.tdesc[tt];
      uint64_t e[LR];
#pragma unroll
      for (int r = 0; r < LR; ++r) {
        const uint64_t* in = (s & 1 ? a.keys[0] : a.keys[1]) + x.at + min(r * TT + t, x.cnt - 1);
        e[r] = FOLD ? load_agent(in) : *in;
      }
      clear_counts(s_cnt);
      block_sync();
#pragma unroll
      for (int r = 0; r < LR; ++r)
        atomicAdd(&s_cnt[((kc.u2_of(e[r]) >> dshift) & (kMaxBins - 1)) * kCountCopies + copy],
                  r * TT + t < x.cnt ? 1u : 0u);
      block_sync();
      write_counts<true>(s_cnt, a.lcount + (size_t)tt * kMaxBins);
      block_sync();  // the counts are read before they are cleared
    }
  });
}

__global__ __launch_bounds__(TT, 8) void l_mid_rows(BArgs a, int s, PhaseKernel kernel) {
  __shared__ WorkLds work;
  __shared__ union {
    uint32_t cnt[kMaxBins * kCountCopies];
    ScanLds<false> scan;
  } sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok || s >= (int)a.plan->nscatter - 1) return;
  for (bool begin = true; next_work(a, kernel, 2, begin, work); begin = false) {
    const uint32_t me = (uint32_t)__builtin_amdgcn_readfirstlane((int)work.me);
    if (work.phase == 0) {  // (uniform)
      uint32_t lo, hi;
      tile_run(tiles, me, lo, hi);
      mid_count<false>(a, s, lo, hi, sh.cnt);
    } else {
      scan_rows<false>(a, me, gridDim.x, sh.scan);
    }
  }
}

__global__ __launch_bounds__(TT) void l_mid_scatter(BArgs a, int s) {
  __shared__ LongFirstLds sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok || s >= (int)a.plan->nscatter - 1) return;
  uint32_t lo, hi;
  tile_run(tiles, blockIdx.x, lo, hi);
  with_codec(a.plan, [&](auto kc) { long_scatter<false, false>(a, kc, s, lo, hi, sh); });
}

// All middle passes of a small batch in one launch: count and scatter of each.
// (Not for larger ones: the scatter is slower here than alone, 96 us against 87
// over 2^24 requests, and the counts have one workgroup per compute unit
// instead of two; four queues of 2^22 with 31-bit lengths 610 us so, 540 in
// separate launches. 70 queues of 20,000 with such lengths 112 us so, 107 in
// separate launches.)
__global__ __launch_bounds__(TT) void l_mid(BArgs a) {
  __shared__ WorkLds work;
  __shared__ union {
    uint32_t cnt[kMaxBins * kCountCopies];
    LongFirstLds scatter;
  } sh;
  const uint32_t tiles = a.ctl->long_run;
  if (tiles == 0 || !a.plan->ok || a.plan->nscatter <= 2) return;
  const uint32_t phases = 2 * (a.plan->nscatter - 2);
  for (bool begin = true; next_work(a, kRunMid, phases, begin, work); begin = false) {
    const uint32_t phase = (uint32_t)__builtin_amdgcn_readfirstlane((int)work.phase);
    const int s = 1 + (int)(phase >> 1);
    uint32_t lo, hi;
    tile_run(tiles, (uint32_t)__builtin_amdgcn_readfirstlane((int)work.me), lo, hi);
    if ((phase & 1) == 0)
      mid_count<true>(a, s, lo, hi, sh.cnt);
    else
      with_codec<true>(a.plan, [&](auto kc) { long_scatter<false, true>(a, kc, s, lo, hi, sh.scatter); });
  }
}

__global__ __launch_bounds__(TT) void l_histF(BArgs a) {
  __shared__ uint64_t s_bin[kFinalSlots];
  const uint32_t tiles = a.ctl->long_run;
  const Plan* pl = a.plan;
  if (tiles == 0 || !pl->ok) return;
  uint32_t lo, hi;
  tile_run(tiles, blockIdx.x, lo, hi);
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

__global__ __launch_bounds__(TT) void l_scanF(BArgs a) {
  __shared__ ScanLds<true> sh;
  if (a.ctl->long_run == 0 || !a.plan->ok) return;
  scan_rows<true>(a, blockIdx.x, gridDim.x, sh);
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
  tile_run(tiles, blockIdx.x, lo, hi);
  if (a.plan->W == 32 && a.plan->sum64) {
    KeyCodec32 kc;
    kc.init(kFirstBits, a.plan);
    long_final<false, FOLD>(a, kc, lo, hi, sh);
  } else {
    with_codec<FOLD>(a.plan, [&](auto kc) { long_final<true, FOLD>(a, kc, lo, hi, sh); });
  }
}

}  // namespace

hipError_t launch_long_queues(const BArgs& a, hipStream_t st) {
  auto grid = [&](int resident) {
    return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(resident, a.max_tiles)));
  };
  auto launch = [&](auto kernel, int resident, auto... more) {
    hipLaunchKernelGGL(kernel, grid(resident), dim3(TT), 0, st, a, more...);
  };
  static const int r_count = resident_groups(l_count), r_first = resident_groups(l_first),
                   r_histF = resident_groups(l_histF);
  const int most = (int)kMaxShares;
  launch(l_count, std::min(r_count, most));
  launch(l_first, r_first);
  if (!a.force_wide && a.max_tiles <= kFoldTiles &&
      a.max_tiles <= kFoldRows * (uint64_t)a.num_segments) {
    static const int r_mid = resident_groups(l_mid), r_final = resident_groups(l_final<true>);
    launch(l_mid, std::min(r_mid, most));
    launch(l_histF, r_histF);
    launch(l_final<true>, r_final);
  } else {
    static const int r_rows = resident_groups(l_mid_rows), r_mid = resident_groups(l_mid_scatter),
                     r_final = resident_groups(l_final<false>);
    static_assert(max_mid_passes(kFirstBits) <= kRunMidLast - kRunMid + 1, "counters per pass");
    for (int s = 1; s <= max_mid_passes(kFirstBits); ++s) {
      launch(l_mid_rows, std::min(r_rows, most), s, (PhaseKernel)(kRunMid + s - 1));
      launch(l_mid_scatter, r_mid, s);
    }
    launch(l_histF, r_histF);
    const int64_t queues =
        std::min<int64_t>(a.num_segments, (int64_t)(a.long_cap / (kSegLargeCap + 1)));
    const unsigned scan = (unsigned)std::min<uint64_t>(1024, long_items_max(a.long_cap, queues));
    hipLaunchKernelGGL(l_scanF, dim3(scan), dim3(TT), 0, st, a);
    launch(l_final<false>, r_final);
  }
  return hipGetLastError();
}

}  // namespace semsched
