// Schedule of one queue of middling length (more than one workgroup's LDS
// holds, at most kTileMaxItems), one tile per workgroup.
//
// The same LSD radix sort as global_sort.hip (Algorithm 1's drained min-heap:
// ids ascending by (priority, length, id); the waits of Eq. 1 and the class
// totals in the last pass), laid out for latency instead of bandwidth: such a
// queue lies in the caches, so what counts is the number of launches and the
// length of each kernel's chain, not the bytes. Tiles of 1024 to 8192
// requests give 17 to 256 workgroups of 16 waves, elements are whole
// u64 (key above id, nothing to look up by position), and the offsets of a
// tile are summed by the workgroup that needs them from the other tiles'
// count rows, so no scan is launched between a count and its scatter:
//   t_count   ranges and first-digit counts of every tile
//   t_first   the plan from the ranges, the tile's offsets, first scatter
//   t_mid     middle passes of wide keys (returns at once for two-pass keys)
//   t_histF   final-digit counts and length sums of every tile
//   t_final   offsets, order, waits; the last workgroup adds up the totals
// Measured: a queue of 50,003 requests 156 us in the big-tile path's nine
// launches (16K-item tiles: 4 workgroups), 26 us here; one of 2^20 76 us (64
// workgroups), 49 us here.
#include "tile_common.h"

namespace semsched {

namespace {

// The count rows of this path: first-digit (or middle-digit) counts, then
// final-digit counts and length sums.
__device__ __forceinline__ uint16_t* count_rows(const GArgs& a) {
  return reinterpret_cast<uint16_t*>(a.block_hist);
}
__device__ __forceinline__ uint64_t* final_rows(const GArgs& a) { return a.block_histw; }
// Per-tile class sums, [tile][P] (lo, hi); unused by this path otherwise.
__device__ __forceinline__ uint64_t* class_parts(const GArgs& a) {
  return reinterpret_cast<uint64_t*>(a.chunk_part);
}
static_assert(kTileRows * 256 * 16 <= kMaxChunks * kMaxBins * 4, "class sums fit chunk_part");

// Ranges and first-digit counts of one tile; workgroup 0 resets the call's state.
template <int R>
__global__ __launch_bounds__(TT) void t_count(GArgs a) {
  __shared__ uint32_t s_cnt[kMaxBins * kCountCopies];
  __shared__ uint32_t s_red[4][TWV];
  const int t = threadIdx.x;
  const int lane = lane_id();
  const int64_t first = (int64_t)blockIdx.x * (TT * R);
  uint32_t pv[R];
  int32_t lv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = min(first + r * TT + t, a.n - 1);
    pv[r] = a.priority[i];
    lv[r] = a.length[i];
  }
  clear_counts(s_cnt);
  if (blockIdx.x == 0) {
    if (t == 0) {
      a.flags[0] = 0;
      a.plan->ok = 0;
      a.plan->pay = 0;
      a.hist_w[0] = 0;  // workgroups done with the final pass
      a.msync->arrive = 0;
      a.msync->release = 0;
    }
    for (int i = t; i < 2 * (1 + a.num_classes); i += TT) a.totals[i] = 0;
  }
  block_sync();
  const uint32_t mask = (1u << a.d0) - 1;
  TileRanges rg;
  const bool carried = a.payload != nullptr;
  uint32_t pay = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool in = first + r * TT + t < a.n;
    rg.add(in, carried ? 0u : pv[r], lv[r], a.num_classes);
    if (in) pay = max(pay, pv[r]);
    atomicAdd(&s_cnt[((uint32_t)lv[r] & mask) * kCountCopies + (lane & (kCountCopies - 1))],
              in ? 1u : 0u);
  }
  if (carried) rg.pmin = pay;
  rg.write(s_red, a.block_ranges + 4 * (size_t)blockIdx.x, carried);  // (holds a barrier)
  write_counts(s_cnt, count_rows(a) + (size_t)blockIdx.x * kMaxBins);
}

// Sums the tiles' count rows: thread t sums digits 4*(t % 256) .. + 3 over every
// fourth row, rows before this tile's apart from the others (a row is the same
// for a whole wave, so the split costs scalar branches only). Four partial
// sums per digit; a barrier must follow.
__device__ __forceinline__ void fold_rows(const GArgs& a, int me, int rows,
                                          uint32_t (*s_before)[kMaxBins],
                                          uint32_t (*s_after)[kMaxBins]) {
  const int t = threadIdx.x;
  const int w = wave_no();
  uint32_t before[4] = {0, 0, 0, 0}, after[4] = {0, 0, 0, 0};
  {
    const ushort4* rowv = reinterpret_cast<const ushort4*>(count_rows(a)) + (t & 255);
    constexpr int U = 16;  // rows in flight per thread
    for (int g0 = w >> 2; g0 < rows; g0 += 4 * U) {
      ushort4 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        x[u] = rowv[(size_t)min(g0 + 4 * u, rows - 1) * (kMaxBins / 4)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = g0 + 4 * u;
        if (g < me) {
          before[0] += x[u].x;
          before[1] += x[u].y;
          before[2] += x[u].z;
          before[3] += x[u].w;
        } else if (g < rows) {
          after[0] += x[u].x;
          after[1] += x[u].y;
          after[2] += x[u].z;
          after[3] += x[u].w;
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    s_before[t >> 8][4 * (t & 255) + k] = before[k];
    s_after[t >> 8][4 * (t & 255) + k] = after[k];
  }
}

// The output position of this tile's first item of the thread's digit, from
// the sums of fold_rows. Holds barriers.
__device__ __forceinline__ uint32_t fold_offset(uint32_t (*s_before)[kMaxBins],
                                                uint32_t (*s_after)[kMaxBins],
                                                uint32_t* scan32) {
  const int t = threadIdx.x;
  uint32_t mine = 0, total = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    mine += s_before[k][t];
    total += s_after[k][t];
  }
  total += mine;
  uint32_t sum;
  return mine + block_excl_scan_u32<TT>(total, scan32, sum);
}

template <int R>
struct TileFirstLds {
  union {
    uint64_t stage[TT * R];
    struct {
      uint32_t before[4][kMaxBins], after[4][kMaxBins];
    } fold;
  } u;
  uint16_t cnt[TWV][kMaxBins];
  uint32_t base[kMaxBins];
  uint32_t red[4][TWV];
  uint32_t scan32[TWV + 1];
  Plan plan;
};

// Stages a ranked tile in digit order and writes it out.
template <int R, typename Codec>
__device__ __forceinline__ void tile_scatter(const GArgs& a, TileFirstLds<R>& sh, int64_t first,
                                             int cv, const uint32_t (&pv)[R],
                                             const uint32_t (&lv)[R], const uint32_t (&dg)[R],
                                             const uint32_t (&rk)[R]) {
  const int w = wave_no();
  const int j0 = w * kWave * R + lane_id();
  const bool carried = a.payload != nullptr;  // the rank rides above the id
  Codec kc;
  kc.init(a.d0, &sh.plan);
#pragma unroll
  for (int r = 0; r < R; ++r)
    sh.u.stage[rk[r] + sh.cnt[w][dg[r]]] =
        kc.make(carried ? 0u : pv[r], lv[r],
                (uint32_t)(first + j0 + r * kWave) | (carried ? pv[r] << kPayIdBits : 0u));
  block_sync();
  uint64_t* out = a.keys[0];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = j0 + r * kWave;
    if (j < cv) {
      const uint64_t e = sh.u.stage[j];
      const uint32_t pos = sh.base[kc.lo_of(e)] + (uint32_t)j;
      if (pos < (uint64_t)a.n) out[pos] = e;  // (always, for consistent counts)
    }
  }
}

template <int R>
__global__ __launch_bounds__(TT) void t_first(GArgs a) {
  __shared__ TileFirstLds<R> sh;
  const int t = threadIdx.x;
  const int lane = lane_id();
  const int w = wave_no();
  const int me = (int)blockIdx.x;
  const int rows = (int)gridDim.x;
  const int64_t first = (int64_t)me * (TT * R);
  const int cv = (int)min((int64_t)(TT * R), a.n - first);
  const int j0 = w * kWave * R + lane;  // the lane's item in round 0
  uint32_t pv[R], lv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = first + min(j0 + r * kWave, cv - 1);
    pv[r] = a.priority[i];
    lv[r] = (uint32_t)a.length[i];
  }
  // ranges of all tiles (rows <= kTileRows <= TT)
  const bool carried = a.payload != nullptr;
  uint4 rg = make_uint4(carried ? 0u : 0xffu, 0u, 0xffffffffu, 0u);
  if (t < rows) rg = reinterpret_cast<const uint4*>(a.block_ranges)[t];
  fold_rows(a, me, rows, sh.u.fold.before, sh.u.fold.after);
  stage_ranges(rg, sh.red, carried);
  clear_row(sh.cnt[w]);
  block_sync();
  if (t == 0) {
    const uint4 all = collect_ranges(sh.red, (rows + kWave - 1) / kWave, carried);
    sh.plan.cglb = 0;
    sh.plan.ok = 0;
    const bool bad = (all.y >> 31) != 0;
    if (bad) {
      if (me == 0) atomicOr(a.flags, kFlagRange);
    } else {
      make_plan((uint32_t)a.d0, (uint32_t)(a.n - 1), false, false, carried ? 0u : all.x, all.y,
                all.z, all.w, &sh.plan);
      if (carried) {  // (keys of lengths alone: at most 31 bits, so W is 32)
        sh.plan.pay = 1;
        sh.plan.pay_max = all.x;
      }
      sh.plan.ok = 1;
    }
    if (me == 0 && !bad) *a.plan = sh.plan;
  }
  // (holds barriers: the plan is written)
  const uint32_t mine = fold_offset(sh.u.fold.before, sh.u.fold.after, sh.scan32);
  if (!sh.plan.ok) return;
  const uint32_t M0 = (1u << a.d0) - 1;

  uint32_t dg[R], rk[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    // items past the end take the last digit, after every real item of it
    dg[r] = j0 + r * kWave < cv ? lv[r] & M0 : M0;
    rk[r] = rank_round_c<10>(dg[r], sh.cnt[w]);
  }
  block_sync();
  const uint32_t ex = tile_positions(sh.cnt, sh.scan32);
  sh.base[t] = mine - ex;
  block_sync();
  if (sh.plan.W == 32) tile_scatter<R, KeyCodec32>(a, sh, first, cv, pv, lv, dg, rk);
  else tile_scatter<R, KeyCodec64>(a, sh, first, cv, pv, lv, dg, rk);
}

// ---- middle passes (keys of more than two digits) --------------------------------

struct TileCountLds {
  uint32_t cnt[kMaxBins * kCountCopies];
};

// Digit counts of one tile of middle pass s.
template <int R, typename Codec>
__device__ void tile_count_mid(const GArgs& a, int s, int me, TileCountLds& sh) {
  const int t = threadIdx.x;
  const uint32_t copy = (uint32_t)lane_id() & (kCountCopies - 1);
  const uint32_t dshift = a.plan->shift[s];
  Codec kc;
  kc.init(a.d0, a.plan);
  const uint64_t* in = a.keys[(s - 1) & 1];
  const int64_t first = (int64_t)me * (TT * R);
  uint64_t e[R];
#pragma unroll
  for (int r = 0; r < R; ++r) e[r] = in[min(first + r * TT + t, a.n - 1)];
  clear_counts(sh.cnt);
  block_sync();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t d = (kc.u2_of(e[r]) >> dshift) & (kMaxBins - 1);
    atomicAdd(&sh.cnt[d * kCountCopies + copy], first + r * TT + t < a.n ? 1u : 0u);
  }
  block_sync();
  write_counts(sh.cnt, count_rows(a) + (size_t)me * kMaxBins);
}

// Scatter of one tile of middle pass s.
template <int R, typename Codec>
__device__ void tile_scatter_mid(const GArgs& a, int s, int me, int rows, TileFirstLds<R>& sh) {
  const int t = threadIdx.x;
  const int w = wave_no();
  const uint32_t dshift = a.plan->shift[s];
  constexpr uint32_t M = kMaxBins - 1;
  Codec kc;
  kc.init(a.d0, a.plan);
  const uint64_t* in = a.keys[(s - 1) & 1];
  uint64_t* out = a.keys[s & 1];
  const int64_t first = (int64_t)me * (TT * R);
  const int cv = (int)min((int64_t)(TT * R), a.n - first);
  const int j0 = w * kWave * R + lane_id();
  uint64_t e[R];
#pragma unroll
  for (int r = 0; r < R; ++r) e[r] = in[first + min(j0 + r * kWave, cv - 1)];
  fold_rows(a, me, rows, sh.u.fold.before, sh.u.fold.after);
  clear_row(sh.cnt[w]);
  block_sync();
  const uint32_t mine = fold_offset(sh.u.fold.before, sh.u.fold.after, sh.scan32);
  uint32_t dg[R], rk[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {  // items past the end take the last digit
    dg[r] = j0 + r * kWave < cv ? (kc.u2_of(e[r]) >> dshift) & M : M;
    rk[r] = rank_round_c<10>(dg[r], sh.cnt[w]);
  }
  block_sync();
  const uint32_t ex = tile_positions(sh.cnt, sh.scan32);
  sh.base[t] = mine - ex;
  block_sync();
#pragma unroll
  for (int r = 0; r < R; ++r) sh.u.stage[rk[r] + sh.cnt[w][dg[r]]] = e[r];
  block_sync();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = j0 + r * kWave;
    if (j < cv) {
      const uint64_t x = sh.u.stage[j];
      const uint32_t pos = sh.base[(kc.u2_of(x) >> dshift) & M] + (uint32_t)j;
      if (pos < (uint64_t)a.n) out[pos] = x;  // (always, for consistent counts)
    }
  }
}

template <int R>
union TileMidLds {
  TileCountLds count;
  TileFirstLds<R> scatter;
};

// A phase of middle pass s over the tiles me, me + step, ...
template <int R>
__device__ void mid_count(const GArgs& a, int s, int me, int step, TileMidLds<R>& sh) {
  const int rows = (int)((a.n + TT * R - 1) / (TT * R));
  for (; me < rows; me += step) {
    if (a.plan->W == 32) tile_count_mid<R, KeyCodec32>(a, s, me, sh.count);
    else tile_count_mid<R, KeyCodec64>(a, s, me, sh.count);
    block_sync();  // the counts are read before they are cleared
  }
}
template <int R>
__device__ void mid_scatter(const GArgs& a, int s, int me, int step, TileMidLds<R>& sh) {
  const int rows = (int)((a.n + TT * R - 1) / (TT * R));
  for (; me < rows; me += step) {
    if (a.plan->W == 32) tile_scatter_mid<R, KeyCodec32>(a, s, me, rows, sh.scatter);
    else tile_scatter_mid<R, KeyCodec64>(a, s, me, rows, sh.scatter);
    block_sync();  // the stage is read before it is written
  }
}

// All middle passes in one launch with bounded grid barriers between their
// phases, as g_mid does for the big tiles; it returns at once for two-pass
// keys. Its grid is tile_mid_groups'.
template <int R>
__global__ __launch_bounds__(TT) void t_mid(GArgs a) {
  __shared__ TileMidLds<R> sh;
  const Plan* pl = a.plan;
  if (!pl->ok || pl->nscatter <= 2) return;
  uint32_t gen = 0;
  for (int s = 1; s < (int)pl->nscatter - 1; ++s) {
    if (s > 1 && !grid_barrier(a, ++gen)) return;
    mid_count<R>(a, s, (int)blockIdx.x, (int)gridDim.x, sh);
    if (!grid_barrier(a, ++gen)) return;
    mid_scatter<R>(a, s, (int)blockIdx.x, (int)gridDim.x, sh);
  }
}

// The middle passes as separate launches (keys known to be wide, and a schedule
// run again after the barrier gave up).
template <int R>
__global__ __launch_bounds__(TT) void t_mid_count(GArgs a, int s) {
  __shared__ TileMidLds<R> sh;
  if (!a.plan->ok || s >= (int)a.plan->nscatter - 1) return;
  mid_count<R>(a, s, (int)blockIdx.x, (int)gridDim.x, sh);
}
template <int R>
__global__ __launch_bounds__(TT) void t_mid_scatter(GArgs a, int s) {
  __shared__ TileMidLds<R> sh;
  if (!a.plan->ok || s >= (int)a.plan->nscatter - 1) return;
  mid_scatter<R>(a, s, (int)blockIdx.x, (int)gridDim.x, sh);
}

// Final-digit counts and length sums of one tile of the last pass's input.
template <int R, typename Codec>
__device__ void tile_histF(const GArgs& a, uint64_t* s_bin) {
  const Plan* pl = a.plan;
  const int s = (int)pl->nscatter - 1;
  Codec kc;
  kc.init(a.d0, pl);
  const uint64_t* in = a.keys[(s - 1) & 1];
  const int64_t first = (int64_t)blockIdx.x * (TT * R);
  const int cv = (int)min((int64_t)(TT * R), a.n - first);
  uint64_t e[R];
#pragma unroll
  for (int r = 0; r < R; ++r) e[r] = in[first + min(r * TT + (int)threadIdx.x, cv - 1)];
  count_final(kc, TileDigit{pl->shift[s], pl->nbits[s]}, (int)pl->nbins[s], e, cv, s_bin,
              final_rows(a) + (size_t)blockIdx.x * kMaxBins);
}

template <int R>
__global__ __launch_bounds__(TT) void t_histF(GArgs a) {
  __shared__ uint64_t s_bin[kFinalSlots];
  if (!a.plan->ok) return;
  if (a.plan->W == 32) tile_histF<R, KeyCodec32>(a, s_bin);
  else tile_histF<R, KeyCodec64>(a, s_bin);
}

template <int R>
struct TileFinalLds : PlaceLds {
  union {
    uint64_t stage[TT * R];
    struct {
      uint64_t bw[kMaxBins], tw[kMaxBins];
      uint32_t bc[kMaxBins], tc[kMaxBins];
    } fold;
  } u;
  uint32_t last;
};

template <bool PAY, int R, typename Codec>
__device__ void tile_final(const GArgs& a, TileFinalLds<R>& sh) {
  const Plan* pl = a.plan;
  const int t = threadIdx.x;
  const int lane = lane_id();
  const int w = wave_no();
  const int me = (int)blockIdx.x;
  const int rows = (int)gridDim.x;
  const int s = (int)pl->nscatter - 1;
  const int nb = (int)pl->nbins[s];
  const TileDigit dig = {pl->shift[s], pl->nbits[s]};
  const uint32_t P = PAY ? pl->pay_max + 1 : pl->P;  // totals to write
  // copies of a carried rank's sum in the 256 class sums
  const uint32_t csh = PAY ? min(4u, 8u - bit_width32(P - 1)) : 0u;
  const bool small = pl->small != 0;
  Codec kc;
  kc.init(a.d0, pl);
  const int64_t first = (int64_t)me * (TT * R);
  const int cv = (int)min((int64_t)(TT * R), a.n - first);
  const int j0 = w * kWave * R + lane;
  const uint64_t* in = a.keys[(s - 1) & 1];
  uint64_t e[R];
#pragma unroll
  for (int r = 0; r < R; ++r) e[r] = in[first + min(j0 + r * kWave, cv - 1)];

  // counts and length sums of the digits: this tile's offsets and the totals.
  // 2^rb >= nb threads (whole waves) take a row, so 1024 >> rb rows are read
  // at a time.
  const uint32_t rb = max(pl->nbits[s], 6u);
  sh.u.fold.bw[t] = 0;
  sh.u.fold.tw[t] = 0;
  sh.u.fold.bc[t] = 0;
  sh.u.fold.tc[t] = 0;
  if (t < 256) {
    sh.clo[t] = 0;
    sh.chi[t] = 0;
  }
  block_sync();
  {
    const int d = t & ((1 << rb) - 1);
    const int step = TT >> rb;
    uint64_t bw = 0, aw = 0;
    uint32_t bc = 0, ac = 0;
    constexpr int U = 8;
    const uint64_t* col = final_rows(a) + min(d, nb - 1);
    for (int g0 = __builtin_amdgcn_readfirstlane(t >> rb); g0 < rows; g0 += step * U) {
      uint64_t x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = col[(size_t)min(g0 + step * u, rows - 1) * kMaxBins];
      uint64_t b = 0, c = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = g0 + step * u;
        if (g < me) b += x[u];
        else if (g < rows) c += x[u];
      }
      bc += (uint32_t)(b >> kSumBits);
      bw += b & kSumMask;
      ac += (uint32_t)(c >> kSumBits);
      aw += c & kSumMask;
    }
    if (d < nb) {
      if (ac + bc) {
        atomicAdd(&sh.u.fold.tc[d], ac + bc);
        atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.fold.tw[d]), aw + bw);
      }
      if (bc) {
        atomicAdd(&sh.u.fold.bc[d], bc);
        atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.fold.bw[d]), bw);
      }
    }
  }
  block_sync();
  uint32_t pos0 = sh.u.fold.bc[t];
  uint64_t wait0 = sh.u.fold.bw[t];
  {
    uint32_t all32;
    uint64_t all64;
    const uint32_t tc = sh.u.fold.tc[t];
    const uint64_t tw = sh.u.fold.tw[t];
    pos0 += block_excl_scan_u32<TT>(tc, sh.scan32, all32);
    wait0 += block_excl_scan_u64<TT>(tw, sh.scan64, all64);
  }

  place_tile<false, PAY>(kc, dig, small, e, cv, pos0, wait0, a.order, a.wait, (uint64_t)a.n, sh,
                         [] {}, csh);
  block_sync();

  // Class totals: every tile publishes its sums, the last workgroup to finish
  // adds them up (atomics of all tiles on the totals' few lines would queue at
  // about 11 ns each). The sums go through agent-scope stores, complete
  // before the counter is advanced, and are read the same way, so no cache
  // has to be written back for them.
  uint64_t* part = class_parts(a);
  for (uint32_t c = t; c < P; c += TT) {
    uint64_t* o = part + 2 * ((size_t)me * P + c);
    U128 v = {0, 0};
    for (uint32_t k = 0; k < (1u << csh); ++k)
      add128(v, U128{sh.clo[(c << csh) | k], sh.chi[(c << csh) | k]});
    __hip_atomic_store(o, v.lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(o + 1, v.hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  wait_stores();
  block_sync();
  if (t == 0)
    sh.last = atomicAdd(reinterpret_cast<unsigned long long*>(a.hist_w), 1ull) ==
              (unsigned long long)(rows - 1);
  for (uint32_t c = t; c < P; c += TT) {
    sh.clo[c] = 0;
    sh.chi[c] = 0;
  }
  block_sync();
  if (!sh.last) return;
  for (uint32_t i = t; i < (uint32_t)rows * P; i += TT) {
    const U128 v = {load_agent(part + 2 * (size_t)i), load_agent(part + 2 * (size_t)i + 1)};
    const uint32_t c = i % P;
    if (v.lo | v.hi) atomic_add128(&sh.clo[c], &sh.chi[c], v);
  }
  block_sync();
  for (uint32_t c = t; c < P; c += TT) {
    uint64_t* o = a.totals + 2 * (1 + (size_t)(PAY ? 0u : pl->pmin) + c);
    o[0] = sh.clo[c];
    o[1] = sh.chi[c];
  }
  if (t == 0) {
    U128 sum = {0, 0};
    for (uint32_t c = 0; c < P; ++c) {
      const U128 v = {sh.clo[c], sh.chi[c]};
      add128(sum, v);
    }
    a.totals[0] = sum.lo;
    a.totals[1] = sum.hi;
  }
}

template <int R>
__global__ __launch_bounds__(TT) void t_final(GArgs a) {
  __shared__ TileFinalLds<R> sh;
  if (!a.plan->ok) return;
  if (a.payload) tile_final<true, R, KeyCodec32>(a, sh);
  else if (a.plan->W == 32) tile_final<false, R, KeyCodec32>(a, sh);
  else tile_final<false, R, KeyCodec64>(a, sh);
}

template <int R>
hipError_t launch_tiles(const GArgs& a, hipStream_t st, const StageEvents* ev) {
  const dim3 g((unsigned)((a.n + TT * R - 1) / (TT * R)));
  mark_stage(ev, 0, false, st);
  hipLaunchKernelGGL(t_count<R>, g, dim3(TT), 0, st, a);
  mark_stage(ev, 0, true, st);
  mark_stage(ev, 1, false, st);
  hipLaunchKernelGGL(t_first<R>, g, dim3(TT), 0, st, a);
  mark_stage(ev, 1, true, st);
  mark_stage(ev, 6, false, st);
  if (a.split_mid) {
    for (int s = 1; s <= max_mid_passes(a.d0); ++s) {
      hipLaunchKernelGGL(t_mid_count<R>, g, dim3(TT), 0, st, a, s);
      hipLaunchKernelGGL(t_mid_scatter<R>, g, dim3(TT), 0, st, a, s);
    }
  } else {
    static const int resident = resident_groups(t_mid<R>);
    hipLaunchKernelGGL(t_mid<R>, dim3((unsigned)tile_mid_groups(a.n, g.x, resident)), dim3(TT), 0,
                       st, a);
  }
  mark_stage(ev, 6, true, st);
  hipLaunchKernelGGL(t_histF<R>, g, dim3(TT), 0, st, a);
  mark_stage(ev, 2, false, st);
  hipLaunchKernelGGL(t_final<R>, g, dim3(TT), 0, st, a);
  mark_stage(ev, 2, true, st);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_schedule(const GArgs& a, hipStream_t st, const StageEvents* ev) {
  switch (tile_rounds(a.n)) {
    case 1: return launch_tiles<1>(a, st, ev);
    case 2: return launch_tiles<2>(a, st, ev);
    case 4: return launch_tiles<4>(a, st, ev);
    default: return launch_tiles<8>(a, st, ev);
  }
}

}  // namespace semsched
