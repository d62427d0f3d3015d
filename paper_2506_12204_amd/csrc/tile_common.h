// One tile of a digit pass in one 1024-thread workgroup: ranking, positions,
// and the last pass's order, waits and class sums. Shared by the queues of
// one tile per workgroup (tile_sort.hip) and the long queues of a batch
// (long_sort.hip).
#pragma once

#include "block_common.h"
#include "kernels.h"
#include "key_plan.h"

namespace semsched {

namespace {

constexpr int TT = 1024;  // threads: one per digit
constexpr int TWV = TT / kWave;
static_assert(TT == kMaxBins, "every thread owns one digit");
constexpr int kCountCopies = 8;  // copies of a count (lane % 8): equal digits in a wave
                                 // (short lengths, few classes) spread over them
constexpr int kFinalSlots = 8192;  // u64 slots of the final digit's counts, all copies

__device__ __forceinline__ int wave_no() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
}

__device__ __forceinline__ void clear_row(uint16_t* cnt) {  // this wave's 1024 counters
  u64_alias* c64 = reinterpret_cast<u64_alias*>(cnt);
#pragma unroll
  for (int i = 0; i < kMaxBins / (kWave * 4); ++i) c64[i * kWave + lane_id()] = 0;
}

// Ranges of the requests a thread has seen; a tile's are four words: smallest
// rank, largest rank (bit 31: a range error), smallest and largest length.
struct TileRanges {
  uint32_t lmin = 0xffffffffu, lmax = 0, pmin = 0xffu, pmax = 0, bad = 0;
  __device__ __forceinline__ void add(bool in, uint32_t p, int32_t l, int num_classes) {
    const bool ok = (l >= 0) & ((int)p < num_classes);
    bad |= (in & !ok) ? 1u : 0u;
    lmin = min(lmin, in ? (uint32_t)l : 0xffffffffu);
    lmax = max(lmax, in ? (uint32_t)l : 0u);
    pmin = min(pmin, in ? p : 0xffu);
    pmax = max(pmax, in ? p : 0u);
  }
  // The workgroup's ranges to out[0 .. 3]. Holds a barrier. (Carried ranks:
  // the caller adds rank 0 and sets pmin to the largest carried rank, which
  // then reduces by its maximum.)
  template <bool AGENT = false>
  __device__ __forceinline__ void write(uint32_t (*red)[TWV], uint32_t* out, bool carried = false);
};

// A wave's ranges to its column of red; a barrier must follow. `carried`: the
// first word is the largest carried rank.
__device__ __forceinline__ void stage_ranges(uint4 rg, uint32_t (*red)[TWV],
                                             bool carried = false) {
  const uint32_t pl = carried ? wave_max_u32(rg.x) : wave_min_u32(rg.x), ph = wave_max_u32(rg.y & 0xffu);
  const uint32_t bad = wave_or_u32(rg.y & 0x80000000u);
  const uint32_t ll = wave_min_u32(rg.z), lh = wave_max_u32(rg.w);
  if (lane_id() == 0) {
    const int w = wave_no();
    red[0][w] = pl;
    red[1][w] = ph | bad;
    red[2][w] = ll;
    red[3][w] = lh;
  }
}

// The ranges of the first `waves` columns (one thread).
__device__ __forceinline__ uint4 collect_ranges(const uint32_t (*red)[TWV], int waves,
                                                bool carried = false) {
  uint4 v = make_uint4(carried ? 0u : 0xffu, 0u, 0xffffffffu, 0u);
  uint32_t bad = 0;
  for (int i = 0; i < waves; ++i) {
    v.x = carried ? max(v.x, red[0][i]) : min(v.x, red[0][i]);
    v.y = max(v.y, red[1][i] & 0xffu);
    bad |= red[1][i] & 0x80000000u;
    v.z = min(v.z, red[2][i]);
    v.w = max(v.w, red[3][i]);
  }
  v.y |= bad;
  return v;
}

template <bool AGENT>
__device__ __forceinline__ void TileRanges::write(uint32_t (*red)[TWV], uint32_t* out,
                                                  bool carried) {
  stage_ranges(make_uint4(pmin, pmax | (bad << 31), lmin, lmax), red, carried);
  block_sync();
  if (threadIdx.x != 0) return;
  const uint4 v = collect_ranges(red, TWV, carried);
  if constexpr (AGENT) {
    store_agent(out, v.x);
    store_agent(out + 1, v.y);
    store_agent(out + 2, v.z);
    store_agent(out + 3, v.w);
  } else {
    *reinterpret_cast<uint4*>(out) = v;
  }
}

// Digit counts of a tile, kCountCopies copies of each: cleared (a barrier must
// follow), and summed into a row of u16 (a tile holds at most 8192 requests;
// a barrier must precede).
__device__ __forceinline__ void clear_counts(uint32_t* s_cnt) {
  for (int i = threadIdx.x; i < kMaxBins * kCountCopies / 4; i += TT)
    reinterpret_cast<uint4*>(s_cnt)[i] = make_uint4(0, 0, 0, 0);
}
template <bool AGENT = false>
__device__ __forceinline__ void write_counts(const uint32_t* s_cnt, uint16_t* row) {
  static_assert(kCountCopies == 8, "two quads per digit");
  const int t = threadIdx.x;
  const uint4 c0 = reinterpret_cast<const uint4*>(s_cnt)[2 * t];
  const uint4 c1 = reinterpret_cast<const uint4*>(s_cnt)[2 * t + 1];
  const uint16_t sum = (uint16_t)(c0.x + c0.y + c0.z + c0.w + c1.x + c1.y + c1.z + c1.w);
  if constexpr (AGENT) store_agent(row + t, sum);
  else row[t] = sum;
}

// Turns the waves' counters of a ranked tile into the positions of each
// wave's first item of a digit in the tile's digit order; the thread's digit
// starts at the returned position. Holds barriers.
__device__ __forceinline__ uint32_t tile_positions(uint16_t (*cnt)[kMaxBins], uint32_t* scan32) {
  const int t = threadIdx.x;
  uint32_t c[TWV], tot = 0;
#pragma unroll
  for (int v = 0; v < TWV; ++v) {
    c[v] = cnt[v][t];
    tot += c[v];
  }
  uint32_t all;
  const uint32_t ex = block_excl_scan_u32<TT>(tot, scan32, all);
  uint32_t run = ex;
#pragma unroll
  for (int v = 0; v < TWV; ++v) {
    cnt[v][t] = (uint16_t)run;
    run += c[v];
  }
  return ex;
}

// Workgroups of a kernel of TT threads that the device holds at once (of it alone).
template <typename K>
int resident_groups(K kernel) {
  int dev = 0, cus = 256, occ = 1;
  if (hipGetDevice(&dev) == hipSuccess) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
  }
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, reinterpret_cast<const void*>(kernel),
                                                   TT, 0) != hipSuccess ||
      occ < 1)
    occ = 1;
  return cus * occ;
}

// Elements that carry a rank have it above the low 24 bits of the id.
constexpr uint32_t kPayIdBits = 24;
constexpr uint32_t kPayIdMask = (1u << kPayIdBits) - 1;

// A digit of the mixed-radix value u2.
struct TileDigit {
  uint32_t shift, bits;
};

// Rows of the final digit's counts hold one u64 per digit: the count above the
// length sum (8192 lengths below 2^31 sum to less than 2^44, so up to eight
// rows can be added as they are).
constexpr uint32_t kSumBits = 47;
constexpr uint64_t kSumMask = (1ull << kSumBits) - 1;

// Counts the final digit of a tile (item r*TT + thread, cv of them valid) into
// such a row of nb digits. Each digit is counted in as many copies (lane
// modulo their number) as the slots hold, at most one per lane: with few
// digits all lanes would otherwise meet on a few words. Holds barriers.
template <int R, typename Codec>
__device__ __forceinline__ void count_final(const Codec& kc, const TileDigit& dig, int nb,
                                            const uint64_t (&e)[R], int cv, uint64_t* s_bin,
                                            uint64_t* row) {
  const int t = threadIdx.x;
  const uint32_t dmask = (1u << dig.bits) - 1;
  const uint32_t cb = min(6u, 13u - dig.bits);
  static_assert(kFinalSlots == 1 << 13, "2^bits digits times 2^cb copies");
  for (int i = t; i < (nb << cb); i += TT) s_bin[i] = 0;
  block_sync();
  const uint32_t copy = (uint32_t)lane_id() & ((1u << cb) - 1);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t d = (kc.u2_of(e[r]) >> dig.shift) & dmask;
    if (r * TT + t < cv)
      atomicAdd(reinterpret_cast<unsigned long long*>(&s_bin[(d << cb) + copy]),
                (1ull << kSumBits) | kc.len_of(e[r]));
  }
  block_sync();
  constexpr int PER = 8;  // copies added by one thread (cb >= 3: at most 1024 digits)
  for (int i = t; i < (nb << cb) / PER; i += TT) {
    uint64_t v = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) v += s_bin[PER * i + k];
    for (uint32_t k = 1; k < (1u << cb) / PER; k <<= 1) v += __shfl_xor(v, (int)k, kWave);
    if ((i & ((1 << cb) / PER - 1)) == 0) row[i >> (cb - 3)] = v;
  }
}

struct PlaceLds {
  uint16_t cnt[TWV][kMaxBins];
  uint64_t wb[kMaxBins];     // wait base of the tile's run of a digit
  uint32_t base[kMaxBins];   // output position of a digit's run minus its tile position
  uint32_t start[kMaxBins];  // the run's tile position
  uint64_t clo[256], chi[256];
  uint64_t scan64[TWV + 1];
  uint32_t scan32[TWV + 1];
};

// Writes order and waits of one tile of the last pass, in its digit order, and
// adds the waits to the class sums clo/chi of LDS (classes relative to pmin).
// e: the tile's elements, item (wave, round, lane) the tile's position
// wave*64*R + round*64 + lane, cv of them valid. pos0, wait0: output position
// and wait of the tile's first item of the thread's digit. Positions of
// `limit` and more are not written. WIDE_SUMS: a wave's waits may add up to
// 2^64 and more (never for queues of at most 2^21 requests: 512 waits below
// 2^52). `staged` is called once e is free to take other elements (the next
// tile's, loaded while this one is placed). The LDS members may be used again
// after the next barrier; clo/chi are complete after it.
// PAY: the ids' bits 24 and up carry the caller's rank, and the totals are
// split by it: its sums go to copies of the class sums (rank << pay_shift |
// lane), 16 of them for up to 16 ranks, which 64 bits hold.
template <bool WIDE_SUMS, bool PAY, int R, typename Codec, typename Lds, typename Staged>
__device__ __forceinline__ void place_tile(const Codec& kc, const TileDigit& dig, bool small,
                                           const uint64_t (&e)[R], int cv, uint32_t pos0,
                                           uint64_t wait0, int32_t* order, int64_t* wait,
                                           uint64_t limit, Lds& sh, Staged&& staged,
                                           uint32_t pay_shift = 0) {
  const int t = threadIdx.x;
  const int lane = lane_id();
  const int w = wave_no();
  const int j0 = w * kWave * R + lane;
  const uint32_t dmask = (1u << dig.bits) - 1;
  uint64_t* stage = sh.u.stage;
  clear_row(sh.cnt[w]);
  uint32_t dg[R], rk[R];
#pragma unroll
  for (int r = 0; r < R; ++r)  // items past the end take the last digit
    dg[r] = j0 + r * kWave < cv ? (kc.u2_of(e[r]) >> dig.shift) & dmask : dmask;
  if (dig.bits <= 6) {
#pragma unroll
    for (int r = 0; r < R; ++r) rk[r] = rank_round_c<6>(dg[r], sh.cnt[w]);
  } else if (dig.bits <= 8) {
#pragma unroll
    for (int r = 0; r < R; ++r) rk[r] = rank_round_c<8>(dg[r], sh.cnt[w]);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) rk[r] = rank_round_c<10>(dg[r], sh.cnt[w]);
  }
  block_sync();
  const uint32_t ex = tile_positions(sh.cnt, sh.scan32);
  sh.base[t] = pos0 - ex;
  sh.start[t] = ex;
  sh.wb[t] = wait0;
  block_sync();
#pragma unroll
  for (int r = 0; r < R; ++r) stage[rk[r] + sh.cnt[w][dg[r]]] = e[r];
  staged();
  block_sync();

  // lengths in the tile's digit order, scanned; the first item of a run turns
  // its digit's wait base into the base of the whole run (the elements are
  // read from the stage again in every step: kept, they would take 2R
  // registers that the next tile's need)
  uint64_t lp[R];
  uint64_t run = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = j0 + r * kWave;
    const uint32_t l = j < cv ? kc.len_of(stage[j]) : 0u;
    const uint64_t inc = small ? (uint64_t)wave_incl_scan_u32(l) : wave_incl_scan_len(l);
    lp[r] = run + inc - l;
    run += last_lane_u64(inc);
  }
  if (lane == 0) sh.scan64[w] = run;
  block_sync();
  uint64_t wave0 = 0;
  for (int v = 0; v < w; ++v) wave0 += sh.scan64[v];  // (w is uniform)
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = j0 + r * kWave;
    lp[r] += wave0;
    dg[r] = j < cv ? (kc.u2_of(stage[j]) >> dig.shift) & dmask : dmask;
    if (j < cv && (uint32_t)j == sh.start[dg[r]]) sh.wb[dg[r]] -= lp[r];
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  block_sync();
  // order and waits; the tile is class-major, so a lane's classes do not
  // decrease over its rounds
  uint32_t cur = 0xffffffffu;
  U128 acc = {0, 0};
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = j0 + r * kWave;
    if (j < cv) {
      const uint32_t pos = sh.base[dg[r]] + (uint32_t)j;
      const uint64_t wt = sh.wb[dg[r]] + lp[r];
      const uint64_t x = stage[j];
      if (pos < limit) {  // (always, for consistent counts)
        order[pos] = (int32_t)(PAY ? kc.id(x) & kPayIdMask : kc.id(x));
        wait[pos] = (int64_t)wt;
      }
      if constexpr (PAY) {
        const uint32_t at = (kc.id(x) >> kPayIdBits << pay_shift) | (lane & ((1u << pay_shift) - 1));
        if (pay_shift >= 4)  // (uniform) 512 waits at most per copy and tile
          atomicAdd(reinterpret_cast<unsigned long long*>(&sh.clo[at]), (unsigned long long)wt);
        else
          atomic_add128(&sh.clo[at], &sh.chi[at], U128{wt, 0});
        continue;
      }
      const uint32_t c = kc.pp_of(x);
      if (c != cur) {
        if (cur != 0xffffffffu) atomic_add128(&sh.clo[cur], &sh.chi[cur], acc);
        cur = c;
        acc = {0, 0};
      }
      if constexpr (WIDE_SUMS) add128(acc, wt);
      else acc.lo += wt;
    }
    // (all rounds' reads and addresses at once would take the registers of
    // the next tile's elements)
    if (r % 2 == 1) __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (PAY) return;
  // lanes that end in one class (nearly all waves) add up first
  const uint32_t c0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cur);
  if (__builtin_amdgcn_ballot_w64(cur != c0) == 0) {
    if (c0 != 0xffffffffu) {
      if constexpr (WIDE_SUMS) acc = wave_sum128(acc);
      else acc.lo = last_lane_u64(wave_incl_scan_u64(acc.lo));
      if (lane == 0) atomic_add128(&sh.clo[c0], &sh.chi[c0], acc);
    }
  } else if (cur != 0xffffffffu) {
    atomic_add128(&sh.clo[cur], &sh.chi[cur], acc);
  }
}

}  // namespace

}  // namespace semsched
