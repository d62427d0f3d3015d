// The plan of one long queue's sort (key layout and digits, from the measured
// ranges), the packed key it describes and the grid barrier of the middle
// passes, shared by the big-tile path
// (global_sort.hip) and the one-tile-per-workgroup path (tile_sort.hip).
#pragma once

#include "block_common.h"
#include "kernels.h"

namespace semsched {

// Fills every field of the plan but `ok` and `cglb` from the ranges of valid
// queues (one thread); no ranks are carried. d0: width of the first digit;
// max_id: the largest request id; force_wide, chunked: as in GArgs.
__device__ __forceinline__ void make_plan(uint32_t d0, uint32_t max_id, bool force_wide,
                                          bool chunked, uint32_t gpmin, uint32_t gpmax,
                                          uint32_t glmin, uint32_t glmax, Plan* pl) {
  const uint32_t P = gpmax - gpmin + 1;
  const uint32_t hmin = glmin >> d0;
  const uint32_t H = (glmax >> d0) - hmin + 1;
  const uint32_t wp = bit_width32(P - 1);
  const uint32_t wh = bit_width32(H - 1);
  const uint32_t wid = bit_width32(max_id);
  const uint32_t kb = wp + wh + d0;  // live key bits
  pl->pmin = gpmin;
  pl->P = P;
  pl->hmin = hmin;
  pl->H = H;
  pl->wp = wp;
  pl->wh = wh;
  // A key of at most 32 bits sits in the high word above a 32-bit id, so no
  // shifts across words are needed to take an element apart.
  pl->W = (!force_wide && kb <= 32) ? 32u : wid;
  pl->packed = (!force_wide && kb + pl->W <= 64) ? 1u : 0u;
  pl->small = glmax < (1u << 26) ? 1u : 0u;
  const uint64_t R = (uint64_t)P * H;  // <= 2^31 because d0 >= 8
  pl->shift[0] = 0;
  pl->nbits[0] = d0;
  pl->nbins[0] = 1u << d0;
  uint32_t mids = 0;
  if (R > (uint64_t)kMaxBins) {
    const uint32_t b2 = bit_width32((uint32_t)(R - 1));
    mids = (b2 - 10 + 9) / 10;
  }
  for (uint32_t s = 1; s <= mids; ++s) {
    pl->shift[s] = 10 * (s - 1);
    pl->nbits[s] = 10;
    pl->nbins[s] = kMaxBins;
  }
  const uint32_t sf = 10 * mids;
  const uint32_t fb = (uint32_t)((R - 1) >> sf) + 1;
  pl->shift[1 + mids] = sf;
  pl->nbins[1 + mids] = fb;
  pl->nbits[1 + mids] = bit_width32(fb - 1);
  pl->nscatter = 2 + mids;
  // compact layout: two passes, at most 256 final digits (the big-tile final
  // pass), lengths below 2^26, and the sub-bucket starts were counted
  pl->compact = (chunked && !force_wide && mids == 0 && fb <= 256 && pl->small) ? 1u : 0u;
  pl->pay = 0;
  pl->pay_shift = 32;
}

// Grid barrier of the middle-pass kernel, a normal launch whose grid is the
// number of workgroups that fit on the device at once. Workgroup leaders add
// to the arrival count; the last to arrive resets it and publishes the
// barrier's generation in the release word, which the others poll. The wait
// is bounded: if the workgroups were not all resident (another program
// holding CUs), a leader gives up after a.mid_spin polls, records
// kFlagDevice, clears the plan's ok word (so the kernels after this one do
// nothing) and every workgroup leaves at its next barrier; the blocking
// calls then run the schedule again with the middle passes as separate
// launches per phase, which need no residency.
static __device__ bool grid_barrier(const GArgs& a, uint32_t gen) {
  __shared__ uint32_t s_ok;
  // Every wave's stores are in the caches (vmcnt 0) before the barrier; then
  // one thread's fence writes this XCD's L2 back for the whole workgroup, and
  // one thread's fence after the wait drops the CU's and L2's stale lines for
  // it. (A fence in every wave made sixteen write-backs of the L2 per
  // workgroup and barrier: a middle pass over 2^20 requests took 82 us.)
  wait_stores();
  block_sync();
  if (threadIdx.x == 0) {
    uint32_t ok = 1;
    __threadfence();  // release
    if (atomicAdd(&a.msync->arrive, 1u) == gridDim.x - 1) {
      __hip_atomic_store(&a.msync->arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.msync->release, gen, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      // relaxed polls: an acquire load would invalidate this XCD's L2 at
      // every poll, under the workgroups still working there; the fence
      // after the wait orders what follows
      for (uint32_t spin = 0; __hip_atomic_load(&a.msync->release, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) < gen;
           ++spin) {
        if (spin >= a.mid_spin || ((spin & 63) == 63 && (load_agent(a.flags) & kFlagDevice))) {
          atomicOr(a.flags, kFlagDevice);
          // the later kernels of this schedule then return at once
          __hip_atomic_store(&a.plan->ok, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    if (load_agent(a.flags) & kFlagDevice) ok = 0;
    __threadfence();  // acquire the other workgroups' writes
    s_ok = ok;
  }
  block_sync();
  return s_ok != 0;
}

struct KeyCodec {
  uint32_t d0, wh, W, hmin, H, pmin;
  uint64_t m0, mh, idmask;
  __device__ __forceinline__ void init(int first_bits, const Plan* pl) {
    d0 = (uint32_t)first_bits;
    wh = pl->wh;
    W = pl->W;
    hmin = pl->hmin;
    H = pl->H;
    pmin = pl->pmin;
    m0 = (1ull << d0) - 1;
    mh = (1ull << wh) - 1;
    idmask = (1ull << W) - 1;
  }
  __device__ __forceinline__ uint32_t lo(uint64_t key) const { return (uint32_t)(key & m0); }
  __device__ __forceinline__ uint32_t h(uint64_t key) const {
    return (uint32_t)((key >> d0) & mh);
  }
  __device__ __forceinline__ uint32_t pp(uint64_t key) const {
    return (uint32_t)(key >> (d0 + wh));
  }
  __device__ __forceinline__ uint32_t u2(uint64_t key) const { return pp(key) * H + h(key); }
  __device__ __forceinline__ uint32_t len(uint64_t key) const {
    return ((h(key) + hmin) << d0) | lo(key);
  }
  __device__ __forceinline__ uint64_t make(uint32_t p, uint32_t l) const {
    return ((uint64_t)(p - pmin) << (d0 + wh)) | ((uint64_t)((l >> d0) - hmin) << d0) |
           (l & (uint32_t)m0);
  }
};

// Element forms of the one-tile-per-workgroup sorts (tile_common.h): what a
// packed element holds, each with make / id / lo_of / u2_of / pp_of / len_of.
//
// Keys of at most 32 bits in the element's high word (Plan::W = 32): no 64-bit
// shifts.
struct KeyCodec32 {
  uint32_t d0, ph, hoff, H, pmin, m0, mh, ml;
  __device__ __forceinline__ void init(int first_bits, const Plan* pl) {
    d0 = (uint32_t)first_bits;
    ph = d0 + pl->wh;  // at most 31: lengths are below 2^31
    hoff = pl->hmin << d0;
    H = pl->H;
    pmin = pl->pmin;
    m0 = (1u << d0) - 1;
    mh = pl->wh ? 0xffffffffu >> (32 - pl->wh) : 0u;
    ml = 0xffffffffu >> (32 - ph);
  }
  __device__ __forceinline__ static uint32_t id(uint64_t e) { return (uint32_t)e; }
  __device__ __forceinline__ uint32_t lo_of(uint64_t e) const { return (uint32_t)(e >> 32) & m0; }
  __device__ __forceinline__ uint32_t pp_of(uint64_t e) const { return (uint32_t)(e >> 32) >> ph; }
  __device__ __forceinline__ uint32_t u2_of(uint64_t e) const {
    return pp_of(e) * H + (((uint32_t)(e >> 32) >> d0) & mh);
  }
  __device__ __forceinline__ uint32_t len_of(uint64_t e) const {
    return ((uint32_t)(e >> 32) & ml) + hoff;
  }
  __device__ __forceinline__ uint64_t make(uint32_t p, uint32_t l, uint32_t i) const {
    return ((uint64_t)(((p - pmin) << ph) + (l - hoff)) << 32) | i;
  }
};

// Any key above an id of W bits.
struct KeyCodec64 : KeyCodec {
  __device__ __forceinline__ uint32_t id(uint64_t e) const { return (uint32_t)(e & idmask); }
  __device__ __forceinline__ uint32_t lo_of(uint64_t e) const { return lo(e >> W); }
  __device__ __forceinline__ uint32_t pp_of(uint64_t e) const { return pp(e >> W); }
  __device__ __forceinline__ uint32_t u2_of(uint64_t e) const { return u2(e >> W); }
  __device__ __forceinline__ uint32_t len_of(uint64_t e) const { return len(e >> W); }
  using KeyCodec::make;
  __device__ __forceinline__ uint64_t make(uint32_t p, uint32_t l, uint32_t i) const {
    return (make(p, l) << W) | i;
  }
};

// Key and id beyond 64 bits together (39-bit keys in queues of more than 2^25
// requests): the element leaves the first digit out, which no pass after the
// first orders by, and lengths are read through the id.
struct KeyCodecGather {
  uint32_t d0, wh, W, hmin, H, pmin;
  uint64_t mh, idmask;
  const int32_t* lengths;  // the queue's
  __device__ __forceinline__ void init(int first_bits, const Plan* pl) {
    d0 = (uint32_t)first_bits;
    wh = pl->wh;
    W = pl->W;
    hmin = pl->hmin;
    H = pl->H;
    pmin = pl->pmin;
    mh = (1ull << wh) - 1;
    idmask = (1ull << W) - 1;
    lengths = nullptr;
  }
  __device__ __forceinline__ uint32_t id(uint64_t e) const { return (uint32_t)(e & idmask); }
  __device__ __forceinline__ uint32_t len_of(uint64_t e) const { return (uint32_t)lengths[id(e)]; }
  __device__ __forceinline__ uint32_t lo_of(uint64_t e) const {
    return len_of(e) & ((1u << d0) - 1);
  }
  __device__ __forceinline__ uint32_t pp_of(uint64_t e) const { return (uint32_t)(e >> (W + wh)); }
  __device__ __forceinline__ uint32_t u2_of(uint64_t e) const {
    return pp_of(e) * H + (uint32_t)((e >> W) & mh);
  }
  __device__ __forceinline__ uint64_t make(uint32_t p, uint32_t l, uint32_t i) const {
    return ((((uint64_t)(p - pmin) << wh) | ((l >> d0) - hmin)) << W) | i;
  }
};

}  // namespace semsched
