// Batch selection with stage awareness (Algorithm 2) and priority-based
// eviction (Algorithms 3 and 4) of Section 3.3.
//
// Both work on the few requests of one scheduling iteration (candidates,
// ongoing requests, cached requests), so each is one workgroup over LDS.
// A request's key is (rank << 32 | length, id): the scheduling order of
// Algorithm 1; the smallest key is the most urgent request.
//
//   b_select  sorts the candidates (the heap's first b entries and the
//             unsorted buffer) and the ongoing requests (an LDS radix sort
//             over the key bits that vary); the candidates C are the first
//             b. The most urgent of C and O decides the stage filter; every
//             element's place in the merged list M (C's surviving members and O) and in the
//             pushed-back list (C's filtered members and M beyond b) comes
//             from binary searches in the other sorted lists.
//   b_evict   sorts the cached requests; the eviction order is that order
//             reversed (least urgent, longest first; the later arrival
//             first among equal keys). A scan of their KV sizes in that
//             order gives, for each incoming request, the number of
//             victims after its step: the shortest prefix covering
//             usage + (demands so far) - capacity.
#include <algorithm>

#include "block_common.h"
#include "kernels.h"

namespace semsched {

namespace {

constexpr int BT = 1024;
constexpr int kCandCap = 2 * kSelectCap;  // heap's first b plus the buffer

__device__ __forceinline__ bool less(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return ka < kb || (ka == kb && ia < ib);
}

// Scratch of the block radix sort: per-wave digit counters (then the waves'
// offsets) and the wave partials of the key range reduction and the scans.
constexpr int kSortWaves = BT / kWave;
struct SortScratch {
  uint16_t cnt[kSortWaves][256];
  uint32_t red[kSortWaves * 6];
};

// Stable LSD radix sort by (key, id) of the first n of the BT * E entries of
// key / id (and a u32 payload that moves with them) in LDS, 8 bits at a time,
// the id's digits first, then the key's; digits that are the same for all n
// entries are skipped (the bitwise AND and OR of all keys and ids tell which
// vary). Every pass ranks the rounds of each wave by ballot matching
// (entries (wave, round, lane) in index order, so ranks follow the current
// order: stable), turns the waves' counts into digit-major offsets and
// scatters through LDS. Entries n .. BT*E-1 take (OR of the keys, OR of the
// ids): no real entry sorts after them. Every thread of the block must call
// it.
template <int E, bool PAYLOAD>
__device__ __forceinline__ void block_sort(uint64_t* key, uint32_t* id, uint32_t* pay, uint32_t n,
                           SortScratch& sc) {
  if (n <= 1) return;  // (uniform) nothing to order
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  auto at = [&](int r) { return (uint32_t)(w * kWave * E + r * kWave + lane); };
  uint64_t xk[E];
  uint32_t xi[E], xp[E];
  uint32_t kand_lo = ~0u, kand_hi = ~0u, kor_lo = 0, kor_hi = 0, iand = ~0u, ior = 0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t i = at(r);
    xk[r] = key[i];
    xi[r] = id[i];
    xp[r] = PAYLOAD ? pay[i] : 0u;
    if (i < n) {
      kand_lo &= (uint32_t)xk[r];
      kand_hi &= (uint32_t)(xk[r] >> 32);
      kor_lo |= (uint32_t)xk[r];
      kor_hi |= (uint32_t)(xk[r] >> 32);
      iand &= xi[r];
      ior |= xi[r];
    }
  }
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) {
    kand_lo &= (uint32_t)__shfl_xor((int)kand_lo, off, kWave);
    kand_hi &= (uint32_t)__shfl_xor((int)kand_hi, off, kWave);
    kor_lo |= (uint32_t)__shfl_xor((int)kor_lo, off, kWave);
    kor_hi |= (uint32_t)__shfl_xor((int)kor_hi, off, kWave);
    iand &= (uint32_t)__shfl_xor((int)iand, off, kWave);
    ior |= (uint32_t)__shfl_xor((int)ior, off, kWave);
  }
  if (lane == 0) {
    uint32_t* r6 = sc.red + 6 * w;
    r6[0] = kand_lo, r6[1] = kand_hi, r6[2] = kor_lo, r6[3] = kor_hi, r6[4] = iand, r6[5] = ior;
  }
  block_sync();
#pragma unroll
  for (int v = 0; v < kSortWaves; ++v) {
    const uint32_t* r6 = sc.red + 6 * v;
    kand_lo &= r6[0], kand_hi &= r6[1], kor_lo |= r6[2], kor_hi |= r6[3];
    iand &= r6[4], ior |= r6[5];
  }
  block_sync();  // (the partials' words are the scans' scratch below)
  const uint64_t kor = (uint64_t)kor_hi << 32 | kor_lo;
  uint64_t kvary = kor ^ ((uint64_t)kand_hi << 32 | kand_lo);
  uint32_t ivary = ior ^ iand;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    if (at(r) >= n) {
      xk[r] = kor;
      xi[r] = ior;
    }
  }
  // Packed form: the spans of varying bits of the id, the key's low word and
  // its high word, laid end to end in one u64 (id lowest), when they fit. Its
  // order is the order by (key, id), and its bytes take the passes, in place
  // of the id's and the key's varying bytes (41 bits and 6 passes against 7
  // bytes for ids of 26 bits, lengths of 12 and ranks of 3). The key array
  // then carries the packed value, and the keys are rebuilt from it (and the
  // bits that do not vary) after the last pass.
  const uint32_t v0 = ivary, v1 = (uint32_t)kvary, v2 = (uint32_t)(kvary >> 32);
  const uint32_t l0 = v0 ? __builtin_ctz(v0) : 0, w0 = v0 ? 32 - __builtin_clz(v0) - l0 : 0;
  const uint32_t l1 = v1 ? __builtin_ctz(v1) : 0, w1 = v1 ? 32 - __builtin_clz(v1) - l1 : 0;
  const uint32_t l2 = v2 ? __builtin_ctz(v2) : 0, w2 = v2 ? 32 - __builtin_clz(v2) - l2 : 0;
  const uint32_t pbits = w0 + w1 + w2;
  auto low_mask = [](uint32_t wd) { return wd >= 32 ? ~0u : (1u << wd) - 1u; };
  const uint32_t m0 = low_mask(w0), m1 = low_mask(w1), m2 = low_mask(w2);
  uint32_t vbytes = 0;  // passes of the byte form
#pragma unroll
  for (int b = 0; b < 4; ++b)
    vbytes += ((v0 >> (8 * b)) & 0xffu ? 1u : 0u) + ((v1 >> (8 * b)) & 0xffu ? 1u : 0u) +
              ((v2 >> (8 * b)) & 0xffu ? 1u : 0u);
  const bool packed = pbits <= 64 && (pbits + 7) / 8 < vbytes;
  const uint32_t s2 = w0 + w1;  // below 64 when the high word's span is not empty
  bool packed_moved = false;  // the key array holds packed values
  if (packed) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint64_t f0 = (xi[r] >> l0) & m0;
      const uint64_t f1 = ((uint32_t)xk[r] >> l1) & m1;
      const uint64_t f2 = ((uint32_t)(xk[r] >> 32) >> l2) & m2;
      xk[r] = f0 | (f1 << w0) | (w2 ? f2 << s2 : 0ull);
    }
    kvary = pbits >= 64 ? ~0ull : (1ull << pbits) - 1;
    ivary = 0;
  }
  uint16_t* mycnt = sc.cnt[w];
  for (int pass = 0; pass < 12; ++pass) {
    const bool on_id = pass < 4;
    const int sh = 8 * (on_id ? pass : pass - 4);
    const uint32_t vary = on_id ? (ivary >> sh) & 0xffu : (uint32_t)(kvary >> sh) & 0xffu;
    if (vary == 0) continue;  // (uniform)
    for (int b = lane; b < 256; b += kWave) mycnt[b] = 0;
    uint32_t dg[E], rk[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      dg[r] = on_id ? (xi[r] >> sh) & 0xffu : (uint32_t)(xk[r] >> sh) & 0xffu;
      rk[r] = rank_round_c<8>(dg[r], mycnt);
    }
    block_sync();  // every wave's counts are in
    // digit-major offsets: thread d < 256 owns digit d
    uint32_t c[kSortWaves], tot = 0;
#pragma unroll
    for (int v = 0; v < kSortWaves; ++v) {
      c[v] = t < 256 ? sc.cnt[v][t] : 0u;
      tot += c[v];
    }
    uint32_t all;
    uint32_t run = block_excl_scan_u32<BT>(tot, sc.red, all);
    if (t < 256) {
#pragma unroll
      for (int v = 0; v < kSortWaves; ++v) {
        sc.cnt[v][t] = (uint16_t)run;
        run += c[v];
      }
    }
    block_sync();  // offsets are written
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t q = rk[r] + mycnt[dg[r]];
      key[q] = xk[r];
      id[q] = xi[r];
      if (PAYLOAD) pay[q] = xp[r];
    }
    packed_moved = packed;
    block_sync();  // the pass is scattered
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t i = at(r);
      xk[r] = key[i];
      xi[r] = id[i];
      if (PAYLOAD) xp[r] = pay[i];
    }
  }
  if (packed_moved) {  // (uniform) the keys back from the packed values
    const uint32_t keep_lo = kand_lo & ~(m1 << l1), keep_hi = kand_hi & ~(m2 << l2);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t f1 = (uint32_t)(xk[r] >> w0) & m1;
      const uint32_t f2 = w2 ? (uint32_t)(xk[r] >> s2) & m2 : 0u;
      key[at(r)] = (uint64_t)(keep_hi | (f2 << l2)) << 32 | (keep_lo | (f1 << l1));
    }
  }
  block_sync();  // (the last pass's reads are done before callers write)
}

// Sorts the first n entries (n <= 8 * BT) of key / id (and pay), with E
// entries per thread, the fewest of 1, 2, 4, 5, 6 or 8 that hold n (each
// pass costs about E rounds per wave, padding included; the sort with a
// payload keeps to 1, 2, 4 and 8, whose kernel the other widths made spill).
template <bool PAYLOAD>
__device__ void sort_pairs(uint64_t* key, uint32_t* id, uint32_t* pay, uint32_t n,
                           SortScratch& sc) {
  if (n <= (uint32_t)BT) block_sort<1, PAYLOAD>(key, id, pay, n, sc);
  else if (n <= 2u * BT) block_sort<2, PAYLOAD>(key, id, pay, n, sc);
  else if (n <= 4u * BT) block_sort<4, PAYLOAD>(key, id, pay, n, sc);
  else if (!PAYLOAD && n <= 5u * BT) block_sort<5, PAYLOAD>(key, id, pay, n, sc);
  else if (!PAYLOAD && n <= 6u * BT) block_sort<6, PAYLOAD>(key, id, pay, n, sc);
  else block_sort<8, PAYLOAD>(key, id, pay, n, sc);
}

template <bool PAYLOAD>
__device__ __forceinline__ uint32_t sort_size(uint32_t n) {
  return n <= (uint32_t)BT ? BT : n <= 2u * BT ? 2 * BT : n <= 4u * BT ? 4 * BT
         : !PAYLOAD && n <= 5u * BT ? 5 * BT : !PAYLOAD && n <= 6u * BT ? 6 * BT : 8 * BT;
}

// Number of entries of a sorted list below (k, i).
__device__ __forceinline__ uint32_t count_below(const uint64_t* key, const uint32_t* id,
                                                uint32_t n, uint64_t k, uint32_t i) {
  uint32_t lo = 0, hi = n;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (less(key[mid], id[mid], k, i)) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Number of entries of a sorted list not above (k, i).
__device__ __forceinline__ uint32_t count_not_above(const uint64_t* key, const uint32_t* id,
                                                    uint32_t n, uint64_t k, uint32_t i) {
  uint32_t lo = 0, hi = n;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (!less(k, i, key[mid], id[mid])) lo = mid + 1; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint64_t key_of(const SelArgs& a, uint32_t id) {
  return (uint64_t)a.priority[id] << 32 | (uint32_t)a.length[id];
}

// Output of entry idx of C (idx < nc) or of O (idx - nc), given both sorted
// and dec[i] = kept (decoding, or every, when the most urgent entry is in
// prefill) members of C before index i, for i <= nc. M = kept members of C
// and O merged by key; the batch is M's first b; pushed back are C's
// filtered members and M beyond b, merged by key.
template <typename D>
__device__ __forceinline__ void select_place(const SelArgs& a, const uint64_t* ckey,
                                             const uint32_t* cid, uint32_t nc,
                                             const uint64_t* okey, const uint32_t* oid,
                                             uint32_t no, const D* dec, uint32_t idx) {
  // (|M| < 2^31: a larger b places the same way)
  const uint32_t b = (uint32_t)min(a.b, (int64_t)1 << 31);
  // members of M below (k, i): kept members of C and members of O
  auto m_below = [&](uint64_t k, uint32_t i) {
    const uint32_t c = count_below(ckey, cid, nc, k, i);
    return (uint32_t)dec[c] + count_below(okey, oid, no, k, i);
  };
  // filtered (prefill) members of C below (k, i)
  auto pre_below = [&](uint64_t k, uint32_t i) {
    const uint32_t c = count_below(ckey, cid, nc, k, i);
    return c - (uint32_t)dec[c];
  };
  auto place_m = [&](uint32_t q, uint32_t id, uint64_t k) {  // q = position in M
    if (q < b) {
      a.batch[q] = (int32_t)id;
    } else {
      a.pushed[(q - b) + pre_below(k, id)] = (int32_t)id;
    }
  };
  if (idx < nc) {
    const uint32_t i = idx;
    const uint64_t k = ckey[i];
    const uint32_t id = cid[i];
    const uint32_t rk = (uint32_t)dec[i];
    const bool kept = (uint32_t)dec[i + 1] != rk;
    if (kept) {
      place_m(rk + count_below(okey, oid, no, k, id), id, k);
    } else {
      const uint32_t mb = m_below(k, id);
      a.pushed[(i - rk) + (mb > b ? mb - b : 0)] = (int32_t)id;
    }
  } else {
    const uint32_t j = idx - nc;
    const uint64_t k = okey[j];
    const uint32_t id = oid[j];
    place_m(j + (uint32_t)dec[count_below(ckey, cid, nc, k, id)], id, k);
  }
}

// ---- the few that matter: narrowing, and the sort of at most 1024 entries ------
// Both kernels need the order of few of their entries only (the b smallest
// candidates; the victims): a radix select over the packed entries' bits,
// 11 at a time from the top, finds a bound that leaves those and few others,
// and only they are sorted.

constexpr int kPickBits = 11;
constexpr int kPickBins = 1 << kPickBits;
constexpr uint32_t kKept = BT;         // most entries kept (one per thread)
// Entries of the small sort (a wave per run of 64, every run searched by every
// other): its LDS reads grow with the square; 1,000 entries in 16 runs took
// 14 us, the radix sort of 1024 8 us. Narrowing goes on above this many.
constexpr uint32_t kSmall = BT / 2;
static_assert(kPickBins == 2 * BT, "two bins per thread");

// Rank, length and id of one entry, packed in schedule order: id in wid bits,
// the length in wl, the rank above.
struct Packer {
  uint32_t wid, wl, bits;
  __device__ __forceinline__ uint64_t pack(uint32_t p, uint32_t l, uint32_t id) const {
    return ((((uint64_t)p << wl) | l) << wid) | id;
  }
  __device__ __forceinline__ uint32_t id(uint64_t v) const {
    return (uint32_t)(v & ((1ull << wid) - 1));
  }
  __device__ __forceinline__ uint64_t key(uint64_t v) const {
    const uint64_t k = v >> wid;
    return ((k >> wl) << 32) | (k & ((1ull << wl) - 1));
  }
};

// The packing that holds every id below n_ids and the block's largest rank
// and length. Holds barriers; red: 2 * kSortWaves words.
__device__ __forceinline__ Packer make_packer(int64_t n_ids, uint32_t pmax, uint32_t lmax,
                                              uint32_t* red) {
  const int w = threadIdx.x / kWave;
  pmax = wave_max_u32(pmax);
  lmax = wave_max_u32(lmax);
  if (lane_id() == 0) {
    red[w] = pmax;
    red[kSortWaves + w] = lmax;
  }
  block_sync();
#pragma unroll
  for (int v = 0; v < kSortWaves; ++v) {
    pmax = max(pmax, red[v]);
    lmax = max(lmax, red[kSortWaves + v]);
  }
  block_sync();  // (the words are scratch again)
  Packer pk;
  pk.wid = bit_width32((uint32_t)max(n_ids - 1, (int64_t)1));
  pk.wl = max(bit_width32(lmax), 1u);
  pk.bits = pk.wid + pk.wl + bit_width32(pmax);
  return pk;
}

// Ascending sort of one (value, payload) per lane over the wave: a bitonic
// network of lane exchanges.
__device__ __forceinline__ void wave_sort(uint64_t& v, uint32_t& pay) {
  const int lane = lane_id();
#pragma unroll
  for (int k = 2; k <= kWave; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      const uint64_t o = __shfl_xor((unsigned long long)v, j, kWave);
      const uint32_t op = __shfl_xor(pay, j, kWave);
      const bool up = (lane & k) == 0 || k == kWave;  // this block ascends
      const bool low = (lane & j) == 0;               // this lane keeps the smaller if so
      const bool take = (up == low) ? o < v : v < o;
      v = take ? o : v;
      pay = take ? op : pay;
    }
  }
}

// The rank of this lane's value among the runs of 64 sorted values
// buf[64 * r0 .. 64 * r1), its own run `mine` at its lane's place. Equal
// values (none for distinct ids) rank by run, so that ranks are distinct.
__device__ __forceinline__ uint32_t rank_in_runs(const uint64_t* buf, int r0, int r1, int mine,
                                                 uint64_t v) {
  uint32_t rank = (uint32_t)lane_id();
  for (int r = r0; r < r1; ++r) {
    if (r == mine) continue;  // (uniform)
    const uint64_t* run = buf + r * kWave;
    const bool ties = r < mine;
    uint32_t p = 0;
#pragma unroll
    for (int step = kWave / 2; step > 0; step >>= 1) {
      const uint64_t x = run[p + step - 1];
      if (x < v || (ties && x == v)) p += step;
    }
    const uint64_t x = run[p];
    if (x < v || (ties && x == v)) ++p;
    rank += p;
  }
  return rank;
}

// Places for the kept entries of the block's E rounds in LDS arrays (order
// arbitrary), one counter addition per wave: place[r] is the place of this
// lane's entry of round r, if kept.
template <int E>
__device__ __forceinline__ void append_places(const bool (&keep)[E], uint32_t* count,
                                              uint32_t (&place)[E]) {
  uint32_t n = 0;  // (uniform)
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint64_t m = __ballot(keep[r]);
    place[r] = n + (uint32_t)__popcll(m & lanes_below());
    n += (uint32_t)__popcll(m);
  }
  uint32_t base = 0;
  if (lane_id() == 0 && n) base = atomicAdd(count, n);
  base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
  for (int r = 0; r < E; ++r) place[r] += base;
}

struct Pick {
  uint32_t bin, before, count;  // the bin, entries in the bins before it, entries in it
  uint64_t weight_before;
  uint32_t found;
};

struct SelectShared {
  uint64_t ckey[kCandCap];
  uint32_t cid[kCandCap];
  uint64_t okey[kSelectCap];
  uint32_t oid[kSelectCap];
  union {  // (the sorts are done before dec_excl is written)
    uint16_t dec_excl[kSelectCap + 1];  // kept members of C before each index (<= 4096)
    SortScratch sort;
    uint32_t hist[kPickBins];
  };
  uint32_t scan32[BT / kWave + 1];
  uint32_t red[2 * kSortWaves];
  Pick pick;
  uint32_t bad, count;
};

// One workgroup: the b smallest candidates (narrowed, then sorted), the
// ongoing requests sorted, the stage filter and the merged places. What
// bounds it is its chain of dependent steps: two gathers (ids, then their
// ranks and lengths), about ten barriers per narrowing round and sort, one
// gather of stages. Sorting all 4,352 candidates of an iteration over 2^20
// requests in six radix passes took 45 us; narrowing them to about 260 first,
// 16 us (over 2^26, where the gathers miss the caches, 57 and 23).
__global__ __launch_bounds__(BT) void b_select(SelArgs a) {
  __shared__ SelectShared sh;
  constexpr int EC = kCandCap / BT;
  const uint32_t t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane((int)(t / kWave));
  const uint32_t nh = (uint32_t)min(a.b, a.n_heap);
  const uint32_t nc_in = nh + (uint32_t)a.n_buffer;
  const uint32_t no = (uint32_t)a.n_ongoing;
  if (t == 0) {
    sh.bad = 0;
    sh.count = 0;
    a.flags[0] = 0;
    wait_stores();  // before any other thread's error bit
  }
  const uint32_t need = min((uint32_t)min(a.b, (int64_t)kCandCap), nc_in);
  // The lists are sorted whole where they are known to need it: more than kKept
  // of either to order, or between 513 and 1024 of at most 2048 candidates,
  // where narrowing costs what it saves.
  const bool whole = need > kKept || no > kKept ||
                     (need > kSmall && nc_in > kKept && nc_in <= 2 * kKept);
  uint32_t m = nc_in;
  bool kept = false;
  if (!whole) {
    // the ids of both lists, then their ranks and lengths, each in one go
    int32_t ci[EC];
#pragma unroll
    for (int r = 0; r < EC; ++r) {
      const uint32_t i = r * BT + t;
      ci[r] = 0;
      if (i < nc_in) ci[r] = i < nh ? a.heap_order[i] : a.buffer[i - nh];
    }
    static_assert(kKept == BT, "an ongoing request per thread");
    const int32_t oi = t < no ? a.ongoing[t] : 0;
    const bool o_ok = t < no && oi >= 0 && oi < a.n_ids;
    bool bad = t < no && !o_ok;
    uint32_t cp[EC], cl[EC];
#pragma unroll
    for (int r = 0; r < EC; ++r) {
      const bool in = (uint32_t)(r * BT + t) < nc_in, ok = in && ci[r] >= 0 && ci[r] < a.n_ids;
      bad |= in && !ok;
      cp[r] = ok ? a.priority[ci[r]] : 0u;
      cl[r] = ok ? (uint32_t)a.length[ci[r]] : 0u;
    }
    const uint32_t op = o_ok ? a.priority[oi] : 0u;
    const uint32_t ol = o_ok ? (uint32_t)a.length[oi] : 0u;
    uint32_t pmax = op, lmax = ol;
#pragma unroll
    for (int r = 0; r < EC; ++r) {
      pmax = max(pmax, cp[r]);
      lmax = max(lmax, cl[r]);
    }
    block_sync();
    if (bad) sh.bad = 1u;
    const Packer pk = make_packer(a.n_ids, pmax, lmax, sh.red);  // (holds barriers)
    uint64_t cv[EC];  // the candidates, packed (meaningless beyond 63 bits, then not used)
#pragma unroll
    for (int r = 0; r < EC; ++r) cv[r] = pk.pack(cp[r], cl[r], (uint32_t)ci[r]);
    const uint64_t mine_o = pk.pack(op, ol, (uint32_t)oi);
    if (sh.bad) {
      if (t == 0) {
        atomicOr(a.flags, kFlagInval);
        a.counts[0] = a.counts[1] = 0;
      }
      return;
    }
    m = nc_in;  // candidates kept for the sort
    uint32_t top_shift = pk.bits;  // kept: (v >> top_shift) <= bound
    uint64_t bound = 0;
    kept = pk.bits <= 63;
    if (need == 0) m = 0;
    if (kept && need > 0 && nc_in > (need <= kSmall ? kSmall : kKept)) {
      uint32_t below = 0;  // candidates below the bound's group
      while (top_shift > 0) {
        const uint32_t sh_ = top_shift > kPickBits ? top_shift - kPickBits : 0u;
        const uint32_t mask = (1u << (top_shift - sh_)) - 1;
        sh.hist[2 * t] = 0;
        sh.hist[2 * t + 1] = 0;
        block_sync();
#pragma unroll
        for (int r = 0; r < EC; ++r) {
          if ((uint32_t)(r * BT + t) < nc_in && (cv[r] >> top_shift) == bound)
            atomicAdd(&sh.hist[(uint32_t)(cv[r] >> sh_) & mask], 1u);
        }
        block_sync();
        const uint32_t c0 = sh.hist[2 * t], c1 = sh.hist[2 * t + 1];
        uint32_t all;
        const uint32_t ex = below + block_excl_scan_u32<BT>(c0 + c1, sh.scan32, all);
        if (ex < need && need <= ex + c0) sh.pick = {2 * t, ex, c0, 0, 1};
        else if (ex + c0 < need && need <= ex + c0 + c1) sh.pick = {2 * t + 1, ex + c0, c1, 0, 1};
        block_sync();
        bound = (bound << (top_shift - sh_)) | sh.pick.bin;
        below = sh.pick.before;
        m = below + sh.pick.count;
        top_shift = sh_;
        // (uniform) above kSmall the radix sort of one entry per thread takes any
        // number up to kKept
        if (m <= (need <= kSmall ? kSmall : kKept)) break;
        block_sync();  // the pick is read before the next round's
      }
    }
    kept = kept && m <= kKept;
    if (kept) {
      // The kept candidates to the first runs of ckey, the ongoing ones to okey:
      // lists of at most kSmall entries as packed values in runs of 64, waves
      // 0 .. 7 the candidates and 8 .. 15 the ongoing ones, longer ones as the
      // radix sort takes them.
      const bool small_c = m <= kSmall, small_o = no <= kSmall;
      sh.ckey[t] = ~0ull;
      sh.okey[t] = t < no && small_o ? mine_o : ~0ull;
      block_sync();
      bool keep[EC];
      uint32_t place[EC];
#pragma unroll
      for (int r = 0; r < EC; ++r)
        keep[r] = m > 0 && (uint32_t)(r * BT + t) < nc_in && (cv[r] >> top_shift) <= bound;
      append_places(keep, &sh.count, place);
#pragma unroll
      for (int r = 0; r < EC; ++r) {
        if (keep[r] && place[r] < kKept) {
          sh.ckey[place[r]] = small_c ? cv[r] : pk.key(cv[r]);
          if (!small_c) sh.cid[place[r]] = pk.id(cv[r]);
        }
      }
      if (!small_o && t < no) {
        sh.okey[t] = pk.key(mine_o);
        sh.oid[t] = pk.id(mine_o);
      }
      block_sync();
      const bool of_c = w < kSortWaves / 2;
      const int mine = of_c ? w : w - kSortWaves / 2;  // this wave's run
      const uint32_t count = of_c ? m : no;
      const int runs = (int)((count + kWave - 1) / kWave);
      const bool used = (of_c ? small_c : small_o) && mine < runs;  // (uniform in the wave)
      uint64_t* buf = of_c ? sh.ckey : sh.okey;
      uint64_t v = 0;
      if (used) {
        v = buf[mine * kWave + lane_id()];
        uint32_t none = 0;
        wave_sort(v, none);
        buf[mine * kWave + lane_id()] = v;
      }
      block_sync();
      const uint32_t rank = used ? rank_in_runs(buf, 0, runs, mine, v) : ~0u;
      block_sync();  // the runs are read before the sorted lists are written
      if (rank < count) {
        buf[rank] = pk.key(v);
        (of_c ? sh.cid : sh.oid)[rank] = pk.id(v);
      }
      block_sync();
      if (!small_c) {  // (the sort's padding: entries m .. 1023)
        if (t >= m) sh.cid[t] = ~0u;
        block_sync();
        block_sort<1, false>(sh.ckey, sh.cid, nullptr, m, sh.sort);
      }
      if (!small_o) {
        if (t >= no) sh.oid[t] = ~0u;
        block_sync();
        block_sort<1, false>(sh.okey, sh.oid, nullptr, no, sh.sort);
      }
    }
  }
  if (!kept) {
    // (also when more candidates tie than the kept list takes, and ids, lengths
    // and ranks beyond 63 bits)
    m = nc_in;
    const uint32_t NC = sort_size<false>(nc_in), NO = sort_size<false>(no);
    block_sync();
    bool bad = false;
    for (uint32_t i = t; i < NC; i += BT) {
      const int32_t v = i >= nc_in ? 0 : i < nh ? a.heap_order[i] : a.buffer[i - nh];
      const bool ok = i < nc_in && v >= 0 && v < a.n_ids;
      bad |= i < nc_in && !ok;
      sh.ckey[i] = ok ? key_of(a, (uint32_t)v) : ~0ull;
      sh.cid[i] = ok ? (uint32_t)v : ~0u;
    }
    for (uint32_t i = t; i < NO; i += BT) {
      const int32_t v = i < no ? a.ongoing[i] : 0;
      const bool ok = i < no && v >= 0 && v < a.n_ids;
      bad |= i < no && !ok;
      sh.okey[i] = ok ? key_of(a, (uint32_t)v) : ~0ull;
      sh.oid[i] = ok ? (uint32_t)v : ~0u;
    }
    if (bad) sh.bad = 1u;
    block_sync();
    if (sh.bad) {
      if (t == 0) {
        atomicOr(a.flags, kFlagInval);
        a.counts[0] = a.counts[1] = 0;
      }
      return;
    }
    sort_pairs<false>(sh.ckey, sh.cid, nullptr, nc_in, sh.sort);
    sort_pairs<false>(sh.okey, sh.oid, nullptr, no, sh.sort);
  }
  const uint32_t nc = min((uint32_t)min(a.b, (int64_t)kCandCap), m);  // C = the first nc
  if (nc == 0 && no == 0) {
    if (t == 0) a.counts[0] = a.counts[1] = 0;
    return;
  }
  // the most urgent of C and O decides whether prefill candidates stay
  bool top_in_c = nc > 0 && (no == 0 || less(sh.ckey[0], sh.cid[0], sh.okey[0], sh.oid[0]));
  const uint32_t top = top_in_c ? sh.cid[0] : sh.oid[0];
  const uint8_t top_stage = a.stage[top];
  // decoding (kept) members of C before each index, a round of the block at a
  // time
  uint32_t ndec = 0;
  for (uint32_t i0 = 0; i0 < nc; i0 += BT) {
    const uint32_t i = i0 + t;
    const uint8_t st = i < nc ? a.stage[sh.cid[i]] : 0;
    const uint32_t kept = i < nc && (top_stage == 0 || st != 0) ? 1u : 0u;
    uint32_t all;
    const uint32_t ex = ndec + block_excl_scan_u32<BT>(kept, sh.scan32, all);
    if (i < nc) sh.dec_excl[i] = (uint16_t)ex;
    ndec += all;
  }
  if (t == 0) sh.dec_excl[nc] = (uint16_t)ndec;
  block_sync();
  const uint32_t nm = ndec + no;  // |M|
  const uint32_t b = (uint32_t)min(a.b, (int64_t)1 << 31);
  const uint32_t npre = nc - ndec;
  const uint32_t over = nm > b ? nm - b : 0;  // M beyond the batch
  for (uint32_t i = t; i < nc + no; i += BT)
    select_place(a, sh.ckey, sh.cid, nc, sh.okey, sh.oid, no, sh.dec_excl, i);
  if (t == 0) {
    a.counts[0] = min(b, nm);
    a.counts[1] = npre + over;
  }
}

// Victims after each incoming request j: the first k of the eviction order
// whose KV prefix psum[k - 1] reaches need_j = usage + (demands 0..j) -
// capacity (all nr if none does); then the victims of the last request, in
// eviction order, from eorder. `last` is a u32 of LDS.
__device__ __forceinline__ void evict_demands(const EvictArgs& a, const uint64_t* psum,
                                              const uint32_t* eorder, uint32_t nr,
                                              uint64_t* scan64, uint32_t* last) {
  const uint32_t t = threadIdx.x;
  bool bad = false;
  int64_t carry = 0;  // demands of the earlier chunks
  for (int64_t j0 = 0; j0 < a.n_demands; j0 += BT) {
    const int64_t j = j0 + t;
    const int64_t s = j < a.n_demands ? a.demands[j] : 0;
    bad |= s < 0;
    uint64_t tot;
    const uint64_t before = block_excl_scan_u64<BT>(s < 0 ? 0 : (uint64_t)s, scan64, tot);
    const int64_t need = a.usage + carry + (int64_t)before + (s < 0 ? 0 : s) - a.capacity;
    uint32_t k = 0;
    if (need > 0) {
      uint32_t lo = 0, hi = nr;  // first index whose inclusive sum reaches need
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((int64_t)psum[mid] >= need) hi = mid; else lo = mid + 1;
      }
      k = lo < nr ? lo + 1 : nr;
    }
    if (j < a.n_demands) a.upto[j] = k;
    if (j == a.n_demands - 1) *last = k;
    carry += (int64_t)tot;  // (every thread holds the chunk's total)
    block_sync();
  }
  if (__ballot(bad) && lane_id() == 0) atomicOr(a.flags, kFlagRange);
  const uint32_t k_last = a.n_demands > 0 ? *last : 0;
  for (uint32_t e = t; e < k_last; e += BT) a.victims[e] = (int32_t)eorder[e];
}

struct EvictShared {
  uint64_t key[kEvictCap];
  uint32_t id[kEvictCap];
  uint32_t src[kEvictCap];    // index into the caller's cached / kv arrays
  uint64_t scan64[BT / kWave + 1];
  uint32_t scan32[BT / kWave + 1];
  union {
    SortScratch sort;
    struct {
      uint64_t kv[kPickBins];  // KV of the entries of a bin
      uint32_t n[kPickBins];   // their number
    } hist;
  };
  uint32_t red[2 * kSortWaves];
  Pick pick;
  uint32_t bad, count;
};

// One workgroup. The victims are the last entries of the schedule order whose
// KV sizes cover the last demand's need: a radix select weighted by KV finds
// a bound that keeps those and few others, and only they are sorted (all of
// them, as before, when the need takes everything or more than fit the small
// sort). Sorting the 8,192 cached requests of an iteration over 2^20 requests
// took 53 us, this 21 us (over 2^26, where the gathers miss the caches, 71 and
// 32).
__global__ __launch_bounds__(BT) void b_evict(EvictArgs a) {
  __shared__ EvictShared sh;
  constexpr int E = kEvictCap / BT;
  const uint32_t t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane((int)(t / kWave));
  const uint32_t nr = (uint32_t)a.n_cached;
  if (t == 0) {
    sh.bad = 0;
    sh.count = 0;
    a.flags[0] = 0;
    wait_stores();  // before any other thread's error bit
  }
  // Up to kKept entries the radix sort takes 8 us; narrowing pays there only when
  // few victims are likely, about one per demand.
  const bool whole = nr > kSmall && nr <= kKept && 2 * a.n_demands > nr;
  uint32_t m = nr;
  bool packed = false;
  if (!whole) {
    // ids and KV sizes, the demands' sum, then ranks and lengths
    int32_t ci[E];
    int64_t kv[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t i = r * BT + t;
      ci[r] = i < nr ? a.cached[i] : 0;
      kv[r] = i < nr ? a.kv[i] : 0;
    }
    uint64_t want = 0;  // (negative demands end in an error, whatever they select)
    for (int64_t j = t; j < a.n_demands; j += BT) want += (uint64_t)max(a.demands[j], (int64_t)0);
    uint32_t bad = 0, cp[E], cl[E], pmax = 0, lmax = 0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool in = (uint32_t)(r * BT + t) < nr, ok = in && ci[r] >= 0 && ci[r] < a.n_ids;
      if (in && !ok) bad |= 1u;
      else if (kv[r] < 0) bad |= 2u;  // 2: negative KV size
      cp[r] = ok ? a.priority[ci[r]] : 0u;
      cl[r] = ok ? (uint32_t)a.length[ci[r]] : 0u;
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      pmax = max(pmax, cp[r]);
      lmax = max(lmax, cl[r]);
    }
    block_sync();
    if (bad) atomicOr(&sh.bad, bad);
    uint64_t total;
    (void)block_excl_scan_u64<BT>(want, sh.scan64, total);
    const Packer pk = make_packer(a.n_ids, pmax, lmax, sh.red);  // (holds barriers)
    uint64_t cv[E];  // packed (meaningless beyond 63 bits, then not used)
#pragma unroll
    for (int r = 0; r < E; ++r) cv[r] = pk.pack(cp[r], cl[r], (uint32_t)ci[r]);
    if (sh.bad) {
      if (t == 0) atomicOr(a.flags, (sh.bad & 1u) ? kFlagInval : kFlagRange);
      return;
    }
    const int64_t need = a.usage + (int64_t)total - a.capacity;
    // kept: (v >> low_shift) >= bound, the entries that leave first
    m = nr;
    uint32_t low_shift = min(pk.bits, 63u);
    uint64_t bound = 0;
    if (need <= 0) {
      m = 0;
      bound = ~0ull;  // (none)
    } else if (pk.bits <= 63 && nr > kSmall) {
      uint64_t freed = 0;  // KV of the entries above the bound's group
      uint32_t above = 0;  // their number
      while (low_shift > 0) {
        const uint32_t sh_ = low_shift > kPickBits ? low_shift - kPickBits : 0u;
        const uint32_t mask = (1u << (low_shift - sh_)) - 1;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          sh.hist.kv[2 * t + k] = 0;
          sh.hist.n[2 * t + k] = 0;
        }
        if (t == 0) sh.pick.found = 0;
        block_sync();
#pragma unroll
        for (int r = 0; r < E; ++r) {
          if ((uint32_t)(r * BT + t) < nr && (cv[r] >> low_shift) == bound) {
            const uint32_t d = (uint32_t)(cv[r] >> sh_) & mask;
            atomicAdd(reinterpret_cast<unsigned long long*>(&sh.hist.kv[d]),
                      (unsigned long long)kv[r]);
            atomicAdd(&sh.hist.n[d], 1u);
          }
        }
        block_sync();
        // bins from the top: thread t takes bins 2047 - 2t and 2046 - 2t
        const uint32_t b0 = kPickBins - 1 - 2 * t, b1 = b0 - 1;
        const uint64_t k0 = sh.hist.kv[b0], k1 = sh.hist.kv[b1];
        const uint32_t n0 = sh.hist.n[b0], n1 = sh.hist.n[b1];
        uint64_t all;
        uint32_t alln;
        const uint64_t ex = freed + block_excl_scan_u64<BT>(k0 + k1, sh.scan64, all);
        const uint32_t en = above + block_excl_scan_u32<BT>(n0 + n1, sh.scan32, alln);
        const uint64_t nd = (uint64_t)need;
        if (ex < nd && nd <= ex + k0) sh.pick = {b0, en, n0, ex, 1};
        else if (ex + k0 < nd && nd <= ex + k0 + k1) sh.pick = {b1, en + n0, n1, ex + k0, 1};
        block_sync();
        if (!sh.pick.found) break;  // (uniform; first round only) everything leaves
        bound = (bound << (low_shift - sh_)) | sh.pick.bin;
        freed = sh.pick.weight_before;
        above = sh.pick.before;
        m = above + sh.pick.count;
        low_shift = sh_;
        // (uniform) done, or more leave for certain than the small sort takes and
        // the radix sort of those would be as wide as of all kept
        if (m <= kSmall || (above >= kSmall && sort_size<true>(above + 1) == sort_size<true>(m)))
          break;
        block_sync();  // the pick is read before the next round's
      }
    }
    bool keep[E];
    uint32_t place[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
      keep[r] = (uint32_t)(r * BT + t) < nr && (cv[r] >> low_shift) >= bound;
    const bool small = pk.bits <= 63 && m <= kSmall;
    if (small) {
      // runs of 64 at the start of key, the kept entries' KV sizes after them,
      // then the sizes in eviction order
      uint64_t* kept_kv = sh.key + BT;
      uint64_t* order_kv = sh.key + 2 * BT;
      sh.key[t] = ~0ull;
      block_sync();
      append_places(keep, &sh.count, place);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        if (keep[r] && place[r] < kSmall) {
          sh.key[place[r]] = cv[r];
          kept_kv[place[r]] = (uint64_t)kv[r];
        }
      }
      block_sync();
      const int runs = (int)((m + kWave - 1) / kWave);
      uint64_t v = sh.key[t];
      uint32_t from = t;
      if (w < runs) {
        wave_sort(v, from);
        sh.key[t] = v;
      }
      block_sync();
      if (w < runs) {
        const uint32_t rank = rank_in_runs(sh.key, 0, runs, w, v);
        if (rank < m) {
          order_kv[m - 1 - rank] = kept_kv[from];
          sh.id[m - 1 - rank] = pk.id(v);
        }
      }
      block_sync();
      const uint64_t x = t < m ? order_kv[t] : 0;
      uint64_t all;
      const uint64_t ex = block_excl_scan_u64<BT>(x, sh.scan64, all);
      sh.key[t] = ex + x;  // KV evicted by the first t + 1 victims
      block_sync();
      evict_demands(a, sh.key, sh.id, m, sh.scan64, &sh.bad);
      return;
    }
    // more victims than the small sort holds
    packed = pk.bits <= 63;
    if (packed) {
      append_places(keep, &sh.count, place);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        if (keep[r]) {
          sh.key[place[r]] = pk.key(cv[r]);
          sh.id[place[r]] = pk.id(cv[r]);
          sh.src[place[r]] = (uint32_t)(r * BT + t);
        }
      }
    }
  }
  if (!packed) {  // all of them (also when they do not pack)
    m = nr;
    block_sync();
    uint32_t bad = 0;
    for (uint32_t i = t; i < nr; i += BT) {
      const int32_t v = a.cached[i];
      const bool ok = v >= 0 && v < a.n_ids;
      if (!ok) bad |= 1u;
      else if (a.kv[i] < 0) bad |= 2u;  // 2: negative KV size
      sh.key[i] = ok ? (uint64_t)a.priority[v] << 32 | (uint32_t)a.length[v] : 0ull;
      sh.id[i] = (uint32_t)v;
      sh.src[i] = i;
    }
    if (bad) atomicOr(&sh.bad, bad);
    block_sync();
    if (sh.bad) {
      if (t == 0) atomicOr(a.flags, (sh.bad & 1u) ? kFlagInval : kFlagRange);
      return;
    }
  }
  for (uint32_t i = m + t; i < sort_size<true>(m); i += BT) {
    sh.key[i] = ~0ull;
    sh.id[i] = ~0u;
    sh.src[i] = 0;
  }
  block_sync();
  sort_pairs<true>(sh.key, sh.id, sh.src, m, sh.sort);
  // KV sizes in eviction order (the sorted order read backwards), inclusive
  // prefix sums over a contiguous chunk per thread, kept in sh.key
  constexpr uint32_t PER = (kEvictCap + BT - 1) / BT;
  const uint32_t e0 = min(m, t * PER), e1 = min(m, e0 + PER);
  uint64_t kvs[PER];
  uint64_t mine = 0;
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint32_t e = e0 + u;
    kvs[u] = e < e1 ? (uint64_t)a.kv[sh.src[m - 1 - e]] : 0;
    mine += kvs[u];
  }
  uint32_t ids[PER];
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) ids[u] = e0 + u < e1 ? sh.id[m - 1 - (e0 + u)] : 0;
  uint64_t sum;
  uint64_t run = block_excl_scan_u64<BT>(mine, sh.scan64, sum);  // (ends with a barrier)
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    if (e0 + u < e1) {
      run += kvs[u];
      sh.key[e0 + u] = run;      // KV evicted by the first e0+u+1 victims
      sh.id[e0 + u] = ids[u];    // the eviction order
    }
  }
  block_sync();
  evict_demands(a, sh.key, sh.id, m, sh.scan64, &sh.bad);
}

// ---- lists beyond one workgroup's LDS -----------------------------------------
// The lists are sorted in chunks of kWideChunk entries, one workgroup each
// (the LDS sort above), and the sorted runs are then merged pairwise, one
// launch per round: an entry's place in the merged run is its index in its
// own run plus the number of entries of the other run before it, found by
// binary search (entries of the first run go before equal entries of the
// second, so the merge keeps the order of equal keys).

__device__ __forceinline__ int64_t list_size(const WideList& l) { return l.n0 + l.n1; }
__device__ __forceinline__ int64_t list_chunks(const WideList& l) {
  return (list_size(l) + kWideChunk - 1) / kWideChunk;
}

template <bool PAY>
struct ChunkShared {
  uint64_t key[kWideChunk];
  uint32_t id[kWideChunk];
  uint32_t pay[PAY ? kWideChunk : 1];
  SortScratch sort;
};

// PAY (eviction): entries carry their index in the caller's arrays, and a
// negative KV size is a range error. Ids outside [0, n_ids) are reported and
// sort last; the outputs of a call with an error are not written.
template <bool PAY>
__global__ __launch_bounds__(BT) void w_chunk_sort(WideSort a) {
  __shared__ ChunkShared<PAY> sh;
  __shared__ uint32_t s_bad;
  int64_t c = blockIdx.x;
  const bool second = a.nlists > 1 && c >= list_chunks(a.list[0]);
  const WideList l = second ? a.list[1] : a.list[0];
  if (second) c -= list_chunks(a.list[0]);
  const int64_t c0 = c * kWideChunk;
  const uint32_t nc = (uint32_t)min((int64_t)kWideChunk, list_size(l) - c0);
  const uint32_t t = threadIdx.x;
  if (t == 0) s_bad = 0;
  block_sync();
  uint32_t bad = 0;
  for (uint32_t i = t; i < nc; i += BT) {
    const int64_t gi = c0 + i;
    const int32_t v = gi < l.n0 ? l.src0[gi] : l.src1[gi - l.n0];
    uint64_t k = ~0ull;
    uint32_t id = ~0u;
    if (v < 0 || v >= a.n_ids) {
      bad |= 1u;
    } else if (PAY && a.kv[gi] < 0) {
      bad |= 2u;  // negative KV size
    } else {
      id = (uint32_t)v;
      k = (uint64_t)a.priority[id] << 32 | (uint32_t)a.length[id];
    }
    sh.key[i] = k;
    sh.id[i] = id;
    if (PAY) sh.pay[i] = (uint32_t)gi;
  }
  if (bad) atomicOr(&s_bad, bad);
  block_sync();
  if (t == 0 && s_bad) atomicOr(a.flags, (s_bad & 1u) ? kFlagInval : kFlagRange);
  block_sort<kWideChunk / BT, PAY>(sh.key, sh.id, sh.pay, nc, sh.sort);
  for (uint32_t i = t; i < nc; i += BT) {
    const int64_t o = l.base + c0 + i;
    a.key[0][o] = sh.key[i];
    a.id[0][o] = sh.id[i];
    if (PAY) a.pay[0][o] = sh.pay[i];
  }
}

// One merge round: runs of `run` entries (sorted) in buffer `from` become
// runs of 2 * run in the other buffer.
template <bool PAY>
__global__ __launch_bounds__(BT) void w_merge(WideSort a, int64_t run, int from) {
  const uint64_t* kin = a.key[from];
  const uint32_t* iin = a.id[from];
  const int to = from ^ 1;
  for (int64_t g = (int64_t)blockIdx.x * BT + threadIdx.x; g < a.total;
       g += (int64_t)gridDim.x * BT) {
    const bool second = a.nlists > 1 && g >= a.list[1].base;
    const int64_t base = second ? a.list[1].base : a.list[0].base;
    const int64_t n = list_size(second ? a.list[1] : a.list[0]);
    const int64_t i = g - base;
    const int64_t ps = i / (2 * run) * (2 * run);   // the pair's first entry
    const int64_t am = min(ps + run, n);             // end of its first run
    const int64_t be = min(ps + 2 * run, n);         // end of its second run
    const uint64_t k = kin[g];
    const uint32_t id = iin[g];
    int64_t pos;
    if (i < am)
      pos = i + count_below(kin + base + am, iin + base + am, (uint32_t)(be - am), k, id);
    else
      pos = ps + (i - am) + count_not_above(kin + base + ps, iin + base + ps, (uint32_t)(am - ps),
                                            k, id);
    a.key[to][base + pos] = k;
    a.id[to][base + pos] = id;
    if (PAY) a.pay[to][base + pos] = a.pay[from][g];
  }
}

// Selection on the sorted candidates (list 0; C = their first nc) and ongoing
// requests (list 1): the stage filter, the kept members of C before each
// index (dec), and the counts.
__global__ __launch_bounds__(BT) void w_select_scan(SelArgs a, WideSort w, int buf,
                                                    uint32_t* dec) {
  __shared__ uint32_t scan32[BT / kWave + 1];
  const uint32_t t = threadIdx.x;
  if (load_agent(a.flags) != 0) {  // an id outside [0, n_ids)
    if (t == 0) a.counts[0] = a.counts[1] = 0;
    return;
  }
  const uint64_t* ck = w.key[buf];
  const uint32_t* ci = w.id[buf];
  const uint64_t* ok = ck + w.list[1].base;
  const uint32_t* oi = ci + w.list[1].base;
  const uint32_t nc = (uint32_t)min(a.b, list_size(w.list[0]));
  const uint32_t no = (uint32_t)list_size(w.list[1]);
  if (nc == 0 && no == 0) {
    if (t == 0) a.counts[0] = a.counts[1] = 0;
    return;
  }
  const bool top_in_c = nc > 0 && (no == 0 || less(ck[0], ci[0], ok[0], oi[0]));
  const bool keep_all = a.stage[top_in_c ? ci[0] : oi[0]] == 0;
  const uint32_t per = (nc + BT - 1) / BT;
  const uint32_t c0 = min(nc, t * per), c1 = min(nc, c0 + per);
  uint32_t mine = 0;
  for (uint32_t i = c0; i < c1; ++i) mine += (keep_all || a.stage[ci[i]] != 0) ? 1u : 0u;
  uint32_t ndec;
  uint32_t run = block_excl_scan_u32<BT>(mine, scan32, ndec);
  for (uint32_t i = c0; i < c1; ++i) {
    dec[i] = run;
    run += (keep_all || a.stage[ci[i]] != 0) ? 1u : 0u;
  }
  if (t == 0) {
    dec[nc] = ndec;
    const uint64_t b = (uint64_t)a.b, nm = (uint64_t)ndec + no;
    a.counts[0] = (int64_t)min(b, nm);
    a.counts[1] = (int64_t)((nc - ndec) + (nm > b ? nm - b : 0));
  }
}

__global__ __launch_bounds__(BT) void w_select_place(SelArgs a, WideSort w, int buf,
                                                     const uint32_t* dec) {
  if (load_agent(a.flags) != 0) return;
  const uint64_t* ck = w.key[buf];
  const uint32_t* ci = w.id[buf];
  const uint32_t nc = (uint32_t)min(a.b, list_size(w.list[0]));
  const uint32_t no = (uint32_t)list_size(w.list[1]);
  for (uint32_t g = blockIdx.x * BT + threadIdx.x; g < nc + no; g += gridDim.x * BT)
    select_place(a, ck, ci, nc, ck + w.list[1].base, ci + w.list[1].base, no, dec, g);
}

// Eviction on the sorted cached requests: KV prefix sums in eviction order
// (the sorted order read backwards) and the eviction order itself, then the
// victims of every incoming request.
__global__ __launch_bounds__(BT) void w_evict(EvictArgs a, WideSort w, int buf, uint64_t* psum,
                                              uint32_t* eorder) {
  __shared__ uint64_t scan64[BT / kWave + 1];
  __shared__ uint32_t last;
  if (load_agent(a.flags) != 0) return;  // a bad id or KV size
  const uint32_t t = threadIdx.x;
  const uint32_t nr = (uint32_t)a.n_cached;
  const uint32_t* id = w.id[buf];
  const uint32_t* src = w.pay[buf];
  const uint32_t per = (nr + BT - 1) / BT;
  const uint32_t e0 = min(nr, t * per), e1 = min(nr, e0 + per);
  uint64_t mine = 0;
  for (uint32_t e = e0; e < e1; ++e) mine += (uint64_t)a.kv[src[nr - 1 - e]];
  uint64_t total;
  uint64_t run = block_excl_scan_u64<BT>(mine, scan64, total);
  for (uint32_t e = e0; e < e1; ++e) {
    run += (uint64_t)a.kv[src[nr - 1 - e]];
    psum[e] = run;            // KV evicted by the first e + 1 victims
    eorder[e] = id[nr - 1 - e];
  }
  block_sync();  // (orders this workgroup's global writes before its reads)
  evict_demands(a, psum, eorder, nr, scan64, &last);
}

// Chunk sort and merge rounds; returns the buffer that holds the result.
template <bool PAY>
int wide_sort(const WideSort& w, hipStream_t st) {
  int64_t chunks = 0, longest = 0;
  for (int l = 0; l < w.nlists; ++l) {
    const int64_t n = w.list[l].n0 + w.list[l].n1;
    chunks += (n + kWideChunk - 1) / kWideChunk;
    longest = std::max(longest, n);
  }
  if (chunks == 0) return 0;
  hipLaunchKernelGGL(w_chunk_sort<PAY>, dim3((unsigned)chunks), dim3(BT), 0, st, w);
  const unsigned grid = (unsigned)std::min<int64_t>((w.total + BT - 1) / BT, 4096);
  int from = 0;
  for (int64_t run = kWideChunk; run < longest; run *= 2) {
    hipLaunchKernelGGL(w_merge<PAY>, dim3(grid), dim3(BT), 0, st, w, run, from);
    from ^= 1;
  }
  return from;
}

}  // namespace

hipError_t launch_select_wide(const SelArgs& a, WideSort w, uint32_t* dec, hipStream_t st) {
  const int buf = wide_sort<false>(w, st);
  hipLaunchKernelGGL(w_select_scan, dim3(1), dim3(BT), 0, st, a, w, buf, dec);
  const int64_t nc = std::min(a.b, w.list[0].n0 + w.list[0].n1);
  const int64_t m = nc + w.list[1].n0 + w.list[1].n1;
  if (m > 0) {
    const unsigned grid = (unsigned)std::min<int64_t>((m + BT - 1) / BT, 4096);
    hipLaunchKernelGGL(w_select_place, dim3(grid), dim3(BT), 0, st, a, w, buf, dec);
  }
  return hipGetLastError();
}

hipError_t launch_evict_wide(const EvictArgs& a, WideSort w, uint64_t* psum, uint32_t* eorder,
                             hipStream_t st) {
  const int buf = wide_sort<true>(w, st);
  hipLaunchKernelGGL(w_evict, dim3(1), dim3(BT), 0, st, a, w, buf, psum, eorder);
  return hipGetLastError();
}

hipError_t launch_select(const SelArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(b_select, dim3(1), dim3(BT), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_evict_victims(const EvictArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(b_evict, dim3(1), dim3(BT), 0, st, a);
  return hipGetLastError();
}

}  // namespace semsched
