// Tile binning: stable LSD radix sort of the key words on their tile id,
// carrying the record id, with the key count read from device memory (so the
// host never synchronises), and the per-tile [start, end) ranges.  Small
// inputs are latency bound: blocks of 1024 keys, walked once, and the whole
// tile id in one pass where it has at most 12 bits.  Otherwise digits are at
// most 8 bits (256 per pass).
#include <algorithm>

#include "ug_kernels.h"

namespace ug {

constexpr int kSortThreads = 256;
constexpr uint32_t kSortMaxBlocks = 2048;

// Small inputs: up to kSmallKeys keys (by capacity) take blocks of 1024 keys,
// each walked once, and the whole tile id in one pass where it has at most 11
// bits, or 12 up to kWideKeys keys.  Times of the sort's kernels with the
// ranges kernel that one pass does not need (launch gaps included): 11 bits,
// 315 K keys 53 us in two passes with blocks of 2048, 26 so; 950 K keys 53 and
// 37 (the wide histograms' column scan grows with the keys: 15 of the 37);
// 12 bits, 78 K keys 45 and 24, 640 K keys 53 and 48, 950 K keys 54 and 57.
constexpr uint32_t kSmallKeys = 1024u * 1024u, kWideKeys = 512u * 1024u;
constexpr uint32_t kSmallChunk = 1024;

// Contiguous chunk of the n keys owned by block b of G (multiple of 256).
__device__ __forceinline__ void sort_chunk(uint32_t n, uint32_t G, uint32_t b, uint32_t& s, uint32_t& e) {
  uint64_t C = ((uint64_t)n + G - 1) / G;
  C = (C + 255) & ~(uint64_t)255;
  const uint64_t s64 = (uint64_t)b * C;
  s = (uint32_t)(s64 < n ? s64 : n);
  const uint64_t e64 = s64 + C;
  e = (uint32_t)(e64 < n ? e64 : n);
}

// Per-block digit histogram, block-major: cnt[b * D + d] (D digit slots).
template <int D>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const Ctrl* __restrict__ ctrl,
                                                              const uint32_t* __restrict__ keys, uint32_t G,
                                                              int shift, uint32_t dmask, uint32_t* __restrict__ cnt) {
  constexpr int kCopies = D > 256 ? 1 : 4;  // counts per wave where that is cheap
  __shared__ uint32_t h[kCopies][D];
  for (int j = threadIdx.x; j < kCopies * D; j += kSortThreads) (&h[0][0])[j] = 0u;
  __syncthreads();
  uint32_t s, e;
  sort_chunk(ctrl->n_key_eff, G, blockIdx.x, s, e);
  const int copy = kCopies > 1 ? (int)(threadIdx.x >> 6) : 0;
  // eight loads in flight per thread, then their counts
  for (uint32_t i0 = s + threadIdx.x; i0 < e; i0 += 8 * kSortThreads) {
    uint32_t kv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t i = i0 + (uint32_t)(j * kSortThreads);
      kv[j] = i < e ? keys[i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (i0 + (uint32_t)(j * kSortThreads) < e) atomicAdd(&h[copy][(kv[j] >> shift) & dmask], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < D; d += kSortThreads) {
    uint32_t c = h[0][d];
#pragma unroll
    for (int q = 1; q < kCopies; ++q) c += h[q][d];
    cnt[(size_t)blockIdx.x * D + d] = c;
  }
}

// Exclusive scan of every digit's column over the G blocks (in place), and
// the column totals.  A block takes eight neighbouring digits, so a row of
// theirs is 32 bytes; its threads are (row group, digit), each with up to
// kScanRows consecutive rows in flight at once.  Bound by that round trip and
// the one of the stores.  (A block per digit read four bytes of every row:
// 2048 rows of 256 digits 15 us, 11 so.)
constexpr int kScanDigits = 8, kScanGroups = 128;
constexpr int kScanRows = kSortMaxBlocks / kScanGroups;
__global__ __launch_bounds__(kScanDigits* kScanGroups) void k_radix_colscan(uint32_t* __restrict__ cnt, uint32_t G,
                                                                          uint32_t D, uint32_t* __restrict__ coltot) {
  __shared__ uint32_t sh[kScanDigits][kScanGroups + 1];
  const uint32_t d = threadIdx.x % kScanDigits, grp = threadIdx.x / kScanDigits;
  const uint32_t rows = (G + kScanGroups - 1u) / kScanGroups, r0 = grp * rows;
  uint32_t* col = cnt + blockIdx.x * kScanDigits + d;
  uint32_t v[kScanRows];
  uint32_t sum = 0;
#pragma unroll
  for (uint32_t j = 0; j < (uint32_t)kScanRows; ++j) v[j] = j < rows && r0 + j < G ? col[(size_t)(r0 + j) * D] : 0u;
#pragma unroll
  for (int j = 0; j < kScanRows; ++j) sum += v[j];
  sh[d][grp] = sum;
  __syncthreads();
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  if (wave < (uint32_t)kScanDigits) {
    static_assert(kScanGroups == 128, "two groups per lane");
    const uint32_t a = sh[wave][2 * lane], b = sh[wave][2 * lane + 1];
    const uint32_t incl = wave_incl_sum(a + b);
    sh[wave][2 * lane] = incl - b - a;
    sh[wave][2 * lane + 1] = incl - b;
    if (lane == 63) coltot[blockIdx.x * kScanDigits + wave] = incl;
  }
  __syncthreads();
  uint32_t run = sh[d][grp];
#pragma unroll
  for (uint32_t j = 0; j < (uint32_t)kScanRows; ++j) {
    if (j < rows && r0 + j < G) col[(size_t)(r0 + j) * D] = run;
    run += v[j];
  }
}

// Stable scatter.  The block's chunk is walked in rounds of NT kItems keys; in
// a round every wave owns an equal share of the round's keys (whole loads of
// 64).  Each wave ranks its keys on its own: lanes holding the same digit are
// found with one ballot per digit bit, and a per-wave digit counter in LDS
// orders the wave's loads.  One block step then orders the waves and the
// digits, the round is reordered by digit in LDS, keys and record ids
// together, and written out as contiguous runs per digit, so the global
// writes coalesce.  The next round's loads are in flight during the writes.
// (A second payload word, the emission index, cost a third of the traffic and
// of the LDS work: 823 us for two passes over 42M keys with it.)
struct SortSet {
  uint32_t* key;
  uint32_t* rec;
};

template <int kItems, int NT>
__device__ __forceinline__ void radix_scatter(const Ctrl* __restrict__ ctrl, SortSet in, SortSet out,
                                              const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ coltot,
                                              uint32_t G, int shift, int dbits, uint32_t* __restrict__ tile_start,
                                              uint32_t T) {
  constexpr int kRound = NT * kItems, D = 256, NW = NT / 64;
  static_assert(NT >= D, "a digit per thread");
  __shared__ uint32_t s_key[kRound], s_rec[kRound];  // the round reordered by digit
  __shared__ uint32_t first[D];                      // output position of a digit's next key, less its first slot
  __shared__ uint32_t wcnt[NW][D];                   // per-wave digit counts, then the slots of their first keys
  __shared__ uint32_t sh[NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t dmask = (1u << dbits) - 1u;
  uint32_t s, e;
  sort_chunk(ctrl->n_key_eff, G, blockIdx.x, s, e);
  uint32_t kk[kItems], rr[kItems], rc[kItems];
  // a round's keys, split evenly over the waves in whole loads of 64
  auto segment = [&](uint32_t base) { return ((min((uint32_t)kRound, e - base) + NT - 1u) / NT) * 64u; };
  auto load_round = [&](uint32_t base) {
    const uint32_t seg = segment(base), w0 = base + (uint32_t)wave * seg;
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
      const uint32_t i = w0 + (uint32_t)(it * 64 + lane);
      const bool valid = (uint32_t)(it * 64) < seg && i < e;
      kk[it] = valid ? in.key[i] : 0u;
      rc[it] = valid ? in.rec[i] : 0u;
    }
  };
  if (s < e) load_round(s);
  uint32_t run = 0u;  // thread d: global output position of the next key of digit d
  {
    const uint32_t tot = tid < D ? coltot[tid] : 0u;
    const uint32_t mine = tid < D ? cnt[(size_t)blockIdx.x * D + tid] : 0u;
    const uint32_t incl = wave_incl_sum(tot);
    if (lane == 63) sh[wave] = incl;
    __syncthreads();
    uint32_t at = incl - tot;
    for (int w = 0; w < wave; ++w) at += sh[w];
    // one pass over the whole tile id: a digit's first output position is its
    // tile's start
    if (tile_start && blockIdx.x == 0 && tid < D && (uint32_t)tid < T) tile_start[tid] = at;
    if (tile_start && blockIdx.x == 0 && tid == 0) tile_start[T] = ctrl->n_key_eff;
    run = at + mine;
  }
  for (uint32_t base = s; base < e; base += kRound) {
    // ---- per wave: ranks of its keys among its own keys of each digit
#pragma unroll
    for (int j = 0; j < D / 64; ++j) wcnt[wave][lane + 64 * j] = 0u;
    wave_lds_sync();
    const uint32_t n_round = min((uint32_t)kRound, e - base), seg = segment(base);
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
      const uint32_t i = base + (uint32_t)wave * seg + (uint32_t)(it * 64 + lane);
      const bool valid = (uint32_t)(it * 64) < seg && i < e;
      const uint32_t d = (kk[it] >> shift) & dmask;
      unsigned long long peers = __ballot(valid);
      for (int bit = 0; bit < dbits; ++bit) {
        const bool on = (d >> bit) & 1u;
        const unsigned long long bm = __ballot(on);
        peers &= on ? bm : ~bm;
      }
      const uint32_t before = valid ? wcnt[wave][d] : 0u;
      wave_lds_sync();
      if (valid && lanemask_lt_popc(peers) == 0) wcnt[wave][d] = before + (uint32_t)__popcll(peers);
      wave_lds_sync();
      rr[it] = valid ? before + lanemask_lt_popc(peers) : 0xffffffffu;
    }
    __syncthreads();
    // ---- thread d: the slots of digit d's keys, wave by wave
    uint32_t c[NW], sum = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      c[w] = tid < D ? wcnt[w][tid] : 0u;
      sum += c[w];
    }
    const uint32_t incl = wave_incl_sum(sum);
    if (lane == 63) sh[wave] = incl;
    __syncthreads();
    if (tid < D) {
      uint32_t slot = incl - sum;
      for (int w = 0; w < wave; ++w) slot += sh[w];
      first[tid] = run - slot;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        wcnt[w][tid] = slot;
        slot += c[w];
      }
      run += sum;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
      if (rr[it] != 0xffffffffu) {
        const uint32_t slot = rr[it] + wcnt[wave][(kk[it] >> shift) & dmask];
        s_key[slot] = kk[it];
        s_rec[slot] = rc[it];
      }
    }
    __syncthreads();
    if (base + kRound < e) load_round(base + kRound);  // in flight while this round is written
    // keys and record ids out, as contiguous runs per digit
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const uint32_t i = (uint32_t)(tid + j * NT);
      if (i < n_round) {
        const uint32_t k = s_key[i];
        const uint32_t o = first[(k >> shift) & dmask] + i;
        out.key[o] = k;
        out.rec[o] = s_rec[i];
      }
    }
    __syncthreads();
  }
}

// The same for small inputs: a block's at most kSmallChunk keys in one round,
// up to 4096 digits.  Everything the block reads is in flight at once (keys,
// record ids, its row of the column scan, the totals), the digits' first
// positions and the round's LDS slots come out of one packed block scan, and
// keys and record ids are reordered together: four barriers in all.
template <int D>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter_small(
    const Ctrl* __restrict__ ctrl, SortSet in, SortSet out, const uint32_t* __restrict__ cnt,
    const uint32_t* __restrict__ coltot, uint32_t G, int shift, int dbits, uint32_t* __restrict__ tile_start,
    uint32_t T) {
  constexpr int kItems = kSmallChunk / kSortThreads, kPer = D / kSortThreads;
  constexpr int kSlotBits = 11;  // a round's slot count, 0 .. 1024
  static_assert(kSmallChunk < (1u << kSlotBits) && ((uint64_t)kSmallKeys << kSlotBits) < (1ull << 32), "packed scan");
  __shared__ uint32_t s_key[kSmallChunk], s_rec[kSmallChunk];
  __shared__ uint32_t first[D];                       // output position of a digit's keys, less their first slot
  __shared__ __align__(16) uint16_t wcnt[4][D];       // per-wave digit counts, then the slots of their first keys
  __shared__ uint32_t sh[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t dmask = (1u << dbits) - 1u;
  const uint32_t n = ctrl->n_key_eff;
  uint32_t s, e;
  sort_chunk(n, G, blockIdx.x, s, e);
  const uint32_t n_round = e - s, seg = ((n_round + 255u) / 256u) * 64u;
  uint32_t kk[kItems], rc[kItems], rr[kItems], tot[kPer], row[kPer];
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const uint32_t i = s + (uint32_t)wave * seg + (uint32_t)(it * 64 + lane);
    const bool valid = (uint32_t)(it * 64) < seg && i < e;
    kk[it] = valid ? in.key[i] : 0u;
    rc[it] = valid ? in.rec[i] : 0u;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    tot[k] = coltot[tid * kPer + k];
    row[k] = cnt[(size_t)blockIdx.x * D + tid * kPer + k];
  }
#pragma unroll
  for (int j = 0; j < D / 128; ++j) reinterpret_cast<uint32_t*>(wcnt[wave])[lane + 64 * j] = 0u;
  wave_lds_sync();
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const uint32_t i = s + (uint32_t)wave * seg + (uint32_t)(it * 64 + lane);
    const bool valid = (uint32_t)(it * 64) < seg && i < e;
    const uint32_t d = (kk[it] >> shift) & dmask;
    unsigned long long peers = __ballot(valid);
    for (int bit = 0; bit < dbits; ++bit) {
      const bool on = (d >> bit) & 1u;
      const unsigned long long bm = __ballot(on);
      peers &= on ? bm : ~bm;
    }
    const uint32_t before = valid ? wcnt[wave][d] : 0u;
    wave_lds_sync();
    if (valid && lanemask_lt_popc(peers) == 0) wcnt[wave][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
    wave_lds_sync();
    rr[it] = valid ? before + lanemask_lt_popc(peers) : 0xffffffffu;
  }
  __syncthreads();
  uint32_t c[4][kPer], sum = 0u;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
#pragma unroll
    for (int w = 0; w < 4; ++w) c[w][k] = wcnt[w][tid * kPer + k];
    sum += tot[k] << kSlotBits | (c[0][k] + c[1][k] + c[2][k] + c[3][k]);
  }
  const uint32_t incl = wave_incl_sum(sum);
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  uint32_t at = incl - sum;
  for (int w = 0; w < wave; ++w) at += sh[w];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int d = tid * kPer + k;
    const uint32_t pos = at >> kSlotBits;
    uint32_t slot = at & ((1u << kSlotBits) - 1u);
    // one pass over the whole tile id: a digit's first output position is its
    // tile's start
    if (tile_start && blockIdx.x == 0 && (uint32_t)d < T) tile_start[d] = pos;
    first[d] = pos + row[k] - slot;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      wcnt[w][d] = (uint16_t)slot;
      slot += c[w][k];
    }
    at += tot[k] << kSlotBits | (c[0][k] + c[1][k] + c[2][k] + c[3][k]);
  }
  if (tile_start && blockIdx.x == 0 && tid == 0) tile_start[T] = n;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    if (rr[it] != 0xffffffffu) {
      const uint32_t slot = rr[it] + wcnt[wave][(kk[it] >> shift) & dmask];
      s_key[slot] = kk[it];
      s_rec[slot] = rc[it];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = (uint32_t)(tid + j * kSortThreads);
    if (i < n_round) {
      const uint32_t k = s_key[i];
      const uint32_t o = first[(k >> shift) & dmask] + i;
      out.key[o] = k;
      out.rec[o] = s_rec[i];
    }
  }
}

// Kernels around the scatter body: rounds of 2048 keys while the chunks are
// about that long (more blocks, less LDS), of 4096 above, and from kLongChunk
// keys per block on of 8192, whose runs of 32 keys per digit are whole lines.
// Bound by the ranking (VALU 57% of the issue) between barriers and the
// scattered writes (address unit 44% busy).  Two passes:
// 33M keys 398 us with rounds of 4096 that moved keys and record ids one after
// the other, 378 with both together and the next round's loads early, 327 with
// 8192; 69M keys 553, 532, 464; 25M keys (15 K per block) 165, 151, 151; 11.8M
// (7 K) 125, 116, 121; 5.7M (3.5 K) 80, 78, 107.  (Rounds of 16384 by 1024
// threads: 366 and 557.)
constexpr uint32_t kLongChunk = 12288;

__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(const Ctrl* __restrict__ ctrl, SortSet in,
                                                                SortSet out,
                                                                const uint32_t* __restrict__ cnt,
                                                                const uint32_t* __restrict__ coltot, uint32_t G,
                                                                int shift, int dbits, uint32_t* __restrict__ tile_start,
                                                                uint32_t T) {
  radix_scatter<8, kSortThreads>(ctrl, in, out, cnt, coltot, G, shift, dbits, tile_start, T);
}

template <int NT>
__global__ __launch_bounds__(NT, 4) void k_radix_scatter_large(
    const Ctrl* __restrict__ ctrl, SortSet in, SortSet out, const uint32_t* __restrict__ cnt,
    const uint32_t* __restrict__ coltot, uint32_t G, int shift, int dbits, uint32_t* __restrict__ tile_start,
    uint32_t T) {
  radix_scatter<16, NT>(ctrl, in, out, cnt, coltot, G, shift, dbits, tile_start, T);
}

// tile_start[t] = first sorted key index whose tile id is >= t (t in [0, T]).
// kRangeLanes lanes per tile search for it: each step probes the interval at
// kRangeLanes evenly spaced keys and keeps the part between the last smaller
// one and the next.  Eight steps at 30M keys, each one round trip; reading
// every key for the places where the tile changes took 29 us at 33M keys and
// 32 K tiles (16 here), 42 at 69M and 65 K (25).
constexpr int kRangeLanes = 8;
__global__ __launch_bounds__(256) void k_tile_ranges(const Ctrl* __restrict__ ctrl,
                                                     const uint32_t* __restrict__ skeys, uint32_t T, uint32_t tmask,
                                                     uint32_t* __restrict__ tile_start) {
  const uint32_t t = (blockIdx.x * 256u + threadIdx.x) / kRangeLanes;
  const uint32_t i = threadIdx.x % kRangeLanes, shift = threadIdx.x & 63u & ~(uint32_t)(kRangeLanes - 1);
  uint32_t lo = 0, hi = t <= T ? ctrl->n_key_eff : 0u;
  while (__ballot(lo < hi)) {
    const uint32_t step = (hi - lo + kRangeLanes) / (kRangeLanes + 1u);
    const uint32_t at = lo + (i + 1u) * step - 1u;  // (kRangeLanes + 1) step < hi - lo + 9: no overflow
    const bool less = lo < hi && at < hi && (skeys[at] & tmask) < t;
    const uint32_t c = (uint32_t)__popcll(__ballot(less) >> shift & ((1u << kRangeLanes) - 1u));
    if (lo < hi) {
      if (c < (uint32_t)kRangeLanes) hi = min(hi, lo + (c + 1u) * step - 1u);
      lo += c * step;
    }
  }
  if (i == 0 && t <= T) tile_start[t] = lo;
}

// Small inputs (see kSmallKeys): chunks of kSmallChunk keys.  Otherwise
// chunks of at least 2048 keys (half a round), at most 2048 blocks (larger
// inputs walk several full rounds per block), and the tile id's bits split
// evenly over passes of at most 8 bits, so small tile counts get fewer digits
// and longer runs per digit.
SortShape sort_shape(int bits, uint32_t key_cap) {
  if (bits < 1) bits = 1;
  SortShape S;
  S.bits = bits;
  S.small = key_cap <= kSmallKeys;
  const uint32_t chunk = S.small ? kSmallChunk : 2048u;
  S.blocks = std::min(std::max((key_cap + chunk - 1u) / chunk, 1u), kSortMaxBlocks);
  const bool one = S.small && (bits <= 11 || (bits == 12 && key_cap <= kWideKeys));
  S.chunk = key_cap / S.blocks;
  S.passes = one ? 1 : (bits + 7) / 8;
  S.digit_bits = (bits + S.passes - 1) / S.passes;
  S.slots = S.digit_bits <= 8 ? 256u : S.digit_bits <= 10 ? 1024u : S.digit_bits <= 11 ? 2048u : 4096u;
  return S;
}

// Digit bits of one pass: the last takes what is left of the tile id (the
// bits above it belong to the key's other fields).
static int pass_bits(const SortShape& S, int pass) { return std::min(S.digit_bits, S.bits - S.digit_bits * pass); }

hipError_t launch_radix_hist(const Ctrl* ctrl, const uint32_t* keys, uint32_t* hist, const SortShape& S, int pass,
                             hipStream_t s) {
  const int shift = S.digit_bits * pass;
  const uint32_t dmask = (1u << pass_bits(S, pass)) - 1u;
#define UG_HIST(D) \
  if (S.slots == D) hipLaunchKernelGGL(k_radix_hist<D>, dim3(S.blocks), dim3(kSortThreads), 0, s, ctrl, keys, S.blocks, shift, dmask, hist);
  UG_HIST(256)
  UG_HIST(1024)
  UG_HIST(2048)
  UG_HIST(4096)
#undef UG_HIST
  return hipGetLastError();
}

hipError_t launch_radix_colscan(uint32_t* hist, const SortShape& S, hipStream_t s) {
  hipLaunchKernelGGL(k_radix_colscan, dim3(S.slots / kScanDigits), dim3(kScanDigits * kScanGroups), 0, s, hist,
                     S.blocks, S.slots, hist + (size_t)S.slots * S.blocks);
  return hipGetLastError();
}

hipError_t launch_radix_scatter(const Ctrl* ctrl, const uint32_t* const in[2], uint32_t* const out[2],
                                const uint32_t* hist, const SortShape& S, int pass, uint32_t* tile_start,
                                uint32_t num_tiles, hipStream_t s) {
  const int shift = S.digit_bits * pass, pb = pass_bits(S, pass);
  const SortSet si{const_cast<uint32_t*>(in[0]), const_cast<uint32_t*>(in[1])};
  const SortSet so{out[0], out[1]};
  const uint32_t* coltot = hist + (size_t)S.slots * S.blocks;
#define UG_SCATTER(kernel, NT) \
  hipLaunchKernelGGL(kernel, dim3(S.blocks), dim3(NT), 0, s, ctrl, si, so, hist, coltot, S.blocks, shift, pb, tile_start, num_tiles)
  if (S.small && S.slots == 4096u)
    UG_SCATTER(k_radix_scatter_small<4096>, kSortThreads);
  else if (S.small && S.slots == 2048u)
    UG_SCATTER(k_radix_scatter_small<2048>, kSortThreads);
  else if (S.small && S.slots == 1024u)
    UG_SCATTER(k_radix_scatter_small<1024>, kSortThreads);
  else if (S.small)
    UG_SCATTER(k_radix_scatter_small<256>, kSortThreads);
  else if (S.chunk >= kLongChunk)
    UG_SCATTER(k_radix_scatter_large<512>, 512);
  else if (S.blocks >= kSortMaxBlocks)
    UG_SCATTER(k_radix_scatter_large<256>, 256);
  else
    UG_SCATTER(k_radix_scatter, kSortThreads);
#undef UG_SCATTER
  return hipGetLastError();
}

hipError_t launch_tile_ranges(const Ctrl* ctrl, const uint32_t* skeys, uint32_t num_tiles, int bits,
                              uint32_t* tile_start, hipStream_t s) {
  const uint32_t tmask = bits >= 32 ? 0xffffffffu : (1u << bits) - 1u;
  const uint32_t per = 256u / kRangeLanes, blocks = num_tiles / per + 1u;  // num_tiles + 1 starts
  hipLaunchKernelGGL(k_tile_ranges, dim3(blocks), dim3(256), 0, s, ctrl, skeys, num_tiles, tmask, tile_start);
  return hipGetLastError();
}

}  // namespace ug
