// Per-tile accumulation of the ultrasound image formation (Eq. 5-8, 12) and
// its adjoint.
//
// Tiles are split into 8x8-pixel sub-blocks; every key carries the mask of
// the sub-blocks its record's ellipse touches (Eq. 12 support, computed at
// key emission), so both passes evaluate (record, pixel) pairs only inside
// touched sub-blocks.
//
// Forward: one workgroup per tile, one wave per band of 8 pixel rows (or two,
// SPLIT = 2, taking alternate rounds of the tile's records and adding their
// sums at the end), lanes = pixels (a lane owns one pixel in each of the
// band's TW/8 sub-blocks).
// Each wave streams the tile's records (sorted by record id, so every pixel
// sums its Gaussians in the same order whatever the launch shape), keeps
// those whose mask touches its band in a wave-private LDS list and walks the
// list: per pixel-record pair two FMAs give the exponent, one compare
// applies the cut-off and one v_exp_f32 gives the weight.  The masks of eight
// list entries travel in one scalar word, so an entry costs its LDS reads and
// its evaluated sub-blocks: with a mask read back from LDS and broadcast per
// entry the kernel issued 12% more (33M keys on 32x16 tiles 1254 us, 1163 so;
// 25M on 16x16 799, 723; 11.8M needles 667, 592).  Bound by its VALU issue.
//
// Adjoint: a block takes keys of one tile, its waves up to 64 each at a time,
// and expands them into (key, four-column strip) items; lanes = items, each
// walking its strip's rows and accumulating the record's seven partial
// derivatives in registers.  The items of a key are summed in strip order
// into the key's partial, so no atomic is needed and the result is
// deterministic.
#include <algorithm>
#include <cfloat>

#include "ug_kernels.h"

namespace ug {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// A pair's weight 2^(e0 - t1^2 - t2^2) (Eq. 8 in log2 units) is evaluated as
// s 2^x with x = d - t1^2 - t2^2, d = e0 - sig and s = 2^sig per record.
// Under a cut-off (Eq. 12) sig = emin, so the support is x >= 0, and one
// signed-integer max of x's bits against the bits of -inf (kCutBits) maps
// every x < 0 to -inf, whose 2^x is 0: the compare and select of the test
// become one instruction.  sig stays within 64 of e0, so the scaled weights
// stay below 2^64 (for chi^2 > 64 / (log2(e) / 2) = 88.7 the cut then drops
// only weights below 2^-64 of the Gaussian's peak instead of those beyond
// chi^2).  Without a cut-off sig = e0 and the max is against INT_MIN (no
// operation).  A record whose sig is -inf (zero amplitude) gets d = -inf.
constexpr int kCutBits = (int)0xff800000u;  // bits of -inf
constexpr int kNoCutBits = (int)0x80000000u;

struct WeightScale {
  float d, s;
};

__device__ __forceinline__ WeightScale weight_scale(float e0, float emin, bool cut) {
  const float sig = cut ? fmaxf(emin, e0 - 64.f) : e0;
  if (!(sig > -INFINITY)) return {-INFINITY, 0.f};
  return {e0 - sig, exp2f(sig)};
}

// x with every value outside the support mapped to -inf (see above).
__device__ __forceinline__ float support_clamp(float x, int kcut) {
  return __int_as_float(max(__float_as_int(x), kcut));
}

// ---------------------------------------------------------------- forward
// CNT: also count the in-support pairs of pixels inside the plane and the
// evaluated pairs (64 per evaluated wave sub-block) into counters[0] and
// counters[1] (a measurement variant; one more VALU op per pair).  BG records
// are staged per wave and round (PER per lane; lanes beyond BG idle when
// BG < 64).
template <int TW, int TH, int BG, bool CNT, int SPLIT>
__global__ __launch_bounds__(64 * (TH / kSubBlock) * SPLIT) void k_accum_fwd(
    const PlaneInt* __restrict__ pint, const uint32_t* __restrict__ tile_plane,
    const uint32_t* __restrict__ tile_start, const uint32_t* __restrict__ skey, const uint32_t* __restrict__ srec,
    const Rec* __restrict__ recs, float* __restrict__ image,
    float* __restrict__ dsave, float bg_alpha, float bg_color, int kcut, unsigned long long* __restrict__ counters) {
  constexpr int K = TW / kSubBlock;   // pixels per lane = sub-blocks per band
  constexpr int NB = TH / kSubBlock;  // bands = waves
  constexpr int PER = BG >= 64 ? BG / 64 : 1;
  constexpr int CAP = PER * 64;
  static_assert(TW % kSubBlock == 0 && TH % kSubBlock == 0 && K * NB <= 32, "tile shape");
  static_assert(SPLIT == 1 || SPLIT == 2, "waves per band");
  // per kept record: (t11, s, s c, mask) and, per pixel row of the band,
  // (scaled exponent d - t2^2 at the row, t1 offset of the row) -- the row
  // set-up is done once per record while staging instead of once per record
  // and lane
  __shared__ float4 cA[NB * SPLIT][CAP];
  __shared__ float2 cR[NB * SPLIT][CAP][kSubBlock];

  const uint32_t t = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t p = tile_plane[t];
  const PlaneInt PI = pint[p];
  const uint32_t lt = t - PI.tile_off;
  const int x0 = (int)(lt % (uint32_t)PI.ntx) * TW, y0 = (int)(lt / (uint32_t)PI.ntx) * TH;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int band = wv % NB, half = wv / NB;  // half: which alternate rounds
  const int lrow = lane / kSubBlock, col0 = lane % kSubBlock;
  const int row = band * kSubBlock + lrow;
  constexpr int kMaskShift = key_mask_shift(TW, TH);
  const uint32_t bshift = (uint32_t)(kMaskShift + band * K), bmask = (1u << K) - 1u;
  float ucol[K], Nacc[K], Dacc[K];
  uint32_t cnt[K];
  uint32_t nexec = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    ucol[k] = (float)(col0 + k * kSubBlock);
    Nacc[k] = 0.f;
    Dacc[k] = 0.f;
    cnt[k] = 0u;
  }
  const bool cut = kcut != kNoCutBits;
  const uint32_t s = tile_start[t], e = tile_start[t + 1];
  RecAcc pa[PER];
  RecGeo pg[PER];
  uint32_t pm[PER];
  // key words and record ids are loaded together (not the id behind the
  // mask test), then the records whose mask touches the band
  auto fetch = [&](uint32_t base) {
    uint32_t kw[PER], rid[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t j = base + (uint32_t)(q * 64 + lane);
      const bool in = q * 64 + lane < BG && j < e;
      kw[q] = in ? skey[j] : 0u;
      rid[q] = in ? srec[j] : 0u;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t m = (kw[q] >> bshift) & bmask;
      pm[q] = m;
      if (m) {
        pa[q] = recs[rid[q]].acc;
        pg[q] = recs[rid[q]].geo;
      }
    }
  };
  const uint32_t s0 = s + (uint32_t)(half * BG);
  if (s0 < e) fetch(s0);
  for (uint32_t base = s0; base < e; base += SPLIT * BG) {
    // keep this round's records that touch the band, in order
    uint32_t n = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t m = pm[q];
      const unsigned long long bal = __ballot(m != 0u);
      if (m) {
        const uint32_t slot = n + lanemask_lt_popc(bal);
        const RecAcc& A = pa[q];
        const float du0 = (float)(pg[q].ub - x0) + A.fu;
        const float dv0 = (float)(pg[q].vb - y0) + A.fv;
        const float P = -A.t11 * du0;
        const WeightScale ws = weight_scale(A.e0, A.emin, cut);
        cA[wv][slot] = make_float4(A.t11, ws.s, ws.s * A.c, __uint_as_float(m));
#pragma unroll
        for (int y = 0; y < kSubBlock; ++y) {
          const float dv = (float)(band * kSubBlock + y) - dv0;
          const float t2 = A.t22 * dv;
          cR[wv][slot][y] = make_float2(fmaf(-t2, t2, ws.d), fmaf(A.t12, dv, P));
        }
      }
      n += (uint32_t)__popcll(bal);
    }
    if (base + SPLIT * BG < e) fetch(base + SPLIT * BG);
    wave_lds_sync();
    auto eval_rec = [&](const float4& a, const float2& rb, uint32_t m) {
      const float erow = rb.x, B = rb.y;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (K > 1 && !((m >> k) & 1u)) continue;  // uniform
        const float t1 = fmaf(a.x, ucol[k], B);
        const float xs = support_clamp(fmaf(-t1, t1, erow), kcut);
        const float w = fast_exp2(xs);  // the weight over s
        Dacc[k] = fmaf(w, a.y, Dacc[k]);
        Nacc[k] = fmaf(w, a.z, Nacc[k]);
        if constexpr (CNT) {
          cnt[k] += xs != -INFINITY ? 1u : 0u;
          ++nexec;
        }
      }
    };
    // K == 1: an entry's one sub-block is always evaluated.  Four entries at a
    // time: a dense tile is one wave's chain of LDS round trips (half of
    // 100,000 Gaussians in a point on 8x8 tiles: 2580 us two at a time with
    // 16-byte reads, 2290 with 12-byte ones, 2240 so; even scenes 250, 320 and
    // 250 us at 300,000 on 128 planes of 256 x 256).
    if constexpr (K == 1) {
      uint32_t j = 0;
      for (; j + 3 < n; j += 4) {
        const float4 a0 = cA[wv][j], a1 = cA[wv][j + 1], a2 = cA[wv][j + 2], a3 = cA[wv][j + 3];
        const float2 r0 = cR[wv][j][lrow], r1 = cR[wv][j + 1][lrow], r2 = cR[wv][j + 2][lrow], r3 = cR[wv][j + 3][lrow];
        asm volatile("" ::"v"(a0.w), "v"(a1.w), "v"(a2.w), "v"(a3.w));  // 16-byte reads (see below)
        eval_rec(a0, r0, 1u);
        eval_rec(a1, r1, 1u);
        eval_rec(a2, r2, 1u);
        eval_rec(a3, r3, 1u);
      }
      if (n & 2u) {
        const float4 a0 = cA[wv][j], a1 = cA[wv][j + 1];
        const float2 r0 = cR[wv][j][lrow], r1 = cR[wv][j + 1][lrow];
        asm volatile("" ::"v"(a0.w), "v"(a1.w));
        eval_rec(a0, r0, 1u);
        eval_rec(a1, r1, 1u);
        j += 2;
      }
      if (n & 1u) eval_rec(cA[wv][j], cR[wv][j][lrow], 1u);
      n = 0;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if ((uint32_t)(64 * q) >= n) break;  // uniform
      // the masks of eight neighbouring records in one word (K <= 4 bits each;
      // zero behind the list's end), in every lane of the eight
      const uint32_t nq = min(n - (uint32_t)(64 * q), 64u);
      uint32_t mw = (uint32_t)lane < nq ? __float_as_uint(cA[wv][64 * q + lane].w) << (4 * (lane & 7)) : 0u;
      mw |= (uint32_t)__builtin_amdgcn_mov_dpp((int)mw, 0xb1, 0xf, 0xf, true);   // lanes 1 0 3 2
      mw |= (uint32_t)__builtin_amdgcn_mov_dpp((int)mw, 0x4e, 0xf, 0xf, true);   // lanes 2 3 0 1
      mw |= (uint32_t)__builtin_amdgcn_mov_dpp((int)mw, 0x141, 0xf, 0xf, true);  // mirrored in the eight
      for (uint32_t j = 0; j < nq; j += 8) {
        const uint32_t m8 = (uint32_t)__builtin_amdgcn_readlane((int)mw, (int)j);
        const float4* ca = &cA[wv][64 * q + j];
        const float2(*cr)[kSubBlock] = &cR[wv][64 * q + j];
        // two records at a time so that their LDS reads overlap
#pragma unroll
        for (uint32_t i = 0; i < 8; i += 2) {
          if (j + i >= nq) break;  // uniform
          const float4 a0 = ca[i], a1 = ca[i + 1];
          const float2 r0 = cr[i][lrow], r1 = cr[i + 1][lrow];
          asm volatile("" ::"v"(a0.w), "v"(a1.w));  // 16-byte reads: 12-byte ones hold the LDS longer
          eval_rec(a0, r0, m8 >> (4 * i));
          eval_rec(a1, r1, m8 >> (4 * i + 4));
        }
      }
    }
    wave_lds_sync();
  }
  if constexpr (SPLIT == 2) {
    // the band's second wave hands its sums over through its own staging
    // area; the first adds them to its own (first half + second half)
    float* xch = reinterpret_cast<float*>(&cR[NB + band][0][0]);
    if (half == 1) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        xch[(2 * k) * 64 + lane] = Nacc[k];
        xch[(2 * k + 1) * 64 + lane] = Dacc[k];
      }
    }
    __syncthreads();
    if (half == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        Nacc[k] += xch[(2 * k) * 64 + lane];
        Dacc[k] += xch[(2 * k + 1) * 64 + lane];
      }
    }
  }
  const int v = y0 + row;
  if (v < PI.H) {
    const size_t rowbase = (((size_t)PI.pix_off_hi << 32) | PI.pix_off_lo) + (size_t)v * PI.W;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int u = x0 + col0 + k * kSubBlock;
      if (u < PI.W) {
        if (half == 0) {
          const float Dt = Dacc[k] + bg_alpha;
          image[rowbase + u] = (Nacc[k] + bg_alpha * bg_color) / Dt;
          dsave[rowbase + u] = Dt;
        }
        c += cnt[k];
      }
    }
    if constexpr (CNT) {
      if (c) atomicAdd(&counters[0], (unsigned long long)c);
    }
  }
  if constexpr (CNT) {
    if (lane == 0 && nexec) atomicAdd(&counters[1], 64ull * nexec);
  }
}

// ---------------------------------------------------------------- backward
// nsplit blocks of NW waves per tile for the tile's first keys, up to twice
// the mean of all tiles, and blocks for the rest of the tiles that have more:
// the sorted keys are cut into chunks, and each of those blocks looks at its
// chunks' first keys (whose words name their tiles) for chunks behind a tile's
// dealt keys.  With nsplit blocks for every tile, however many keys it has, a
// dense tile's walk alone set the time: half of 100,000 Gaussians in a
// fiftieth of the volume, 64 planes of 256 x 256, 6.88 ms per step, 3.37 so;
// shells and a core in 160 x 160 planes (50,000 on 16 planes, one wave per
// tile) 217 and 160 us.  Where no tile has more it costs 0.1 to 0.4% of a step.
// Each wave has a contiguous share of its block's keys and takes up to 64 of
// them per pass.  The block forms the tile's per-pixel inputs, gamma =
// dL/dc_hat / D and gamma c_hat, in LDS (every row the evaluation reads comes
// from there); the loss gradient takes the
// float operations of the separate kernel.  A kernel of its own that wrote
// them tile by tile took 61 us and this one 14 us less at 16.8M pixels (step
// 4948 -> 4885 us); at 16 planes of 160 x 160 it was a launch more (99 -> 96 us).
//
// A key's ellipse touches a range of four-column strips of the tile; each
// becomes an item (key, strip over the whole tile height).  lanes = items: a
// closed form gives the rows of the strip that can hold a pixel inside the
// ellipse, and the pass's items are ranked by their row count over the whole
// block, largest first.  The evaluation (lanes = items in that order, groups
// of 64 taken by the waves as they get free) walks items with similar row
// counts together, each lane summing its record's seven derivatives over its
// rows in registers into the item's LDS slot; then each key adds its slots in
// strip order.  Pixels an item skips would only add exact zeros, so the sums
// are those of walking all pixels of the tile, and neither the order of the
// ranks nor an atomic touches them: deterministic.
//
// Bound by its VALU issue: about 54 instructions per four-pixel row, three
// quarters of the evaluated pixels inside the support (four-column strips
// with trimmed rows; 0.57 with eight columns).  Ranking 64 keys' items (three
// groups) left 0.62 of the evaluation's lanes at work, 256 keys' (eleven
// groups) 0.85.  Measured, against (key, 8 x 8 sub-block) items ranked per
// wave with the rows found by testing all eight: 33M keys of 32x16 tiles 2300
// -> 1755 us (1,760 instead of 2,500 VALU instructions per 64 keys), 25M of
// 16x16 1567 -> 1115 us, 160,000 of 16x32 28 -> 23 us.
constexpr int kStrip = 4;  // columns per item
// items of one wave's keys per pass: four blocks' LDS fit a CU (three with
// the 9 KB of a 32 x 32 tile's gamma)
__host__ __device__ constexpr int slots_wave(int tw, int th) { return tw * th <= 256 || tw * th > 512 ? 224 : 208; }

// What the item stage needs of a key.  The ellipse t1^2 + t2^2 <= d has at
// column offset du from its centre the rows dv = -m du -/+ sqrt(D - E du^2)
// with S = t12^2 + t22^2, m = t11 t12 / S, D = d / S, E = (t11 t22 / S)^2; its
// bottom row sits at du = us (t1 = 0), its top row at -us.
struct StripGeo {
  float m, D, E, us;
};

// The key's StripGeo, its row padding py and the strips [sa, sa + return) of
// a TW x TH tile its ellipse reaches.  The strips are the column counterpart
// of strip_rows over the tile's rows: at row offset dv the ellipse spans
// du = -(t12 / t11) dv -/+ sqrt(d - t22^2 dv^2) / t11, with its right end at
// dvr and its left at -dvr.  Every bound is widened far above the float
// rounding of these forms: d by 1e-4 (the cancellation near the ellipse's
// ends), the offsets by 1e-3 of a pixel and more far from the centre.
// Without a cut-off, or where a constant is not finite, every strip and row
// passes; a record without support (d < 0, or d = -inf for a zero amplitude)
// has no strip.
template <int TW, int TH>
__device__ __forceinline__ int key_strips(float t11, float t12, float t22, float d, float du0, float dv0, bool cut,
                                          StripGeo& g, float& py, int& sa) {
  const float iS = __builtin_amdgcn_rcpf(fmaf(t12, t12, t22 * t22));
  const float i11 = __builtin_amdgcn_rcpf(t11), i22 = __builtin_amdgcn_rcpf(t22);
  const float vext = __builtin_amdgcn_sqrtf(d) * i22, a = t12 * i11, dw = d * 1.0001f;
  const float e = t11 * t22 * iS;
  g.m = t11 * t12 * iS;
  g.D = dw * iS;
  g.E = e * e;
  g.us = -a * vext;
  py = fmaf(1e-5f, vext + fabsf(dv0), 2e-3f);
  const float dvr = -t12 * vext * __builtin_amdgcn_sqrtf(iS);
  const float pv = fmaf(2e-6f, fabsf(dv0), 1e-3f);
  const float lo = -dv0 - pv, hi = ((float)(TH - 1) - dv0) + pv;
  const float vr = __builtin_amdgcn_fmed3f(dvr, lo, hi), vl = __builtin_amdgcn_fmed3f(-dvr, lo, hi);
  const float tr = t22 * vr, tl = t22 * vl;
  const float qr = fmaf(-tr, tr, dw), ql = fmaf(-tl, tl, dw);
  const float hr = __builtin_amdgcn_sqrtf(fmaxf(qr, 0.f)) * i11, hl = __builtin_amdgcn_sqrtf(fmaxf(ql, 0.f)) * i11;
  const float ur = fmaf(-a, vr, hr), ul = fmaf(-a, vl, -hl);
  const float px = fmaf(1e-5f, (ur - ul) + fabsf(du0), 2e-3f);
  const float fa = fmaxf(floorf((ul + du0 - px) * (1.f / kStrip)), 0.f);
  const float fz = fminf(floorf((ur + du0 + px) * (1.f / kStrip)), (float)(TW / kStrip - 1));
  const bool any = qr >= 0.f && fz >= fa;  // qr < 0: the tile's rows lie beside the ellipse
  sa = any ? (int)fa : 0;
  int ns = any ? (int)fz - sa + 1 : 0;
  // finite and far from overflow: m du and E du^2 stay finite over any tile
  const bool fin = fabsf(g.m) < 1e12f && g.D < 1e30f && g.E < 1e24f && fabsf(g.us) < 1e12f && py < 1e12f &&
                   fabsf(a) < 1e12f && fabsf(dvr) < 1e12f;
  if (!cut || !fin) {
    g.m = g.D = g.E = g.us = 0.f;
    py = INFINITY;
    sa = 0;
    ns = TW / kStrip;
  }
  return d >= 0.f ? ns : 0;  // NaN: no pixel passes its cut-off either
}

// First row and number of rows (0: none) of the strip of kStrip columns from
// tile column xa that can hold a pixel of the key's support.
template <int TH>
__device__ __forceinline__ int strip_rows(const StripGeo& g, float du0, float dv0, float py, float xa, int& ya) {
  const float px = fmaf(2e-6f, fabsf(du0), 1e-3f);
  const float lo = (xa - px) - du0, hi = fmaf(2.f, px, lo + (float)(kStrip - 1));
  const float db = __builtin_amdgcn_fmed3f(g.us, lo, hi), dt = __builtin_amdgcn_fmed3f(-g.us, lo, hi);
  const float qb = fmaf(-g.E * db, db, g.D), qt = fmaf(-g.E * dt, dt, g.D);
  const float vb = fmaf(-g.m, db, __builtin_amdgcn_sqrtf(fmaxf(qb, 0.f)));
  const float vt = fmaf(-g.m, dt, -__builtin_amdgcn_sqrtf(fmaxf(qt, 0.f)));
  const float fa = fmaxf(ceilf((vt + dv0) - py), 0.f);
  const float fb = fminf(floorf((vb + dv0) + py), (float)(TH - 1));
  // qb < 0 with both clamped ends on one side: the strip lies beside the ellipse
  const bool any = qb >= 0.f && fb >= fa;
  ya = any ? (int)fa : 0;
  return any ? (int)fb - ya + 1 : 0;
}

// Place of record rid's key for tile t in emission order (its keys start at
// k0 and ascend in tile id), for keys whose index did not fit the key word.
__device__ __noinline__ uint32_t find_emitted(const uint32_t* __restrict__ emitted,
                                              const uint32_t* __restrict__ rec_koff, uint32_t rid, uint32_t k0,
                                              uint32_t t, uint32_t tmask) {
  uint32_t a = k0, b = rec_koff[rid + 1] - 1u;  // the key is in [a, b]
  while (a < b) {
    const uint32_t m = a + (b - a) / 2u;
    if ((emitted[m] & tmask) < t) a = m + 1u;
    else b = m;
  }
  return a;
}

// The block's keys: [lo, hi) of the keys of tile t, `share` to a wave; with
// loss also the tile's sum of squared differences (loss_part also tells that
// `second` is the target).
template <int TW, int TH, int NW>
__device__ __forceinline__ void accum_bwd_keys(
    const uint32_t* __restrict__ tile_org, const uint32_t* __restrict__ tile_start, const uint32_t* __restrict__ skey,
    const uint32_t* __restrict__ srec, const uint32_t* __restrict__ emitted, const uint32_t* __restrict__ rec_koff,
    const uint32_t* __restrict__ run_koff, const Rec* __restrict__ recs, const PlaneInt* __restrict__ pint,
    const uint32_t* __restrict__ tile_plane, const float* __restrict__ image, const float* __restrict__ second,
    const float* __restrict__ dsave, float scale, float* __restrict__ loss_part, float4* __restrict__ partial, int kcut,
    int tile_bits, uint32_t t, uint32_t lo, uint32_t hi, uint32_t share, bool loss) {
  constexpr int kMaskShift = key_mask_shift(TW, TH);
  constexpr int kSlotsWave = slots_wave(TW, TH), kGroups = (kSlotsWave + 63) / 64;
  constexpr int kMaxStrips = TW / kStrip, kThreads = 64 * NW;
  // float4 per tile row of (gamma, gamma c_hat) in LDS: one more than it
  // needs, so that the rows of a column strip start in different banks
  constexpr int kRow = TW / 2 + 1;
  static_assert(kMaxStrips <= 8 && TH <= 32 && kSlotsWave <= 256, "item fields");
  __shared__ float4 gt[(TH + 1) * kRow];        // the tile's gamma, then a row of zeros
  __shared__ float4 kpA[kThreads];                   // t11, t12, t22, -t11 du0
  __shared__ float4 kpB[kThreads];                   // du0, dv0, d, c
  __shared__ uint32_t bucket[TH + 1];           // items per row count
  __shared__ uint32_t more[NW];                 // whether the wave has keys left after the pass
  __shared__ float quarter_sq[4];               // squared differences of every fourth 64 pixels
  __shared__ uint32_t grab;                     // next group of 64 items to evaluate
  __shared__ uint32_t sorted[NW * kSlotsWave];   // slot | wave << 8 | key << 10 | strip << 18 | first row << 21 | rows << 26
  // the items' sums; before a wave's items are evaluated its part holds what
  // the item stage needs of its keys (read by the same wave only)
  struct ItemStage {
    float4 geo[64];                // StripGeo of the wave's keys
    float py[64];                  // and their row padding
    uint16_t queue[kSlotsWave];    // lane of the key | strip << 8
  };
  union Slots {
    float f[7][kSlotsWave];
    ItemStage in;
  };
  __shared__ Slots slot[NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float ln2 = (float)kLn2;
  const bool cut = kcut != kNoCutBits;
  const uint32_t tmask = (1u << tile_bits) - 1u;
  const uint32_t s = tile_start[t], n = tile_start[t + 1] - s;
  if (threadIdx.x <= TH) bucket[threadIdx.x] = 0u;
  if (threadIdx.x == 0) grab = 0u;
  const PlaneInt& PI = pint[tile_plane[t]];
  const uint32_t org = tile_org[t];  // x0 | y0 << 16
  const int x0 = (int)(org & 0xffffu), y0 = (int)(org >> 16);
  uint32_t k = min(lo + (uint32_t)wave * share, hi);  // the wave's next key
  const uint32_t ke = min(k + share, hi);             // its last
  // A pass's keys are loaded during the pass before it, and their records (a
  // random 64-byte gather per key) before that pass's evaluation.  Lanes past
  // the wave's keys read the tile's last key and are masked off.
  uint32_t kw, rid;
  RecAcc A;
  int ub, vb;
  uint32_t run, koff;
  auto load_keys = [&]() {
    const uint32_t j = s + min(k + (uint32_t)lane, n - 1u);
    kw = skey[j];
    rid = srec[j];
  };
  auto load_recs = [&]() {
    A = recs[rid].acc;
    ub = recs[rid].geo.ub;
    vb = recs[rid].geo.vb;
    run = recs[rid].geo.run;
    koff = recs[rid].geo.koff;
  };
  if (n) load_keys();
  {
    // The tile's gamma and gamma c_hat (zero outside the plane) from the
    // image, the upstream gradient or the target, and the denominators; the
    // loads are in flight with the first keys and records.
    constexpr int kPer = (TW * TH + kThreads - 1) / kThreads;
    const int W = PI.W, H = PI.H;
    const size_t base = ((size_t)PI.pix_off_hi << 32) | PI.pix_off_lo;
    float im[kPer], sc[kPer], dt[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int j = (int)threadIdx.x + kThreads * i, u = x0 + j % TW, v = y0 + j / TW;
      im[i] = sc[i] = 0.f;
      dt[i] = 1.f;
      if (j < TW * TH && u < W && v < H) {
        const size_t idx = base + (size_t)v * W + u;
        im[i] = image[idx];
        sc[i] = second[idx];
        dt[i] = dsave[idx];
      }
    }
    if (n) load_recs();
    float2* g2 = reinterpret_cast<float2*>(gt);
    // The squared differences are added by quarters (every fourth 64 pixels of
    // the tile: one wave's of four), then over the lanes, then the quarters in
    // order, whatever the number of waves: the loss does not depend on it.
    // The lanes are added over DPP: four quarters over LDS shuffles held one
    // wave's block up (10,800 tiles of some keys 69 -> 74 us, 70 so).
    constexpr int kSums = 4 / NW;
    float sq[kSums];
#pragma unroll
    for (int q = 0; q < kSums; ++q) sq[q] = 0.f;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int j = (int)threadIdx.x + kThreads * i;
      float dI = sc[i];
      if (loss_part) {  // uniform
        const float d = im[i] - dI;
        dI = scale * d;
        sq[i % kSums] = fmaf(d, d, sq[i % kSums]);
      }
      const float gam = dI / dt[i];
      if (j < TW * TH) g2[j / TW * (2 * kRow) + j % TW] = make_float2(gam, gam * im[i]);
    }
    if (threadIdx.x < kRow) gt[TH * kRow + threadIdx.x] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (loss) {  // uniform
#pragma unroll
      for (int q = 0; q < kSums; ++q) {
        const float sum = wave_total(sq[q]);
        if (lane == 63) quarter_sq[wave * kSums + q] = sum;
      }
    }
  }
  __syncthreads();  // gt, bucket and grab are ready
  if (loss) {  // uniform
    if (threadIdx.x == 0) loss_part[t] = ((quarter_sq[0] + quarter_sq[1]) + quarter_sq[2]) + quarter_sq[3];
    if (n == 0) return;
  }
  for (;;) {
    // where the key's partial goes: its place in emission order, the record's
    // offset plus the key's index among the record's keys
    const uint32_t last_index = (1u << (kMaskShift - tile_bits)) - 1u;
    const uint32_t index = (kw >> tile_bits) & last_index;
    uint32_t dst = run_koff[run] + koff + index;
    if (index == last_index) dst = find_emitted(emitted, rec_koff, rid, dst - index, t, tmask);
    const uint32_t left = ke - k;
    // at most 64 keys per pass, the last two passes alike
    const uint32_t want = left > 128u ? 64u : (left > 64u ? (left + 1u) / 2u : left);
    const float du0 = (float)(ub - x0) + A.fu, dv0 = (float)(vb - y0) + A.fv;
    const WeightScale ws = weight_scale(A.e0, A.emin, cut);
    ItemStage& in = slot[wave].in;
    int sa;
    uint32_t pc;  // the key's items
    {
      StripGeo g;
      float py;
      const int ns = key_strips<TW, TH>(A.t11, A.t12, A.t22, ws.d, du0, dv0, cut, g, py, sa);
      pc = (uint32_t)lane < want && (kw >> kMaskShift) != 0u ? (uint32_t)ns : 0u;
      kpA[threadIdx.x] = make_float4(A.t11, A.t12, A.t22, -A.t11 * du0);
      kpB[threadIdx.x] = make_float4(du0, dv0, ws.d, A.c);
      in.geo[lane] = make_float4(g.m, g.D, g.E, g.us);
      in.py[lane] = py;
    }
    const float t11k = A.t11, t12k = A.t12, t22k = A.t22;
    uint32_t off = 0u;  // the key's first item
#pragma unroll
    for (int bit = 0; bit < 4; ++bit) off += lanemask_lt_popc(__ballot((pc >> bit) & 1u)) << bit;
    // the leading keys whose items fit the slots (nearly always all of them)
    const bool mine = (uint32_t)lane < want && off + pc <= (uint32_t)kSlotsWave;
    const uint32_t took = (uint32_t)__popcll(__ballot(mine));
    if (!mine) pc = 0u;
    const uint32_t L = (uint32_t)__builtin_amdgcn_readlane((int)(off + pc), (int)(took ? took - 1u : 0u));
#pragma unroll
    for (uint32_t i = 0; i < kMaxStrips; ++i)
      if (i < pc) in.queue[off + i] = (uint16_t)((uint32_t)lane | ((uint32_t)sa + i) << 8);
    k += took;
    if (lane == 0) more[wave] = ke - k;
    if (k < ke) load_keys();
    wave_lds_sync();
    // ---- lanes = items: the rows each can reach, ranked by their count (an
    // item without rows is ranked last and its sums come out as zeros)
    uint32_t ent[kGroups], rank[kGroups];
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
      ent[i] = 0u;
      rank[i] = 0xffffffffu;
      const uint32_t q = (uint32_t)(i * 64 + lane);
      if (q < L) {
        const uint32_t e = in.queue[q];
        const int kl = (int)(e & 63u);
        const float4 kb = kpB[wave * 64 + kl], kd = in.geo[kl];
        int ya;
        const int nr = strip_rows<TH>(StripGeo{kd.x, kd.y, kd.z, kd.w}, kb.x, kb.y, in.py[kl],
                                      (float)((e >> 8) * kStrip), ya);
        ent[i] = q | (uint32_t)wave << 8 | (e | (uint32_t)wave << 6) << 10 | (uint32_t)ya << 21 | (uint32_t)nr << 26;
        rank[i] = atomicAdd(&bucket[nr], 1u);
      }
    }
    __syncthreads();
    // first rank of every row count, largest first (lane l: TH - l rows)
    const uint32_t bv = lane <= TH ? bucket[TH - lane] : 0u;
    const uint32_t bx = wave_incl_sum(bv);
    const uint32_t Ls = (uint32_t)__builtin_amdgcn_readlane((int)bx, 63);  // items of the pass
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
      const uint32_t f = __shfl(bx - bv, TH - (int)(ent[i] >> 26), 64);
      if (rank[i] != 0xffffffffu) sorted[f + rank[i]] = ent[i];
    }
    uint32_t any_more = more[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) any_more |= more[w];
    const bool again = any_more != 0u;
    __syncthreads();
    if (threadIdx.x <= TH) bucket[threadIdx.x] = 0u;
    if (k < ke) load_recs();  // in flight during the evaluation
    // ---- lanes = items by row count: the rows of one key's strip.  Each wave
    // takes the next group of 64 when it is done with its last one.
    for (;;) {
      uint32_t taken = 0u;
      if (lane == 0) taken = atomicAdd(&grab, 1u);
      const uint32_t s0 = 64u * __builtin_amdgcn_readfirstlane(taken);
      if (s0 >= Ls) break;
      const bool has = s0 + (uint32_t)lane < Ls;
      const uint32_t e = has ? sorted[s0 + (uint32_t)lane] : 0u;
      const int kl = (int)((e >> 10) & 255u), st = (int)((e >> 18) & 7u), by = (int)((e >> 21) & 31u);
      const int nr = (int)(e >> 26);  // 0 for a lane without an item
      const float4 ka = kpA[kl];
      const float4 kb = kpB[kl];
      const float t11 = ka.x, t12 = ka.y, t22 = ka.z, P = ka.w;
      const float dvo = kb.y, d = kb.z, c = kb.w;
      const float bxf = (float)((st >> 1) * kSubBlock);  // the sub-block's first column
      // t1 as over the whole sub-block: B0 at its first column, column j
      // from there at B0 + t11 j, j = 0..3 or 4..7
      const float j0 = (float)((st & 1) * kStrip);
      const float j1 = j0 + 1.f, j2 = j0 + 2.f, j3 = j0 + 3.f;
      float rowf = (float)by;
      int at = (by * kRow + st * (kStrip / 2)) * (int)sizeof(float4);
      const int stop = at + nr * kRow * (int)sizeof(float4);  // rows past the item's read zeros: they add exact zeros
      const int nmax = __builtin_amdgcn_readfirstlane(nr);  // the group's first item has the most rows
      float Sge = 0.f, Sa = 0.f, Sau = 0.f, S12 = 0.f, S22 = 0.f, Sb = 0.f, Sdc = 0.f;
      for (int r = 0; r < nmax; ++r) {
        const float4* row = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(gt) +
                                                            (at < stop ? at : TH * kRow * (int)sizeof(float4)));
        const float4 g0 = row[0], g1 = row[1];
        at += kRow * (int)sizeof(float4);
        const float dv = rowf - dvo;
        rowf += 1.f;
        const float B0 = fmaf(t11, bxf, fmaf(t12, dv, P));
        const float t2 = t22 * dv;
        const float erow = fmaf(-t2, t2, d);
        const float ta = fmaf(t11, j0, B0), tb = fmaf(t11, j1, B0), tc = fmaf(t11, j2, B0), td = fmaf(t11, j3, B0);
        // weights over s; dL/dw = gamma (c - c_hat)
        const float wa = fast_exp2(support_clamp(fmaf(-ta, ta, erow), kcut));
        const float wb = fast_exp2(support_clamp(fmaf(-tb, tb, erow), kcut));
        const float wc = fast_exp2(support_clamp(fmaf(-tc, tc, erow), kcut));
        const float wd = fast_exp2(support_clamp(fmaf(-td, td, erow), kcut));
        const float ga = wa * fmaf(g0.x, c, -g0.y), gb = wb * fmaf(g0.z, c, -g0.w);
        const float gc = wc * fmaf(g1.x, c, -g1.y), gd = wd * fmaf(g1.z, c, -g1.w);
        Sdc = fmaf(g0.x, wa, Sdc);
        Sdc = fmaf(g0.z, wb, Sdc);
        Sdc = fmaf(g1.x, wc, Sdc);
        Sdc = fmaf(g1.z, wd, Sdc);
        // the row's sums of ge, ge i, ge i^2 over i = 0..3; with t1 = ta +
        // t11 i they give its sums of ge t1 and ge t1 i
        const float rge = (ga + gb) + (gc + gd);
        const float rj = fmaf(3.f, gd, fmaf(2.f, gc, gb));
        const float rjj = fmaf(9.f, gd, fmaf(4.f, gc, gb));
        const float ra = fmaf(t11, rj, ta * rge);
        Sau = fmaf(t11, rjj, Sau);
        Sau = fmaf(ta, rj, Sau);
        Sge += rge;
        Sa += ra;
        S12 = fmaf(dv, ra, S12);
        const float u = t2 * rge;
        Sb += u;
        S22 = fmaf(dv, u, S22);
      }
      if (has) {
        float* o = &slot[(e >> 8) & 3u].f[0][e & 255u];
        o[0 * kSlotsWave] = Sge;
        o[1 * kSlotsWave] = Sa;
        o[2 * kSlotsWave] = fmaf((float)(st * kStrip), Sa, Sau);  // sum ge t1 x, x the tile column
        o[3 * kSlotsWave] = S12;
        o[4 * kSlotsWave] = S22;
        o[5 * kSlotsWave] = Sb;
        o[6 * kSlotsWave] = Sdc;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) grab = 0u;  // every wave has left the loop above
    // ---- each key adds its items in strip order
    float acc[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (uint32_t i = 0; i < kMaxStrips; ++i) {
      if (i < pc) {
#pragma unroll
        for (int f = 0; f < 7; ++f) acc[f] += slot[wave].f[f][off + i];
      }
    }
    if (mine) {
      // every sum is linear in the weights: scale them back by s once
      const float Sge = acc[0] * ws.s, Sa = acc[1] * ws.s, Sau = acc[2] * ws.s, S12 = acc[3] * ws.s,
                  S22 = acc[4] * ws.s, Sb = acc[5] * ws.s, Sdc = acc[6] * ws.s;
      // w = 2^(e0 - t1^2 - t2^2):  dL/ds = -ln2 w dL/dw, s = t1^2 + t2^2.
      const float k2 = 2.f * ln2;
      partial[2 * (size_t)dst] = make_float4(-k2 * (Sau - du0 * Sa), -k2 * S12, -k2 * S22, k2 * t11k * Sa);
      partial[2 * (size_t)dst + 1] = make_float4(k2 * (t12k * Sa + t22k * Sb), ln2 * Sge, Sdc, 0.f);
    }
    if (!again) break;  // uniform over the block
    wave_lds_sync();    // the next pass's item stage takes the slots' place
  }
}

template <int TW, int TH, int NW>
__global__ __launch_bounds__(64 * NW, NW > 1 && TW * TH > 512 ? 3 : 4) void k_accum_bwd(
    const uint32_t* __restrict__ tile_org, const uint32_t* __restrict__ tile_start, const uint32_t* __restrict__ skey,
    const uint32_t* __restrict__ srec, const uint32_t* __restrict__ emitted, const uint32_t* __restrict__ rec_koff,
    const uint32_t* __restrict__ run_koff, const Rec* __restrict__ recs, const PlaneInt* __restrict__ pint,
    const uint32_t* __restrict__ tile_plane, const float* __restrict__ image, const float* __restrict__ second,
    const float* __restrict__ dsave, float scale, float* __restrict__ loss_part, float4* __restrict__ partial, int kcut,
    int tile_bits, uint32_t num_tiles, uint32_t nsplit, uint32_t min_deal, float twice, uint32_t chunk) {
  auto keys = [&](uint32_t t, uint32_t lo, uint32_t hi, uint32_t share, bool loss) {
    accum_bwd_keys<TW, TH, NW>(tile_org, tile_start, skey, srec, emitted, rec_koff, run_koff, recs, pint, tile_plane,
                               image, second, dsave, scale, loss_part, partial, kcut, tile_bits, t, lo, hi, share,
                               loss);
  };
  const uint32_t n_all = tile_start[num_tiles];
  // keys of a tile that its own blocks take
  const uint32_t deal = max(min_deal, (uint32_t)fminf((float)n_all * twice, 4e9f));
  if (blockIdx.x < num_tiles * nsplit) {
    // all tiles' first parts, then their second ...: the blocks left without
    // keys come last, instead of every few (which left the same CUs idle)
    const uint32_t part = blockIdx.x / num_tiles, t = xcd_remap(blockIdx.x - part * num_tiles, num_tiles);
    const uint32_t dealt = min(tile_start[t + 1] - tile_start[t], deal);
    // at least 32 each (fewer, fuller waves where a tile has few)
    const uint32_t share = max((dealt + NW * nsplit - 1u) / (NW * nsplit), 32u);
    const uint32_t lo = min(part * NW * share, dealt), hi = min(lo + NW * share, dealt);
    const bool loss = loss_part && part == 0;
    if (lo < hi || loss) keys(t, lo, hi, share, loss);  // uniform
    return;
  }
  // The rest: 64 chunks at a time, a lane each (every wave of the block the
  // same ones), neighbouring chunks in different blocks.  A chunk holds keys
  // behind a tile's dealt ones only if it starts in that tile (chunk <= deal).
  const uint32_t nrest = gridDim.x - num_tiles * nsplit, lane = threadIdx.x & 63u;
  for (uint32_t c = blockIdx.x - num_tiles * nsplit; (uint64_t)c * chunk < n_all; c += 64u * nrest) {
    const uint64_t at = (uint64_t)(c + lane * nrest) * chunk;
    const bool in = at < n_all;
    const uint32_t pos = in ? (uint32_t)at : 0u, tile = skey[pos] & ((1u << tile_bits) - 1u);
    const uint32_t ts = tile_start[tile], te = tile_start[tile + 1];
    const uint32_t a = max(pos - ts, deal), z = pos - ts + min(chunk, te - pos);
    for (unsigned long long todo = __ballot(in && a < z); todo; todo &= todo - 1ull) {
      const int l = __builtin_ctzll(todo);
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)a, l);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)z, l);
      keys((uint32_t)__builtin_amdgcn_readlane((int)tile, l), lo, hi, max((hi - lo + NW - 1u) / NW, 32u), false);
      wave_lds_sync();  // as between two passes
    }
  }
}

// ---------------------------------------------------------------- dispatch
template <int TW, int TH, int SPLIT>
static hipError_t fwd_bg(int bg, dim3 grid, hipStream_t s, const PlaneInt* pint, const uint32_t* tp,
                         const uint32_t* ts, const uint32_t* skey, const uint32_t* srec, const Rec* rc,
                         float* img, float* ds, float ba, float bc, int kcut, unsigned long long* n_eval) {
  constexpr int NT = 64 * (TH / kSubBlock) * SPLIT;
  switch (bg) {
#define UG_BG(B)                                                                                                   \
  case B:                                                                                                          \
    if (n_eval)                                                                                                    \
      hipLaunchKernelGGL((k_accum_fwd<TW, TH, B, true, SPLIT>), grid, dim3(NT), 0, s, pint, tp, ts, skey, srec,    \
                         rc, img, ds, ba, bc, kcut, n_eval);                                                       \
    else                                                                                                           \
      hipLaunchKernelGGL((k_accum_fwd<TW, TH, B, false, SPLIT>), grid, dim3(NT), 0, s, pint, tp, ts, skey, srec,   \
                         rc, img, ds, ba, bc, kcut, n_eval);                                                       \
    return hipGetLastError();
    UG_BG(32)
    UG_BG(64)
    UG_BG(128)
    UG_BG(256)
#undef UG_BG
    default:
      return hipErrorInvalidValue;
  }
}

int accum_default_ppl(int tile_w, int tile_h) {
  (void)tile_h;
  return tile_w / kSubBlock;
}

bool accum_config_supported(int tile_w, int tile_h, int ppl, int lds_batch) {
  if (!(lds_batch == 32 || lds_batch == 64 || lds_batch == 128 || lds_batch == 256)) return false;
  if (ppl != tile_w / kSubBlock) return false;
#define UG_OK_SHAPE(W, H) \
  if (tile_w == W && tile_h == H) return true;
  UG_TILE_SHAPES(UG_OK_SHAPE)
#undef UG_OK_SHAPE
  return false;
}

hipError_t launch_accum_fwd(int tile_w, int tile_h, int lds_batch, int split, const PlaneInt* pint,
                            const uint32_t* tile_plane, const uint32_t* tile_start, const uint32_t* skey,
                            const uint32_t* srec, const Rec* recs, float* image, float* dsave,
                            float bg_alpha, float bg_color, bool cut, uint32_t num_tiles,
                            unsigned long long* n_eval, hipStream_t s) {
  const dim3 grid(num_tiles);
  const int kcut = cut ? kCutBits : kNoCutBits;
#define UG_LAUNCH_SHAPE(W, H)                                                                                    \
  if (tile_w == W && tile_h == H)                                                                                \
    return split == 2 ? fwd_bg<W, H, 2>(lds_batch, grid, s, pint, tile_plane, tile_start, skey, srec, recs,       \
                                        image, dsave, bg_alpha, bg_color, kcut, n_eval)                          \
                      : fwd_bg<W, H, 1>(lds_batch, grid, s, pint, tile_plane, tile_start, skey, srec, recs,       \
                                        image, dsave, bg_alpha, bg_color, kcut, n_eval);
  UG_TILE_SHAPES(UG_LAUNCH_SHAPE)
#undef UG_LAUNCH_SHAPE
  return hipErrorInvalidValue;
}

// Blocks per tile: about 1,024 keys each (four passes of a block, so its
// start-up is a small part; measured at 3,700 keys per tile: one block per
// tile 787 us, four 739, sixteen 824), and where that leaves fewer than 1,024
// blocks (four per CU) down to 128 keys each (84 tiles of 1,025 keys: one
// block per tile 41 us, eight 13; 600 tiles of 150: one 11, two 15).
constexpr uint32_t kBwdBlockKeys = 1024, kBwdMinBlocks = 1024, kBwdMinKeys = 128;

// A tile's own blocks take kBwdDealKeys keys each (a quarter of that with one
// wave) or twice the mean of all tiles, if that is more; the keys behind go to
// up to kBwdRestWaves waves in chunks of about a 1,024th of the capacity,
// kBwdMinChunk to kBwdDealKeys keys (kBwdMinChunk with one wave).  Fewer dealt
// keys share better, but cut the even scenes' blocks up, whose fullest tiles
// hold 1.3 times the mean.  The kernel's time, half of these, these, twice
// these, then 1.3 and 4 times the mean: a core of 500,000 in 256 x 256 planes
// (32x16 tiles) 639, 631, 720, 629, 712 us; shells and a core, 80 planes of
// 160 x 160 (16x16) 186, 189, 215, 191, 192; the same on 16 planes (one wave)
// 49, 51, 72, 48, 87.
constexpr uint32_t kBwdDealKeys = 1024, kBwdMinChunk = 256, kBwdRestWaves = 4096;

// One wave per block where a tile has few keys: 40 KB of LDS let four blocks
// of four waves on a CU, and with a wave's worth of keys in a tile their time
// is the block's start-up, which a block of one wave (10 to 18 KB) repeats
// less and overlaps more.  With many keys the four waves win: they form the
// tile's per-pixel inputs once for all and rank their items together.  Both
// ways, keys per tile at many tiles: 16x16 pixels 16 140 us / 69, 100 157 /
// 120, 240 184 / 207; 32x16 57 91 / 61, 174 103 / 117; 8x8 24 410 / 138, 240
// 563 / 432; 32x32 168 85 / 102.  The lines lie near 3584 / sqrt(pixels) keys
// of capacity.  With fewer tiles than kBwdOneTiles the chip is not full and
// the four waves shorten each tile.
constexpr uint32_t kBwdOneTiles = 1024;
constexpr uint64_t kBwdOneKeys = 3584;

hipError_t launch_accum_bwd(int tile_w, int tile_h, int tile_bits, const uint32_t* tile_org,
                            const uint32_t* tile_start, const uint32_t* skey, const uint32_t* srec,
                            const uint32_t* emitted, const uint32_t* rec_koff, const uint32_t* run_koff,
                            const Rec* recs, const PlaneInt* pint, const uint32_t* tile_plane, const float* image,
                            const float* second, const float* dsave, float scale, float* loss_part, float* partial,
                            bool cut, uint32_t num_tiles, uint32_t key_cap, hipStream_t s) {
  float4* p4 = reinterpret_cast<float4*>(partial);
  if (num_tiles == 0) return hipSuccess;
  const uint32_t avg = key_cap / num_tiles;
  const uint64_t px = (uint64_t)(tile_w * tile_h);
  const bool one = num_tiles >= kBwdOneTiles && (uint64_t)avg * avg * px < kBwdOneKeys * kBwdOneKeys;
  const uint32_t fill = std::min((kBwdMinBlocks + num_tiles - 1u) / num_tiles, avg / kBwdMinKeys);
  const uint32_t nsplit = std::max(std::max(avg / kBwdBlockKeys, fill), 1u);
  const uint32_t waves = one ? 1u : 4u;
  const uint32_t min_deal = nsplit * (kBwdDealKeys / 4u * waves);
  const uint32_t chunk = one ? kBwdMinChunk : std::min(std::max(key_cap / kBwdMinBlocks, kBwdMinChunk), kBwdDealKeys);
  const uint32_t nrest =
      key_cap > min_deal ? std::min(key_cap / chunk + 1u, kBwdRestWaves / waves) : 0u;  // else no tile has more
  const float twice = 2.f / (float)num_tiles;
  const dim3 grid(num_tiles * nsplit + nrest);
  const int kcut = cut ? kCutBits : kNoCutBits;
#define UG_BWD_NW(W, H, NW)                                                                                     \
  hipLaunchKernelGGL((k_accum_bwd<W, H, NW>), grid, dim3(64 * NW), 0, s, tile_org, tile_start, skey, srec,      \
                     emitted, rec_koff, run_koff, recs, pint, tile_plane, image, second, dsave, scale,          \
                     loss_part, p4, kcut, tile_bits, num_tiles, nsplit, min_deal, twice, chunk)
#define UG_BWD(W, H)                                                                                            \
  if (tile_w == W && tile_h == H) {                                                                             \
    if (one)                                                                                                    \
      UG_BWD_NW(W, H, 1);                                                                                       \
    else                                                                                                        \
      UG_BWD_NW(W, H, 4);                                                                                       \
    return hipGetLastError();                                                                                   \
  }
  UG_TILE_SHAPES(UG_BWD)
#undef UG_BWD
#undef UG_BWD_NW
  return hipErrorInvalidValue;
}

}  // namespace ug
