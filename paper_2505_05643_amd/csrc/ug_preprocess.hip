// Preprocess kernels: plane set-up, the Phase-1 cull with record compaction
// (Section 4.4: reject the pairs whose box misses the plane, then compact
// the accepted ones), the per-record in-plane conic with key offsets and key
// emission (tile binning), and the adjoint of the record construction.
//
// Each compaction is a count kernel and a write kernel.  The count kernel
// leaves one total per block; a block of the write kernel adds up the totals
// of the blocks before it (at most 2048 of them, read coalesced), so offsets
// never depend on scheduling and no block waits on another: records are
// Gaussian-major with planes in order, and keys are in record order.
#include <cfloat>

#include "ug_conic.h"
#include "ug_kernels.h"

namespace ug {

// ---------------------------------------------------------------- plane set-up
// FP64 constants of plane p's pose (an invalid pose is marked and skipped; the
// cull raises the flag) and the float constants of its cull.
__device__ __forceinline__ PlaneCull plane_setup(const ug_planes& pl, const PlaneInt* __restrict__ pint, int p,
                                                 PlaneConst* __restrict__ pc, bool write) {
  double R[9];
  bool fin = true;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    R[k] = (double)pl.rot[9 * p + k];
    fin = fin && isfinite_d(R[k]);
  }
  PlaneConst c;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c.o[k] = (double)pl.origin[3 * p + k];
    fin = fin && isfinite_d(c.o[k]);
    c.e1[k] = R[3 * k + 0];
    c.e2[k] = R[3 * k + 1];
  }
  c.sx = (double)pl.spacing[2 * p + 0];
  c.sy = (double)pl.spacing[2 * p + 1];
  fin = fin && isfinite_d(c.sx) && isfinite_d(c.sy) && c.sx > 0.0 && c.sy > 0.0;
  // R^-1 = adj(R) / det(R)
  const double a = R[0], b = R[1], cc = R[2], d = R[3], e = R[4], f = R[5], g = R[6], h = R[7], i = R[8];
  const double A = e * i - f * h, B = -(d * i - f * g), C = d * h - e * g;
  const double det = a * A + b * B + cc * C;
  fin = fin && isfinite_d(det) && det > 0.0;
  const double id = 1.0 / det;
  c.rinv[0] = A * id;
  c.rinv[1] = -(b * i - cc * h) * id;
  c.rinv[2] = (b * f - cc * e) * id;
  c.rinv[3] = B * id;
  c.rinv[4] = (a * i - cc * g) * id;
  c.rinv[5] = -(a * f - cc * d) * id;
  c.rinv[6] = C * id;
  c.rinv[7] = -(a * h - b * g) * id;
  c.rinv[8] = (a * e - b * d) * id;
  c.absdet = fabs(det);
  c.cu = 0.5 * (double)pint[p].W - 0.5;
  c.cv = 0.5 * (double)pint[p].H - 0.5;
  c.valid = fin ? 1 : 0;
  c.pad = 0;
  if (write) pc[p] = c;
  PlaneCull q;
  for (int k = 0; k < 3; ++k) {
    q.o[k] = pl.origin[3 * p + k];
    q.r3[k] = (float)c.rinv[6 + k] + 0.f;  // -0 as +0 (same test; one group key per normal)
  }
  q.valid = c.valid;
  q.pad = 0;
  return q;
}

// Bits of a float in the order of its value (-0 before +0).
__device__ __forceinline__ uint32_t float_order(float x) {
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Whether two planes' group keys (validity, r3, o[0], o[1]) agree bit for bit.
__device__ __forceinline__ bool group_key_eq(const PlaneCull& a, const PlaneCull& b) {
  return a.valid == b.valid && __float_as_uint(a.r3[0]) == __float_as_uint(b.r3[0]) &&
         __float_as_uint(a.r3[1]) == __float_as_uint(b.r3[1]) && __float_as_uint(a.r3[2]) == __float_as_uint(b.r3[2]) &&
         __float_as_uint(a.o[0]) == __float_as_uint(b.o[0]) && __float_as_uint(a.o[1]) == __float_as_uint(b.o[1]);
}

// A 32-bit mix of the group key's bits (equal keys, equal hashes).
__device__ __forceinline__ uint32_t group_key_hash(const PlaneCull& q) {
  const uint32_t w[6] = {(uint32_t)q.valid, __float_as_uint(q.r3[0]), __float_as_uint(q.r3[1]),
                         __float_as_uint(q.r3[2]), __float_as_uint(q.o[0]), __float_as_uint(q.o[1])};
  uint32_t h = 0x811c9dc5u;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    h = (h ^ w[i]) * 0x9e3779b1u;
    h ^= h >> 15;
  }
  return h;
}

// Sum over the quad of lanes, in every lane of it.
__device__ __forceinline__ uint32_t quad_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xb1, 0xf, 0xf, true);  // lanes 1 0 3 2
  x += (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4e, 0xf, 0xf, true);  // lanes 2 3 0 1
  return x;
}

// Groups of at least this many planes are searched by the cull.
constexpr uint32_t kGroupSearch = 8;

// One thread per plane; thread 0 clears the control block.  With group (a
// launch of one block, at most kGroupMaxPlanes planes) the planes are also
// ordered by (hash of the group key, o[2], index): each plane counts the
// planes before it in that order (its position), those with a smaller hash
// (its group's first position) and those with its hash (the group's size).
// Every plane then checks that its key equals that of its group's first
// plane; if two keys ever share a hash, the cull tests every plane instead.
// Four neighbouring lanes share a plane's counts (a quarter of the planes
// each), which are the kernel's longest chain: 256 planes 16 us with one lane
// per plane, 12.9 so.
template <bool GROUP>
__global__ __launch_bounds__(GROUP ? 4 * kGroupMaxPlanes : 256) void k_init(ug_planes pl,
                                                                         const PlaneInt* __restrict__ pint,
                                                                         PlaneConst* __restrict__ pc,
                                                                         PlaneCull* __restrict__ pcf,
                                                                         PlaneGroups* __restrict__ pg,
                                                                         Ctrl* __restrict__ ctrl) {
  __shared__ PlaneCull s_q[kGroupMaxPlanes];
  __shared__ unsigned long long s_hz[kGroupMaxPlanes];  // hash << 32 | order bits of o[2]
  __shared__ uint32_t s_first[kGroupMaxPlanes];         // plane at each group's first position
  __shared__ uint32_t s_big, s_bad;
  const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
  if (gid == 0) {
    ctrl->n_rec = 0;
    ctrl->n_key = 0;
    ctrl->n_eval = 0;
    ctrl->n_exec = 0;
    ctrl->flags = 0;
    ctrl->n_rec_eff = 0;
    ctrl->n_key_eff = 0;
  }
  const int p = (int)(GROUP ? gid / 4u : gid);
  const uint32_t part = GROUP ? gid % 4u : 0u;
  const bool has = p < pl.p, mine = has && part == 0;
  PlaneCull q{};
  if (has) q = plane_setup(pl, pint, p, pc, mine);
  if (mine) pcf[p] = q;
  if (!GROUP) {
    if (gid == 0) pg->use = 0u;
    return;
  }
  const uint32_t h = group_key_hash(q);
  const unsigned long long hz = (unsigned long long)h << 32 | float_order(q.o[2]);
  if (mine) {
    s_q[p] = q;
    s_hz[p] = hz;
  }
  if (threadIdx.x == 0) {
    s_big = 0u;
    s_bad = 0u;
  }
  __syncthreads();
  uint32_t rank = 0u, below = 0u, same = 0u;
  if (has) {
#pragma unroll 8
    for (int j = (int)part; j < pl.p; j += 4) {
      const unsigned long long o = s_hz[j];
      rank += (o < hz || (o == hz && j < p)) ? 1u : 0u;
      const uint32_t oh = (uint32_t)(o >> 32);
      below += oh < h ? 1u : 0u;
      same += oh == h ? 1u : 0u;
    }
  }
  rank = quad_sum(rank);
  below = quad_sum(below);
  same = quad_sum(same);
  if (mine) {
    pg->perm[rank] = (uint32_t)p;
    pg->oz[rank] = q.o[2];
    pg->end[rank] = below + same;
    if (rank == below) s_first[below] = (uint32_t)p;
    if (q.valid && same >= kGroupSearch) atomicOr(&s_big, 1u);
  }
  __syncthreads();
  if (mine && !group_key_eq(q, s_q[s_first[below]])) atomicOr(&s_bad, 1u);
  __syncthreads();
  if (threadIdx.x == 0) pg->use = (s_big && !s_bad) ? 1u : 0u;
}

// Conservative float pre-test of Phase 1: false only if the exact (double)
// test surely rejects the pair.  The float m3 is off by at most a few ulps of
// sum |r3_i (mu_i - o_i)|, the float Sigma'_33 by a few ulps relative; the
// margins below are ten times larger.
// Split in two: Sigma'_33 depends on the plane through r3 only, so planes
// sharing r3 share it.
__device__ __forceinline__ float cull_s33(const GaussT<float>& G, const PlaneCull& P) {
  float g3[3];
  fsub(G, P.r3[0], P.r3[1], P.r3[2], g3);
  return g3[0] * g3[0] + g3[1] * g3[1] + g3[2] * g3[2];
}
__device__ __forceinline__ bool cull_test(const GaussT<float>& G, const PlaneCull& P, float S33, float chi2) {
  const float d0 = G.mu[0] - P.o[0], d1 = G.mu[1] - P.o[1], d2 = G.mu[2] - P.o[2];
  const float m3 = P.r3[0] * d0 + P.r3[1] * d1 + P.r3[2] * d2;
  const float slack = 2e-6f * (fabsf(P.r3[0] * d0) + fabsf(P.r3[1] * d1) + fabsf(P.r3[2] * d2));
  const float a = fmaxf(fabsf(m3) - slack, 0.f);
  return a * a <= chi2 * S33 * 1.0002f;  // false for NaN as well
}
__device__ __forceinline__ bool cull_maybe(const GaussT<float>& G, const PlaneCull& P, float chi2) {
  return cull_test(G, P, cull_s33(G, P), chi2);
}

// Sorted positions [lo, hi) of a plane group (planes sharing r3, o[0] and
// o[1], sorted by o[2]; P0 one of them) outside which cull_maybe rejects G.
// It accepts only if |m3| - slack <= sqrt(chi2 S33 1.0002) up to float
// rounding, where |m3| >= |r3_2 d2| - A with A = |r3_0 d0| + |r3_1 d1| (the
// same for the whole group) and slack <= 2e-6 (A + |r3_2 d2|), so
// |mu_2 - o_2| <= (sqrt(chi2 S33 1.0002) + A) (1 + 3e-6) / |r3_2|; the factors
// below widen that well beyond every rounding of this bound, and an infinite
// or undefined bound (no cut-off, r3_2 = 0) keeps the whole group.
__device__ __forceinline__ void group_window(const GaussT<float>& G, const PlaneCull& P0, float S33, float chi2,
                                             const float* oz, int& lo, int& hi) {
  const float d0 = G.mu[0] - P0.o[0], d1 = G.mu[1] - P0.o[1];
  const float A = fabsf(P0.r3[0] * d0) + fabsf(P0.r3[1] * d1);
  const float D = (sqrtf(chi2 * S33 * 1.0002f) + A) * 1.001f / fabsf(P0.r3[2]);
  const float mu = G.mu[2];
  const float Dw = D * 1.001f + 1e-6f * fabsf(mu);
  if (!(Dw <= FLT_MAX)) return;
  const float vlo = mu - Dw, vhi = mu + Dw;
  int a = lo, b = hi;  // first position with oz >= vlo
  while (a < b) {
    const int m = (a + b) >> 1;
    if (oz[m] < vlo) a = m + 1; else b = m;
  }
  int c = a, d = hi;  // first position with oz > vhi
  while (c < d) {
    const int m = (c + d) >> 1;
    if (oz[m] <= vhi) c = m + 1; else d = m;
  }
  lo = a;
  hi = c;
}

// ---------------------------------------------------------------- block scan
// Exclusive scan of one value per thread over a 256-thread block.
template <typename T>
__device__ __forceinline__ T block_exscan_256(T v, T* sh /*[4]*/, T& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  T before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const T s = sh[w];
    if (w < wave) before += s;
    total += s;
  }
  __syncthreads();
  return before + x - v;
}

// Sum of the first b block totals, by the whole block (coalesced reads).
__device__ __forceinline__ unsigned long long block_prefix(const uint32_t* __restrict__ tot, uint32_t b,
                                                           unsigned long long* sh /*[4]*/, uint32_t mask = ~0u) {
  unsigned long long s = 0;
  for (uint32_t i = threadIdx.x; i < b; i += 256) s += tot[i] & mask;
  unsigned long long t;
  block_exscan_256<unsigned long long>(s, sh, t);
  return t;
}

// ---------------------------------------------------------------- cull pass
// A group of LPG lanes per Gaussian, lane k of a group testing planes k,
// k + LPG, ...; the group ORs its bits.  A block covers gpb Gaussians in
// rounds of 256 / LPG.  Small inputs spread a Gaussian over several lanes
// (and blocks over fewer Gaussians) so enough waves run; large ones use one
// lane per Gaussian, whose plane loads are then uniform (scalar).  A pair
// becomes a record iff the conservative float test
// of Phase 1 (Eq. 13's box along the normal meets the plane, i.e. the plane
// meets the Eq. 12 ellipsoid) passes; the test only errs towards accepting a
// pair whose plane narrowly misses the ellipsoid, and such a record has an
// empty support, so it adds exactly zero everywhere.  Acceptance is kept as
// one bit per (Gaussian, plane), 64 planes per word.
//
// INIT (up to kInitPlanes planes, and no groups to search): the launch's
// planes are set up here, by every block for itself, instead of by a kernel
// before it (3 us and the wait for it: the setup takes the time of the
// Gaussians' loads).  The first block writes the constants the later kernels
// read, and what the setup kernel would have cleared, the control block, is
// written whole by the write pass; until then a block's flag travels in the
// top bit of its total.
constexpr int kInitPlanes = 64;
constexpr uint32_t kTotFlag = 0x80000000u;
template <int LPG, bool INIT>
__global__ __launch_bounds__(256) void k_cull_count(ug_gaussians g, ug_planes pl, const PlaneInt* __restrict__ pint,
                                                    PlaneConst* __restrict__ pc, const PlaneCull* __restrict__ pcf,
                                                    const PlaneGroups* __restrict__ pg, RenderParams rp, int gpb,
                                                    uint32_t* __restrict__ cnt_rec,
                                                    unsigned long long* __restrict__ accbits,
                                                    uint32_t* __restrict__ blk_tot, Ctrl* __restrict__ ctrl) {
  __shared__ uint32_t s_tot, s_flag;
  __shared__ PlaneCull s_pcf[INIT ? kInitPlanes : 1];
  // grouped planes (one lane per Gaussian): each group is searched for the
  // window of planes the pre-test can accept, and only those are tested
  __shared__ uint16_t s_perm[kGroupMaxPlanes], s_end[kGroupMaxPlanes];
  __shared__ float s_oz[kGroupMaxPlanes];
  const bool grouped = !INIT && LPG == 1 && pg->use != 0u;  // uniform
  if (grouped) {
    for (int j = (int)threadIdx.x; j < rp.p; j += 256) {
      s_perm[j] = (uint16_t)pg->perm[j];
      s_end[j] = (uint16_t)pg->end[j];
      s_oz[j] = pg->oz[j];
    }
  }
  if (threadIdx.x == 0) s_tot = s_flag = 0;
  if (INIT) {
    __syncthreads();
    const int p = (int)threadIdx.x;
    if (p < rp.p) {
      s_pcf[p] = plane_setup(pl, pint, p, pc, blockIdx.x == 0);
      if (!s_pcf[p].valid) s_flag = 1u;
    }
  } else if (blockIdx.x == 0 && threadIdx.x == 0) {
    for (int p = 0; p < rp.p; ++p)
      if (!pcf[p].valid) {
        atomicOr(&ctrl->flags, kFlagNonfinite);
        break;
      }
  }
  __syncthreads();
  const int nch = (rp.p + 63) / 64;
  const int sub = LPG == 1 ? 0 : (int)threadIdx.x % LPG;
  uint32_t mine = 0;
  for (int r0 = 0; r0 < gpb; r0 += 256 / LPG) {
    const int gi = blockIdx.x * gpb + r0 + (int)threadIdx.x / LPG;
    const bool has = gi < rp.n;
    GaussT<float> G;
    G.finite = false;
    if (has) load_gauss<float>(g, gi, rp.beta, G, true);
    if (has && sub == 0 && !G.finite) {
      if (INIT) s_flag = 1u;
      else atomicOr(&ctrl->flags, kFlagNonfinite);
    }
    const bool live = has && G.finite;
    uint32_t count = 0;
    if (grouped) {
      // at most 256 planes: four acceptance words, the word of plane q picked
      // by compares (no indexed register array)
      unsigned long long w0 = 0ull, w1 = 0ull, w2 = 0ull, w3 = 0ull;
      if (live) {
        for (int i = 0; i < rp.p;) {  // uniform: the groups in order
          const int e = min(max((int)s_end[i], i + 1), rp.p);  // a group ends past its start
          // the group's shared constants; each plane differs only in o[2]
          PlaneCull pf = pcf[s_perm[i]];
          const float S33 = cull_s33(G, pf);
          int lo = i, hi = pf.valid ? e : i;
          if ((uint32_t)(e - i) >= kGroupSearch) group_window(G, pf, S33, rp.chi2, s_oz, lo, hi);
          for (int j = lo; j < hi; ++j) {
            const int q = s_perm[j];
            pf.o[2] = s_oz[j];
            if (cull_test(G, pf, S33, rp.chi2)) {
              const unsigned long long bit = 1ull << (q & 63);
              const int w = q >> 6;
              w0 |= w == 0 ? bit : 0ull;
              w1 |= w == 1 ? bit : 0ull;
              w2 |= w == 2 ? bit : 0ull;
              w3 |= w == 3 ? bit : 0ull;
            }
          }
          i = e;
        }
      }
      if (has) {
        for (int c = 0; c < nch; ++c)
          accbits[(size_t)gi * nch + c] = c == 0 ? w0 : (c == 1 ? w1 : (c == 2 ? w2 : w3));
        count = (uint32_t)(__popcll(w0) + __popcll(w1) + __popcll(w2) + __popcll(w3));
        cnt_rec[gi] = count;
        mine += count;
      }
      continue;
    }
    for (int c = 0; c < nch; ++c) {
      const int pend = min(64, rp.p - c * 64);
      unsigned long long bits = 0;
      for (int j = sub; j < pend; j += LPG) {
        const PlaneCull pf = INIT ? s_pcf[j] : pcf[c * 64 + j];
        if (live && pf.valid && cull_maybe(G, pf, rp.chi2)) bits |= 1ull << j;
      }
#pragma unroll
      for (int o = 1; o < LPG; o <<= 1) bits |= __shfl_xor(bits, o, 64);
      if (has && sub == 0) accbits[(size_t)gi * nch + c] = bits;
      count += (uint32_t)__popcll(bits);
    }
    if (has && sub == 0) {
      cnt_rec[gi] = count;
      mine += count;
    }
  }
  if (mine) atomicAdd(&s_tot, mine);
  __syncthreads();
  if (threadIdx.x == 0) blk_tot[blockIdx.x] = s_tot | (s_flag ? kTotFlag : 0u);
}

// Offsets and the compact (Gaussian, plane) list, Gaussian-major with planes
// ascending.  A block covers m consecutive count blocks (gpb Gaussians in
// all).  The last block publishes the total and the capacity check; with INIT
// (see the count pass) it writes the whole control block.
template <bool INIT>
__global__ __launch_bounds__(256) void k_cull_write(RenderParams rp, int gpb, uint32_t m, uint32_t nblk, uint32_t ncnt,
                                                    const uint32_t* __restrict__ cnt_rec,
                                                    const unsigned long long* __restrict__ accbits,
                                                    const uint32_t* __restrict__ blk_tot,
                                                    unsigned long long* __restrict__ off_rec,
                                                    uint2* __restrict__ rec_pair, Ctrl* __restrict__ ctrl) {
  __shared__ unsigned long long s_sh[4];
  const int nch = (rp.p + 63) / 64;
  // the first round's counts and first acceptance word do not depend on the
  // block prefix: load them before it so the two round trips overlap
  const int gi0 = blockIdx.x * gpb + threadIdx.x;
  const bool has0 = (int)threadIdx.x < gpb && gi0 < rp.n;
  const unsigned long long cnt0 = has0 ? cnt_rec[gi0] : 0ull;
  const unsigned long long bits0 = has0 ? accbits[(size_t)gi0 * nch] : 0ull;
  unsigned long long carry = block_prefix(blk_tot, blockIdx.x * m, s_sh, INIT ? ~kTotFlag : ~0u);
  for (int r0 = 0; r0 < gpb; r0 += 256) {
    const int gi = blockIdx.x * gpb + r0 + threadIdx.x;
    const bool has = r0 + (int)threadIdx.x < gpb && gi < rp.n;
    const unsigned long long cnt = r0 == 0 ? cnt0 : (has ? cnt_rec[gi] : 0ull);
    unsigned long long tot;
    const unsigned long long base = carry + block_exscan_256<unsigned long long>(cnt, s_sh, tot);
    carry += tot;
    if (!has) continue;
    off_rec[gi] = base;
    unsigned long long r = base;
    for (int c = 0; c < nch; ++c) {
      unsigned long long bits = (r0 == 0 && c == 0) ? bits0 : accbits[(size_t)gi * nch + c];
      while (bits) {
        const int j = __builtin_ctzll(bits);
        bits &= bits - 1ull;
        if (r < rp.rec_cap) rec_pair[r] = make_uint2((uint32_t)gi, (uint32_t)(c * 64 + j));
        ++r;
      }
    }
  }
  uint32_t flag = 0u;
  if (INIT && blockIdx.x == nblk - 1) {  // uniform
    for (uint32_t i = threadIdx.x; i < ncnt; i += 256) flag |= blk_tot[i] & kTotFlag;
    flag = __syncthreads_or((int)flag) ? kFlagNonfinite : 0u;
  }
  if (blockIdx.x == nblk - 1 && threadIdx.x == 0) {
    ctrl->n_rec = carry;
    if (INIT) {
      ctrl->n_key = 0;
      ctrl->n_eval = 0;
      ctrl->n_exec = 0;
      ctrl->n_key_eff = 0;
      ctrl->flags = flag | (carry > rp.rec_cap ? kFlagRecCap : 0u);
    } else if (carry > rp.rec_cap) {
      atomicOr(&ctrl->flags, kFlagRecCap);
    }
    ctrl->n_rec_eff = carry <= rp.rec_cap ? (uint32_t)carry : 0u;
  }
}

// ---------------------------------------------------------------- record pass
// Lanes = records (every lane an accepted pair: no divergence); a block
// covers rpb consecutive records in rounds of 256.

// Records per block from the device-side record count: whole rounds of 256
// spread evenly over the grid (sized by the host for the capacity), so every
// block has a share whatever the head-room.  The record and emission kernels
// use the same split (the emission's block prefix reads the record blocks'
// totals).
__device__ __forceinline__ uint32_t record_rpb_dev(uint32_t nrec, uint32_t grid) {
  const uint32_t rounds = (nrec + 255u) / 256u;
  const uint32_t per = (rounds + grid - 1u) / grid;
  return (per < 1u ? 1u : per) * 256u;
}

// Records per run: whole waves of 64, in up to kRuns runs per block (four at 256
// records per block: an eighth of a block, 32, left half of every wave's lanes
// idle up to 524,288 records).
__device__ __forceinline__ uint32_t record_run_dev(uint32_t rpb) {
  return (rpb / kRuns + 63u) & ~63u;
}

// What the emission's items need of a record, in LDS (80 bytes, read 16 at a
// time).
struct EmitRec {
  float4 mask0;  // BandMask: t22, a, i11, d
  float4 mask1;  // dvr, fu, fv, and ub's bits
  uint4 at;      // vb's bits, first key, one past the last, first item
  uint4 geo;     // tx0 | tx1 << 16, ty0, RowSpans
  uint4 plane;   // first tile, tile columns, W | H << 16, flags: 1 no cut-off, 2 has support
};

// Writes the keys of a wave's records (its lanes'): lanes = items (record,
// tile row), 64 at a time in record order, so a record with many rows does
// not hold up the others and the keys of neighbouring lanes are neighbours in
// memory.  A lane walking its record's rows took 418 us at 16.2M records with
// 33.5M keys (398 so, 2.8 TB/s of slots read and keys written), 198 at 3.6M
// needles with 11.8M keys (135), 123 at 2.1M with 25M (96); bound by its VALU
// instructions (72 to 77% of the issue) beside those stores.  The tile shape is a
// template argument: band loops and masks without run-time bounds gave 475 ->
// 441 us at 69M keys.  nr = the lane's record's tile rows (0: no keys), key = the wave's
// first key; an item's first key is the number of keys of the items before
// it.  Of every PARTS chunks of 64 items only the part-th is written.
template <uint32_t PARTS, int TW, int TH>
__device__ __forceinline__ void emit_items(const EmitRec* __restrict__ s_rec, uint32_t* __restrict__ s_mark,
                                           const Rec* __restrict__ recs, const RenderParams& rp, uint32_t r0,
                                           uint32_t nr, uint32_t first_item, uint32_t items, uint32_t key,
                                           uint32_t part, uint32_t* __restrict__ key_tile,
                                           uint32_t* __restrict__ rec_of_key) {
  constexpr int NB = TH / kSubBlock, K = TW / kSubBlock;
  constexpr int mshift = key_mask_shift(TW, TH);
  const uint32_t last_index = (1u << (mshift - rp.tile_bits)) - 1u;  // indices from here on: looked up
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t open = 0u;  // 1 + the record whose items the chunk starts with
  for (uint32_t base = 0, chunk = 0; base < items; base += 64, ++chunk) {
    // the lane's record: the last one that starts at or before its item
    s_mark[lane] = 0u;
    wave_lds_sync();
    if (nr > 0 && first_item - base < 64u) s_mark[first_item - base] = lane + 1u;
    wave_lds_sync();
    uint32_t m = s_mark[lane];
    if (lane == 0) m = max(m, open);
    m = wave_incl_max(m);
    open = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
    wave_lds_sync();
    const bool has = base + lane < items;
    const uint32_t rl = m - 1u;  // the first item starts a record: m > 0
    const EmitRec& R = s_rec[rl];
    const uint4 at = R.at, geo = R.geo, plane = R.plane;
    const int gx0 = (int)(geo.x & 0xffffu), gx1 = (int)(geo.x >> 16);
    const int W = (int)(plane.z & 0xffffu), H = (int)(plane.z >> 16);
    const int i = (int)(base + lane - at.w), ty = (int)geo.y + i;
    const int umin = gx0 * TW, umax = min(gx1 * TW + TW - 1, W - 1);
    int tx0 = gx0, tx1 = has ? gx1 : gx0 - 1;
    if (rp.by_rows && has) {
      // the record kernel's span for the rows it kept, else recomputed
      const int bits = span_bits(gx1 - gx0), at_bit = bits * i;
      if (at_bit + bits <= 32) {
        const uint32_t mask = (1u << bits) - 1u;
        tx0 = gx0 + (int)(geo.z >> at_bit & mask);
        tx1 = gx0 + (int)(geo.w >> at_bit & mask);
      } else {
        BandPrep bp;
        if (!band_prep(recs[r0 + rl].acc, (int)__float_as_uint(R.mask1.w), (int)at.x, bp) ||
            !rows_span(bp, ty, TW, TH, H, umin, umax, tx0, tx1))
          tx1 = tx0 - 1;
      }
    }
    const uint32_t len = (uint32_t)max(tx1 - tx0 + 1, 0);
    const uint32_t incl = wave_incl_sum(len);
    uint32_t e = key + incl - len;
    key += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    if (PARTS > 1 && chunk % PARTS != part) continue;  // uniform
    const float4 m0 = R.mask0, m1 = R.mask1;
    const BandMask bm{m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, (int)__float_as_uint(m1.w), (int)at.x,
                      (plane.w & 1u) != 0u};
    // rows below the centre's: the tile row's first and the plane's last
    const float y0 = (float)(ty * TH - bm.vb) - bm.fv, yl = (float)(H - 1 - bm.vb) - bm.fv;
    int ca[NB], cz[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float ya = y0 + (float)(b * kSubBlock), yb = fminf(ya + (float)(kSubBlock - 1), yl);
      band_mask_cols(bm, ya, yb, umin, umax, ca[b], cz[b]);
      if (!(plane.w & 2u) || ty * TH + b * kSubBlock >= H) cz[b] = ca[b] - 1;
    }
    const uint32_t tile0 = plane.x + (uint32_t)ty * plane.y;
    const uint32_t r = r0 + rl;
    for (int tx = tx0; tx <= tx1; ++tx, ++e) {
      const uint32_t index = e - at.y;
      if (index < at.z - at.y) {
        key_tile[e] = (tile0 + (uint32_t)tx) | min(index, last_index) << rp.tile_bits |
                      (tile_mask<NB, K>(ca, cz, tx) << mshift);
        rec_of_key[e] = r;
      }
    }
  }
}

// Launches with up to kStagePlanes planes give the record kernel and the
// record adjoint their planes' constants from LDS (copied once per block)
// instead of gathering each record's plane from memory: a wave's 64 records
// touch many planes, and those gathers queue on the vector-memory address
// path.
constexpr int kStagePlanes = 256;

// A plane's PlaneRec in LDS: an odd number of doubles, so that the lanes'
// planes (mostly consecutive) start in different banks (24 of them put four
// planes in all banks between them, and the conflicts set the record kernel's
// time), then its size.
constexpr int kPlaneDoubles = 25;
constexpr size_t kPlaneLds = kPlaneDoubles * sizeof(double) + sizeof(int2);

__device__ __forceinline__ PlaneRec plane_rec(const PlaneConst& c, const PlaneInt& i) {
  return PlaneRec{plane_as<double>(c), c.cu, c.cv, 1.0 / c.sx, 1.0 / c.sy, i.W, i.H};
}
__device__ __forceinline__ void plane_rec_to_lds(const PlaneRec& q, double* d, int2* wh) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    d[k] = q.pose.o[k];
    d[12 + k] = q.pose.e1[k];
    d[15 + k] = q.pose.e2[k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) d[3 + k] = q.pose.rinv[k];
  d[18] = q.pose.absdet;
  d[19] = q.pose.sx;
  d[20] = q.pose.sy;
  d[21] = q.cu;
  d[22] = q.cv;
  d[23] = q.isx;
  d[24] = q.isy;
  *wh = make_int2(q.W, q.H);
}
__device__ __forceinline__ PlaneRec plane_rec_from_lds(const double* d, const int2& wh) {
  PlaneRec q;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    q.pose.o[k] = d[k];
    q.pose.e1[k] = d[12 + k];
    q.pose.e2[k] = d[15 + k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) q.pose.rinv[k] = d[3 + k];
  q.pose.absdet = d[18];
  q.pose.sx = d[19];
  q.pose.sy = d[20];
  q.cu = d[21];
  q.cv = d[22];
  q.isx = d[23];
  q.isy = d[24];
  q.W = wh.x;
  q.H = wh.y;
  return q;
}

// FP64 in-plane conic and footprint of each record; key counts and the
// block's total.  STAGE (launches of up to kStagePlanes planes): the planes'
// constants are copied to LDS once per block (512 threads: the 52 KB of a
// 256-plane launch and the slots' 20 KB leave the 16 waves per CU the
// registers allow)
// instead of being gathered per record from memory.
//
// Bound by its FP64 arithmetic (760 VALU instructions per 64 records, 78% of
// the issue).  16.2M records on 256 planes: 575 us with exact divisions and
// roots, plane constants 24 doubles apart and every lane storing its own
// slot; 567 without the exact forms, 548 without the bank conflicts too, 443
// with the slots stored through LDS (2.5 TB/s written).
// BOX: the paper-literal box support (a template argument, so that its exact
// divisions take none of the other records' registers, which are at the limit).
// chi2 is passed as the double it is used as, in scalar registers.
template <bool STAGE, bool BOX>
__global__ __launch_bounds__(STAGE ? 512 : 256, STAGE ? 4 : 3) void k_record(ug_gaussians g, const PlaneConst* __restrict__ pc,
                                                              const PlaneInt* __restrict__ pint, RenderParams rp,
                                                              const uint2* __restrict__ rec_pair,
                                                              Rec* __restrict__ recs, uint32_t* __restrict__ rec_nkey,
                                                              uint32_t* __restrict__ blk_tot,
                                                              Ctrl* __restrict__ ctrl, double chi2_arg) {
  constexpr uint32_t NT = STAGE ? 512u : 256u;
  extern __shared__ double s_planes[];  // STAGE: rp.p x kPlaneDoubles, then rp.p sizes
  constexpr int kSlotPitch = 5;  // float4 per slot in LDS: four and one of padding
  __shared__ float4 s_slot[NT / 64][32 * kSlotPitch];
  __shared__ uint32_t s_tot, s_counted;
  const uint32_t nrec = ctrl->n_rec_eff;
  const uint32_t rpb = record_rpb_dev(nrec, gridDim.x);
  const uint32_t r_begin = blockIdx.x * rpb;
  if (r_begin >= nrec) return;  // uniform
  int2* s_wh = reinterpret_cast<int2*>(s_planes + (size_t)kPlaneDoubles * rp.p);
  if (STAGE) {
    for (int q = (int)threadIdx.x; q < rp.p; q += (int)NT)
      plane_rec_to_lds(plane_rec(pc[q], pint[q]), s_planes + kPlaneDoubles * q, s_wh + q);
  }
  if (threadIdx.x == 0) s_tot = s_counted = 0;
  __syncthreads();
  const bool rows = rp.by_rows != 0;  // the records carry their row spans
  uint32_t mine = 0, counted = 0;
  const uint32_t r_end = min(r_begin + rpb, nrec);
  // A wave builds whole runs, so a record's key offset within its run needs
  // no other wave (a barrier per round for offsets within the block made the
  // kernel 25% slower).
  const uint32_t len = record_run_dev(rpb);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t run = (uint32_t)wave; run < kRuns; run += NT / 64) {
    const uint32_t run_end = min(r_begin + (run + 1u) * len, r_end);
    uint32_t carry = 0;  // keys of the run so far
    for (uint32_t r0 = r_begin + run * len; r0 < run_end; r0 += 64) {
      const uint32_t r = r0 + (uint32_t)lane;
      Rec out{};
      uint32_t nk = 0;
      if (r < run_end) {
        Footprint f;
        const uint2 gp = rec_pair[r];
        GaussIn G;
        load_gauss(g, (int)gp.x, (double)rp.beta, G, BOX);
        double chi2 = chi2_arg;
        asm volatile("" : "+s"(chi2));  // its products are not kept from record to record in vector registers
        const PlaneRec Q = STAGE ? plane_rec_from_lds(s_planes + kPlaneDoubles * gp.y, s_wh[gp.y])
                                 : plane_rec(pc[gp.y], pint[gp.y]);
        Conic k;
        const bool meets = conic_cull(G, Q.pose, chi2, k);
        conic_full(G, Q.pose, k);
        // Box support: the FP64 Phase-1 decision is final (a pair the
        // conservative float cull let through would otherwise fill its box).
        const bool ok = BOX ? (meets && make_box_record(G, Q, k, chi2, f))
                            : make_footprint(G, Q, k, chi2, rp.box_mode, rows, rp.tile_w, rp.tile_h, f);
        if (!ok) {
          // the plane cuts the ellipsoid (or box) outside the image: a record with no keys
          f.keys = f.counted = 0;
          f.acc = RecAcc{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          f.geo = RecGeo{0, 0, 0, 0, 1, 0, 1, 0};
          f.spans = RowSpans{0u, 0u};
        }
        rec_nkey[r] = nk = f.keys;
        counted += f.counted;
        out = Rec{f.acc, f.geo, f.spans};
      }
      const uint32_t incl = wave_incl_sum(nk);
      out.geo.run = blockIdx.x * kRuns + run;
      out.geo.koff = carry + incl - nk;
      carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      // The slots go out through LDS, half the wave's at a time: every store
      // then writes whole 64-byte slots side by side.  A lane storing its own
      // slot sixteen bytes at a time makes four requests of it, and the L2's
      // write requests set the kernel's time.
      const float4* src = reinterpret_cast<const float4*>(&out);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        wave_lds_sync();
        if ((lane >> 5) == h) {
#pragma unroll
          for (int q = 0; q < 4; ++q) s_slot[wave][(lane & 31) * kSlotPitch + q] = src[q];
        }
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const uint32_t rr = (uint32_t)(i * 16 + (lane >> 2)), to = r0 + (uint32_t)(32 * h) + rr;
          if (to < run_end) reinterpret_cast<float4*>(recs + to)[lane & 3] = s_slot[wave][rr * kSlotPitch + (lane & 3)];
        }
      }
    }
    mine += carry;
  }
  // with PAPER boxes binned by rows the reported key count is the rectangles'
  const bool rect = rows && rp.box_mode == UG_BOX_PAPER;
  if (lane == 0 && mine) atomicAdd(&s_tot, mine);
  if (rect && counted) atomicAdd(&s_counted, counted);
  __syncthreads();
  if (threadIdx.x == 0) {
    blk_tot[blockIdx.x] = s_tot;
    if (rect && s_counted) atomicAdd(&ctrl->n_key, (unsigned long long)s_counted);
  }
}

// Launches of up to kEmitPartBlocks record blocks give every block's records
// to kEmitParts blocks, each writing the part-th of every kEmitParts chunks of
// items: so few blocks leave most CUs idle, and a CU that has one spends its
// time on the stores of its records' keys.  9 K records with 90 K keys (36
// blocks): 14 us with one block each, 9.5 with four.  The line: at 400 blocks
// the four repeat the prefix and the scan for nothing (10.8 us against 14.7 at
// 79 K records with 160 K keys).
constexpr uint32_t kEmitParts = 4, kEmitPartBlocks = 128;

// Key offsets (block prefix + in-block scan) and key emission.  The last
// active block publishes the key total and the capacity check.
template <uint32_t PARTS, int TW, int TH>
__global__ __launch_bounds__(256) void k_emit(const PlaneInt* __restrict__ pint, RenderParams rp,
                                              const uint2* __restrict__ rec_pair, const Rec* __restrict__ recs,
                                              const uint32_t* __restrict__ rec_nkey,
                                              const uint32_t* __restrict__ blk_tot, uint32_t* __restrict__ rec_koff,
                                              uint32_t* __restrict__ run_koff, Ctrl* __restrict__ ctrl, uint32_t* __restrict__ key_tile,
                                              uint32_t* __restrict__ rec_of_key) {
  __shared__ unsigned long long s_sh[4];
  __shared__ EmitRec s_rec[256];
  __shared__ uint32_t s_mark[256];
  const uint32_t nrec = ctrl->n_rec_eff;
  const uint32_t blk = blockIdx.x / PARTS, part = blockIdx.x % PARTS;
  const uint32_t rpb = record_rpb_dev(nrec, gridDim.x / PARTS);
  const uint32_t r_begin = blk * rpb;
  if (r_begin >= nrec) return;  // uniform
  const uint32_t nact = (nrec + rpb - 1) / rpb;
  const uint32_t r_end = min(r_begin + rpb, nrec);
  // Each round's record data is loaded one round ahead (the first round's
  // before the block prefix), so its round trip overlaps the previous
  // round's scan and emission.  Lanes past the block's records load its last
  // record and drop it (no branch around the loads: the wait at a branch's
  // join would take every load in flight).  The plane lookup needs the plane
  // index first; it is issued at the end of the previous round, before the
  // next prefetch, so the emission waits for it and not for the prefetch
  // (loads complete in issue order as far as the waits can tell).
  uint32_t r = r_begin + threadIdx.x;
  bool act = r < r_end;
  uint32_t pl, nk;
  RecAcc ra;
  RecGeo ge;
  RowSpans sp;
  {
    const uint32_t rl = act ? r : r_end - 1u;
    pl = rec_pair[rl].y;
    ra = recs[rl].acc;
    ge = recs[rl].geo;
    sp = recs[rl].spans;
    nk = act ? rec_nkey[rl] : 0u;
  }
  unsigned long long carry = block_prefix(blk_tot, blk, s_sh);
  PlaneInt PI = pint[pl];
  for (uint32_t r0 = r_begin; r0 < r_end; r0 += 256) {
    const uint32_t rn = r + 256u;
    const bool actn = rn < r_end;
    const uint32_t rl = actn ? rn : r_end - 1u;
    const uint32_t pln = rec_pair[rl].y;
    const RecAcc ran = recs[rl].acc;
    const RecGeo gen = recs[rl].geo;
    const RowSpans spn = recs[rl].spans;
    const uint32_t nkl = rec_nkey[rl];
    const uint32_t nkn = actn ? nkl : 0u;
    unsigned long long tot;
    const unsigned long long koff = carry + block_exscan_256<unsigned long long>(nk, s_sh, tot);
    carry += tot;
    if (act) {
      if (part == 0) rec_koff[r] = (uint32_t)(koff < rp.key_cap ? koff : rp.key_cap);
    }
    // (key offsets only grow: the records that fit come first)
    const uint32_t nr = act && nk > 0 && koff + nk <= rp.key_cap ? (uint32_t)(ge.ty1 - ge.ty0 + 1) : 0u;
    const uint32_t rows_incl = wave_incl_sum(nr);
    const uint32_t items = (uint32_t)__builtin_amdgcn_readlane((int)rows_incl, 63);
    if (items) {  // uniform over the wave
      BandMask bm;
      const bool ok = band_mask_prep(ra, ge.ub, ge.vb, bm);
      EmitRec& R = s_rec[threadIdx.x];
      R.mask0 = make_float4(bm.t22, bm.a, bm.i11, bm.d);
      R.mask1 = make_float4(bm.dvr, bm.fu, bm.fv, __uint_as_float((uint32_t)ge.ub));
      R.at = make_uint4((uint32_t)ge.vb, (uint32_t)koff, (uint32_t)koff + nk, rows_incl - nr);
      R.geo = make_uint4((uint32_t)ge.tx0 | (uint32_t)ge.tx1 << 16, ge.ty0, sp.first, sp.last);
      R.plane = make_uint4(PI.tile_off, (uint32_t)PI.ntx, (uint32_t)PI.W | (uint32_t)PI.H << 16,
                           (bm.all ? 1u : 0u) | (ok ? 2u : 0u));
      const uint32_t w0 = threadIdx.x & ~63u;
      emit_items<PARTS, TW, TH>(s_rec + w0, s_mark + w0, recs, rp, r0 + w0, nr, rows_incl - nr, items,
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)koff), part, key_tile, rec_of_key);
    }
    r = rn;
    act = actn;
    nk = nkn;
    ra = ran;
    ge = gen;
    sp = spn;
    PI = pint[pln];
  }
  if (part != 0) return;
  __syncthreads();  // rec_koff of the block's records
  if (threadIdx.x < kRuns) {
    const uint32_t rr = r_begin + threadIdx.x * record_run_dev(rpb);
    if (rr < r_end) run_koff[blk * kRuns + threadIdx.x] = rec_koff[rr];
  }
  if (blk == nact - 1 && threadIdx.x == 0) {
    const unsigned long long counted = rp.by_rows && rp.box_mode == UG_BOX_PAPER ? ctrl->n_key : carry;
    ctrl->n_key = counted;
    const bool ok = counted <= rp.key_cap;
    if (!ok) atomicOr(&ctrl->flags, kFlagKeyCap);
    ctrl->n_key_eff = ok ? (uint32_t)carry : 0u;
    rec_koff[nrec] = ok ? (uint32_t)carry : 0u;
  }
}

// ---------------------------------------------------------------- adjoint
// Final gradient of Gaussian i from the sum of its records' contributions
// (dmu[3], dL[6], da, dc): dL_kk / dl_kk = 2 l_kk (Eq. 11).
__device__ __forceinline__ void write_gauss_grad(const ug_gaussians& g, int i, const float (&acc)[kGradFields],
                                                 float* __restrict__ d_means, float* __restrict__ d_lraw,
                                                 float* __restrict__ d_int, float* __restrict__ d_op, int accumulate) {
  float v[kGradFields];
#pragma unroll
  for (int j = 0; j < kGradFields; ++j) v[j] = acc[j];
  v[3] *= 2.f * g.lraw[6 * i + 0];
  v[6] *= 2.f * g.lraw[6 * i + 3];
  v[8] *= 2.f * g.lraw[6 * i + 5];
  if (accumulate) {
    for (int j = 0; j < 3; ++j) d_means[3 * i + j] += v[j];
    for (int j = 0; j < 6; ++j) d_lraw[6 * i + j] += v[3 + j];
    d_op[i] += v[9];
    d_int[i] += v[10];
  } else {
    for (int j = 0; j < 3; ++j) d_means[3 * i + j] = v[j];
    for (int j = 0; j < 6; ++j) d_lraw[6 * i + j] = v[3 + j];
    d_op[i] = v[9];
    d_int[i] = v[10];
  }
}

// Lanes = records, 64 consecutive records per wave: the sum of the record's
// keys' partial derivatives (contiguous in emission order), the chain rule
// through the record construction (FP32: the adjoint's tolerance is 1e-3),
// then the per-Gaussian sum.  A Gaussian's records are contiguous, so equal
// Gaussian ids are added with a segmented scan across the wave; a Gaussian
// whose records all sit in one wave gets its gradient here.  Each wave also
// leaves its first and last segment sums in side[] for the Gaussians that
// span waves (k_gauss_grad).  Deterministic, no atomics.
// Float plane constants as the record adjoint stages them in LDS (o, R^-1,
// e1, e2, |det R|, sx, sy).
constexpr int kPlaneFloats = 21;

__device__ __forceinline__ void plane_to_lds(const PlaneT<float>& P, float* d) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    d[k] = P.o[k];
    d[12 + k] = P.e1[k];
    d[15 + k] = P.e2[k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) d[3 + k] = P.rinv[k];
  d[18] = P.absdet;
  d[19] = P.sx;
  d[20] = P.sy;
}

__device__ __forceinline__ PlaneT<float> plane_from_lds(const float* d) {
  PlaneT<float> P;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    P.o[k] = d[k];
    P.e1[k] = d[12 + k];
    P.e2[k] = d[15 + k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) P.rinv[k] = d[3 + k];
  P.absdet = d[18];
  P.sx = d[19];
  P.sy = d[20];
  return P;
}


// How a record's partials are added (always in emission order, so all three
// give the same bits):
//  - COOP, launches of up to kCoopBlocks waves of records: a block per 64
//    records, eight lanes to a record, one value each.  Few waves have the
//    chip to themselves and the time is the longest one's.  The block brings
//    its keys through LDS, 256 at a time: 9 K records with 90 K keys, some with
//    hundreds each, 29 us with a lane walking its record's keys, 12.5 here.
//    Where that takes many rounds and the records' lengths are alike (the
//    longest's kCoopEven times or more in the block), it would leave all but a
//    group or two waiting, and each group reads its own records' keys instead,
//    eight in flight: 3,840 records of 256 keys 68 us a lane each, 184 staged,
//    34 so; 24,000 of 100 keys 33, 40 and 20; 400 of 13,375 keys 5.1 ms, 9.2
//    and 1.9.  (A round of 256 keys takes 2.7 us if they are one record's and
//    under 1 if they are ten's; eight keys of every group 1.1, more out of cold
//    caches.  So it takes kCoopEvenKeys keys in the block: with a quarter of
//    that line the 9 K records above are 3 us slower on new inputs, with none
//    79 K records of two keys 0.6.  kCoopEven: at ten, 200,000 Gaussians on one
//    plane of 4000 x 3000 with records of uneven lengths took 318 us, 263 so.)
//  - kStagedKeys or more keys per record on average: the wave brings its keys
//    through LDS, loaded side by side while the ones before are added, a lane
//    per record.  25M keys of 2.1M records 138 us (190 with each lane reading
//    its record's from memory), 11.8M of 3.6M 124 (144).
//  - else each lane reads its own, two per step: 33M keys of 16M records 395
//    us, 420 through LDS (two round trips per wave there as well, and the LDS
//    on top).
// Bound by its 640 VALU instructions per 64 records (a third of them the
// segmented scan) and the round trips before them: 16M records 410 us with
// exact divisions and the scan over LDS shuffles.
constexpr uint32_t kCoopBlocks = 2048;
constexpr uint32_t kCoopEven = 24, kCoopEvenKeys = 4096;
constexpr uint32_t kStagedKeys = 3;

// Adds to every value that of the lane the DPP control names, where that lane
// holds the same Gaussian (rows outside the mask, and lanes it names no lane
// for, see id ~0).
template <int kCtrl, int kRows>
__device__ __forceinline__ void seg_add(uint32_t gid, float (&v)[kGradFields]) {
  const uint32_t gu = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)gid, kCtrl, kRows, 0xf, false);
  const bool add = gu == gid;
#pragma unroll
  for (int j = 0; j < kGradFields; ++j) {
    const float y = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v[j]), kCtrl, kRows, 0xf, true));
    v[j] += add ? y : 0.f;
  }
}

template <bool COOP>
__global__ __launch_bounds__(256) void k_record_adjoint(ug_gaussians g, const PlaneConst* __restrict__ pc,
                                                        RenderParams rp, const Ctrl* __restrict__ ctrl,
                                                        const uint2* __restrict__ rec_pair,
                                                        const uint32_t* __restrict__ rec_koff,
                                                        const float4* __restrict__ partial,
                                                        const uint32_t* __restrict__ cnt_rec,
                                                        const unsigned long long* __restrict__ off_rec,
                                                        float* __restrict__ side, float* __restrict__ d_means,
                                                        float* __restrict__ d_lraw, float* __restrict__ d_int,
                                                        float* __restrict__ d_op, int accumulate) {
  extern __shared__ float s_plane[];  // rp.p x kPlaneFloats when staged
  constexpr int kKeyPitch = 3;        // float4 per key in LDS: two and one of padding (banks)
  constexpr int kSumPitch = 9;
  __shared__ float4 s_key[COOP ? 512 : 4 * 64 * kKeyPitch];
  __shared__ float s_sum[COOP ? 64 * kSumPitch : 1];
  const bool staged = rp.p <= kStagePlanes;
  if (staged) {
    for (int q = threadIdx.x; q < rp.p; q += 256) plane_to_lds(plane_as<float>(pc[q]), s_plane + q * kPlaneFloats);
    __syncthreads();
  }
  const bool ok = (ctrl->flags & (kFlagRecCap | kFlagKeyCap)) == 0;
  const uint32_t nrec = ok ? ctrl->n_rec_eff : 0u;
  const uint32_t nw = (nrec + 63u) / 64u;
  const float chi2 = rp.chi2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool many = COOP || (unsigned long long)(ok ? ctrl->n_key_eff : 0u) >= (unsigned long long)kStagedKeys * nrec;
  uint32_t w = COOP ? blockIdx.x : blockIdx.x * 4u + (uint32_t)wave;
  for (; w < nw; w += COOP ? gridDim.x : gridDim.x * 4u) {
    if (COOP) {
      // eight neighbouring lanes add a record's keys, one value each, in order
      const uint32_t rb = w * 64u;
      const uint32_t ka = rec_koff[rb], kb = rec_koff[min(rb + 64u, nrec)];
      const int fq = (int)(threadIdx.x & 7u), q0 = (int)(threadIdx.x >> 3);
      uint32_t qa[2], qz[2];
      float acc[2] = {0.f, 0.f};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t rq = min(rb + (uint32_t)(q0 + 32 * h), nrec);
        qa[h] = rec_koff[rq];
        qz[h] = rq < nrec ? rec_koff[rq + 1] : qa[h];
      }
      // the first chunk, in flight while the form is decided
      const float4* p4 = partial + 2 * (size_t)ka;
      const uint32_t n4 = 2u * (kb - ka);
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
      if (threadIdx.x < n4) x = p4[threadIdx.x];
      if (threadIdx.x + 256u < n4) y = p4[threadIdx.x + 256u];
      bool even = false;  // uniform over the block
      if (kb - ka > kCoopEvenKeys) {
        const uint32_t rm = min(rb + (uint32_t)lane, nrec), len = rm < nrec ? rec_koff[rm + 1] - rec_koff[rm] : 0u;
        const uint32_t longest = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_max(len), 63);
        even = (uint64_t)(kb - ka) > (uint64_t)kCoopEven * longest;
      }
      if (even) {
        // each group reads its records' keys itself, eight at a time (an add
        // of zero behind the last)
        const float* p = reinterpret_cast<const float*>(partial) + fq;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          for (uint32_t k = qa[h]; k < qz[h]; k += 8) {
            float t[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) t[u] = p[8 * (size_t)min(k + u, qz[h] - 1u)];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) acc[h] += k + u < qz[h] ? t[u] : 0.f;
          }
        }
      } else {  // 256 keys at a time through LDS
        for (uint32_t kc = ka; kc < kb; kc += 256) {
          __syncthreads();  // the chunk before, and the block's sums before, are read
          s_key[threadIdx.x] = x;
          s_key[threadIdx.x + 256] = y;
          __syncthreads();
          const uint32_t nx = 2u * (kc + 256u - ka) + threadIdx.x;
          if (nx < n4) x = p4[nx];
          if (nx + 256u < n4) y = p4[nx + 256u];
          const float* sk = reinterpret_cast<const float*>(s_key);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t ke = min(qz[h], kc + 256u);
            uint32_t k = max(qa[h], kc);
            for (; k + 8u <= ke; k += 8) {
              float t[8];
#pragma unroll
              for (uint32_t u = 0; u < 8; ++u) t[u] = sk[8u * (k + u - kc) + (uint32_t)fq];
#pragma unroll
              for (int u = 0; u < 8; ++u) acc[h] += t[u];
            }
            for (; k < ke; ++k) acc[h] += sk[8u * (k - kc) + (uint32_t)fq];
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 2; ++h) s_sum[(q0 + 32 * h) * kSumPitch + fq] = acc[h];
      __syncthreads();
      if (wave != 0) continue;
    }
    const uint32_t r = w * 64u + (uint32_t)lane;
    const bool act = r < nrec;
    float v[kGradFields];
#pragma unroll
    for (int j = 0; j < kGradFields; ++j) v[j] = 0.f;
    uint32_t gid = 0xffffffffu;
    // lanes past the last record take it and no key of it; the Gaussian's
    // parameters are loaded with the key range, so the two round trips overlap
    const uint32_t rl = act ? r : nrec - 1u;
    const uint2 gp = rec_pair[rl];
    const uint32_t kend = rec_koff[rl + 1];
    const uint32_t k0 = act ? rec_koff[rl] : kend, k1 = kend;
    const GaussRaw gr = load_gauss_raw(g, (int)gp.x);
    const uint64_t goff = off_rec[gp.x];
    const uint32_t gcnt = cnt_rec[gp.x];
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), c = a;
    const uint32_t ka = (uint32_t)__builtin_amdgcn_readfirstlane((int)k0);
    const uint32_t kb = (uint32_t)__builtin_amdgcn_readlane((int)k1, 63);
    if constexpr (COOP) {
      const float* f = s_sum + lane * kSumPitch;
      a = make_float4(f[0], f[1], f[2], f[3]);
      c = make_float4(f[4], f[5], f[6], 0.f);
    } else if (!many) {
      // two keys per step, both loaded before either is added
      for (uint32_t k = k0; k < k1; k += 2) {
        const float4 x0 = partial[2 * (size_t)k], y0 = partial[2 * (size_t)k + 1];
        const bool two = k + 1 < k1;
        float4 x1 = make_float4(0.f, 0.f, 0.f, 0.f), y1 = x1;
        if (two) {
          x1 = partial[2 * (size_t)k + 2];
          y1 = partial[2 * (size_t)k + 3];
        }
        a.x += x0.x; a.y += x0.y; a.z += x0.z; a.w += x0.w;
        c.x += y0.x; c.y += y0.y; c.z += y0.z;
        a.x += x1.x; a.y += x1.y; a.z += x1.z; a.w += x1.w;
        c.x += y1.x; c.y += y1.y; c.z += y1.z;
      }
    } else if (ka < kb) {
      // the wave's keys are contiguous: 64 at a time
      float4* s_wave = s_key + wave * 64 * kKeyPitch;
      const size_t j = min(ka + (uint32_t)lane, kb - 1u);
      float4 x = partial[2 * j], y = partial[2 * j + 1];
      for (uint32_t kc = ka; kc < kb; kc += 64) {
        s_wave[lane * kKeyPitch] = x;
        s_wave[lane * kKeyPitch + 1] = y;
        if (kc + 64u < kb) {
          const size_t jn = min(kc + 64u + (uint32_t)lane, kb - 1u);
          x = partial[2 * jn];
          y = partial[2 * jn + 1];
        }
        wave_lds_sync();
        const uint32_t ke = min(k1, kc + 64u);
        for (uint32_t k = max(k0, kc); k < ke; ++k) {
          const float4 x0 = s_wave[(k - kc) * kKeyPitch], y0 = s_wave[(k - kc) * kKeyPitch + 1];
          a.x += x0.x; a.y += x0.y; a.z += x0.z; a.w += x0.w;
          c.x += y0.x; c.y += y0.y; c.z += y0.z;
        }
        wave_lds_sync();
      }
    }
    if (act) {
      gid = gp.x;
      if (k1 > k0) {
        const float dr[7] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z};
        GaussT<float> G;
        gauss_setup(gr, rp.beta, G);
        const PlaneT<float> P = staged ? plane_from_lds(s_plane + gp.y * kPlaneFloats) : plane_as<float>(pc[gp.y]);
        ConicT<float> k;
        conic_cull(G, P, chi2, k);
        conic_full(G, P, k);
        float dmu[3] = {0, 0, 0}, dL[6] = {0, 0, 0, 0, 0, 0}, da = 0.f, dc = 0.f;
        footprint_adjoint(G, P, k, dr, dmu, dL, da, dc);
        v[0] = dmu[0]; v[1] = dmu[1]; v[2] = dmu[2];
        for (int j = 0; j < 6; ++j) v[3 + j] = dL[j];
        v[9] = da;
        v[10] = dc;
      }
    }
    // segmented inclusive scan over equal Gaussian ids (ids are sorted): within
    // rows of 16 lanes, then over the rows
    seg_add<0x111, 0xf>(gid, v);  // lane - 1
    seg_add<0x112, 0xf>(gid, v);  // lane - 2
    seg_add<0x114, 0xf>(gid, v);  // lane - 4
    seg_add<0x118, 0xf>(gid, v);  // lane - 8
    seg_add<0x142, 0xa>(gid, v);  // the previous row's last lane, rows 1 and 3
    seg_add<0x143, 0xc>(gid, v);  // lane 31, rows 2 and 3
    const uint32_t gnext = __shfl_down(gid, 1, 64);
    const uint32_t g0 = __shfl(gid, 0, 64);
    const bool seg_end = act && (lane == 63 || gnext != gid);
    if (seg_end) {
      const uint64_t o = goff, e = o + gcnt;
      if (o >= (uint64_t)w * 64u && e <= (uint64_t)w * 64u + 64u)
        write_gauss_grad(g, (int)gid, v, d_means, d_lraw, d_int, d_op, accumulate);
      float* sd = side + (size_t)w * 2 * kGradFields;
      if (gid == g0) {
#pragma unroll
        for (int j = 0; j < kGradFields; ++j) sd[j] = v[j];
      }
      if (lane == 63 || r + 1 == nrec) {
#pragma unroll
        for (int j = 0; j < kGradFields; ++j) sd[kGradFields + j] = v[j];
      }
    }
  }
}

// One thread per Gaussian: zero gradient for a Gaussian without records,
// and the sum of the wave pieces for one whose records span waves (the
// first wave's last segment, whole middle waves, the last wave's first
// segment); the others were written by k_record_adjoint.
// With loss_out, block 0 also adds the adjoint accumulate's per-tile squared
// differences (nparts floats, in order, in FP64) into the mean squared error.
__global__ __launch_bounds__(256) void k_gauss_grad(ug_gaussians g, RenderParams rp, const Ctrl* __restrict__ ctrl,
                                                    const uint32_t* __restrict__ cnt_rec,
                                                    const unsigned long long* __restrict__ off_rec,
                                                    const float* __restrict__ side, float* __restrict__ d_means,
                                                    float* __restrict__ d_lraw, float* __restrict__ d_int,
                                                    float* __restrict__ d_op, int accumulate,
                                                    const float* __restrict__ loss_part, uint32_t nparts,
                                                    double inv_m, float* __restrict__ loss_out) {
  if (loss_out && blockIdx.x == 0) {  // uniform
    __shared__ double s_l[256];
    double a = 0.0;
    // 16 bytes per load (the array is aligned), eight loads in flight: the
    // block's round trips are the kernel's tail
    const float4* part4 = reinterpret_cast<const float4*>(loss_part);
    const uint32_t n4 = nparts / 4u;
    uint32_t k = threadIdx.x;
    for (; k + 7u * 256u < n4; k += 8u * 256u) {
      float4 x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = part4[k + 256u * (uint32_t)q];
#pragma unroll
      for (int q = 0; q < 8; ++q) a += ((double)x[q].x + (double)x[q].y) + ((double)x[q].z + (double)x[q].w);
    }
    for (; k < n4; k += 256) {
      const float4 x = part4[k];
      a += ((double)x.x + (double)x.y) + ((double)x.z + (double)x.w);
    }
    if (threadIdx.x < nparts % 4u) a += (double)loss_part[4u * n4 + threadIdx.x];
    s_l[threadIdx.x] = a;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) s_l[threadIdx.x] += s_l[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss_out[0] = (float)(s_l[0] * inv_m);
  }
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rp.n) return;
  const bool ok = (ctrl->flags & (kFlagRecCap | kFlagKeyCap)) == 0;
  const uint32_t nr = ok ? cnt_rec[i] : 0u;
  float acc[kGradFields];
#pragma unroll
  for (int j = 0; j < kGradFields; ++j) acc[j] = 0.f;
  if (nr > 0) {
    const uint64_t o = off_rec[i];
    const uint64_t wa = o / 64u, wb = (o + nr - 1u) / 64u;
    if (wa == wb) return;  // finished by k_record_adjoint
    const float* sa = side + (size_t)wa * 2 * kGradFields + kGradFields;
#pragma unroll
    for (int j = 0; j < kGradFields; ++j) acc[j] = sa[j];
    for (uint64_t w = wa + 1; w <= wb; ++w) {
      const float* sw = side + (size_t)w * 2 * kGradFields;
#pragma unroll
      for (int j = 0; j < kGradFields; ++j) acc[j] += sw[j];
    }
  }
  write_gauss_grad(g, i, acc, d_means, d_lraw, d_int, d_op, accumulate);
}

// ---------------------------------------------------------------- launchers
constexpr uint32_t kMaxScanBlocks = 2048;

// Lanes per Gaussian (log2) in the cull count: doubled while the lanes stay
// under 2^18 (a few waves per SIMD), up to one lane per plane and 64.
int cull_lpg_log2(int n, int p) {
  int l = 0;
  while (l < 6 && (1 << l) < p && ((long)n << l) < (1L << 18)) ++l;
  return l;
}

// Gaussians per cull block: whole count rounds (256 lanes), at most 2048
// blocks.
int cull_gpb(int n, int p) {
  const long unit = 256 >> cull_lpg_log2(n, p);
  const long rounds = ((long)n + unit - 1) / unit;
  const long per = (rounds + kMaxScanBlocks - 1) / kMaxScanBlocks;
  return (int)((per < 1 ? 1 : per) * unit);
}

uint32_t cull_blocks(int n, int p) {
  const int gpb = cull_gpb(n, p);
  return (uint32_t)((n + gpb - 1) / gpb);
}

// Records per record block: whole rounds of 256, at most 2048 blocks.
int record_rpb(uint32_t rec_cap) {
  const uint32_t rounds = (rec_cap + 255u) / 256u;
  const uint32_t per = (rounds + kMaxScanBlocks - 1) / kMaxScanBlocks;
  return (int)((per < 1 ? 1 : per) * 256u);
}

uint32_t record_blocks(uint32_t rec_cap) {
  const uint32_t rpb = (uint32_t)record_rpb(rec_cap);
  const uint32_t nb = (rec_cap + rpb - 1) / rpb;
  return nb < 1 ? 1 : nb;
}

hipError_t launch_init(const ug_planes& pl, const PlaneInt* pint, PlaneConst* pc, PlaneCull* pcf, PlaneGroups* pg,
                       bool group, Ctrl* ctrl, hipStream_t s) {
  const bool grp = group && pl.p >= 1 && pl.p <= kGroupMaxPlanes;  // one block
  const uint32_t blocks = grp ? 1u : ((uint32_t)pl.p + 255) / 256;
  if (grp)
    hipLaunchKernelGGL(k_init<true>, dim3(1), dim3(4 * kGroupMaxPlanes), 0, s, pl, pint, pc, pcf, pg, ctrl);
  else
    hipLaunchKernelGGL(k_init<false>, dim3(blocks < 1 ? 1 : blocks), dim3(256), 0, s, pl, pint, pc, pcf, pg, ctrl);
  return hipGetLastError();
}

size_t accbits_words(int n, int p) { return (size_t)n * (size_t)((p + 63) / 64); }

// The count pass sets the planes up itself (and the write pass the control
// block) where it tests every plane for every Gaussian anyway.
bool cull_inits(int n, int p) {
  return n > 0 && p <= kInitPlanes && (cull_lpg_log2(n, p) > 0 || p < (int)kGroupSearch);
}

hipError_t launch_cull_count(const ug_gaussians& g, const ug_planes& pl, const PlaneInt* pint, PlaneConst* pc,
                             const PlaneCull* pcf, const PlaneGroups* pg, const RenderParams& rp, uint32_t* cnt_rec,
                             unsigned long long* accbits, uint32_t* blk_tot, Ctrl* ctrl, hipStream_t s) {
  const uint32_t nb = cull_blocks(rp.n, rp.p);
  if (nb == 0) return hipGetLastError();  // no Gaussians: the zeroed totals stand
  const int gpb = cull_gpb(rp.n, rp.p);
  const bool init = cull_inits(rp.n, rp.p);
  switch (cull_lpg_log2(rp.n, rp.p)) {
#define UG_CULL(L)                                                                                                    \
  case L:                                                                                                             \
    if (init)                                                                                                         \
      hipLaunchKernelGGL((k_cull_count<(1 << L), true>), dim3(nb), dim3(256), 0, s, g, pl, pint, pc, pcf, pg, rp,     \
                         gpb, cnt_rec, accbits, blk_tot, ctrl);                                                       \
    else                                                                                                              \
      hipLaunchKernelGGL((k_cull_count<(1 << L), false>), dim3(nb), dim3(256), 0, s, g, pl, pint, pc, pcf, pg, rp,    \
                         gpb, cnt_rec, accbits, blk_tot, ctrl);                                                       \
    break;
    UG_CULL(0)
    UG_CULL(1)
    UG_CULL(2)
    UG_CULL(3)
    UG_CULL(4)
    UG_CULL(5)
    UG_CULL(6)
#undef UG_CULL
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_cull_write(const RenderParams& rp, const uint32_t* cnt_rec, const unsigned long long* accbits,
                             const uint32_t* blk_tot, unsigned long long* off_rec, uint2* rec_pair, Ctrl* ctrl,
                             hipStream_t s) {
  const uint32_t nb = cull_blocks(rp.n, rp.p);
  if (nb == 0) return hipGetLastError();
  // count blocks of fewer than 256 Gaussians are written m at a time
  const int gpb = cull_gpb(rp.n, rp.p);
  const uint32_t m = gpb < 256 ? (uint32_t)(256 / gpb) : 1u;
  const uint32_t nbw = (nb + m - 1) / m;
  if (cull_inits(rp.n, rp.p))
    hipLaunchKernelGGL(k_cull_write<true>, dim3(nbw), dim3(256), 0, s, rp, gpb * (int)m, m, nbw, nb, cnt_rec, accbits,
                       blk_tot, off_rec, rec_pair, ctrl);
  else
    hipLaunchKernelGGL(k_cull_write<false>, dim3(nbw), dim3(256), 0, s, rp, gpb * (int)m, m, nbw, nb, cnt_rec,
                       accbits, blk_tot, off_rec, rec_pair, ctrl);
  return hipGetLastError();
}

hipError_t launch_record(const ug_gaussians& g, const PlaneConst* pc, const PlaneInt* pint, const RenderParams& rp,
                         const uint2* rec_pair, Rec* recs, uint32_t* rec_nkey, uint32_t* blk_tot,
                         Ctrl* ctrl, hipStream_t s) {
  const bool stage = rp.p <= kStagePlanes;
  const size_t lds = stage ? (size_t)rp.p * kPlaneLds : 0;
  const dim3 grid(record_blocks(rp.rec_cap)), block(stage ? 512 : 256);
#define UG_RECORD(STAGE, BOX)                                                                                      \
  if (stage == STAGE && (rp.box_support != 0) == BOX)                                                              \
    hipLaunchKernelGGL((k_record<STAGE, BOX>), grid, block, lds, s, g, pc, pint, rp, rec_pair, recs, rec_nkey,     \
                       blk_tot, ctrl, (double)rp.chi2);
  UG_RECORD(true, false)
  UG_RECORD(false, false)
  UG_RECORD(true, true)
  UG_RECORD(false, true)
#undef UG_RECORD
  return hipGetLastError();
}

hipError_t launch_emit(const PlaneInt* pint, const RenderParams& rp, const uint2* rec_pair, const Rec* recs,
                       const uint32_t* rec_nkey, const uint32_t* blk_tot, uint32_t* rec_koff, uint32_t* run_koff,
                       Ctrl* ctrl, uint32_t* key_tile, uint32_t* rec_of_key, hipStream_t s) {
  const uint32_t blocks = (uint32_t)record_blocks(rp.rec_cap);
#define UG_EMIT_PARTS(PARTS, W, H)                                                                                   \
  hipLaunchKernelGGL((k_emit<PARTS, W, H>), dim3(blocks * PARTS), dim3(256), 0, s, pint, rp, rec_pair, recs, rec_nkey, \
                     blk_tot, rec_koff, run_koff, ctrl, key_tile, rec_of_key)
#define UG_EMIT(W, H)                            \
  if (rp.tile_w == W && rp.tile_h == H) {        \
    if (blocks <= kEmitPartBlocks)               \
      UG_EMIT_PARTS(kEmitParts, W, H);           \
    else                                         \
      UG_EMIT_PARTS(1, W, H);                    \
    return hipGetLastError();                    \
  }
  UG_TILE_SHAPES(UG_EMIT)
#undef UG_EMIT
#undef UG_EMIT_PARTS
  return hipErrorInvalidValue;
}

size_t adjoint_side_floats(uint32_t rec_cap) { return ((size_t)rec_cap + 63) / 64 * 2 * kGradFields; }

hipError_t launch_record_adjoint(const ug_gaussians& g, const PlaneConst* pc, const RenderParams& rp,
                                 const Ctrl* ctrl, const uint2* rec_pair, const uint32_t* rec_koff,
                                 const float* partial, const uint32_t* cnt_rec, const unsigned long long* off_rec,
                                 float* side, float* d_means, float* d_lraw, float* d_int, float* d_op,
                                 int accumulate, hipStream_t s) {
  uint32_t want = (rp.rec_cap + 255u) / 256u;
  // with staged planes every block loads them once: fewer, longer blocks
  const bool staged = rp.p <= kStagePlanes;
  const uint32_t cap = staged ? 2048u : 8192u;
  const uint32_t blocks = want < 1 ? 1 : (want > cap ? cap : want);
  const size_t lds = staged ? (size_t)rp.p * kPlaneFloats * sizeof(float) : 0;
  const uint32_t coop = (rp.rec_cap + 63u) / 64u;
  if (coop <= kCoopBlocks)
    hipLaunchKernelGGL(k_record_adjoint<true>, dim3(coop < 1 ? 1 : coop), dim3(256), lds, s, g, pc, rp, ctrl, rec_pair,
                       rec_koff, reinterpret_cast<const float4*>(partial), cnt_rec, off_rec, side, d_means, d_lraw,
                       d_int, d_op, accumulate);
  else
    hipLaunchKernelGGL(k_record_adjoint<false>, dim3(blocks), dim3(256), lds, s, g, pc, rp, ctrl, rec_pair, rec_koff,
                       reinterpret_cast<const float4*>(partial), cnt_rec, off_rec, side, d_means, d_lraw, d_int, d_op,
                       accumulate);
  return hipGetLastError();
}

hipError_t launch_gauss_grad(const ug_gaussians& g, const RenderParams& rp, const Ctrl* ctrl, const uint32_t* cnt_rec,
                             const unsigned long long* off_rec, const float* side, float* d_means, float* d_lraw,
                             float* d_int, float* d_op, int accumulate, const float* loss_part, uint32_t nparts,
                             double inv_m, float* loss_out, hipStream_t s) {
  int blocks = (rp.n + 255) / 256;
  if (loss_out && blocks < 1) blocks = 1;  // the loss is written even with no Gaussians
  if (blocks > 0)
    hipLaunchKernelGGL(k_gauss_grad, dim3(blocks), dim3(256), 0, s, g, rp, ctrl, cnt_rec, off_rec, side, d_means,
                       d_lraw, d_int, d_op, accumulate, loss_part, nparts, inv_m, loss_out);
  return hipGetLastError();
}

}  // namespace ug
