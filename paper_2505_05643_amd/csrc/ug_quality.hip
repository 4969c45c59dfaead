// Image-quality scores of rendered planes against references, for
// evaluating reconstructions (Section 5.2 reports SSIM and PSNR).  Per
// plane: the mean SSIM (Wang et al. 2004; 11 x 11 Gaussian window of
// standard deviation 1.5, weighted population moments, C1 = (0.01 L)^2,
// C2 = (0.03 L)^2) over the window positions that lie inside the image, and
// the MSE over every pixel, from which PSNR = 10 log10(L^2 / MSE).
//
// One wave per strip of 64 input columns (54 output columns) and chunk of
// rows, sliding down it four rows at a time, lanes = columns.  Four moments
// are enough (x, y, x^2 + y^2, x y: the two variances only enter as their
// sum), all in FP64.  The column pass comes first and stays in registers: per
// moment ten partial sums, one per window the row is in, each moving one
// place with every row (a fused multiply-add whose result goes one register
// down), so a row costs its two loads and 44 multiply-adds, with nothing
// re-read.  The four rows' column sums go to LDS, where each lane takes four
// neighbouring outputs of a row: 14 sums read per moment instead of 44.  The
// next four rows are loaded meanwhile.  Each wave writes its two sums (SSIM
// over its window positions, squared differences over its own pixels) to a
// partial array, and a second launch adds each plane's waves in a fixed
// order: the result is deterministic.
//
// Bound by its FP64 instructions (three quarters of what it issues; 65% of the
// issue slots at three waves per SIMD).  480 planes of 160 x 160: 79 us, where
// 8-column strips with five moments, a ring of row sums in LDS and eleven LDS
// reads per moment and output took 152.  (Twenty rows per turn, so that the
// partial sums need no copying back, is no faster; twice as many chunks filter
// a quarter more rows and gain nothing.)
#include <algorithm>

#include "ug_kernels.h"
#include "ug_quality_tile.h"

namespace ug {

constexpr int kQMom = 4;  // x, y, x^2 + y^2, x y

// Strips and row chunks of a plane (at least one: a plane too small for a
// window still has its squared differences).
__device__ __host__ __forceinline__ int q_strips(int W) { return W - 2 * kQRad > kQOut ? (W - 2 * kQRad + kQOut - 1) / kQOut : 1; }
__device__ __host__ __forceinline__ int q_chunks(int H, int rows) {
  return H - 2 * kQRad > rows ? (H - 2 * kQRad + rows - 1) / rows : 1;
}

__global__ __launch_bounds__(64, 3) void k_quality_strip(const PlaneInt* __restrict__ pint, int chunk_rows,
                                                         uint32_t max_strips, const float* __restrict__ img,
                                                         const float* __restrict__ ref, QualityConst q,
                                                         double2* __restrict__ part) {
  __shared__ double2 s_h[kQRows][kQMom][kQPitch / 2];
  const PlaneInt PI = pint[blockIdx.y];
  const int strip = (int)(blockIdx.x % max_strips), chunk = (int)(blockIdx.x / max_strips);
  const int ns = q_strips(PI.W), nc = q_chunks(PI.H, chunk_rows);
  if (strip >= ns || chunk >= nc) return;  // uniform
  const int lane = (int)threadIdx.x;
  const int x = strip * kQOut + lane;
  const int ya = chunk * chunk_rows, yb = chunk == nc - 1 ? PI.H : ya + chunk_rows + 2 * kQRad;
  // the pixels whose squared differences are this wave's
  const int own_y = chunk == nc - 1 ? PI.H : ya + chunk_rows;
  const bool own_x = x < PI.W && (strip == ns - 1 || lane < kQOut);
  const size_t base = ((size_t)PI.pix_off_hi << 32) | PI.pix_off_lo;
  // columns and rows past the plane's (or chunk's) last read the last: no
  // window that counts holds them
  const uint32_t xl = (uint32_t)min(x, PI.W - 1);
  float a[kQRows], b[kQRows];
  auto load_rows = [&](int y) {
#pragma unroll
    for (int r = 0; r < kQRows; ++r) {
      const size_t row = base + (size_t)min(y + r, yb - 1) * (size_t)PI.W;  // uniform
      a[r] = (img + row)[xl];
      b[r] = (ref + row)[xl];
    }
  };
  double acc[kQMom][kQWin - 1];  // [i]: the window that ends i + 1 rows further down
#pragma unroll
  for (int f = 0; f < kQMom; ++f)
#pragma unroll
    for (int i = 0; i < kQWin - 1; ++i) acc[f][i] = 0.0;
  static_assert(kQCols == 64 && kQRows * (64 / kQRows) == 64, "lanes = columns, then (row, group) pairs");
  double s_ssim = 0.0, s_se = 0.0;
  const int place = 2 * q_pair(lane >> 1) + (lane & 1);
  const int orow = lane >> 4, og = lane & 15;  // the lane's outputs: row, group of four columns (the last two groups have none)
  load_rows(ya);
  for (int y0 = ya; y0 < yb; y0 += kQRows) {
#pragma unroll
    for (int r = 0; r < kQRows; ++r) {
      const double A = a[r], B = b[r];
      const double d = own_x && y0 + r < own_y ? A - B : 0.0;
      s_se = fma(d, d, s_se);
      const double h[kQMom] = {A, B, fma(A, A, B * B), A * B};
#pragma unroll
      for (int f = 0; f < kQMom; ++f) {
        reinterpret_cast<double*>(&s_h[r][f][0])[place] = fma(q.taps[0], h[f], acc[f][0]);
#pragma unroll
        for (int i = 0; i + 1 < kQWin - 1; ++i) acc[f][i] = fma(q.taps[i + 1], h[f], acc[f][i + 1]);
        acc[f][kQWin - 2] = q.taps[kQWin - 1] * h[f];
      }
    }
    load_rows(y0 + kQRows);
    if (y0 + kQRows - 1 - ya < 2 * kQRad) continue;  // uniform: no window is complete yet
    wave_lds_sync();
    double m[kQMom][kQPer];
#pragma unroll
    for (int f = 0; f < kQMom; ++f) {
#pragma unroll
      for (int j = 0; j < kQPairs; ++j) {
        const double2 t = s_h[orow][f][q_read_pair(og, j)];
        const double v[2] = {t.x, t.y};
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int o = 0; o < kQPer; ++o) {
            const int tap = 2 * j + k - o;
            if (tap == 0) m[f][o] = q.taps[0] * v[k];
            else if (tap > 0 && tap < kQWin) m[f][o] = fma(q.taps[tap], v[k], m[f][o]);
          }
      }
      // computed here and not behind the bounds test of the output they serve
      // (which keeps all the sums read alive until then)
#pragma unroll
      for (int o = 0; o < kQPer; ++o) asm volatile("" : "+v"(m[f][o]));
    }
    const int y = y0 + orow;  // the windows' last row
    const bool row_ok = y - ya >= 2 * kQRad && y < yb;
#pragma unroll
    for (int o = 0; o < kQPer; ++o) {
      const double t = m[0][o] * m[1][o], e = fma(m[0][o], m[0][o], m[1][o] * m[1][o]);
      const double s = (fma(2.0, t, q.c1) * fma(2.0, m[3][o] - t, q.c2)) / ((e + q.c1) * ((m[2][o] - e) + q.c2));
      const int c = kQPer * og + o;
      s_ssim += row_ok && c < kQOut && strip * kQOut + c + 2 * kQRad < PI.W ? s : 0.0;
    }
    wave_lds_sync();  // the next rows take the sums' place
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s_ssim += __shfl_xor(s_ssim, o, 64);
    s_se += __shfl_xor(s_se, o, 64);
  }
  if (lane == 0) part[(size_t)blockIdx.y * gridDim.x + (size_t)chunk * ns + strip] = make_double2(s_ssim, s_se);
}

// One wave per plane: its strips' and chunks' sums added in a fixed order.
__global__ __launch_bounds__(64) void k_quality_plane(const PlaneInt* __restrict__ pint,
                                                      const double2* __restrict__ part, uint32_t max_parts,
                                                      int chunk_rows, double* __restrict__ ssim,
                                                      double* __restrict__ mse) {
  const PlaneInt PI = pint[blockIdx.x];
  const int n = q_strips(PI.W) * q_chunks(PI.H, chunk_rows);
  const double2* pp = part + (size_t)blockIdx.x * max_parts;
  double a = 0.0, b = 0.0;
  for (int i = (int)threadIdx.x; i < n; i += 64) {
    a += pp[i].x;
    b += pp[i].y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  if (threadIdx.x == 0) {
    const double nw = (double)(PI.W - 2 * kQRad) * (double)(PI.H - 2 * kQRad);
    ssim[blockIdx.x] = (PI.W >= kQWin && PI.H >= kQWin) ? a / nw : __builtin_nan("");
    mse[blockIdx.x] = b / ((double)PI.W * (double)PI.H);
  }
}

// Output rows per chunk: as few chunks as fill the chip (three waves per
// SIMD, what the registers allow), each at least kQMinRows rows; a chunk
// filters ten rows more than it puts out.
constexpr int kQWaves = 3 * 1024, kQMinRows = 16;
int quality_chunk_rows(int32_t p, int32_t max_w, int32_t max_h) {
  const int rows = std::max(max_h - 2 * kQRad, 1);
  const int64_t strips = (int64_t)q_strips(max_w) * std::max(p, 1);
  const int chunks = (int)std::max<int64_t>(std::min<int64_t>(kQWaves / strips, rows / kQMinRows), 1);
  return (rows + chunks - 1) / chunks;
}

uint32_t quality_parts(int32_t p, int32_t max_w, int32_t max_h) {
  return (uint32_t)q_strips(max_w) * (uint32_t)q_chunks(max_h, quality_chunk_rows(p, max_w, max_h));
}

hipError_t launch_quality(const PlaneInt* pint, int32_t p, int32_t max_w, int32_t max_h, const float* img,
                          const float* ref, const QualityConst& q, double2* part, double* ssim, double* mse,
                          hipStream_t s) {
  if (p <= 0) return hipSuccess;
  const int rows = quality_chunk_rows(p, max_w, max_h);
  const uint32_t parts = quality_parts(p, max_w, max_h);
  hipLaunchKernelGGL(k_quality_strip, dim3(parts, (uint32_t)p), dim3(64), 0, s, pint, rows, (uint32_t)q_strips(max_w),
                     img, ref, q, part);
  hipLaunchKernelGGL(k_quality_plane, dim3((uint32_t)p), dim3(64), 0, s, pint, part, parts, rows, ssim, mse);
  return hipGetLastError();
}

}  // namespace ug
