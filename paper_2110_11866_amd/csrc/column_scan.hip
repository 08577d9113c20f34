// Column scan (gfx950): the granule scan's arithmetic along the columns of a row-major float32 matrix,
// for the second axis of the separable image filters, without transposing the image.
//
// A wave takes 32 columns and a piece of the rows, 16 rows (one run per column) at a time. Lane
// 16 q + c loads rows 4 q .. 4 q + 3 of columns 2 c, 2 c + 1 (128 bytes of a row per 16 lanes); column
// 2 c + g is run c of product g. With the runs as matrix columns, the lane's loads are its operands as
// they are, the run sums land in the lane that owns the states q, q + 4, q + 8 of the column, and the
// outputs in the lane that stores them: no scan across lanes and no LDS. A state before a piece is the
// sum over the window before it, as in the granule scan.
//
// It replaces a transpose, the row scan and a transpose back. On 4096 x 4096 float32 (K = 4, 2L = 54)
// the columns take 50 us against 39 + 2 x 37; with 64 columns per wave 81 us (two waves per SIMD instead
// of four, loads exposed), with 16 columns 100 us (half lines).
#include <hip/hip_runtime.h>

#include "granule.h"
#include "launch.h"
#include "scan_common.h"

namespace mk {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kCols = kColWave;   // columns per wave
constexpr int kG = kCols / 16;    // columns per lane
typedef float vg __attribute__((ext_vector_type(kG)));
typedef float vg_any __attribute__((ext_vector_type(kG), aligned(4)));   // any column alignment

// REV: the adjoint, rows from the last to the first
template <int NS, bool REV>
__global__ __launch_bounds__(64) void column_kernel(ColumnLaunch P) {
  constexpr int MB = NS > 2 ? 2 : 1;
  const int lane = threadIdx.x, q = lane >> 4, c = lane & 15;
  const int64_t N = P.rows, W = P.cols;
  const int64_t cb = (int64_t)blockIdx.x * kCols + kG * c;   // the lane's first column
  const bool full = (int64_t)(blockIdx.x + 1) * kCols <= W;
  const int64_t n0 = (int64_t)blockIdx.y * P.piece;         // the piece's first output row
  const int64_t n1 = n0 + P.piece < N ? n0 + P.piece : N;

  const GranLayout lay{4 * NS};
  const float* tf = reinterpret_cast<const float*>(P.tabs);
  const double* td = reinterpret_cast<const double*>(tf + lay.nFloats());
  float T[4], C[2 * NS];
  double Pm[MB][4], ar[NS], ai[NS];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    T[k] = tf[lay.fTre(k) + lane];
#pragma unroll
    for (int b = 0; b < MB; ++b) Pm[b][k] = td[lay.dP(b, k) + lane];
  }
#pragma unroll
  for (int k = 0; k < 2 * NS; ++k) C[k] = tf[lay.fCre(k) + lane];
#pragma unroll
  for (int s = 0; s < NS; ++s) { ar[s] = td[lay.dSC(0, s, 0) + q]; ai[s] = td[lay.dSC(0, s, 1) + q]; }
  const float Y = tf[lay.fYre()];
  const double D = td[lay.dD()];

  // rows j .. j + 3 (position order) of the lane's columns, zero outside [lo, hi)
  auto load = [&](int64_t j, int64_t lo, int64_t hi, vg (&v)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t p = j + k;
      v[k] = (vg)0.0f;
      if (p >= lo && p < hi) {
        const float* x = P.x + (REV ? N - 1 - p : p) * W + cb;
        if (full) {
          v[k] = *reinterpret_cast<const vg_any*>(x);
        } else {
#pragma unroll
          for (int g = 0; g < kG; ++g)
            if (cb + g < W) v[k][g] = x[g];
        }
      }
    }
  };
  auto run_sums = [&](const double (&d)[4], double (&br)[NS], double (&bi)[NS]) {
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      v4d acc = {0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Pm[b][k], d[k], acc, 0, 0, 0);
      br[2 * b] = acc[0]; bi[2 * b] = acc[1];
      if (2 * b + 1 < NS) { br[2 * b + 1] = acc[2]; bi[2 * b + 1] = acc[3]; }
    }
  };

  // states before position js of the lane's two columns
  double zr[kG][NS], zi[kG][NS];
#pragma unroll
  for (int g = 0; g < kG; ++g)
#pragma unroll
    for (int s = 0; s < NS; ++s) { zr[g][s] = 0; zi[g][s] = 0; }
  auto step = [&](int g, const double (&br)[NS], const double (&bi)[NS]) {   // z <- a^16 z + B
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const double nr = fma(ar[s], zr[g][s], fma(-ai[s], zi[g][s], br[s]));
      zi[g][s] = fma(ar[s], zi[g][s], fma(ai[s], zr[g][s], bi[s]));
      zr[g][s] = nr;
    }
  };
  const int64_t js = n0 + P.jout0, L2 = 2 * P.L;
  {
    const int64_t lo = js - L2 > 0 ? js - L2 : 0;
    const int64_t nw = js > lo && lo < N ? (js - lo + kRun - 1) / kRun : 0;
    vg y[4];
    if (nw > 0) load(js - kRun * nw + 4 * q, lo, N, y);
    for (int64_t i = nw; i > 0; --i) {
      double d[kG][4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int g = 0; g < kG; ++g) d[g][k] = (double)y[k][g];
      if (i > 1) load(js - kRun * (i - 1) + 4 * q, lo, N, y);
#pragma unroll
      for (int g = 0; g < kG; ++g) {
        double br[NS], bi[NS];
        run_sums(d[g], br, bi);
        step(g, br, bi);
      }
    }
  }

  vg ya[4], yb[4];
  load(js + 4 * q, 0, N, ya);
  load(js - L2 + 4 * q, 0, N, yb);
  for (int64_t n = n0; n < n1; n += kRun) {
    v4f o[kG];
    double d[kG][4];
    bool odd = false;   // some input is infinite or NaN
#pragma unroll
    for (int g = 0; g < kG; ++g) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        d[g][k] = fma(-D, (double)yb[k][g], (double)ya[k][g]);
        o[g][k] = Y * yb[k][g];
      }
      odd = odd || !__builtin_isfinite((d[g][0] + d[g][1]) + (d[g][2] + d[g][3]));
    }
    const bool slow = __ballot(odd) != 0;
    if (n + kRun < n1) {   // the next run's rows, in flight during this one
      const int64_t j = n + kRun + P.jout0 + 4 * q;
      load(j, 0, N, ya);
      load(j - L2, 0, N, yb);
    }
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      if (!slow) {
#pragma unroll
        for (int k = 0; k < 4; ++k) o[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(T[k], (float)d[g][k], o[g], 0, 0, 0);
      } else {
#pragma unroll 1
        for (int r = 0; r < kRun; ++r) {   // output row r from the inputs up to it
          v4f t = o[g];
#pragma unroll
          for (int k = 0; k < 4; ++k)
            t = __builtin_amdgcn_mfma_f32_16x16x4f32(T[k], 4 * q + k <= r ? (float)d[g][k] : 0.0f, t, 0, 0, 0);
#pragma unroll
          for (int k = 0; k < 4; ++k) o[g][k] = 4 * q + k == r ? t[k] : o[g][k];
        }
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        o[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(C[2 * s], (float)zr[g][s], o[g], 0, 0, 0);
        o[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(C[2 * s + 1], (float)zi[g][s], o[g], 0, 0, 0);
      }
      double br[NS], bi[NS];
      run_sums(d[g], br, bi);
      step(g, br, bi);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t r = n + 4 * q + k;
      if (r < n1) {
        float* y = P.out + (REV ? N - 1 - r : r) * W + cb;
        if (full) {
          vg t;
#pragma unroll
          for (int g = 0; g < kG; ++g) t[g] = o[g][k];
          *reinterpret_cast<vg_any*>(y) = t;
        } else {
#pragma unroll
          for (int g = 0; g < kG; ++g)
            if (cb + g < W) y[g] = o[g][k];
        }
      }
    }
  }
}

}  // namespace

hipError_t launch_columns(const ColumnLaunch& a, hipStream_t s) {
  if (a.rows <= 0 || a.cols <= 0) return hipSuccess;
  const int64_t bx = (a.cols + kCols - 1) / kCols, by = a.piece > 0 ? (a.rows + a.piece - 1) / a.piece : 0;
  if (a.K < 1 || a.K > kMaxTerms || by < 1 || by > 65535 || !launchable(bx, 64)) return hipErrorInvalidValue;
  const int ns = GranLayout{a.K}.NS();
  void (*fn)(ColumnLaunch) = a.adjoint ? (ns == 1 ? column_kernel<1, true> : ns == 2 ? column_kernel<2, true> : column_kernel<3, true>)
                                       : (ns == 1 ? column_kernel<1, false> : ns == 2 ? column_kernel<2, false> : column_kernel<3, false>);
  hipLaunchKernelGGL(fn, dim3((unsigned)bx, (unsigned)by), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace mk
