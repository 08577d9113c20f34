// Carrier kernels of the Morlet transform by the multiplication method (Sec. III-B).
//
// The method's sum over the real frequencies xi + beta p of the envelope's Fourier terms is the
// carrier times the fitted envelope, sum_p a'_p e^{i (xi + beta p) k} = e^{i xi k} G_hat[k], so
//   x_M[n] = C' [ e^{i xi n} (G_hat * u)[n] - kappa (G_hat * x)[n] ],   u[m] = e^{-i xi m} x[m].
// The three real Gaussian smoothings (Re u, Im u, x) run as three rows of one scan launch;
// these two elementwise kernels form the rows before it and combine them after it. The
// phase xi m is formed and reduced in float64 (sincos of the float64 product), so it stays
// exact to float32 for any index.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "launch.h"
#include "multiply.h"
#include "scan_common.h"

namespace mk {
namespace {

constexpr int kMmThreads = 256;

// A thread takes four consecutive samples with 16-byte accesses (at any sample alignment: the rows of
// an odd length are not aligned) and one sincos: the phases of the other three are float64 rotations
// by constants. With a sincos and 4-byte accesses per sample the kernels were bound by its 100 float64
// instructions (N = 2^22: demodulation 16 us, remodulation 24; now 11.5 and 16.6, 5.8 and 5.0 TB/s).
struct Turns {   // e^{i xi k}, k = 1, 2, 3
  double c[3], s[3];
};

// cos and sin of xi (m + k), k < 4
__device__ __forceinline__ void phases(double xi, const Turns& r, int64_t m, double (&c)[4], double (&s)[4]) {
  sincos(xi * (double)m, &s[0], &c[0]);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c[k + 1] = fma(c[0], r.c[k], -(s[0] * r.s[k]));
    s[k + 1] = fma(s[0], r.c[k], c[0] * r.s[k]);
  }
}

__device__ __forceinline__ void load4_row(const float* p, int64_t m, int64_t N, float (&v)[4]) {
  if (m + 4 <= N) {
    const v4f_any t = *reinterpret_cast<const v4f_any*>(p + m);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = t[k];
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = m + k < N ? p[m + k] : 0.0f;
  }
}
__device__ __forceinline__ void store4_row(float* p, int64_t m, int64_t N, const float (&v)[4]) {
  if (m + 4 <= N) {
    *reinterpret_cast<v4f_any*>(p + m) = v4f_any{v[0], v[1], v[2], v[3]};
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (m + k < N) p[m + k] = v[k];
  }
}

// u[m] = x[m] cos(xi m), u[N + m] = -x[m] sin(xi m), u[2N + m] = x[m]
__global__ __launch_bounds__(kMmThreads) void mm_demodulate_kernel(const void* x, int dtype, float* u, int64_t N,
                                                                     double xi, Turns r) {
  const int64_t stride = (int64_t)gridDim.x * kMmThreads * 4;
  for (int64_t m = ((int64_t)blockIdx.x * kMmThreads + threadIdx.x) * 4; m < N; m += stride) {
    float v[4], a[4], b[4];
    if (dtype == 0) {
      load4_row(static_cast<const float*>(x), m, N, v);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = m + k < N ? load1(x, dtype, m + k) : 0.0f;
    }
    double c[4], s[4];
    phases(xi, r, m, c, s);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[k] = (float)((double)v[k] * c[k]);
      b[k] = (float)(-(double)v[k] * s[k]);
    }
    store4_row(u, m, N, a);
    store4_row(u + N, m, N, b);
    store4_row(u + 2 * N, m, N, v);
  }
}

// W[n] = ce (e^{i xi n} (g[n] + i g[N + n]) - kappa g[2N + n])
__global__ __launch_bounds__(kMmThreads) void mm_remodulate_kernel(const float* g, float* W, int64_t N, double xi,
                                                                     double ce, double cek, Turns r) {
  const int64_t stride = (int64_t)gridDim.x * kMmThreads * 4;
  for (int64_t n = ((int64_t)blockIdx.x * kMmThreads + threadIdx.x) * 4; n < N; n += stride) {
    float gc[4], gs[4], gx[4], o[2][4];
    load4_row(g, n, N, gc);
    load4_row(g + N, n, N, gs);
    load4_row(g + 2 * N, n, N, gx);
    double c[4], s[4];
    phases(xi, r, n, c, s);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double pc = gc[k], ps = gs[k];
      o[k / 2][2 * (k % 2)] = (float)(ce * (c[k] * pc - s[k] * ps) - cek * (double)gx[k]);
      o[k / 2][2 * (k % 2) + 1] = (float)(ce * (s[k] * pc + c[k] * ps));
    }
    store4_row(W, 2 * n, 2 * N, o[0]);
    store4_row(W, 2 * n + 4, 2 * N, o[1]);
  }
}

// Transposes for the backward (real loss, gW = dLoss/dRe W + i dLoss/dIm W):
//   g[n] = ce (gWr cos + gWi sin), g[N + n] = ce (gWi cos - gWr sin), g[2N + n] = -ce kappa gWr
__global__ __launch_bounds__(kMmThreads) void mm_remodulate_t_kernel(const float* gW, float* g, int64_t N, double xi,
                                                                       double ce, double cek, Turns r) {
  const int64_t stride = (int64_t)gridDim.x * kMmThreads * 4;
  for (int64_t n = ((int64_t)blockIdx.x * kMmThreads + threadIdx.x) * 4; n < N; n += stride) {
    float w[2][4], a[4], b[4], d[4];
    load4_row(gW, 2 * n, 2 * N, w[0]);
    load4_row(gW, 2 * n + 4, 2 * N, w[1]);
    double c[4], s[4];
    phases(xi, r, n, c, s);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double gr = w[k / 2][2 * (k % 2)], gi = w[k / 2][2 * (k % 2) + 1];
      a[k] = (float)(ce * (gr * c[k] + gi * s[k]));
      b[k] = (float)(ce * (gi * c[k] - gr * s[k]));
      d[k] = (float)(-cek * gr);
    }
    store4_row(g, n, N, a);
    store4_row(g + N, n, N, b);
    store4_row(g + 2 * N, n, N, d);
  }
}

//   gx[m] = cos(xi m) gu[m] - sin(xi m) gu[N + m] + gu[2N + m]
__global__ __launch_bounds__(kMmThreads) void mm_demodulate_t_kernel(const float* gu, float* gx, int64_t N, double xi,
                                                                       Turns r) {
  const int64_t stride = (int64_t)gridDim.x * kMmThreads * 4;
  for (int64_t m = ((int64_t)blockIdx.x * kMmThreads + threadIdx.x) * 4; m < N; m += stride) {
    float a[4], b[4], d[4], o[4];
    load4_row(gu, m, N, a);
    load4_row(gu + N, m, N, b);
    load4_row(gu + 2 * N, m, N, d);
    double c[4], s[4];
    phases(xi, r, m, c, s);
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = (float)(c[k] * (double)a[k] - s[k] * (double)b[k] + (double)d[k]);
    store4_row(gx, m, N, o);
  }
}

int mm_grid(int64_t N) {
  const int64_t blocks = (N + 4 * kMmThreads - 1) / (4 * kMmThreads);
  return (int)std::max<int64_t>(1, std::min<int64_t>(blocks, 8192));
}

Turns turns(double xi) {
  Turns r;
  for (int k = 0; k < 3; ++k) {
    r.c[k] = std::cos(xi * (k + 1));
    r.s[k] = std::sin(xi * (k + 1));
  }
  return r;
}

}  // namespace

hipError_t launch_mm_demodulate(const void* x, int dtype, float* u, int64_t N, double xi, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  hipLaunchKernelGGL(mm_demodulate_kernel, dim3(mm_grid(N)), dim3(kMmThreads), 0, s, x, dtype, u, N, xi, turns(xi));
  return hipGetLastError();
}

hipError_t launch_mm_remodulate(const float* g, float2* W, int64_t N, double xi, double ce, double cek,
                                hipStream_t s) {
  if (N <= 0) return hipSuccess;
  hipLaunchKernelGGL(mm_remodulate_kernel, dim3(mm_grid(N)), dim3(kMmThreads), 0, s, g, reinterpret_cast<float*>(W), N, xi, ce, cek, turns(xi));
  return hipGetLastError();
}

hipError_t launch_mm_remodulate_t(const float2* gW, float* g, int64_t N, double xi, double ce, double cek,
                                  hipStream_t s) {
  if (N <= 0) return hipSuccess;
  hipLaunchKernelGGL(mm_remodulate_t_kernel, dim3(mm_grid(N)), dim3(kMmThreads), 0, s, reinterpret_cast<const float*>(gW), g, N, xi, ce, cek, turns(xi));
  return hipGetLastError();
}

hipError_t launch_mm_demodulate_t(const float* gu, float* gx, int64_t N, double xi, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  hipLaunchKernelGGL(mm_demodulate_t_kernel, dim3(mm_grid(N)), dim3(kMmThreads), 0, s, gu, gx, N, xi, turns(xi));
  return hipGetLastError();
}

}  // namespace mk
