// Device pieces that the granule kernels share: loads of quads of samples, exact thirds of float32
// values and their products, moves along the 16 lanes of a DPP row.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "granule.h"
#include "scan_common.h"

namespace mk {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v6i __attribute__((ext_vector_type(6)));
typedef __bf16 v2b __attribute__((ext_vector_type(2)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));

template <int SH, typename T>
__device__ __forceinline__ T row_shr(T v) {   // lane c of each 16-lane row reads lane c - SH, else 0
  return __builtin_amdgcn_update_dpp((T)0, v, 0x110 + SH, 0xF, 0xF, true);
}
template <typename T>
__device__ __forceinline__ T row_last(T v) {  // every lane of a row reads its lane 15
  return __builtin_amdgcn_update_dpp((T)0, v, 0x15F, 0xF, 0xF, true);
}

// order of a wave's own LDS accesses (the hardware keeps it; this keeps the compiler's)
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The wave's quads of samples p0 + 4 lane .. + 3 of ST real streams, zero outside [lo, hi), in the
// type they are stored in. IN 0, 1, 2: one stream of float32, float16, bfloat16 samples at index p.
// IN 3, 4: the cotangent of the adjoint, read backwards, sample p at index N - 1 - p: complex64 (its
// real and imaginary parts two streams) or float32.
enum { kInRev = 3 };
template <int IN>
struct Quad {
  using E = typename std::conditional<IN == 1 || IN == 2, unsigned short, typename std::conditional<IN == 3, v2f, float>::type>::type;
  using V = typename std::conditional<IN == 1 || IN == 2, v4h_any, v4f_any>::type;
  V v[IN == 3 ? 2 : 1];
  // INNER: the whole granule lies inside [lo, hi)
  template <bool INNER = false>
  __device__ __forceinline__ void load(const void* xs, int64_t p0, int64_t lo, int64_t hi, int64_t N, int lane) {
    const E* x = static_cast<const E*>(xs);
    const E* p = IN >= kInRev ? x + (N - 4 - p0) : x + p0;   // wave-uniform; the lane's quad starts at p -+ 4 lane
    const int o = IN >= kInRev ? -4 * lane : 4 * lane;
    if (INNER || (p0 >= lo && p0 + kGran <= hi)) {
      v[0] = *reinterpret_cast<const V*>(p + o);
      if constexpr (IN == 3) v[1] = *reinterpret_cast<const V*>(p + o + 2);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t j = p0 + 4 * lane + (IN >= kInRev ? 3 - e : e);
        const bool in = j >= lo && j < hi;
        if constexpr (IN == 3) {
          const v2f t = in ? p[o + e] : v2f{0.0f, 0.0f};
          v[e / 2][2 * (e % 2)] = t[0];
          v[e / 2][2 * (e % 2) + 1] = t[1];
        } else {
          v[0][e] = in ? p[o + e] : (E)0;
        }
      }
    }
  }
  __device__ __forceinline__ v4f f32(int st) const {   // stream st in scan order
    if constexpr (IN == 0) return v[0];
    else if constexpr (IN == 1) return v4f{cvt_f16(v[0][0]), cvt_f16(v[0][1]), cvt_f16(v[0][2]), cvt_f16(v[0][3])};
    else if constexpr (IN == 2) return v4f{cvt_bf16(v[0][0]), cvt_bf16(v[0][1]), cvt_bf16(v[0][2]), cvt_bf16(v[0][3])};
    else if constexpr (IN == 3) return v4f{v[1][2 + st], v[1][st], v[0][2 + st], v[0][st]};
    else return v4f{v[0][3], v[0][2], v[0][1], v[0][0]};
  }
};

// Four float32 values as bfloat16 thirds, middle, high, low (two registers each): every value is the
// exact sum of its thirds, if its nearest bfloat16 is finite and the lowest third does not vanish
// (no_thirds). The remainder after a third is one
// dot product with (-1, 0) or (0, -1).
__device__ __forceinline__ int bf16_pair(float a, float b) {
  return __builtin_bit_cast(int, __builtin_convertvector(v2f{a, b}, v2b));
}
__device__ __forceinline__ v6i thirds(const float (&x)[4]) {
  int lo;   // (-1, 0): as a register, an inline constant would stand for another pair
  asm("s_mov_b32 %0, 0xbf80" : "=s"(lo));
  const v2b n0 = __builtin_bit_cast(v2b, lo), n1 = __builtin_bit_cast(v2b, (int)0xbf800000);
  auto left = [&](int p, float a, float b, float& ra, float& rb) {
    ra = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2b, p), n0, a, false);
    rb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2b, p), n1, b, false);
  };
  float r[4], t[4];
  const int h0 = bf16_pair(x[0], x[1]), h1 = bf16_pair(x[2], x[3]);
  left(h0, x[0], x[1], r[0], r[1]);
  left(h1, x[2], x[3], r[2], r[3]);
  const int m0 = bf16_pair(r[0], r[1]), m1 = bf16_pair(r[2], r[3]);
  left(m0, r[0], r[1], t[0], t[1]);
  left(m1, r[2], r[3], t[2], t[3]);
  return v6i{m0, m1, h0, h1, bf16_pair(t[0], t[1]), bf16_pair(t[2], t[3])};
}
// The largest sum of four magnitudes that a lane has seen, as bits (an infinite or NaN one is above all others).
__device__ __forceinline__ void keep_top(uint32_t& top, const float (&x)[4]) {
  const uint32_t m = __float_as_uint((fabsf(x[0]) + fabsf(x[1])) + (fabsf(x[2]) + fabsf(x[3])));
  top = m > top ? m : top;
}
// Whether some value of the wave's is infinite, NaN or so near the end of the range that its high third may be
// infinite, or all are so small (not all zero) that their low thirds fall below bfloat16's smallest value, 2^-133:
// from 2^-110 down thirds are not exact (signals of 1e-36 gave outputs off by 3e-5).
__device__ __forceinline__ bool all_small(uint32_t top) { return __ballot(top >= __float_as_uint(0x1p-106f)) == 0; }
__device__ __forceinline__ bool no_thirds(uint32_t top) {
  return __ballot(top >= __float_as_uint(0x1p126f)) != 0 || (all_small(top) && __ballot(top != 0) != 0);
}
// The same of states, which make the outputs where the inputs are zeros (off by up to 7e-4 after a signal of 1e-36).
template <int NS>
__device__ __forceinline__ bool no_thirds(const double (&zr)[NS], const double (&zi)[NS]) {
  float m = 0;
#pragma unroll
  for (int s = 0; s < NS; ++s) m = fmaxf(m, fmaxf(fabsf((float)zr[s]), fabsf((float)zi[s])));
  return no_thirds(__float_as_uint(m));
}
// Weights of four inputs per lane as thirds: middle, high, low.
struct Weights {
  v6i w;
  __device__ __forceinline__ float at(int e) const {   // the weight of input e
    auto part = [&](int i) {
      asm volatile("" : "+v"(i));   // formed where it is used, not kept in registers through the loop
      return __int_as_float(e % 2 ? i & (int)0xffff0000 : i << 16);
    };
    return (part(w[4 + e / 2]) + part(w[e / 2])) + part(w[2 + e / 2]);
  }
  __device__ __forceinline__ void load(const v2i* t, int h, int m, int l) {
    const v2i vh = t[h], vm = t[m], vl = t[l];
    w = v6i{vm[0], vm[1], vh[0], vh[1], vl[0], vl[1]};
  }
};
// acc + x w to float32 accuracy: the products of thirds down to 2^-16 of the largest (middle x low and
// low x low, below 2^-25, are left out), smallest first
__device__ __forceinline__ v4f product(const v6i& x, const Weights& w, v4f acc) {
  const v8b wmh = __builtin_bit_cast(v8b, __builtin_shufflevector(w.w, w.w, 0, 1, 2, 3));
  const v8b whl = __builtin_bit_cast(v8b, __builtin_shufflevector(w.w, w.w, 2, 3, 4, 5));
  const v8b lh = __builtin_bit_cast(v8b, __builtin_shufflevector(x, x, 4, 5, 2, 3));
  const v8b mm = __builtin_bit_cast(v8b, __builtin_shufflevector(x, x, 0, 1, 0, 1));
  const v8b hh = __builtin_bit_cast(v8b, __builtin_shufflevector(x, x, 2, 3, 2, 3));
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lh, whl, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mm, wmh, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(hh, wmh, acc, 0, 0, 0);
}

// the same in float32, for any x (an infinite or NaN value must not meet a zero weight)
__device__ __forceinline__ v4f product_unsplit(const float (&x)[4], const Weights& w, v4f acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], w.at(e), acc, 0, 0, 0);
  return acc;
}

// product() and product_unsplit() with the weights as rows
__device__ __forceinline__ v4f product_t_unsplit(const Weights& w, const float (&x)[4], v4f acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.at(e), x[e], acc, 0, 0, 0);
  return acc;
}
__device__ __forceinline__ v4f product_t(const Weights& w, const v6i& x, v4f acc) {
  const v8b wmh = __builtin_bit_cast(v8b, __builtin_shufflevector(w.w, w.w, 0, 1, 2, 3));
  const v8b whl = __builtin_bit_cast(v8b, __builtin_shufflevector(w.w, w.w, 2, 3, 4, 5));
  const v8b lh = __builtin_bit_cast(v8b, __builtin_shufflevector(x, x, 4, 5, 2, 3));
  const v8b mm = __builtin_bit_cast(v8b, __builtin_shufflevector(x, x, 0, 1, 0, 1));
  const v8b hh = __builtin_bit_cast(v8b, __builtin_shufflevector(x, x, 2, 3, 2, 3));
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(whl, lh, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wmh, mm, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(wmh, hh, acc, 0, 0, 0);
}

// Granule slot of quad q of run c: 4 c + (q ^ swz(c)), so 8 lanes of consecutive runs reading one
// quad index, and 16 of them, hit different 16-byte banks.
__device__ __forceinline__ int swz(int c) { return (((c >> 1) ^ (c >> 3)) & 1) | (((c >> 2) & 1) << 1); }

// (xr, xi) <- (cr, ci) (yr, yi) + (xr, xi)
__device__ __forceinline__ void mac(double cr, double ci, double yr, double yi, double& xr, double& xi) {
  xr = fma(cr, yr, fma(-ci, yi, xr));
  xi = fma(cr, yi, fma(ci, yr, xi));
}

// Run sums of one run per lane column, from the lane's operand quad d (WIDE, float64 product) or its thirds x:
// real and imaginary part of state 4 s + q of the column in slot s.
template <int NS, bool WIDE>
struct RunSums {
  static constexpr int MB = NS > 2 ? 2 : 1;
  using sum_t = typename std::conditional<WIDE, double, float>::type;
  using acc_t = typename std::conditional<WIDE, v4d, v4f>::type;
  double p[WIDE ? MB : 1][4];
  Weights w[WIDE ? 1 : MB];
  // c: -1, or the stream of the complex adjoint
  __device__ __forceinline__ void load(const GranLayout& lay, const double* td, const v2i* tq, int lane, int c = -1) {
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      if constexpr (WIDE) {
#pragma unroll
        for (int k = 0; k < 4; ++k) p[b][k] = td[(c < 0 ? lay.dP(b, k) : lay.dPA(c, b, k)) + lane];
      } else if (c < 0) {
        w[b].load(tq, lay.bP(b, 0), lay.bP(b, 1), lay.bP(b, 2));
      } else {
        w[b].load(tq, lay.bPA(c, b, 0), lay.bPA(c, b, 1), lay.bPA(c, b, 2));
      }
    }
  }
  __device__ __forceinline__ void add(const double (&d)[4], const v6i& x, acc_t (&acc)[MB]) const {
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      if constexpr (WIDE) {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[b][k], d[k], acc[b], 0, 0, 0);
      } else {
        acc[b] = product_t(w[b], x, acc[b]);
      }
    }
  }
  __device__ __forceinline__ void add_unsplit(const float (&x)[4], acc_t (&acc)[MB]) const {
    if constexpr (!WIDE)
#pragma unroll
      for (int b = 0; b < MB; ++b) acc[b] = product_t_unsplit(w[b], x, acc[b]);
  }
  static __device__ __forceinline__ void states(const acc_t (&acc)[MB], sum_t (&br)[NS], sum_t (&bi)[NS]) {
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      br[2 * b] = acc[b][0]; bi[2 * b] = acc[b][1];
      if (2 * b + 1 < NS) { br[2 * b + 1] = acc[b][2]; bi[2 * b + 1] = acc[b][3]; }
    }
  }
};

}  // namespace
}  // namespace mk
