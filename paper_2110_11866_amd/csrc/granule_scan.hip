// Granule scan (gfx950): the forward transform on the matrix cores, one wave per piece of a row.
//
// The state of the scan (scan_kernel.h: v_p[j] = a v_p[j-1] + dy[j], dy[j] = y[j] - a^{2L} y[j-2L])
// is the windowed sum v_p[j] = sum_{q = j-2L+1}^{j} a^{j-q} y[q]: it can be formed at any position
// from the 2L samples before it. So a row is cut into pieces that never wait on each other: a wave
// sums the window before its piece (run sums only, no outputs), then runs the piece granule by
// granule, 256 positions as 16 runs of 16:
//   1. dy of run c as operand: lane 16 q + c holds dy[4 q .. 4 q + 3] of run c. The quads are loaded
//      coalesced, lane l the l-th quad (16-byte loads at any sample alignment), and change lanes
//      through 1 KB of LDS, swizzled so neither side conflicts;
//   2. run sums B = P dy (2K x 16 by 16 x 16) in float64: lane 16 q + c receives the components of states
//      q, q + 4, q + 8 of run c;
//   3. float64 scan of the 16 runs along the 16 lanes of a DPP row (4 levels, constants a^{16 2^d}), the
//      state at the granule's start entering run 0;
//   4. outputs of run c, position r: o = T dy + C S + Y y[j-2L], one product per component with the
//      runs as rows and the positions as columns, so lane 16 q + r holds position r of runs
//      4 q .. 4 q + 3 and a store instruction writes whole 128-byte lines.
// The recurrence over the 16 positions and the K-term combination, 36 vector operations per position
// at K = 5, become 40 matrix multiply-adds, which issue beside the vector work of other waves.
//
// Zeros of T meet inputs of the same run at later positions: a run with an infinite or NaN input
// takes the product masked position by position, so no output depends on a later input.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "granule.h"
#include "launch.h"
#include "scan_common.h"

namespace mk {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));            // any sample alignment
typedef unsigned short v4h_any __attribute__((ext_vector_type(4), aligned(2)));

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
  __device__ __forceinline__ void load(const void* xs, int64_t p0, int64_t lo, int64_t hi, int64_t N, int lane) {
    const E* x = static_cast<const E*>(xs);
    const E* p = IN >= kInRev ? x + (N - 4 - p0) : x + p0;   // wave-uniform; the lane's quad starts at p -+ 4 lane
    const int o = IN >= kInRev ? -4 * lane : 4 * lane;
    if (p0 >= lo && p0 + kGran <= hi) {
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

// Granule slot of quad q of run c: 4 c + (q ^ swz(c)), so 8 lanes of consecutive runs reading one
// quad index, and 16 of them, hit different 16-byte banks.
__device__ __forceinline__ int swz(int c) { return (((c >> 1) ^ (c >> 3)) & 1) | (((c >> 2) & 1) << 1); }

// IN: the input (Quad). CPLX: the transform's outputs are complex (IN < 3: complex64 out; IN 3: their
// cotangent comes in). An output component k is formed from stream k of the adjoint's two, or from
// the only stream; the adjoint adds its components, Re sum conj(h) g = (h_re * g_re) + (h_im * g_im).
template <int NS, bool CPLX, int IN>
__global__ __launch_bounds__(64) void granule_kernel(GranLaunch P) {
  constexpr bool REV = IN >= kInRev;
  constexpr int ST = IN == 3 ? 2 : 1, NC = CPLX ? 2 : 1, MB = NS > 2 ? 2 : 1;
  static_assert(!REV || CPLX == (IN == 3), "the adjoint's input is the cotangent of the transform's output");
  __shared__ __align__(16) float s_y[ST][kGran];   // y[j], by run and quad
  __shared__ __align__(16) float s_b[ST][kGran];   // y[j - 2L]
  const int lane = threadIdx.x, q = lane >> 4, c = lane & 15;

  Row row = P.row0;
  int64_t g0, gn;
  if (P.segs) {
    const cptr<GranSeg> sp = (cptr<GranSeg>)P.segs + blockIdx.x;
    const cptr<Row> rp = (cptr<Row>)P.rows + sp->row;
    row.x_off = rp->x_off; row.w_off = rp->w_off; row.N = rp->N; row.L = rp->L;
    row.jout0 = rp->jout0; row.scale = rp->scale;
    g0 = sp->g0; gn = sp->n;
  } else {
    const uint32_t r = blockIdx.x / (uint32_t)P.pieces;
    g0 = (int64_t)(blockIdx.x - r * (uint32_t)P.pieces) * P.seg_n; gn = P.seg_n;
    if (P.nrows != 1) {
      const cptr<Row> rp = (cptr<Row>)P.rows + r;
      row.x_off = rp->x_off; row.w_off = rp->w_off; row.N = rp->N; row.L = rp->L;
      row.jout0 = rp->jout0; row.scale = rp->scale;
    }
  }
  const int64_t N = row.N, L2 = 2 * row.L;
  constexpr int IB = IN == 0 || IN == 4 ? 4 : IN == 3 ? 8 : 2;   // bytes per input element
  constexpr int OB = CPLX && !REV ? 8 : 4;                       // bytes per output
  const void* xs = static_cast<const char*>(P.x) + (REV ? row.w_off : row.x_off) * IB;
  unsigned char* W = static_cast<unsigned char*>(P.out) + row.w_off * OB;
  // granules start on the output's 128-byte lines (the adjoint writes from the row's end)
  const int64_t m = REV ? (int64_t)((-reinterpret_cast<uintptr_t>(W + N * OB) & 127) / OB)
                        : (int64_t)((reinterpret_cast<uintptr_t>(W) & 127) / OB);
  {
    const int64_t left = (N + m + kGran - 1) / kGran - g0;   // granules from g0 to the row's end
    gn = left < gn ? left : gn;
  }
  if (gn <= 0) return;

  const GranLayout lay{4 * NS};   // layouts differ by the slot count only
  const float* tf = reinterpret_cast<const float*>(P.tabs + (int64_t)row.scale * P.tab_stride);
  const double* td = reinterpret_cast<const double*>(tf + lay.nFloats());
  float T[NC][4], C[NC][2 * NS], Y[NC];
  double Pm[MB][4], scr[4][NS], sci[4][NS];
  double gr[NS], gi[NS];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    T[0][k] = tf[lay.fTre(k) + lane];
    if constexpr (NC == 2) T[NC - 1][k] = tf[lay.fTim(k) + lane];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      Pm[b][k] = td[lay.dP(b, k) + lane];
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      scr[k][s] = td[lay.dSC(k, s, 0) + q];
      sci[k][s] = td[lay.dSC(k, s, 1) + q];
    }
  }
#pragma unroll
  for (int k = 0; k < 2 * NS; ++k) {
    C[0][k] = tf[lay.fCre(k) + lane];
    if constexpr (NC == 2) C[NC - 1][k] = tf[lay.fCim(k) + lane];
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    gr[s] = td[lay.dG(1, s, 0) + q]; gi[s] = td[lay.dG(1, s, 1) + q];
  }
  Y[0] = tf[lay.fYre()];
  if constexpr (NC == 2) Y[NC - 1] = tf[lay.fYim()];
  const double Dd = td[lay.dD()];

  const int wslot = 4 * (4 * (lane >> 2) + ((lane & 3) ^ swz(lane >> 2)));
  const int rslot = 4 * (4 * c + (q ^ swz(c)));
  // y[j - 2L] of position c of run 4 q + v: the swizzle of runs 4 q, 4 q + 1; its low bit flips for
  // 4 q + 2, 4 q + 3
  const int bs = (q >> 1) | ((q & 1) << 1);
  const int bslot0 = 64 * q + 4 * ((c >> 2) ^ bs) + (c & 3);
  const int bslot1 = 64 * q + 32 + 4 * ((c >> 2) ^ bs ^ 1) + (c & 3);

  // run sums of a granule from the lane's operand quad d: Re, Im of state 4 s + q of run c in slot s
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

  const int64_t js = kGran * g0 - m + row.jout0;   // position of the piece's first output
  // the states before position js: every lane of row q holds state 4 s + q in slot s
  double zr[ST][NS], zi[ST][NS];
#pragma unroll
  for (int t = 0; t < ST; ++t)
#pragma unroll
    for (int s = 0; s < NS; ++s) { zr[t][s] = 0; zi[t][s] = 0; }
  {
    const int64_t lo = js - L2 > 0 ? js - L2 : 0;
    const int64_t nw = js > lo && lo < N ? (js - lo + kGran - 1) / kGran : 0;
    if (nw > 0) {
      Quad<IN> y;
      int64_t p = js - kGran * nw;
      y.load(xs, p, lo, N, N, lane);
      for (int64_t i = 0; i < nw; ++i) {
#pragma unroll
        for (int t = 0; t < ST; ++t) *reinterpret_cast<v4f*>(s_y[t] + wslot) = y.f32(t);
        p += kGran;
        if (i + 1 < nw) y.load(xs, p, lo, N, N, lane);
        lds_order();
        v4f ya[ST];
#pragma unroll
        for (int t = 0; t < ST; ++t) ya[t] = *reinterpret_cast<const v4f*>(s_y[t] + rslot);
        lds_order();
#pragma unroll
        for (int t = 0; t < ST; ++t) {
          const double d[4] = {(double)ya[t][0], (double)ya[t][1], (double)ya[t][2], (double)ya[t][3]};
          double br[NS], bi[NS];
          run_sums(d, br, bi);
#pragma unroll
          for (int s = 0; s < NS; ++s) {   // per run: acc <- a^256 acc + B
            const double nr = fma(gr[s], zr[t][s], fma(-gi[s], zi[t][s], br[s]));
            zi[t][s] = fma(gr[s], zi[t][s], fma(gi[s], zr[t][s], bi[s]));
            zr[t][s] = nr;
          }
        }
      }
      // sum over the runs, weighted a^{16 (15 - c)}
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double wr = td[lay.dLANE(s, 0) + (lane ^ 15)], wi = td[lay.dLANE(s, 1) + (lane ^ 15)];
#pragma unroll
        for (int t = 0; t < ST; ++t) {
          double vr = wr * zr[t][s] - wi * zi[t][s], vi = wr * zi[t][s] + wi * zr[t][s];
#pragma unroll
          for (int off = 8; off >= 1; off >>= 1) { vr += __shfl_xor(vr, off, 64); vi += __shfl_xor(vi, off, 64); }
          zr[t][s] = vr; zi[t][s] = vi;
        }
      }
    }
  }

  Quad<IN> ya, yb;
  ya.load(xs, js, 0, N, N, lane);
  yb.load(xs, js - L2, 0, N, N, lane);
  for (int64_t g = 0; g < gn; ++g) {
    const int64_t j = js + kGran * g;
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      *reinterpret_cast<v4f*>(s_y[t] + wslot) = ya.f32(t);
      *reinterpret_cast<v4f*>(s_b[t] + wslot) = yb.f32(t);
    }
    if (g + 1 < gn) {   // the next granule's samples, in flight during this one
      ya.load(xs, j + kGran, 0, N, N, lane);
      yb.load(xs, j + kGran - L2, 0, N, N, lane);
    }
    lds_order();
    float df[ST][4], b[ST][4];
    double d[ST][4];
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      const v4f a = *reinterpret_cast<const v4f*>(s_y[t] + rslot), bb = *reinterpret_cast<const v4f*>(s_b[t] + rslot);
#pragma unroll
      for (int k = 0; k < 4; ++k) { d[t][k] = fma(-Dd, (double)bb[k], (double)a[k]); df[t][k] = (float)d[t][k]; }
      b[t][0] = s_b[t][bslot0]; b[t][1] = s_b[t][bslot0 + 16];
      b[t][2] = s_b[t][bslot1]; b[t][3] = s_b[t][bslot1 + 16];
    }
    lds_order();

    double br[ST][NS], bi[ST][NS];
    bool odd = false;   // some input is infinite or NaN (or the run's sum overflows)
#pragma unroll
    for (int t = 0; t < ST; ++t) odd = odd || !__builtin_isfinite((df[t][0] + df[t][1]) + (df[t][2] + df[t][3]));

    v4f o[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[k][v] = Y[k] * b[k % ST][v];
    if (__ballot(odd) == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < NC; ++k) o[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(df[k % ST][i], T[k][i], o[k], 0, 0, 0);
    } else {
#pragma unroll 1
      for (int r = 0; r < kRun; ++r) {   // column r from the inputs up to position r
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          v4f t = o[k];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            t = __builtin_amdgcn_mfma_f32_16x16x4f32(4 * q + i <= r ? df[k % ST][i] : 0.0f, T[k][i], t, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; ++v) o[k][v] = c == r ? t[v] : o[k][v];
        }
      }
    }

#pragma unroll
    for (int t = 0; t < ST; ++t) run_sums(d[t], br[t], bi[t]);

    // states before the runs
    float sf[ST][2 * NS];
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      // the granule's carry enters run 0: B_0 += a^16 Z, then one scan gives the full states
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double fr = c == 0 ? zr[t][s] : 0.0, fi = c == 0 ? zi[t][s] : 0.0;
        br[t][s] = fma(scr[0][s], fr, fma(-sci[0][s], fi, br[t][s]));
        bi[t][s] = fma(scr[0][s], fi, fma(sci[0][s], fr, bi[t][s]));
      }
#define MK_LEVEL(D, SH)                                                              \
  _Pragma("unroll") for (int s = 0; s < NS; ++s) {                                   \
    const double ur = row_shr<SH>(br[t][s]), ui = row_shr<SH>(bi[t][s]);               \
    br[t][s] = fma(scr[D][s], ur, fma(-sci[D][s], ui, br[t][s]));                    \
    bi[t][s] = fma(scr[D][s], ui, fma(sci[D][s], ur, bi[t][s]));                     \
  }
      MK_LEVEL(0, 1) MK_LEVEL(1, 2) MK_LEVEL(2, 4) MK_LEVEL(3, 8)
#undef MK_LEVEL
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double er = row_shr<1>(br[t][s]), ei = row_shr<1>(bi[t][s]);
        sf[t][2 * s] = (float)(c == 0 ? zr[t][s] : er);
        sf[t][2 * s + 1] = (float)(c == 0 ? zi[t][s] : ei);
        zr[t][s] = row_last(br[t][s]);
        zi[t][s] = row_last(bi[t][s]);
      }
    }
#pragma unroll
    for (int i = 0; i < 2 * NS; ++i)
#pragma unroll
      for (int k = 0; k < NC; ++k) o[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(sf[k % ST][i], C[k][i], o[k], 0, 0, 0);

    // lane 16 q + r: position r of runs 4 q + v
    const int64_t n0 = kGran * (g0 + g) - m;
    unsigned char* w = REV ? W + (N - 1 - n0) * OB : W + n0 * OB;   // wave-uniform
    const bool whole = n0 >= 0 && n0 + kGran <= N;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = 64 * q + 16 * v + c;
      if (whole || (n0 + e >= 0 && n0 + e < N)) {
        if constexpr (REV) {
          float* y = reinterpret_cast<float*>(w) - e;
          __builtin_nontemporal_store(CPLX ? o[0][v] + o[NC - 1][v] : o[0][v], y);
        } else if constexpr (CPLX) {
          __builtin_nontemporal_store(v2f{o[0][v], o[NC - 1][v]}, reinterpret_cast<v2f*>(w) + e);
        } else {
          __builtin_nontemporal_store(o[0][v], reinterpret_cast<float*>(w) + e);
        }
      }
    }
  }
}

using GranFn = void (*)(GranLaunch);

template <int NS>
GranFn pick(bool cplx, int in) {
#define MK_PICK(C, D) \
  if (cplx == (C) && in == (D)) return granule_kernel<NS, C, D>;
  MK_PICK(false, 0) MK_PICK(false, 1) MK_PICK(false, 2) MK_PICK(false, 4)
  MK_PICK(true, 0) MK_PICK(true, 1) MK_PICK(true, 2) MK_PICK(true, 3)
#undef MK_PICK
  return nullptr;
}

}  // namespace

hipError_t launch_granules(const GranLaunch& a, hipStream_t s) {
  if (a.nseg <= 0) return hipSuccess;
  if (a.K < 1 || a.K > kMaxTerms || a.nseg > 0x7fffffff || (!a.segs && (a.pieces < 1 || a.nseg != (int64_t)a.nrows * a.pieces)))
    return hipErrorInvalidValue;
  const bool cplx = a.kind == 0;
  const int ns = GranLayout{a.K}.NS();
  const int in = a.adjoint ? (cplx ? 3 : 4) : a.dtype;
  const GranFn fn = ns == 1 ? pick<1>(cplx, in) : ns == 2 ? pick<2>(cplx, in) : pick<3>(cplx, in);
  if (!fn) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fn, dim3((unsigned)a.nseg), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace mk
