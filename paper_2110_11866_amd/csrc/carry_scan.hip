// Carried granule scan (gfx950): rows whose window is much longer than what a wave runs.
//
// The granule scan (granule_scan.hip) lets every piece of a row sum the 2L samples before it. Where the
// window is long against the pieces that fill the device, that sum is most of the work. Here a piece is
// run by a block of 8 waves, 8 consecutive granules (a chunk of 2048 positions) at a time, and two launches
// hand the states on:
//   1. carry_sums_kernel: the state at the end of each piece from a zero state at its start, float64;
//   2. carry_kernel: the state before a piece is sum_e a^{e n} of the earlier pieces' sums (e pieces back, n
//      positions long), one term per lane; then chunk by chunk each wave runs its granule from a zero
//      state, the waves' totals meet in LDS, and what enters the granule is added to its runs' states
//      before the outputs' products.
// No block waits for another: the order of the two launches is the only dependence.
//
// Bound: the latency of the two launches for short rows (N = 102400, 2L = 49152), the issue of
// instructions as in the granule scan for long ones.
#include <hip/hip_runtime.h>

#include "granule.h"
#include "granule_ops.h"
#include "launch.h"
#include "scan_common.h"

namespace mk {
namespace {

constexpr int kCW = kCarryWaves;

template <int SH, typename T>
__device__ __forceinline__ T row_ror(T v) {   // lane c of each 16-lane row reads lane (c - SH) mod 16
  return __builtin_amdgcn_update_dpp((T)0, v, 0x120 + SH, 0xF, 0xF, true);
}
__device__ __forceinline__ double row_sum(double v) {   // sum over the lanes of a row, in all of them
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  return v + row_ror<1>(v);
}

// The row, piece and first position of a block.
struct Place {
  Row row;
  int64_t first;       // output of the row's first granule (<= 0: granules start on 128-byte lines of the output)
  int64_t jd;          // position of the row's first chunk, whole chunks before the first granule's
  const void* xs;
  unsigned char* W;
};
template <bool CPLX, int IN>
__device__ __forceinline__ Place place(const GranLaunch& P) {
  constexpr bool REV = IN >= kInRev;
  constexpr int IB = IN == 0 || IN == 4 ? 4 : IN == 3 ? 8 : 2, OB = CPLX && !REV ? 8 : 4;
  Place a;
  a.row = P.row0;
  if (P.nrows != 1) {
    const cptr<Row> rp = (cptr<Row>)P.rows + blockIdx.y;
    a.row.x_off = rp->x_off; a.row.w_off = rp->w_off; a.row.N = rp->N; a.row.L = rp->L;
    a.row.jout0 = rp->jout0; a.row.scale = rp->scale;
  }
  a.xs = static_cast<const char*>(P.x) + (REV ? a.row.w_off : a.row.x_off) * IB;
  a.W = static_cast<unsigned char*>(P.out) + a.row.w_off * OB;
  const int64_t m = REV ? (int64_t)((-reinterpret_cast<uintptr_t>(a.W + a.row.N * OB) & 127) / OB)
                        : (int64_t)((reinterpret_cast<uintptr_t>(a.W) & 127) / OB);
  a.first = -m;
  const int64_t js = a.row.jout0 - m;
  a.jd = js <= 0 ? js : js - (js + kChunk - 1) / kChunk * kChunk;
  return a;
}

// dy of the lane's quad of the wave's granule, from the staged samples
__device__ __forceinline__ void differences(const float* sy, const float* sb, double Dd, float Df, bool wide, double (&d)[4], float (&f)[4]) {
  const v4f a = *reinterpret_cast<const v4f*>(sy);
  const v4f b = *reinterpret_cast<const v4f*>(sb);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    d[k] = 0;
    if (wide) {
      d[k] = fma(-Dd, (double)b[k], (double)a[k]);
      f[k] = (float)d[k];
    } else {
      f[k] = fmaf(-Df, b[k], a[k]);
    }
  }
}

template <int NS, bool CPLX, int IN, bool WIDE>
__global__ __launch_bounds__(64 * kCW) void carry_sums_kernel(GranLaunch P) {
  constexpr int ST = IN == 3 ? 2 : 1;
  __shared__ __align__(16) float s_y[kCW][ST][kGran], s_b[kCW][ST][kGran];
  __shared__ double2 s_z[kCW][ST][NS * 4];
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Place a = place<CPLX, IN>(P);
  const int64_t N = a.row.N, L2 = 2 * a.row.L;
  const GranLayout lay{4 * NS};
  const unsigned char* tb = P.tabs + (int64_t)a.row.scale * P.tab_stride;
  const double* td = reinterpret_cast<const double*>(reinterpret_cast<const float*>(tb) + lay.nFloats());
  const v2i* tq = reinterpret_cast<const v2i*>(tb + lay.quadOff()) + lane;
  int64_t p = a.jd + kChunk * (int64_t)P.seg_n * blockIdx.x + kGran * w;
  Quad<IN> ya, yb;
  ya.load(a.xs, p, 0, N, N, lane);
  yb.load(a.xs, p - L2, 0, N, N, lane);
  RunSums<NS, WIDE> run_sums;
  run_sums.load(lay, td, tq, lane);
  double gr[NS], gi[NS], zr[ST][NS], zi[ST][NS];   // a^2048; sums per column
#pragma unroll
  for (int s = 0; s < NS; ++s) { gr[s] = td[lay.dG(kCW, s, 0) + q]; gi[s] = td[lay.dG(kCW, s, 1) + q]; }
#pragma unroll
  for (int t = 0; t < ST; ++t)
#pragma unroll
    for (int s = 0; s < NS; ++s) { zr[t][s] = 0; zi[t][s] = 0; }
  const double Dd = td[lay.dD()];
  const float Df = (float)Dd;
  const int w1 = 4 * (4 * (lane >> 2) + ((lane & 3) ^ swz(lane >> 2)));
  const int rslot = 4 * (4 * c + (q ^ swz(c)));
  using Sums = RunSums<NS, WIDE>;
  auto sum = [&](auto split) {   // the piece's chunks, the first loaded; returns whether some input had no thirds
    uint32_t top = 0;
    for (int i = 0; i < P.seg_n; ++i) {
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        *reinterpret_cast<v4f*>(s_y[w][t] + w1) = ya.f32(t);
        *reinterpret_cast<v4f*>(s_b[w][t] + w1) = yb.f32(t);
      }
      p += kChunk;
      if (i + 1 < P.seg_n) {
        ya.load(a.xs, p, 0, N, N, lane);
        yb.load(a.xs, p - L2, 0, N, N, lane);
      }
      lds_order();
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        double d[4];
        float f[4];
        differences(s_y[w][t] + rslot, s_b[w][t] + rslot, Dd, Df, WIDE, d, f);
        typename Sums::acc_t acc[Sums::MB] = {};
        if constexpr (WIDE) {
          run_sums.add(d, v6i{}, acc);
        } else if constexpr (decltype(split)::value) {
          keep_top(top, f);
          run_sums.add(d, thirds(f), acc);
        } else {
          run_sums.add_unsplit(f, acc);
        }
        typename Sums::sum_t br[NS], bi[NS];
        Sums::states(acc, br, bi);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          double xr = br[s], xi = bi[s];
          mac(gr[s], gi[s], zr[t][s], zi[t][s], xr, xi);
          zr[t][s] = xr; zi[t][s] = xi;
        }
      }
      lds_order();
    }
    return no_thirds(top);
  };
  if (sum(std::true_type{})) {
    p -= kChunk * (int64_t)P.seg_n;
    ya.load(a.xs, p, 0, N, N, lane);
    yb.load(a.xs, p - L2, 0, N, N, lane);
#pragma unroll
    for (int t = 0; t < ST; ++t)
#pragma unroll
      for (int s = 0; s < NS; ++s) { zr[t][s] = 0; zi[t][s] = 0; }
    sum(std::false_type{});
  }
  // over the columns, weighted a^{16 (15 - c)}, and the waves, a^{256 (7 - w)}
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const double wr = td[lay.dLANE(s, 0) + (lane ^ 15)], wi = td[lay.dLANE(s, 1) + (lane ^ 15)];
    const double er = td[lay.dG(kCW - 1 - w, s, 0) + q], ei = td[lay.dG(kCW - 1 - w, s, 1) + q];
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      const double vr = row_sum(wr * zr[t][s] - wi * zi[t][s]), vi = row_sum(wr * zi[t][s] + wi * zr[t][s]);
      if (c == 0) s_z[w][t][4 * s + q] = make_double2(er * vr - ei * vi, er * vi + ei * vr);
    }
  }
  __syncthreads();
  const int k = threadIdx.x;
  if (k < ST * P.K) {
    const int t = k / P.K, st = k - t * P.K;
    double vr = 0, vi = 0;
#pragma unroll
    for (int i = 0; i < kCW; ++i) { vr += s_z[i][t][st].x; vi += s_z[i][t][st].y; }
    double* o = P.sums + 2 * (((int64_t)blockIdx.y * (P.pieces - 1) + blockIdx.x) * (ST * P.K) + k);
    o[0] = vr;
    o[1] = vi;
  }
}

template <int NS, bool CPLX, int IN, bool WIDE>
__global__ __launch_bounds__(64 * kCW) void carry_kernel(GranLaunch P) {
  constexpr bool REV = IN >= kInRev;
  constexpr int ST = IN == 3 ? 2 : 1, NC = CPLX ? 2 : 1, SETS = NS > 2 ? 2 : 1, OB = CPLX && !REV ? 8 : 4;
  __shared__ __align__(16) float s_y[kCW][ST][kGran], s_b[kCW][ST][kGran];
  __shared__ double2 s_t[2][kCW + 1][ST][NS * 4];   // totals of the waves' granules; last: the chunk's carry
  __shared__ double2 s_k[4 * NS * 4];               // a^{16 2^d} of slot s, row q, at (d NS + s) 4 + q
  __shared__ double2 s_lane[NS][64];                // a^{16 c}
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int piece = blockIdx.x;
  const Place a = place<CPLX, IN>(P);
  const int64_t N = a.row.N, L2 = 2 * a.row.L, jend = N + a.row.jout0;
  const int64_t j0 = a.jd + kChunk * (int64_t)P.seg_n * piece;
  int64_t chunks = (jend - j0 + kChunk - 1) / kChunk;
  chunks = chunks < P.seg_n ? chunks : P.seg_n;
  if (chunks <= 0 || j0 + kChunk * chunks <= a.row.jout0) return;   // no outputs (the whole block)

  const GranLayout lay{4 * NS};
  const unsigned char* tb = P.tabs + (int64_t)a.row.scale * P.tab_stride;
  const float* tf = reinterpret_cast<const float*>(tb);
  const double* td = reinterpret_cast<const double*>(tf + lay.nFloats());
  const v2i* tq = reinterpret_cast<const v2i*>(tb + lay.quadOff()) + lane;
  int64_t j = j0 + kGran * w;
  Quad<IN> ya, yb;
  ya.load(a.xs, j, 0, N, N, lane);
  yb.load(a.xs, j - L2, 0, N, N, lane);

  // the state before the piece: term e pieces back, e = 16 w + c + 128 i
  double zr[ST][NS], zi[ST][NS];
#pragma unroll
  for (int t = 0; t < ST; ++t)
#pragma unroll
    for (int s = 0; s < NS; ++s) { zr[t][s] = 0; zi[t][s] = 0; }
  if (piece > 0) {
    double pr[NS], pi[NS], vr[NS], vi[NS];   // a^{2048 seg_n 2^b}; the lane's weight
    auto mul = [](double xr, double xi, double& yr, double& yi) {
      const double r = xr * yr - xi * yi;
      yi = xr * yi + xi * yr;
      yr = r;
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      double br = td[lay.dG(kCW, s, 0) + q], bi = td[lay.dG(kCW, s, 1) + q];
      pr[s] = 1; pi[s] = 0;
      for (int n = P.seg_n; n; n >>= 1) {
        if (n & 1) mul(br, bi, pr[s], pi[s]);
        const double tr = br, ti = bi;
        mul(tr, ti, br, bi);
      }
      vr[s] = 1; vi[s] = 0;
#pragma unroll
      for (int b = 0; b < 7; ++b) {
        double tr = vr[s], ti = vi[s];
        mul(pr[s], pi[s], tr, ti);
        const bool on = ((16 * w + c) >> b) & 1;
        vr[s] = on ? tr : vr[s];
        vi[s] = on ? ti : vi[s];
        const double xr = pr[s], xi = pi[s];
        mul(xr, xi, pr[s], pi[s]);
      }
    }
    const double* sums = P.sums + 2 * (int64_t)blockIdx.y * (P.pieces - 1) * (ST * P.K);
    for (int e = 16 * w + c + (piece - 1) / 128 * 128; e >= 0; e -= 128) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const bool in = e < piece && 4 * s + q < P.K;
#pragma unroll
        for (int t = 0; t < ST; ++t) {
          const double* d = sums + 2 * ((int64_t)(piece - 1 - e) * (ST * P.K) + t * P.K + 4 * s + q);
          double xr = in ? d[0] : 0.0, xi = in ? d[1] : 0.0;
          mac(pr[s], pi[s], zr[t][s], zi[t][s], xr, xi);
          zr[t][s] = xr; zi[t][s] = xi;
        }
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        const double xr = row_sum(vr[s] * zr[t][s] - vi[s] * zi[t][s]), xi = row_sum(vr[s] * zi[t][s] + vi[s] * zr[t][s]);
        if (c == 0) s_t[1][w][t][4 * s + q] = make_double2(xr, xi);
      }
  } else {
    for (int i = lane; i < ST * NS * 4; i += 64) (&s_t[1][w][0][0])[i] = make_double2(0.0, 0.0);
  }
  for (int i = threadIdx.x; i < 4 * NS * 4; i += 64 * kCW) {
    const int d = i / (4 * NS), s = i / 4 % NS;
    s_k[i] = make_double2(td[lay.dSC(d, s, 0) + i % 4], td[lay.dSC(d, s, 1) + i % 4]);
  }
  for (int i = threadIdx.x; i < NS * 64; i += 64 * kCW)
    s_lane[i / 64][i % 64] = make_double2(td[lay.dLANE(i / 64, 0) + i % 64], td[lay.dLANE(i / 64, 1) + i % 64]);
  Weights T[NC], C[NC][SETS];
  float Y[NC];
  RunSums<NS, WIDE> run_sums;
  run_sums.load(lay, td, tq, lane);
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    T[k].load(tq, lay.bT(k, 0), lay.bT(k, 1), lay.bT(k, 2));
#pragma unroll
    for (int e = 0; e < SETS; ++e) C[k][e].load(tq, lay.bC(k, e, 0), lay.bC(k, e, 1), lay.bC(k, e, 2));
  }
  Y[0] = tf[lay.fYre()];
  if constexpr (NC == 2) Y[NC - 1] = tf[lay.fYim()];
  const double Dd = td[lay.dD()];
  const float Df = (float)Dd;
  // what enters the wave's granule: lane c < w adds the total of wave c, lane w the chunk's carry
  double gr[NS], gi[NS], hr[NS], hi[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int k = c < w ? w - 1 - c : w;
    gr[s] = td[lay.dG(k, s, 0) + q]; gi[s] = td[lay.dG(k, s, 1) + q];
    hr[s] = td[lay.dG(1, s, 0) + q]; hi[s] = td[lay.dG(1, s, 1) + q];
  }
  __syncthreads();
  if (w == kCW - 1) {
    for (int i = lane; i < ST * NS * 4; i += 64) {
      double vr = 0, vi = 0;
#pragma unroll
      for (int k = 0; k < kCW; ++k) { vr += (&s_t[1][k][0][0])[i].x; vi += (&s_t[1][k][0][0])[i].y; }
      (&s_t[0][kCW][0][0])[i] = make_double2(vr, vi);
    }
  }

  const int w1 = 4 * (4 * (lane >> 2) + ((lane & 3) ^ swz(lane >> 2)));
  const int rslot = 4 * (4 * c + (q ^ swz(c)));
  const int bs = (q >> 1) | ((q & 1) << 1);
  const int bslot0 = 64 * q + 4 * ((c >> 2) ^ bs) + (c & 3);
  const int bslot1 = 64 * q + 32 + 4 * ((c >> 2) ^ bs ^ 1) + (c & 3);
  const int from = c < w ? c : kCW;
  using Sums = RunSums<NS, WIDE>;
  for (int64_t i = 0; i < chunks; ++i, j += kChunk) {
    const int par = (int)(i & 1);
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      *reinterpret_cast<v4f*>(s_y[w][t] + w1) = ya.f32(t);
      *reinterpret_cast<v4f*>(s_b[w][t] + w1) = yb.f32(t);
    }
    if (i + 1 < chunks) {
      ya.load(a.xs, j + kChunk, 0, N, N, lane);
      yb.load(a.xs, j + kChunk - L2, 0, N, N, lane);
    }
    lds_order();
    v6i dx[ST];
    double er[ST][NS], ei[ST][NS], fr[ST][NS], fi[ST][NS];
    uint32_t top = 0;
    unsigned nan = 0;   // the lane's inputs that are infinite or NaN
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      double d[4];
      float f[4];
      differences(s_y[w][t] + rslot, s_b[w][t] + rslot, Dd, Df, WIDE, d, f);
      keep_top(top, f);
      dx[t] = thirds(f);
      typename Sums::acc_t acc[Sums::MB] = {};
      run_sums.add(d, dx[t], acc);
      typename Sums::sum_t br[NS], bi[NS];
      Sums::states(acc, br, bi);
#pragma unroll
      for (int s = 0; s < NS; ++s) { fr[t][s] = br[s]; fi[t][s] = bi[s]; }
    }
    bool slow = no_thirds(top);
    if (slow) {   // the run sums of the inputs as they are
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        double d[4];
        float f[4];
        differences(s_y[w][t] + rslot, s_b[w][t] + rslot, Dd, Df, WIDE, d, f);
        if constexpr (!WIDE) {
          typename Sums::acc_t acc[Sums::MB] = {};
          run_sums.add_unsplit(f, acc);
          typename Sums::sum_t br[NS], bi[NS];
          Sums::states(acc, br, bi);
#pragma unroll
          for (int s = 0; s < NS; ++s) { fr[t][s] = br[s]; fi[t][s] = bi[s]; }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) nan |= __builtin_isfinite(f[k]) ? 0u : 1u << k;
      }
    }
#pragma unroll
    for (int t = 0; t < ST; ++t) {
      // inclusive scan of the runs from a zero state
#define MK_LEVEL(D, SH)                                                                        \
  _Pragma("unroll") for (int s = 0; s < NS; ++s) {                                             \
    const double2 k = s_k[(D * NS + s) * 4 + q];                                               \
    mac(k.x, k.y, row_shr<SH>(fr[t][s]), row_shr<SH>(fi[t][s]), fr[t][s], fi[t][s]);           \
  }
      if (i == 0 && t == 0) __syncthreads();   // s_k, s_lane and the first carry
      MK_LEVEL(0, 1) MK_LEVEL(1, 2) MK_LEVEL(2, 4) MK_LEVEL(3, 8)
#undef MK_LEVEL
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (c == 15) s_t[par][w][t][4 * s + q] = make_double2(fr[t][s], fi[t][s]);
        er[t][s] = row_shr<1>(fr[t][s]);
        ei[t][s] = row_shr<1>(fi[t][s]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < ST; ++t)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double2 v = s_t[par][from][t][4 * s + q];
        const bool in = c <= w;
        const double xr = row_sum(in ? gr[s] * v.x - gi[s] * v.y : 0.0), xi = row_sum(in ? gr[s] * v.y + gi[s] * v.x : 0.0);
        if (w == kCW - 1 && c == 15) {   // the next chunk's carry
          double yr = fr[t][s], yi = fi[t][s];
          mac(hr[s], hi[s], xr, xi, yr, yi);
          s_t[par ^ 1][kCW][t][4 * s + q] = make_double2(yr, yi);
        }
        const double2 l = s_lane[s][lane];
        mac(l.x, l.y, xr, xi, er[t][s], ei[t][s]);
      }
    if (all_small(top) && !slow) {   // zeros: outputs of the entering states
#pragma unroll
      for (int t = 0; t < ST; ++t) slow = slow || no_thirds(er[t], ei[t]);
    }

    auto components = [&](int e, int t, float (&x)[4]) {   // states 2 e, 2 e + 1 of stream t in float32
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int s = 2 * e + k / 2;
        x[k] = s < NS ? (float)(k & 1 ? ei[t][s < NS ? s : 0] : er[t][s < NS ? s : 0]) : 0.0f;
      }
    };
    v4f o[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const float* b = s_b[w][k % ST];
      const float bv[4] = {b[bslot0], b[bslot0 + 16], b[bslot1], b[bslot1 + 16]};
#pragma unroll
      for (int v = 0; v < 4; ++v) o[k][v] = Y[k] * bv[v];
      o[k] = product(dx[k % ST], T[k], o[k]);
    }
    if (slow) {   // from the inputs and states as they are; infinite and NaN inputs count as zeros
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        double d[4];
        float f[4];
        differences(s_y[w][k % ST] + rslot, s_b[w][k % ST] + rslot, Dd, Df, WIDE, d, f);
#pragma unroll
        for (int v = 0; v < 4; ++v) f[v] = __builtin_isfinite(f[v]) ? f[v] : 0.0f;
        const float* b = s_b[w][k % ST];
        o[k] = product_unsplit(f, T[k], v4f{Y[k] * b[bslot0], Y[k] * b[bslot0 + 16], Y[k] * b[bslot1], Y[k] * b[bslot1 + 16]});
#pragma unroll
        for (int e = 0; e < SETS; ++e) {
          float x[4];
          components(e, k % ST, x);
          o[k] = product_unsplit(x, C[k][e], o[k]);
        }
      }
#pragma unroll
      for (int t = 0; t < ST; ++t)
#pragma unroll
        for (int s = 0; s < NS; ++s) { er[t][s] = 0; ei[t][s] = 0; }
      // an infinite or NaN input reaches the outputs of its run from its own position on: bit 16 q' + c'
      // of bad marks input 4 q' + e of column c'
#pragma unroll 1
      for (int e = 0; e < 4; ++e) {
        const unsigned long long bad = __ballot((nan >> e) & 1);
        unsigned long long upto = 0;   // columns 4 q + v, positions 4 q' + e <= c
        for (int r = 0; r < 4; ++r)
          if (4 * r + e <= c) upto |= bad >> (16 * r);
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if ((upto >> (4 * q + v)) & 1)
#pragma unroll
            for (int k = 0; k < NC; ++k) o[k][v] = __builtin_nanf("");
      }
    }
#pragma unroll
    for (int e = 0; e < SETS; ++e) {
      v6i sx[ST];
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        float x[4];
        components(e, t, x);
        sx[t] = thirds(x);
      }
#pragma unroll
      for (int k = 0; k < NC; ++k) o[k] = product(sx[k % ST], C[k][e], o[k]);
    }
    // lane 16 q + r: position r of columns 4 q + v
    const int64_t n0 = j - a.row.jout0;
    unsigned char* out = REV ? a.W + (N - 1 - n0) * OB : a.W + n0 * OB;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = kRun * (4 * q + v) + c;
      if (n0 + e >= 0 && n0 + e < N) {
        if constexpr (REV) {
          __builtin_nontemporal_store(CPLX ? o[0][v] + o[NC - 1][v] : o[0][v], reinterpret_cast<float*>(out) - e);
        } else if constexpr (CPLX) {
          __builtin_nontemporal_store(v2f{o[0][v], o[NC - 1][v]}, reinterpret_cast<v2f*>(out) + e);
        } else {
          __builtin_nontemporal_store(o[0][v], reinterpret_cast<float*>(out) + e);
        }
      }
    }
    lds_order();   // the next samples overwrite these
  }
}

using GranFn = void (*)(GranLaunch);

template <int NS>
void pick(bool cplx, int in, bool wide, GranFn& sums, GranFn& scan) {
#define MK_PICK(C, D)                                                                       \
  if (cplx == (C) && in == (D)) {                                                           \
    sums = wide ? carry_sums_kernel<NS, C, D, true> : carry_sums_kernel<NS, C, D, false>;   \
    scan = wide ? carry_kernel<NS, C, D, true> : carry_kernel<NS, C, D, false>;             \
  }
  MK_PICK(false, 0) MK_PICK(false, 1) MK_PICK(false, 2) MK_PICK(false, 4)
  MK_PICK(true, 0) MK_PICK(true, 1) MK_PICK(true, 2) MK_PICK(true, 3)
#undef MK_PICK
}

}  // namespace

hipError_t launch_carried(const GranLaunch& a, hipStream_t s) {
  if (a.K < 1 || a.K > kMaxTerms || a.nrows < 1 || a.nrows > 65535 || a.pieces < 1 || a.seg_n < 1 || (a.pieces > 1 && !a.sums))
    return hipErrorInvalidValue;
  const bool cplx = a.kind == 0, wide = a.acc == kAccMixed;
  const int ns = GranLayout{a.K}.NS(), in = a.adjoint ? (cplx ? 3 : 4) : a.dtype;
  GranFn sums = nullptr, scan = nullptr;
  if (ns == 1) pick<1>(cplx, in, wide, sums, scan);
  else if (ns == 2) pick<2>(cplx, in, wide, sums, scan);
  else pick<3>(cplx, in, wide, sums, scan);
  if (!scan) return hipErrorInvalidValue;
  if (a.pieces > 1) {   // the last piece's sum enters nothing
    hipLaunchKernelGGL(sums, dim3(a.pieces - 1, a.nrows), dim3(64 * kCW), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(scan, dim3(a.pieces, a.nrows), dim3(64 * kCW), 0, s, a);
  return hipGetLastError();
}

}  // namespace mk
