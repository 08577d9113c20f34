// Granule scan (gfx950): the forward transform on the matrix cores, one wave per piece of a row.
//
// The state of the scan (scan_kernel.h: v_p[j] = a v_p[j-1] + dy[j], dy[j] = y[j] - a^{2L} y[j-2L])
// is the windowed sum v_p[j] = sum_{q = j-2L+1}^{j} a^{j-q} y[q]: it can be formed at any position
// from the 2L samples before it. So a row is cut into pieces that never wait on each other: a wave
// sums the window before its piece (run sums only, no outputs), then runs the piece granule by
// granule, 256 positions as 16 runs of 16:
//   1. dy of run c as operand: lane 16 q + c holds dy[4 q .. 4 q + 3] of run c. The quads are loaded
//      coalesced, lane l the l-th quad (16-byte loads at any sample alignment), and change lanes
//      through LDS, swizzled so neither side conflicts;
//   2. run sums B = P dy (2K x 16 by 16 x 16): lane 16 q + c receives the components of states q, q + 4,
//      q + 8 of run c. Float64 product for the mixed scan; from float32 to float32 for the float32 scan;
//   3. float64 scan of the runs along the 16 lanes of a DPP row (4 levels, constants a^{16 2^d}), the
//      state before the granule entering run 0;
//   4. outputs of run c, position r: o = T dy + C S + Y y[j-2L], one product per component with the
//      runs as rows and the positions as columns, so lane 16 q + r holds position r of runs
//      4 q .. 4 q + 3 and a store instruction writes whole 128-byte lines.
// The recurrence over the 16 positions and the K-term combination, 36 vector operations per position
// at K = 5, become 42 multiply-adds of matrix products.
//
// Float32 products run on the bfloat16 matrix cores as products of exact thirds (24 bits = 3 x 8): a
// float32 or float64 matrix instruction has the vector units' rate and does not run beside them, the
// bfloat16 one does 14 times the work. Six of the nine products of thirds keep float32 accuracy.
//
// Bound: issue of vector and matrix instructions (about 680 cycles of a SIMD per 256 outputs at K = 5,
// 683 us of a 488e6-output scalogram without its stores), then the stores (3.9 GB at 5.3-5.8 TB/s, 740 us
// without the products); together 910 us back to back (a launch timed alone 1030), the tile scan 1390.
//
// Zeros of T meet inputs of the same run at later positions: where a run has an infinite or NaN input,
// the product takes zero for it and its outputs from that position on are set to NaN, so no output
// depends on a later input. A wave with such inputs, with finite ones so large that their nearest bfloat16 is
// infinite, or with nothing but values below 2^-106 (zeros after such values), repeats its products in float32. The states are held at
// half their size (the weights P at half, C at twice theirs): one that is finite in float32 always has thirds.
#include <hip/hip_runtime.h>

#include "granule.h"
#include "granule_ops.h"
#include "launch.h"
#include "scan_common.h"

namespace mk {
namespace {

// IN: the input (Quad). CPLX: the transform's outputs are complex (IN < 3: complex64 out; IN 3: their
// cotangent comes in). An output component k is formed from stream k of the adjoint's two, or from
// the only stream; the adjoint adds its components, Re sum conj(h) g = (h_re * g_re) + (h_im * g_im). Term
// p's part of the sum is Re a^d w_p with w_p = q_re g_re + q_im g_im (q: the term's complex output weights), so
// the complex adjoint runs one state per term on w_p (with a state for each stream 188 us a launch at
// 64 x 32768 x 16 scales, K = 5, now 142).
// NST: runs per lane column; a wave works on 16 columns of NST consecutive runs (256 NST positions) at a
// time, so that the scan across lanes is done once for NST runs.
// WIDE: run sums in float64 (the mixed scan), else from float32 inputs to float32 (the float32 scan);
// everything that propagates from run to run is float64.
template <int NS, bool CPLX, int IN, int NST, bool WIDE>
__global__ __launch_bounds__(64) void granule_kernel(GranLaunch P) {
  constexpr bool REV = IN >= kInRev;
  constexpr int ST = IN == 3 ? 2 : 1, NC = CPLX ? 2 : 1, SETS = NS > 2 ? 2 : 1;
  constexpr int NO = CPLX && !REV ? 2 : 1;   // outputs of a state: the complex adjoint has one state for its two streams
  using Sums = RunSums<NS, WIDE>;
  constexpr int G = kGran * NST;        // positions at a time
  constexpr int PS = NST == 1 ? kGran : kGran + 16;   // floats from one run of the columns to the next
  constexpr int LV = NST - 1;           // log2 NST
  static_assert(NST == 1 || NST == 2);
  static_assert(!REV || CPLX == (IN == 3), "the adjoint's input is the cotangent of the transform's output");
  __shared__ __align__(16) float s_y[ST][NST * PS];   // y[j], by run of the columns, column and quad
  __shared__ __align__(16) float s_b[ST][NST * PS];   // y[j - 2L]
  __shared__ double2 s_k[4 * NS * 4];                 // a^{16 NST 2^d} of slot s, row q, at (d NS + s) 4 + q
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
  // outputs [n0, nend) of the piece
  const int64_t first = kGran * g0 - m;
  int64_t nend = first + kGran * gn;
  nend = nend < N ? nend : N;
  if (first >= nend) return;

  const GranLayout lay{4 * NS};   // layouts differ by the slot count only
  const unsigned char* tb = P.tabs + (int64_t)row.scale * P.tab_stride;
  const float* tf = reinterpret_cast<const float*>(tb);
  const double* td = reinterpret_cast<const double*>(tf + lay.nFloats());
  const v2i* tq = reinterpret_cast<const v2i*>(tb + lay.quadOff()) + lane;
  Weights T[NC], C[NO][SETS];
  float Y[NC];
  double ar[NS], ai[NS];   // a^16
  Sums run_sums[ST];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    T[k].load(tq, lay.bT(k, 0), lay.bT(k, 1), lay.bT(k, 2));
  }
#pragma unroll
  for (int k = 0; k < NO; ++k)
#pragma unroll
    for (int e = 0; e < SETS; ++e) {
      if constexpr (IN == 3) C[k][e].load(tq, lay.bCA(e, 0), lay.bCA(e, 1), lay.bCA(e, 2));
      else C[k][e].load(tq, lay.bC(k, e, 0), lay.bC(k, e, 1), lay.bC(k, e, 2));
    }
#pragma unroll
  for (int t = 0; t < ST; ++t) run_sums[t].load(lay, td, tq, lane, IN == 3 ? t : -1);
#pragma unroll
  for (int s = 0; s < NS; ++s) { ar[s] = td[lay.dSC(0, s, 0) + q]; ai[s] = td[lay.dSC(0, s, 1) + q]; }
  Y[0] = tf[lay.fYre()];
  if constexpr (NC == 2) Y[NC - 1] = tf[lay.fYim()];
  const double Dd = td[lay.dD()];
  const float Df = (float)Dd;

  for (int i = lane; i < 4 * NS * 4; i += 64) {
    const int d = i / (4 * NS), s = i / 4 % NS;
    s_k[i] = make_double2(td[lay.dSC(LV + d, s, 0) + i % 4], td[lay.dSC(LV + d, s, 1) + i % 4]);
  }

  // quad of run i of column c: i PS + 4 (4 c + (q ^ swz(c))) floats. Written: lane l of load k holds
  // positions 256 k + 4 l .., i.e. column 16 k / NST + l / (4 NST), run (l / 4) % NST, quad l % 4.
  const int lc = lane / (4 * NST), li = (lane >> 2) % NST;
  int wslot[NST];
#pragma unroll
  for (int k = 0; k < NST; ++k) {
    const int cc = k * (16 / NST) + lc;
    wslot[k] = li * PS + 4 * (4 * cc + ((lane & 3) ^ swz(cc)));
  }
  const int rslot = 4 * (4 * c + (q ^ swz(c)));
  // y[j - 2L] of position c of column 4 q + v: the swizzle of columns 4 q, 4 q + 1; its low bit flips
  // for 4 q + 2, 4 q + 3
  const int bs = (q >> 1) | ((q & 1) << 1);
  const int bslot0 = 64 * q + 4 * ((c >> 2) ^ bs) + (c & 3);
  const int bslot1 = 64 * q + 32 + 4 * ((c >> 2) ^ bs ^ 1) + (c & 3);

  using sum_t = typename Sums::sum_t;
  const int64_t js = first + row.jout0;   // position of the piece's first output
  // the states before position js: every lane of row q holds state 4 s + q in slot s
  double zr[NS], zi[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) { zr[s] = 0; zi[s] = 0; }
  {
    const int64_t lo = js - L2 > 0 ? js - L2 : 0;
    const int64_t nw = js > lo && lo < N ? (js - lo + kGran - 1) / kGran : 0;
    if (nw > 0) {   // 256 positions at a time, run c of 16 per lane column
      const int w1 = 4 * (4 * (lane >> 2) + ((lane & 3) ^ swz(lane >> 2)));
      double gr[NS], gi[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) { gr[s] = td[lay.dG(1, s, 0) + q]; gi[s] = td[lay.dG(1, s, 1) + q]; }
      auto window = [&](auto split) {   // returns whether some input had no thirds
        Quad<IN> y;
        int64_t p = js - kGran * nw;
        uint32_t top = 0;
        y.load(xs, p, lo, N, N, lane);
        for (int64_t i = 0; i < nw; ++i) {
#pragma unroll
          for (int t = 0; t < ST; ++t) *reinterpret_cast<v4f*>(s_y[t] + w1) = y.f32(t);
          p += kGran;
          if (i + 1 < nw) y.load(xs, p, lo, N, N, lane);
          lds_order();
          v4f ya[ST];
#pragma unroll
          for (int t = 0; t < ST; ++t) ya[t] = *reinterpret_cast<const v4f*>(s_y[t] + rslot);
          lds_order();
          typename Sums::acc_t acc[Sums::MB] = {};
#pragma unroll
          for (int t = 0; t < ST; ++t) {
            const double d[4] = {(double)ya[t][0], (double)ya[t][1], (double)ya[t][2], (double)ya[t][3]};
            const float f[4] = {ya[t][0], ya[t][1], ya[t][2], ya[t][3]};
            if constexpr (WIDE) {
              run_sums[t].add(d, v6i{}, acc);
            } else if constexpr (decltype(split)::value) {
              keep_top(top, f);
              run_sums[t].add(d, thirds(f), acc);
            } else {
              run_sums[t].add_unsplit(f, acc);
            }
          }
          sum_t br[NS], bi[NS];
          Sums::states(acc, br, bi);
#pragma unroll
          for (int s = 0; s < NS; ++s) {   // per column: z <- a^256 z + B
            double xr = br[s], xi = bi[s];
            mac(gr[s], gi[s], zr[s], zi[s], xr, xi);
            zr[s] = xr; zi[s] = xi;
          }
        }
        return no_thirds(top);
      };
      if (window(std::true_type{})) {
#pragma unroll
        for (int s = 0; s < NS; ++s) { zr[s] = 0; zi[s] = 0; }
        window(std::false_type{});
      }
      // sum over the columns, weighted a^{16 (15 - c)}
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double wr = td[lay.dLANE(s, 0) + (lane ^ 15)], wi = td[lay.dLANE(s, 1) + (lane ^ 15)];
        double vr = wr * zr[s] - wi * zi[s], vi = wr * zi[s] + wi * zr[s];
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) { vr += __shfl_xor(vr, off, 64); vi += __shfl_xor(vi, off, 64); }
        zr[s] = vr; zi[s] = vi;
      }
    }
  }

  Quad<IN> ya[NST], yb[NST];
#pragma unroll
  for (int k = 0; k < NST; ++k) {
    ya[k].load(xs, js + kGran * k, 0, N, N, lane);
    yb[k].load(xs, js + kGran * k - L2, 0, N, N, lane);
  }
  // one step from output n0. INNER: every output is the piece's, and the next step's samples lie inside the
  // signal: the stores and loads are unconditional, so waiting for the loads does not wait for stores
  // that follow them.
  auto step = [&](auto inner, int64_t n0) {
    constexpr bool INNER = decltype(inner)::value;
#pragma unroll
    for (int t = 0; t < ST; ++t)
#pragma unroll
      for (int k = 0; k < NST; ++k) {
        *reinterpret_cast<v4f*>(s_y[t] + wslot[k]) = ya[k].f32(t);
        *reinterpret_cast<v4f*>(s_b[t] + wslot[k]) = yb[k].f32(t);
      }
    if (INNER || n0 + G < nend) {   // the next samples, in flight during these
      const int64_t j = n0 + G + row.jout0;
#pragma unroll
      for (int k = 0; k < NST; ++k) {
        ya[k].template load<INNER>(xs, j + kGran * k, 0, N, N, lane);
        yb[k].template load<INNER>(xs, j + kGran * k - L2, 0, N, N, lane);
      }
    }
    lds_order();

    // float32 dy of run i, for the rare cases
    auto differences = [&](int t, int i, float (&f)[4]) {
      const v4f a = *reinterpret_cast<const v4f*>(s_y[t] + i * PS + rslot);
      const v4f b = *reinterpret_cast<const v4f*>(s_b[t] + i * PS + rslot);
#pragma unroll
      for (int k = 0; k < 4; ++k) f[k] = WIDE ? (float)fma(-Dd, (double)b[k], (double)a[k]) : fmaf(-Df, b[k], a[k]);
    };
    // run sums of the columns' runs, then the state before each column
    float df[WIDE ? ST : 1][NST][4];       // dy (WIDE), or its thirds
    v6i dx[WIDE ? 1 : ST][NST];
    sum_t br[NST][NS], bi[NST][NS];
    double er[NS], ei[NS];
    uint32_t top = 0;
#pragma unroll
    for (int i = 0; i < NST; ++i) {
      typename Sums::acc_t acc[Sums::MB] = {};
#pragma unroll
      for (int t = 0; t < ST; ++t) {
        const v4f a = *reinterpret_cast<const v4f*>(s_y[t] + i * PS + rslot);
        const v4f b = *reinterpret_cast<const v4f*>(s_b[t] + i * PS + rslot);
        double d[4] = {0, 0, 0, 0};
        float f[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if constexpr (WIDE) {
            d[k] = fma(-Dd, (double)b[k], (double)a[k]);
            f[k] = df[t][i][k] = (float)d[k];
          } else {
            f[k] = fmaf(-Df, b[k], a[k]);
          }
        }
        keep_top(top, f);
        if constexpr (!WIDE) dx[t][i] = thirds(f);
        run_sums[t].add(d, dx[WIDE ? 0 : t][i], acc);
        __builtin_amdgcn_sched_barrier(0);   // a run at a time (registers)
      }
      Sums::states(acc, br[i], bi[i]);
    }
    bool slow = no_thirds(top);
    if (all_small(top) && !slow) slow = no_thirds(zr, zi);   // zeros: outputs of the entering state
    if (!WIDE && slow) {   // the run sums of the inputs as they are
#pragma unroll
      for (int i = 0; i < NST; ++i) {
        typename Sums::acc_t acc[Sums::MB] = {};
#pragma unroll
        for (int t = 0; t < ST; ++t) {
          float f[4];
          differences(t, i, f);
          run_sums[t].add_unsplit(f, acc);
          __builtin_amdgcn_sched_barrier(0);
        }
        Sums::states(acc, br[i], bi[i]);
      }
    }
    {
      double fr[NS], fi[NS];   // sum over the column's runs; the carry enters column 0
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        fr[s] = c == 0 ? zr[s] : 0.0;
        fi[s] = c == 0 ? zi[s] : 0.0;
#pragma unroll
        for (int i = 0; i < NST; ++i) {
          double xr = br[i][s], xi = bi[i][s];
          mac(ar[s], ai[s], fr[s], fi[s], xr, xi);
          fr[s] = xr; fi[s] = xi;
        }
      }
      // inclusive scan over the columns, constants a^{16 NST 2^d}
#define MK_LEVEL(D, SH)                                                                        \
  _Pragma("unroll") for (int s = 0; s < NS; ++s) {                                             \
    const double2 a = s_k[(D * NS + s) * 4 + q];                                               \
    mac(a.x, a.y, row_shr<SH>(fr[s]), row_shr<SH>(fi[s]), fr[s], fi[s]);                       \
  }
      MK_LEVEL(0, 1) MK_LEVEL(1, 2) MK_LEVEL(2, 4) MK_LEVEL(3, 8)
#undef MK_LEVEL
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double pr = row_shr<1>(fr[s]), pi = row_shr<1>(fi[s]);
        er[s] = c == 0 ? zr[s] : pr;
        ei[s] = c == 0 ? zi[s] : pi;
        zr[s] = row_last(fr[s]);
        zi[s] = row_last(fi[s]);
      }
    }

    unsigned char* w = REV ? W + (N - 1 - n0) * OB : W + n0 * OB;   // wave-uniform
#pragma unroll
    for (int i = 0; i < NST; ++i) {
      v4f o[NC];
      v6i sx[SETS];
      auto components = [&](int e, float (&x)[4]) {   // states 2 e, 2 e + 1 in float32
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int s = 2 * e + k / 2;
          x[k] = s < NS ? (float)(k & 1 ? ei[s < NS ? s : 0] : er[s < NS ? s : 0]) : 0.0f;
        }
      };
#pragma unroll
      for (int e = 0; e < SETS; ++e) {
        float x[4];
        components(e, x);
        sx[e] = thirds(x);
      }
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const float* b = s_b[k % ST] + i * PS;
        const float bv[4] = {b[bslot0], b[bslot0 + 16], b[bslot1], b[bslot1 + 16]};
#pragma unroll
        for (int v = 0; v < 4; ++v) o[k][v] = Y[k] * bv[v];
      }
      [[maybe_unused]] v6i wx[ST];
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        if constexpr (WIDE) {
          if (k < ST) wx[k] = thirds(df[k % ST][i]);
          o[k] = product(wx[k % ST], T[k], o[k]);
        } else {
          o[k] = product(dx[k % ST][i], T[k], o[k]);
        }
      }
      if (slow) {   // from the inputs and states as they are; infinite and NaN inputs count as zeros
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          float f[4];
          differences(k % ST, i, f);
#pragma unroll
          for (int v = 0; v < 4; ++v) f[v] = __builtin_isfinite(f[v]) ? f[v] : 0.0f;
          const float* b = s_b[k % ST] + i * PS;
          __builtin_amdgcn_sched_barrier(0);
          o[k] = product_unsplit(f, T[k], v4f{Y[k] * b[bslot0], Y[k] * b[bslot0 + 16], Y[k] * b[bslot1], Y[k] * b[bslot1 + 16]});
        }
#pragma unroll
        for (int e = 0; e < SETS; ++e) {
          float x[4];
          __builtin_amdgcn_sched_barrier(0);
          components(e, x);
          sx[e] = v6i{};
#pragma unroll
          for (int k = 0; k < NO; ++k) o[k] = product_unsplit(x, C[k][e], o[k]);
        }
        // an infinite or NaN input reaches the outputs of its run from its own position on: bit 16 q' + c'
        // of bad marks input 4 q' + e of column c'
#pragma unroll 1
        for (int e = 0; e < 4; ++e) {
          bool mine = false;
#pragma unroll
          for (int t = 0; t < ST; ++t) {
            float f[4];
            differences(t, i, f);
            const float fe = e == 0 ? f[0] : e == 1 ? f[1] : e == 2 ? f[2] : f[3];
            mine = mine || !__builtin_isfinite(fe);
          }
          const unsigned long long bad = __ballot(mine);
          // columns 4 q + v, positions 4 q' + e <= c
          unsigned long long upto = 0;
          for (int r = 0; r < 4; ++r)
            if (4 * r + e <= c) upto |= bad >> (16 * r);
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if ((upto >> (4 * q + v)) & 1)
#pragma unroll
              for (int k = 0; k < NC; ++k) o[k][v] = __builtin_nanf("");
        }
      }
      if (i + 1 < NST) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {   // on to the next run of the column
          double xr = br[i][s], xi = bi[i][s];
          mac(ar[s], ai[s], er[s], ei[s], xr, xi);
          er[s] = xr; ei[s] = xi;
        }
      }
#pragma unroll
      for (int k = 0; k < NO; ++k)
#pragma unroll
        for (int e = 0; e < SETS; ++e) o[k] = product(sx[e], C[k][e], o[k]);

      // lane 16 q + r: position r of run i of columns 4 q + v
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int e = kRun * (NST * (4 * q + v) + i) + c;
        if (INNER || (n0 + e >= 0 && n0 + e < nend)) {
          if constexpr (REV) {
            __builtin_nontemporal_store(CPLX ? o[0][v] + o[NC - 1][v] : o[0][v], reinterpret_cast<float*>(w) - e);
          } else if constexpr (CPLX) {
            __builtin_nontemporal_store(v2f{o[0][v], o[NC - 1][v]}, reinterpret_cast<v2f*>(w) + e);
          } else {
            __builtin_nontemporal_store(o[0][v], reinterpret_cast<float*>(w) + e);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    lds_order();   // the next samples overwrite these
  };
  // steps [inner0, inner1) from the first are INNER: outputs n0 >= 0 and n0 + G <= nend, and for the next
  // step's samples j + G - 2L >= 0 and j + 2 G <= N
  const int64_t steps = (nend - first + G - 1) / G;
  auto up = [](int64_t v) { return v <= 0 ? (int64_t)0 : (v + G - 1) / G; };
  const int64_t inner0 = up(-first) > up(L2 - js - G) ? up(-first) : up(L2 - js - G);
  const int64_t fit = nend - first < N - js - G ? nend - first : N - js - G;   // inner while n0 - first + G <= fit
  const int64_t inner1 = fit < G ? 0 : fit / G;
  int64_t k = 0;
  for (; k < steps && (k < inner0 || k >= inner1); ++k) step(std::false_type{}, first + G * k);
  for (; k < inner1; ++k) step(std::true_type{}, first + G * k);
  for (; k < steps; ++k) step(std::false_type{}, first + G * k);
}

using GranFn = void (*)(GranLaunch);

template <int NS>
GranFn pick(bool cplx, int in, bool two, bool wide) {
#define MK_PICK(C, D) \
  if (cplx == (C) && in == (D)) \
    return wide ? (two ? granule_kernel<NS, C, D, (D) == 3 ? 1 : 2, true> : granule_kernel<NS, C, D, 1, true>) \
                : (two ? granule_kernel<NS, C, D, (D) == 3 ? 1 : 2, false> : granule_kernel<NS, C, D, 1, false>);
  MK_PICK(false, 0) MK_PICK(false, 1) MK_PICK(false, 2) MK_PICK(false, 4)
  MK_PICK(true, 0) MK_PICK(true, 1) MK_PICK(true, 2) MK_PICK(true, 3)
#undef MK_PICK
  return nullptr;
}

}  // namespace

hipError_t launch_granules(const GranLaunch& a, hipStream_t s) {
  if (a.nseg <= 0) return hipSuccess;
  if (a.K < 1 || a.K > kMaxTerms || !launchable(a.nseg, 64) || (!a.segs && (a.pieces < 1 || a.nseg != (int64_t)a.nrows * a.pieces)))
    return hipErrorInvalidValue;
  const bool cplx = a.kind == 0;
  const int ns = GranLayout{a.K}.NS();
  const int in = a.adjoint ? (cplx ? 3 : 4) : a.dtype;
  // two runs per lane column halve the scans across lanes in long pieces (ragged scalogram, each launch
  // timed alone: 1000 us against 1090); four leave two waves per SIMD (1005). In the complex adjoint two already do
  // (202 registers, 166 us at 64 x 32768 x 16 scales): one, three waves (142)
  const bool two = a.two != 0;
  const GranFn fn = ns == 1 ? pick<1>(cplx, in, two, a.acc == kAccMixed) : ns == 2 ? pick<2>(cplx, in, two, a.acc == kAccMixed) : pick<3>(cplx, in, two, a.acc == kAccMixed);
  if (!fn) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fn, dim3((unsigned)a.nseg), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace mk
