// Granule scan (granule_scan.hip): the constants it reads, the pieces of rows it runs and its launch.
#pragma once
#include <hip/hip_runtime.h>

#include "layout.h"

namespace mk {

constexpr int kRun = 16;                 // positions per run
constexpr int kGran = 16 * kRun;         // positions per granule (16 runs)

// Constants of one scale, behind its TabLayout table: powers of a_p laid out for the matrix cores,
// one value per lane. Lane l = 16 q + c of a wave owns run c of a granule and the states q, q + 4,
// q + 8 (slot s holds state 4 s + q; slots past the last term are zero). Float32 part first, then
// float64.
struct GranLayout {
  int K;
  MK_HD int NS() const { return (K + 3) / 4; }            // state slots per lane
  MK_HD int MB() const { return K > 8 ? 2 : 1; }          // matrix blocks of the run sums
  // float32, 64 lanes each: run outputs from run inputs, T[4 q + kb -> r] (lane 16 q + r), of the real component;
  // run outputs from the state before the run, component k = 2 s + (0 re, 1 im)
  MK_HD int fTre(int kb) const { return 64 * kb; }
  MK_HD int fCre(int k) const { return 64 * (4 + k); }
  // scalars: weight of y[j - 2L] in the output (real, imaginary component)
  MK_HD int fYre() const { return 64 * (4 + 2 * NS()); }
  MK_HD int fYim() const { return fYre() + 1; }
  MK_HD int nFloats() const { return (fYre() + 4 + 31) / 32 * 32; }
  // float64: run sums B / 2, B = sum_r a^{15 - r} dy[r] (states are held at half their size, the weights fC*,
  // bC and bCA are for such states), lane 16 q + m holding the weight of input 4 q + kb for
  // row m of the product; a^{16 c} per lane (64); a^{16 2^d}, d < 5, one value per q; a^{256 k},
  // k in [0, 8]; e^{-2 alpha L}. Parts of slot s: 0 real, 1 imaginary
  MK_HD int dP(int mb, int kb) const { return 64 * (4 * mb + kb); }
  MK_HD int dLANE(int s, int part) const { return 64 * (4 * MB() + 2 * s + part); }
  MK_HD int dSC(int d, int s, int part) const { return 64 * (4 * MB() + 2 * NS()) + 4 * ((d * NS() + s) * 2 + part); }
  MK_HD int dG(int k, int s, int part) const { return dSC(5, 0, 0) + 4 * ((k * NS() + s) * 2 + part); }
  MK_HD int dD() const { return dG(9, 0, 0); }
  // run sums of the complex adjoint, from stream c (real, imaginary part of the cotangent): dP times the
  // term's output weight of component c
  MK_HD int dPA(int c, int mb, int kb) const { return (dD() + 64) / 64 * 64 + 64 * (4 * (c * MB() + mb) + kb); }
  MK_HD int nDoubles() const { return dPA(2, 0, 0); }
  // bfloat16 thirds of the float32 weights (value = high + middle + low, exactly), four per lane:
  // T[4 q + e -> r] of component c, and the weights of state components 4 set + e (0 past the last)
  MK_HD int SETS() const { return NS() > 2 ? 2 : 1; }
  MK_HD int bT(int c, int third) const { return 64 * (3 * c + third); }
  MK_HD int bC(int c, int set, int third) const { return 64 * (6 + 3 * (c * SETS() + set) + third); }
  // run sums: lane 16 q + 4 u + v holds the weights of inputs 4 q + e for component v of the states u, u + 4
  // (block 0: real and imaginary parts of slots 0, 1) or u + 8 (block 1)
  MK_HD int bP(int mb, int third) const { return 64 * (6 + 6 * SETS() + 3 * mb + third); }
  // the same for the complex adjoint (dPA), and its output from the state before the run, Re a^{r + 1} V
  MK_HD int bPA(int c, int mb, int third) const { return 64 * (6 + 6 * SETS() + 3 * (MB() + c * MB() + mb) + third); }
  MK_HD int bCA(int set, int third) const { return 64 * (6 + 6 * SETS() + 9 * MB() + 3 * set + third); }
  MK_HD int nQuads() const { return bCA(SETS(), 0); }
  MK_HD size_t quadOff() const { return (size_t)nFloats() * 4 + (size_t)nDoubles() * 8; }
  MK_HD size_t bytes() const { return quadOff() + (size_t)nQuads() * 8; }
};

// A piece of a row for one wave: granules [g0, g0 + n) of the row. Granule g holds the outputs
// [256 g - m, 256 g - m + 256), m the outputs by which the row starts past a 128-byte line.
struct GranSeg {
  int32_t row;
  int32_t n;
  int64_t g0;
};

// Granules that cover a row of N outputs at any alignment.
inline int64_t granules_for(int64_t N) { return N <= 0 ? 0 : (N + 31 + kGran - 1) / kGran; }

// A launch holds fewer than 2^32 threads along its first dimension.
inline bool launchable(int64_t blocks, int threads) { return blocks <= (int64_t)0xffffffff / threads; }

struct GranLaunch {
  int K, acc, kind, dtype;      // acc: kAccF32 or kAccMixed; kind: 0 complex transform, else real
  int adjoint;                  // x is the cotangent, out the float32 gradient
  const void* x;
  void* out;
  // pieces, one wave each: the device list segs, or (segs null, rows of one length) piece k of row
  // r at index r pieces + k, seg_n granules long
  const GranSeg* segs;
  int64_t nseg;
  int32_t pieces, seg_n;
  int two;                      // two granules at a time
  Row row0;                     // the only row when nrows == 1
  const Row* rows;              // device rows
  int nrows;
  const unsigned char* tabs;    // granule constants of scale 0
  int64_t tab_stride;
  double* sums;                 // carried scan: [nrows][pieces - 1][streams][K] complex float64
};
hipError_t launch_granules(const GranLaunch& a, hipStream_t s);

// Carried scan (carry_scan.hip): rows of one length in `pieces` pieces of seg_n chunks, a block each; the
// states pass from piece to piece through sums. A row's first piece starts at a position in (-kChunk, 0], its
// outputs on 128-byte lines (within 31 of jout0 where that is negative); together they reach its last output.
constexpr int kCarryWaves = 8;
constexpr int64_t kChunk = kCarryWaves * kGran;
inline int64_t chunks_for(int64_t N, int64_t jout0) {   // chunks of a row of N outputs at any alignment
  return (jout0 > 0 ? (jout0 + kChunk - 1) / kChunk : 0) + (N + 31 + kChunk - 1) / kChunk;
}
hipError_t launch_carried(const GranLaunch& a, hipStream_t s);

// Column scan (column_scan.hip): a real filter along the columns of a rows x cols float32 matrix.
constexpr int kColWave = 32;    // columns per wave
struct ColumnLaunch {
  int K, adjoint;
  const float* x;
  float* out;                   // not x
  int64_t rows, cols, L, jout0;
  int64_t piece;                // output rows per wave
  const unsigned char* tabs;    // granule constants
};
hipError_t launch_columns(const ColumnLaunch& a, hipStream_t s);

}  // namespace mk
