// Host-side plan object and the host math behind it (fits, order search, tables).
#pragma once
#include <stdint.h>
#include <string>
#include <vector>

#include "granule.h"
#include "layout.h"

namespace mk {
// Pieces of rows for the granule scan: granules per piece of a row of ng granules whose window spans
// nw granules (2L positions), from the load of the whole launch.
struct GranSplit {
  int64_t base = 1;      // granules per piece, at least
  double per_warm = 0;   // and at least this many per granule of the window
  double cost = 0;       // estimated time of the launch, in granule times of a wave on a full device
  double out = 0, window = 0;             // granules of all pieces, with outputs and of the windows before them
  double wave_out = 0, wave_window = 0;   // of the longest wave
  int64_t piece(int64_t nw) const;   // even with two()
  // two granules at a time: halves the scans across lanes, but starts and ends cost more; from pieces of
  // eight granules on (4096^2 image, pieces of four: 98 us with two, 93 with one)
  bool two() const { return base >= 8; }
};
}  // namespace mk

// One scale of a batched plan.
struct ScaleParams {
  double sigma = 0, xi = 0;
  int64_t L = 0;
  int P_S = 0;
  int64_t n0_asft = 0;
  std::vector<double> cc, sc, jac;
  double relrmse = 0;
};

struct morlet_plan_s {
  int kind = 0;           // 0 Morlet, 1 Gaussian family (real output)
  int deriv = 0;          // Gaussian family: 0 smoothing, 1 first differential (sine
                          // components 1..K), 2 second differential (cosine components 0..K-1)
  int64_t N = 0;
  double sigma = 0, xi = 0;
  int K = 0;
  int64_t L = 0;
  int P_S = 0;
  int mode = 0;           // 0 SFT, 1 ASFT
  int64_t n0 = 0;         // ASFT shift (0 for SFT)
  int64_t n0_asft = 0;    // shift used when ASFT is selected
  int accum = 3;          // morlet_accum: 0 float32 tile scan, 1 float64, 2 mixed, 3 by mode
  int boundary = 0;       // single signals: 0 zero extension, 1 edge values (Sec. II)
  std::vector<double> cc, sc;   // cos / sin coefficients (m, l) or (a, 0)
  std::vector<double> jac;      // [4K]: dcc/dsigma, dcc/dxi, dsc/dsigma, dsc/dxi
  double relrmse = 0;
  int R = 16;             // samples per thread
  int row_serial = -1;    // schedule: -1 automatic, 0 tiles with look-back, 1 whole rows, 2 segments
  int seg_tiles = 0;      // segments schedule: tiles per segment (0: about two segments per resident block)
  int device = 0;
  int num_cus = 256;
  void* d_tab = nullptr;  // device copy of the constant table
  size_t tab_bytes = 0;
  std::vector<unsigned char> h_tab;
  // morlet_plan_refit: pinned staging copy of the table for the stream-ordered upload, and the
  // event recorded after that upload (allocated by the first refit, kept until destroy)
  void* h_stage = nullptr;
  size_t stage_bytes = 0;
  void* stage_event = nullptr;            // hipEvent_t
  // batched ragged plans (B signals x S scales); empty for single-signal plans
  bool batched = false;
  int B = 0, S = 0;
  std::vector<int64_t> lengths, offsets;   // per signal (offsets: prefix sums of lengths)
  std::vector<ScaleParams> scales;
  std::vector<mk::Row> rows;               // B*S rows, signal-major
  std::vector<int32_t> tile_row;
  std::vector<int32_t> row_order;          // row-serial schedule: the row queues back to back
  int32_t qstart[mk::kQueues + 1] = {0};   // queue q is row_order[qstart[q] .. qstart[q + 1])
  int64_t max_row_tiles = 0;
  int64_t ntiles = 0, ntiles_max = 0;
  int64_t gran_ng = -1, gran_nw = -1;      // rows of one length: the granules, window granules and split
  mk::GranSplit gran_split;
  bool gran_rows = false;                  // batched plans: whether the split and pieces have been found
  bool equal_rows = false;                 // all rows have one length and one scale (images, the multiplication method)
  bool gran_two = false;                   // granule scan: every piece starts on an even granule
  std::vector<mk::GranSeg> gran_segs;      // granule scan: pieces of the rows in launch order
  void* d_rows = nullptr;                  // device rows, then tile_row, row_order, gran_segs
  size_t rows_bytes = 0;
  // exact taps of the direct-convolution baseline (uploaded on its first call)
  void* d_direct = nullptr;
  int64_t direct_H = -1;
  // Morlet by the multiplication method (Sec. III-B): a batched Gaussian plan over three rows
  // of the signal's length (the demodulated signal's real and imaginary parts, and the signal),
  // the carrier applied around the scan
  bool multiply = false;
  int64_t mult_N = 0;                  // signal length
  double mult_ce = 0, mult_kappa = 0;  // C_xi / (pi^(1/4) sqrt(sigma)) / sqrt(gamma / pi), kappa_xi
  // separable 2-D Gaussian smoothing of an H x W image (Sec. IV: lines filtered independently):
  // axis[0] is a batched Gaussian plan over the H rows (length W), axis[1] one over the W rows
  // of the transposed image (length H); this plan owns both
  bool image2d = false;
  bool gabor = false;   // image plan: Morlet rows (axis 0) then Gaussian columns of both parts
  int64_t img_H = 0, img_W = 0;
  morlet_plan_s* axis[2] = {nullptr, nullptr};
};

namespace mk {

struct Fit {
  std::vector<double> cc, sc;
  double relrmse;
};

// Kernel samples on k = -L..L (index k + L).
void morlet_taps(double sigma, double xi, int64_t L, std::vector<double>& re, std::vector<double>& im);
// G[k] (deriv 0), G_D[k] (1) or G_DD[k] (2) for k = -L..L (Sec. II)
void gauss_taps(double sigma, int64_t L, std::vector<double>& g, int deriv = 0);

// MMSE fit of the given real targets on orders P_S..P_S+K-1 (cos part to `even`,
// sin part to `odd`); relrmse against the combined complex target.
Fit fit_orders(const std::vector<double>& tre, const std::vector<double>& tim, int64_t L, int P_S, int K);

int select_ps(double sigma, double xi, int K, int64_t L, double* best_err);
int64_t select_L(double sigma, double xi, int K, bool gauss);
// kernel relRMSE of the K-term fit on [-L, L] (Morlet: at the best lowest order)
double err_at_L(double sigma, double xi, int K, int64_t L, bool gauss);

void jacobian(morlet_plan_s* p);
// Fill p->h_tab for the plan's current mode and R; returns false on bad parameters.
bool build_table(morlet_plan_s* p, std::string* err);
// Fill one table for arbitrary parameters (used by the scalogram plans as well).
void fill_table(unsigned char* dst, int kind, int K, int R, int64_t L, int P_S, double sigma, double xi,
                int mode, int64_t n0, const std::vector<double>& cc, const std::vector<double>& sc,
                const std::vector<double>& jac);
// Constants of the granule scan for one scale (GranLayout). okind: the launch's kind (0 complex
// output, 1 cosine components, 2 sine components, 3 both).
void fill_granules(unsigned char* dst, int okind, int K, int64_t L, int P_S, double sigma, double xi, int mode,
                   int64_t n0, const std::vector<double>& cc, const std::vector<double>& sc);
// Bytes of one scale's constants: its TabLayout table, then its granule constants.
size_t scale_bytes(int K, int R);
// Output kind of a plan's forward scan.
int out_kind(const morlet_plan_s* p);

struct GranRow {
  int64_t ng, nw, count;   // granules, window granules, rows of this shape
};
// The shapes of the rows of every length at every window (granules), each once.
std::vector<GranRow> gran_shapes(const std::vector<int64_t>& lengths, const std::vector<int64_t>& windows);
// warm: cost of a window granule relative to one with outputs.
GranSplit split_granules(const std::vector<GranRow>& rows, int num_cus, double warm = 0.3);
// Estimated times in us of a launch's three ways. kind: the launch's (0 complex output, else real); wide: float64
// run sums (the mixed scan).
double granule_us(const GranSplit& s, int kind, bool adjoint, bool wide, int K, int num_cus);
double carried_us(double chunks, int kind, bool adjoint, bool wide, int K);   // chunks that a CU runs, in turn or at once
double tiles_us(int64_t ntiles, int kind, bool adjoint, int K, int num_cus);
// The column scan's, in runs of 16 rows on half the device's wave slots, and what the transposed route adds to its
// lines' scan: two transposes of a matrix of `cells` float32 values.
double columns_us(const GranSplit& s, int K, int num_cus);
double transposes_us(double cells);
// The split of `count` rows of N samples with half width L, kept in the plan.
void set_split(morlet_plan_s* p, int64_t N, int64_t L, int64_t count);

}  // namespace mk
