// Host plan math: kernel samples, minimum-squared-error Fourier fits (eq. mmse), the
// lowest-order search of the direct method (Sec. III-A, Sec. V-A), the window choice,
// coefficient Jacobians and the per-scale constant tables of the scan kernels.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>

#include "plan_internal.h"

namespace mk {

namespace {

const double kPi = 3.14159265358979323846;

struct MorletConsts {
  double C, kappa, A;
};

MorletConsts morlet_consts(double sigma, double xi) {
  const double x0 = xi * sigma;  // dimensionless carrier
  MorletConsts c;
  c.C = 1.0 / std::sqrt(1.0 + std::exp(-x0 * x0) - 2.0 * std::exp(-0.75 * x0 * x0));
  c.kappa = std::exp(-0.5 * x0 * x0);
  c.A = c.C / (std::pow(kPi, 0.25) * std::sqrt(sigma));
  return c;
}

// Projections of a target y[k] (k = -L..L, index k + L) on cos(beta p k) and sin(beta p k)
// for p = p_lo..p_hi, with the angle reduced exactly: beta p k = pi ((p k) mod 2L) / L.
// Uses y[k] cos + y[-k] cos = (y[k] + y[-k]) cos (and the odd counterpart for sin).
void project(const std::vector<double>& y, int64_t L, int p_lo, int p_hi, std::vector<double>& bc,
             std::vector<double>& bs) {
  const int n = p_hi - p_lo + 1;
  bc.assign(n, 0.0);
  bs.assign(n, 0.0);
  const int64_t twoL = 2 * L;
  for (int i = 0; i < n; ++i) {
    const int64_t p = p_lo + i;
    double sc = y[L], ss = 0.0;  // k = 0 term
    int64_t m = 0;
    for (int64_t k = 1; k <= L; ++k) {
      m += p;
      if (m >= twoL) m -= twoL * (m / twoL);
      const double ang = kPi * (double)m / (double)L;
      sc += (y[L + k] + y[L - k]) * std::cos(ang);
      ss += (y[L + k] - y[L - k]) * std::sin(ang);
    }
    bc[i] = sc;
    bs[i] = ss;
  }
}

double sumsq(const std::vector<double>& v) {
  double s = 0;
  for (double x : v) s += x * x;
  return s;
}

// Normal equations of the fit. Over k = -L..L the cosines of orders 0..L have Gram matrix
// diag(d) + s s^T with d_p = 2L for p in {0, L} (L otherwise) and s_p = (-1)^p, because the
// end point k = L repeats k = -L of the 2L-periodic grid; the sines of orders 1..L-1 are
// orthogonal with squared norm L and vanish for p in {0, L}.
void solve_cos(const std::vector<double>& b, int64_t L, int P_S, std::vector<double>& c) {
  const int K = (int)b.size();
  std::vector<double> db(K), ds(K);
  double sdb = 0, sds = 0;
  for (int i = 0; i < K; ++i) {
    const int64_t p = P_S + i;
    const double d = (p == 0 || p == L) ? 2.0 * (double)L : (double)L;
    const double s = (p & 1) ? -1.0 : 1.0;
    db[i] = b[i] / d;
    ds[i] = s / d;
    sdb += s * db[i];
    sds += s * ds[i];
  }
  c.resize(K);
  const double f = sdb / (1.0 + sds);
  for (int i = 0; i < K; ++i) c[i] = db[i] - ds[i] * f;
}

void solve_sin(const std::vector<double>& b, int64_t L, int P_S, std::vector<double>& c) {
  const int K = (int)b.size();
  c.assign(K, 0.0);
  for (int i = 0; i < K; ++i) {
    const int64_t p = P_S + i;
    if (p >= 1 && p <= L - 1) c[i] = b[i] / (double)L;
  }
}

double kterm_relrmse(const std::vector<double>& tre, const std::vector<double>& tim, int64_t L, int P_S,
                     const std::vector<double>& cc, const std::vector<double>& sc) {
  const int K = (int)cc.size();
  double num = 0, den = 0;
  for (int64_t k = -L; k <= L; ++k) {
    double fr = 0, fi = 0;
    for (int i = 0; i < K; ++i) {
      const int64_t p = P_S + i;
      int64_t m = (p * k) % (2 * L);
      if (m < 0) m += 2 * L;
      const double ang = kPi * (double)m / (double)L;
      fr += cc[i] * std::cos(ang);
      fi += sc[i] * std::sin(ang);
    }
    const double er = fr - tre[L + k], ei = fi - (tim.empty() ? 0.0 : tim[L + k]);
    num += er * er + ei * ei;
    den += tre[L + k] * tre[L + k] + (tim.empty() ? 0.0 : tim[L + k] * tim[L + k]);
  }
  return std::sqrt(num / den);
}

int ps_hi(double xi, int K, int64_t L) {
  const int64_t carrier = (int64_t)std::ceil(xi * (double)L / kPi);
  const int64_t hi = std::min<int64_t>(L - K + 1, carrier + K);
  return (int)std::max<int64_t>(hi, 0);
}

// Residual^2 of the fit on orders P_S..P_S+K-1 from the projections (index p - p_lo).
double residual2(const std::vector<double>& bc_all, const std::vector<double>& bs_all, int p_lo, int P_S,
                 int K, int64_t L, double yy) {
  std::vector<double> bc(bc_all.begin() + (P_S - p_lo), bc_all.begin() + (P_S - p_lo) + K);
  std::vector<double> bs(bs_all.begin() + (P_S - p_lo), bs_all.begin() + (P_S - p_lo) + K);
  std::vector<double> c, s;
  solve_cos(bc, L, P_S, c);
  solve_sin(bs, L, P_S, s);
  double r = yy;
  for (int i = 0; i < K; ++i) r -= c[i] * bc[i] + s[i] * bs[i];
  return r;
}

}  // namespace

void morlet_taps(double sigma, double xi, int64_t L, std::vector<double>& re, std::vector<double>& im) {
  const MorletConsts mc = morlet_consts(sigma, xi);
  re.resize(2 * L + 1);
  im.resize(2 * L + 1);
  for (int64_t k = -L; k <= L; ++k) {
    const double kk = (double)k;
    const double env = mc.A * std::exp(-kk * kk / (2.0 * sigma * sigma));
    re[L + k] = env * (std::cos(xi * kk) - mc.kappa);
    im[L + k] = env * std::sin(xi * kk);
  }
}

void gauss_taps(double sigma, int64_t L, std::vector<double>& g, int deriv) {
  const double gamma = 1.0 / (2.0 * sigma * sigma);
  const double a = std::sqrt(gamma / kPi);
  g.resize(2 * L + 1);
  for (int64_t k = -L; k <= L; ++k) {
    const double kk = (double)k, G = a * std::exp(-gamma * kk * kk);
    // G, G_D = (-2 gamma k) G, G_DD = (4 gamma^2 k^2 - 2 gamma) G (Sec. II)
    g[L + k] = deriv == 0 ? G : deriv == 1 ? -2.0 * gamma * kk * G : (4.0 * gamma * gamma * kk * kk - 2.0 * gamma) * G;
  }
}

Fit fit_orders(const std::vector<double>& tre, const std::vector<double>& tim, int64_t L, int P_S, int K) {
  std::vector<double> bc, bs, bc2, bs2;
  project(tre, L, P_S, P_S + K - 1, bc, bs2);
  Fit f;
  solve_cos(bc, L, P_S, f.cc);
  if (!tim.empty()) {
    project(tim, L, P_S, P_S + K - 1, bc2, bs);
    solve_sin(bs, L, P_S, f.sc);
  } else {
    f.sc.assign(K, 0.0);
  }
  f.relrmse = kterm_relrmse(tre, tim, L, P_S, f.cc, f.sc);
  return f;
}

int select_ps(double sigma, double xi, int K, int64_t L, double* best_err) {
  std::vector<double> re, im;
  morlet_taps(sigma, xi, L, re, im);
  const int hi = ps_hi(xi, K, L);
  std::vector<double> bc, bs_unused, bc_unused, bs;
  project(re, L, 0, hi + K - 1, bc, bs_unused);
  project(im, L, 0, hi + K - 1, bc_unused, bs);
  const double yy = sumsq(re) + sumsq(im);
  int best = 0;
  double best_r = std::numeric_limits<double>::infinity();
  for (int ps = 0; ps <= hi; ++ps) {
    const double r = std::sqrt(std::max(residual2(bc, bs, 0, ps, K, L, yy), 0.0) / yy);
    if (r < best_r * (1.0 - 1e-12)) {
      best_r = r;
      best = ps;
    }
  }
  if (best_err) *best_err = best_r;
  return best;
}

double err_at_L(double sigma, double xi, int K, int64_t L, bool gauss) {
  if (gauss) {
    std::vector<double> g, none;
    gauss_taps(sigma, L, g);
    std::vector<double> bc, bs;
    project(g, L, 0, K - 1, bc, bs);
    return std::sqrt(std::max(residual2(bc, std::vector<double>(K, 0.0), 0, 0, K, L, sumsq(g)), 0.0) / sumsq(g));
  }
  double e = 0;
  select_ps(sigma, xi, K, L, &e);
  return e;
}

int64_t select_L(double sigma, double xi, int K, bool gauss) {
  // Grid L = round(c sigma), c = 1.50, 1.52, ..., 5.00, searched coarse to fine: every
  // fifth grid point first, then the grid points within 0.10 of the best coarse one.
  auto L_of = [&](int ci) {
    int64_t L = (int64_t)std::llround((1.5 + 0.02 * ci) * sigma);
    return std::max<int64_t>(L, std::max(K, 1));
  };
  int best_ci = 0;
  double best = std::numeric_limits<double>::infinity();
  for (int ci = 0; ci <= 175; ci += 5) {
    const double e = err_at_L(sigma, xi, K, L_of(ci), gauss);
    if (e < best * (1.0 - 1e-12)) {
      best = e;
      best_ci = ci;
    }
  }
  const int c0 = best_ci;
  for (int ci = std::max(0, c0 - 5); ci <= std::min(175, c0 + 5); ++ci) {
    if (ci % 5 == 0) continue;
    const double e = err_at_L(sigma, xi, K, L_of(ci), gauss);
    if (e < best * (1.0 - 1e-12) || (e <= best && ci < best_ci)) {
      best = e;
      best_ci = ci;
    }
  }
  return L_of(best_ci);
}

void jacobian(morlet_plan_s* p) {
  const int K = p->K;
  const int64_t L = p->L;
  p->jac.assign(4 * K, 0.0);
  if (p->deriv != 0) return;   // differential smoothing has no parameter gradients
  std::vector<double> ds_re(2 * L + 1), ds_im(2 * L + 1), dx_re(2 * L + 1), dx_im(2 * L + 1);
  if (p->kind == 0) {
    // d psi / d sigma and d psi / d xi by the product rule on
    //   psi = A(x0) sigma^{-1/2} E (e^{i xi k} - kappa(x0)),  x0 = xi sigma,
    //   A = C(x0) pi^{-1/4}, C = D^{-1/2}, D = 1 + e^{-x0^2} - 2 e^{-3 x0^2/4}, kappa = e^{-x0^2/2}.
    const double sigma = p->sigma, xi = p->xi, x0 = xi * sigma;
    const MorletConsts mc = morlet_consts(sigma, xi);
    const double D = 1.0 + std::exp(-x0 * x0) - 2.0 * std::exp(-0.75 * x0 * x0);
    const double dD = -2.0 * x0 * std::exp(-x0 * x0) + 3.0 * x0 * std::exp(-0.75 * x0 * x0);
    const double dA = (-0.5 * std::pow(D, -1.5) * dD) / std::pow(kPi, 0.25);  // dA/dx0
    const double A = mc.C / std::pow(kPi, 0.25);
    const double dkappa = -x0 * mc.kappa;  // dkappa/dx0
    const double s = 1.0 / std::sqrt(sigma), dsig_s = -0.5 * std::pow(sigma, -1.5);
    for (int64_t k = -L; k <= L; ++k) {
      const double kk = (double)k;
      const double E = std::exp(-kk * kk / (2.0 * sigma * sigma));
      const double dE = E * kk * kk / (sigma * sigma * sigma);
      const double cr = std::cos(xi * kk) - mc.kappa, ci = std::sin(xi * kk);
      // sigma: A and kappa move through x0 (dx0/dsigma = xi), plus sigma^{-1/2} and E
      const double gs = dA * xi * s * E + A * dsig_s * E + A * s * dE;
      ds_re[L + k] = gs * cr + A * s * E * (-dkappa * xi);
      ds_im[L + k] = gs * ci;
      // xi: A and kappa move through x0 (dx0/dxi = sigma); the carrier gives i k e^{i xi k}
      const double gx = dA * sigma * s * E;
      dx_re[L + k] = gx * cr + A * s * E * (-kk * std::sin(xi * kk) - dkappa * sigma);
      dx_im[L + k] = gx * ci + A * s * E * (kk * std::cos(xi * kk));
    }
  } else {
    // Gaussian: dG/dsigma = G (k^2/sigma^3 - 1/sigma); no xi
    std::vector<double> g;
    gauss_taps(p->sigma, L, g);
    for (int64_t k = -L; k <= L; ++k) {
      const double kk = (double)k;
      ds_re[L + k] = g[L + k] * (kk * kk / (p->sigma * p->sigma * p->sigma) - 1.0 / p->sigma);
      ds_im[L + k] = 0.0;
      dx_re[L + k] = 0.0;
      dx_im[L + k] = 0.0;
    }
  }
  const int P_S = p->P_S;
  std::vector<double> bc, bs, c;
  const std::vector<double>* srcs[4] = {&ds_re, &dx_re, &ds_im, &dx_im};
  for (int t = 0; t < 4; ++t) {
    project(*srcs[t], L, P_S, P_S + K - 1, bc, bs);
    if (t < 2) solve_cos(bc, L, P_S, c);
    else if (p->kind == 0) solve_sin(bs, L, P_S, c);
    else c.assign(K, 0.0);
    for (int i = 0; i < K; ++i) p->jac[t * K + i] = c[i];
  }
}

namespace {
// a_p^m = e^{-alpha m} e^{-i beta p m}, angle reduced exactly
inline void apow(int64_t p, int64_t m, int64_t L, double alpha, double& re, double& im) {
  int64_t r = (p % (2 * L)) * (m % (2 * L)) % (2 * L);
  const double ang = -kPi * (double)r / (double)L;
  const double mag = std::exp(-alpha * (double)m);
  re = mag * std::cos(ang);
  im = mag * std::sin(ang);
}
}  // namespace

void fill_table(unsigned char* dst, int kind, int K, int R, int64_t L, int P_S, double sigma, double xi,
                int mode, int64_t n0, const std::vector<double>& cc, const std::vector<double>& sc,
                const std::vector<double>& jac) {
  TabLayout lay{K, R};
  std::memset(dst, 0, lay.bytes());
  float* tf = (float*)dst;
  double* td = (double*)(dst + lay.f32Bytes());
  const double alpha = (mode == 1) ? (double)n0 / (sigma * sigma) : 0.0;
  const int64_t T = (int64_t)R * kThreads;
  const int mo = lay.nComplex();
  // entry e gets a^d, entry mo + e gets d a^d
  auto put = [&](int e, int i, int64_t p, int64_t d) {
    double re, im;
    apow(p, d, L, alpha, re, im);
    const double dd = (double)d;
    tf[(2 * e) * K + i] = (float)re;
    tf[(2 * e + 1) * K + i] = (float)im;
    td[(2 * e) * K + i] = re;
    td[(2 * e + 1) * K + i] = im;
    tf[(2 * (mo + e)) * K + i] = (float)(dd * re);
    tf[(2 * (mo + e) + 1) * K + i] = (float)(dd * im);
    td[(2 * (mo + e)) * K + i] = dd * re;
    td[(2 * (mo + e) + 1) * K + i] = dd * im;
  };
  auto putrow = [&](int row, int i, double v) {
    tf[row * K + i] = (float)v;
    td[row * K + i] = v;
  };
  double cx = 0;
  for (int i = 0; i < K; ++i) {
    const int64_t p = P_S + i;
    put(lay.eA(), i, p, 1);
    for (int r = 0; r < R; ++r) put(lay.eP1(r), i, p, R - 1 - r);
    for (int d = 0; d < 6; ++d) put(lay.eTR(d), i, p, (int64_t)R << d);
    for (int l = 0; l < 64; ++l) put(lay.eLANE(l), i, p, (int64_t)R * l);
    for (int w = 0; w <= kWaves; ++w) put(lay.eWV(w), i, p, (int64_t)64 * R * w);
    for (int k = 0; k <= 64; ++k) put(lay.eLB(k), i, p, T * k);
    for (int k = 0; k <= 64; ++k) put(lay.eLB2(k), i, p, 64 * T * k);
    const double sgn = (p & 1) ? -1.0 : 1.0;
    const double up = std::exp(alpha * (double)L), dn = std::exp(-alpha * (double)L);
    putrow(lay.rMW(), i, sgn * cc[i] * up);
    putrow(lay.rLW(), i, sgn * sc[i] * up);
    putrow(lay.rSGN(), i, sgn);
    putrow(lay.rCC(), i, cc[i]);
    putrow(lay.rSC(), i, sc[i]);
    for (int q = 0; q < 4; ++q) putrow(lay.rJ(q), i, jac.size() == (size_t)4 * K ? jac[q * K + i] : 0.0);
    for (int k = 1; k <= 4; ++k) {
      double re, im;
      apow(p, k, L, alpha, re, im);
      const int v = lay.vHC(i) + 2 * (k - 1);
      tf[v] = (float)re;
      tf[v + 1] = (float)im;
      td[v] = re;
      td[v + 1] = im;
    }
    cx += sgn * cc[i] * dn;
  }
  const double D = std::exp(-2.0 * alpha * (double)L);
  double gre = 1.0, gim = 0.0, dsig = 0.0, dxi = 0.0, dalpha = 0.0;
  if (mode == 1) {
    const double s = std::exp(-(double)n0 * (double)n0 / (2.0 * sigma * sigma));
    if (kind == 0) {
      gre = s * std::cos(xi * (double)n0);
      gim = s * std::sin(xi * (double)n0);
      dxi = (double)n0;
    } else {
      gre = s;
    }
    dsig = (double)n0 * (double)n0 / (sigma * sigma * sigma);
    dalpha = -2.0 * (double)n0 / (sigma * sigma * sigma);
  }
  const double sv[10] = {cx, D, gre, gim, std::exp(alpha * (double)L), std::exp(-alpha * (double)L), (double)L,
                         dsig, dxi, dalpha};
  const int so[10] = {lay.sCX(), lay.sD(), lay.sGre(), lay.sGim(), lay.sUP(), lay.sDN(), lay.sLL(), lay.sDSIG(),
                      lay.sDXI(), lay.sDALPHA()};
  for (int q = 0; q < 10; ++q) {
    tf[so[q]] = (float)sv[q];
    td[so[q]] = sv[q];
  }
  // float32 remainders of every entry, for float-float arithmetic
  float* tl = (float*)(dst + lay.f32Bytes() + lay.f64Bytes());
  for (int v = 0; v < lay.nValues(); ++v) tl[v] = (float)(td[v] - (double)tf[v]);
}

size_t scale_bytes(int K, int R) { return TabLayout{K, R}.bytes() + GranLayout{K}.bytes(); }

int out_kind(const morlet_plan_s* p) {
  // differentials: 2 real output from the sines (SFT, first), 1 from the cosines (SFT, second),
  // 3 from both (ASFT)
  return p->deriv == 0 ? p->kind : p->mode == 1 ? 3 : p->deriv == 1 ? 2 : 1;
}

void fill_granules(unsigned char* dst, int okind, int K, int64_t L, int P_S, double sigma, double xi, int mode,
                   int64_t n0, const std::vector<double>& cc, const std::vector<double>& sc) {
  const GranLayout lay{K};
  std::memset(dst, 0, lay.bytes());
  float* tf = (float*)dst;
  double* td = (double*)(tf + lay.nFloats());
  const double alpha = (mode == 1) ? (double)n0 / (sigma * sigma) : 0.0;
  const double up = std::exp(alpha * (double)L), dn = std::exp(-alpha * (double)L);
  const double s = mode == 1 ? std::exp(-(double)n0 * (double)n0 / (2.0 * sigma * sigma)) : 1.0;
  const double gre = mode == 1 && okind == 0 ? s * std::cos(xi * (double)n0) : s;
  const double gim = mode == 1 && okind == 0 ? s * std::sin(xi * (double)n0) : 0.0;
  // Run sums, and so all states, are held at half their size, and their output weights at twice it: a state that
  // is finite in float32 is then below the values whose nearest bfloat16 is infinite.
  const double kHeld = 0.5;
  // output: (gre + i gim)(A - iB) for the wavelet, gre (A - B) for real output, with
  // A = cx y + sum_t mw_t Re v_t, B = sum_t lw_t Im v_t; weights of Re v, Im v per component
  double T[2][kRun] = {}, cx = 0;
  float ca[8][64] = {};   // outputs of the complex adjoint from its state: component 2 slot + part
  float tim[4][64] = {}, cim[8][64] = {};   // the imaginary component's fTre, fCre
  for (int i = 0; i < K; ++i) {
    const int64_t p = P_S + i;
    const int slot = i / 4, q = i % 4;
    const double sgn = (p & 1) ? -1.0 : 1.0;
    const double mw = okind == 2 ? 0.0 : sgn * cc[i] * up, lw = okind == 1 ? 0.0 : sgn * sc[i] * up;
    const double wr[2] = {gre * mw, gim * mw};
    const double wi[2] = {okind == 0 ? gim * lw : -gre * lw, okind == 0 ? -gre * lw : 0.0};
    if (okind != 2) cx += sgn * cc[i] * dn;
    double re, im, pr[kRun + 1], pi[kRun + 1];   // a^d
    for (int d = 0; d <= kRun; ++d) apow(p, d, L, alpha, pr[d], pi[d]);
    for (int d = 0; d < kRun; ++d) {
      re = pr[d];
      im = pi[d];
      for (int c = 0; c < 2; ++c) T[c][d] += wr[c] * re + wi[c] * im;
      // run sums: input r = 15 - d; lane 16 (r / 4) + row, block kb = r % 4
      const int r = kRun - 1 - d, b = slot / 2, lq = 16 * (r / 4), kb = r % 4;
      const int v = 2 * (slot % 2);   // result registers v, v + 1 of lane row q: rows q + 4 v, q + 4 (v + 1)
      td[lay.dP(b, kb) + lq + q + 4 * v] = kHeld * re;
      td[lay.dP(b, kb) + lq + q + 4 * (v + 1)] = kHeld * im;
      for (int c = 0; c < 2; ++c) {
        td[lay.dPA(c, b, kb) + lq + q + 4 * v] = kHeld * (wr[c] * re + wi[c] * im);
        td[lay.dPA(c, b, kb) + lq + q + 4 * (v + 1)] = kHeld * (wr[c] * im - wi[c] * re);
      }
      // outputs at position d from the state before the run
      re = pr[d + 1] / kHeld;
      im = pi[d + 1] / kHeld;
      ca[2 * slot][16 * q + d] = (float)re;
      ca[2 * slot + 1][16 * q + d] = (float)-im;
      tf[lay.fCre(2 * slot) + 16 * q + d] = (float)(wr[0] * re + wi[0] * im);
      tf[lay.fCre(2 * slot + 1) + 16 * q + d] = (float)(-wr[0] * im + wi[0] * re);
      cim[2 * slot][16 * q + d] = (float)(wr[1] * re + wi[1] * im);
      cim[2 * slot + 1][16 * q + d] = (float)(-wr[1] * im + wi[1] * re);
      apow(p, (int64_t)kRun * d, L, alpha, re, im);
      td[lay.dLANE(slot, 0) + 16 * q + d] = re;
      td[lay.dLANE(slot, 1) + 16 * q + d] = im;
    }
    for (int d = 0; d < 5; ++d) {
      apow(p, (int64_t)kRun << d, L, alpha, re, im);
      td[lay.dSC(d, slot, 0) + q] = re;
      td[lay.dSC(d, slot, 1) + q] = im;
    }
    for (int k = 0; k <= 8; ++k) {
      apow(p, (int64_t)kGran * k, L, alpha, re, im);
      td[lay.dG(k, slot, 0) + q] = re;
      td[lay.dG(k, slot, 1) + q] = im;
    }
  }
  for (int r = 0; r < kRun; ++r)
    for (int rp = 0; rp <= r; ++rp) {
      tf[lay.fTre(rp % 4) + 16 * (rp / 4) + r] = (float)T[0][r - rp];
      tim[rp % 4][16 * (rp / 4) + r] = (float)T[1][r - rp];
    }
  // thirds: the nearest bfloat16 of the value, of what is left, and the rest
  auto thirds = [](float v, uint16_t* h, uint16_t* m, uint16_t* l) {
    auto near = [](float x) {   // round to nearest even
      uint32_t u;
      std::memcpy(&u, &x, 4);
      return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1)) >> 16);
    };
    auto value = [](uint16_t b) {
      const uint32_t u = (uint32_t)b << 16;
      float x;
      std::memcpy(&x, &u, 4);
      return x;
    };
    *h = near(v);
    const float r = v - value(*h);
    *m = near(r);
    *l = near(r - value(*m));
  };
  uint16_t* bq = reinterpret_cast<uint16_t*>(dst + lay.quadOff());
  for (int b = 0; b < lay.MB(); ++b)
    for (int lane = 0; lane < 64; ++lane)
      for (int e = 0; e < 4; ++e) {
        const int u = lane / 4 % 4, v = lane % 4;   // the float64 table has row u + 4 v
        thirds((float)td[lay.dP(b, e) + 16 * (lane / 16) + u + 4 * v], bq + 4 * (lay.bP(b, 0) + lane) + e,
               bq + 4 * (lay.bP(b, 1) + lane) + e, bq + 4 * (lay.bP(b, 2) + lane) + e);
        for (int c = 0; c < 2; ++c)
          thirds((float)td[lay.dPA(c, b, e) + 16 * (lane / 16) + u + 4 * v], bq + 4 * (lay.bPA(c, b, 0) + lane) + e,
                 bq + 4 * (lay.bPA(c, b, 1) + lane) + e, bq + 4 * (lay.bPA(c, b, 2) + lane) + e);
      }
  for (int set = 0; set < lay.SETS(); ++set)
    for (int lane = 0; lane < 64; ++lane)
      for (int e = 0; e < 4; ++e)
        thirds(ca[4 * set + e][lane], bq + 4 * (lay.bCA(set, 0) + lane) + e, bq + 4 * (lay.bCA(set, 1) + lane) + e,
               bq + 4 * (lay.bCA(set, 2) + lane) + e);
  for (int c = 0; c < 2; ++c)
    for (int lane = 0; lane < 64; ++lane)
      for (int e = 0; e < 4; ++e) {
        thirds(c ? tim[e][lane] : tf[lay.fTre(e) + lane], bq + 4 * (lay.bT(c, 0) + lane) + e,
               bq + 4 * (lay.bT(c, 1) + lane) + e, bq + 4 * (lay.bT(c, 2) + lane) + e);
        for (int set = 0; set < lay.SETS(); ++set)
          if (4 * set + e < 2 * lay.NS())
            thirds(c ? cim[4 * set + e][lane] : tf[lay.fCre(4 * set + e) + lane], bq + 4 * (lay.bC(c, set, 0) + lane) + e,
                   bq + 4 * (lay.bC(c, set, 1) + lane) + e, bq + 4 * (lay.bC(c, set, 2) + lane) + e);
      }
  tf[lay.fYre()] = (float)(gre * cx);
  tf[lay.fYim()] = (float)(gim * cx);
  td[lay.dD()] = std::exp(-2.0 * alpha * (double)L);
}

int64_t GranSplit::piece(int64_t nw) const {
  const int64_t n = (int64_t)std::ceil(per_warm * (double)nw);
  const int64_t p = std::min<int64_t>(std::max(base, n), (int64_t)1 << 30);
  return two() ? (p + 1) / 2 * 2 : p;
}

std::vector<GranRow> gran_shapes(const std::vector<int64_t>& lengths, const std::vector<int64_t>& windows) {
  // the split is evaluated over these for every candidate: 20 000 signals at 32 scales are 640 000 rows of a few
  // dozen shapes (plan of 20 000 signals at 32 scales: 341 ms over the rows, 124 over the shapes)
  std::vector<int64_t> ng;
  for (int64_t n : lengths)
    if (n > 0) ng.push_back(granules_for(n));
  std::sort(ng.begin(), ng.end());
  std::vector<int64_t> nw = windows;
  std::sort(nw.begin(), nw.end());
  std::vector<GranRow> shapes;
  for (size_t w = 0; w < nw.size();) {
    size_t w1 = w;
    while (w1 < nw.size() && nw[w1] == nw[w]) ++w1;
    for (size_t g = 0; g < ng.size();) {
      size_t g1 = g;
      while (g1 < ng.size() && ng[g1] == ng[g]) ++g1;
      shapes.push_back({ng[g], nw[w], (int64_t)((g1 - g) * (w1 - w))});
      g = g1;
    }
    w = w1;
  }
  return shapes;
}

GranSplit split_granules(const std::vector<GranRow>& rows, int num_cus, double kWarm) {
  // A granule of the window costs kWarm of one with outputs. Four waves per SIMD share it; a wave
  // alone runs a granule in about 0.4 of the time. Longer pieces sum fewer windows, shorter ones fill
  // the device and end together.
  const double kAlone = 0.4, slots = 16.0 * num_cus;
  GranSplit best;
  best.cost = -1;
  for (double pw : {0.0, 0.5, 2.0})
    for (int64_t base = 1; base <= 1024; base *= 2) {
      GranSplit t;
      t.base = base;
      t.per_warm = pw;
      double work = 0, longest = 0;
      for (const GranRow& r : rows) {
        const int64_t n = t.piece(r.nw), ns = (r.ng + n - 1) / n;
        // windows before the first piece's end reach the row's start
        const int64_t part = std::min<int64_t>(ns, r.nw / n + 1);   // pieces whose window is cut short
        const double o = (double)std::min(n, r.ng), w = ns > part ? (double)r.nw : (double)n * (double)(part - 1);
        work += (double)r.count * ((double)r.ng + kWarm * ((double)n * 0.5 * (double)(part - 1) * (double)part + (double)r.nw * (double)(ns - part)));
        longest = std::max(longest, o + kWarm * w);
        // as the kernel sums them: the first output lies half a window past the row's start
        const double half = 0.5 * (double)r.nw;
        const int64_t cut = std::min<int64_t>(ns, (int64_t)(half / (double)n) + 1);
        const double wave = ns > cut ? (double)r.nw : std::min((double)r.nw, half + (double)n * (double)(cut - 1));
        t.out += (double)r.count * (double)r.ng;
        t.window += (double)r.count * (half * (double)cut + (double)n * 0.5 * (double)(cut - 1) * (double)cut + (double)r.nw * (double)(ns - cut));
        if (o + kWarm * wave > t.wave_out + kWarm * t.wave_window) {
          t.wave_out = o;
          t.wave_window = wave;
        }
      }
      t.cost = std::max(work / slots, kAlone * longest) + 0.25 * longest;
      if (best.cost < 0 || t.cost < best.cost) best = t;
    }
  return best;
}

// The three ways' measured times, fitted over 4400 calls in both directions (1 to 1000 rows of 300 to 2^25
// samples, 1 to 16 scales, K 4 to 12, windows of 60 samples to a whole row), to 10-20 %. A wave's own chain
// bounds the granule scan in short launches, the issue of all waves in long ones; where windows are long against the
// pieces both are mostly windows (one signal of 2^20, 2 scales, 2L up to 2^18, K = 5: 915 us, the tile scan 40).
// Chosen by the least estimate, 6 calls in 1000 take more than 1.05 times the tile scan's time, none 1.6.
double granule_us(const GranSplit& s, int kind, bool adjoint, bool wide, int K, int num_cus) {
  struct Us { double base, out, window, all_out, all_window; };   // a wave's granule, a granule of four waves per SIMD
  static const Us us[3][2][3] = {   // real, complex forward, complex adjoint; float64 run sums; slots of states
      {{{4, 0.8, 0.23, 1.8, 0.58}, {4.1, 0.67, 0.24, 2, 0.62}, {4.8, 0.15, 0.27, 2.8, 0.71}},
       {{3.9, 0.74, 0.28, 2, 0.61}, {4.2, 0.59, 0.29, 2.3, 0.7}, {4.9, 0.22, 0.4, 3.6, 1.1}}},
      {{{3.7, 0.72, 0.22, 2.2, 0.65}, {4.3, 0.29, 0.23, 2.6, 0.73}, {4.8, 0.02, 0.26, 3.7, 0.94}},
       {{4, 0.32, 0.28, 2.4, 0.93}, {4.4, 0.02, 0.29, 2.8, 1}, {4.7, 0.02, 0.4, 4.3, 1.7}}},
      {{{5.3, 0.87, 0.32, 2.9, 1.1}, {5.6, 0.72, 0.34, 3.2, 1.3}, {6.2, 0.02, 0.4, 4.8, 1.7}},
       {{5.4, 0.61, 0.47, 3.3, 1.8}, {5.6, 0.42, 0.48, 3.6, 2}, {5.9, 0.02, 0.7, 6.1, 3.2}}}};
  const Us& u = us[kind != 0 ? 0 : adjoint ? 2 : 1][wide][(K - 1) / 4];
  const double slots = 16.0 * num_cus;
  return u.base + std::hypot(u.out * s.wave_out + u.window * s.wave_window, (u.all_out * s.out + u.all_window * s.window) / slots);
}

double carried_us(double chunks, int kind, bool adjoint, bool wide, int K) {
  struct Us { double base, chunk; };
  static const Us us[3][2][3] = {
      {{{7.3, 1.7}, {7.5, 2.2}, {9, 2.8}},
       {{7, 2}, {7.5, 2.4}, {9.2, 3.3}}},
      {{{7.2, 1.5}, {7.9, 2.1}, {9.9, 2.5}},
       {{7.1, 1.8}, {8, 2.3}, {10, 3}}},
      {{{7.6, 2.4}, {8.5, 3.3}, {11, 4.3}},
       {{7.6, 3}, {8.2, 4.2}, {11, 5.4}}}};
  const Us& u = us[kind != 0 ? 0 : adjoint ? 2 : 1][wide][(K - 1) / 4];
  return u.base + u.chunk * chunks;
}

double tiles_us(int64_t ntiles, int kind, bool adjoint, int K, int num_cus) {
  struct Us { double base, base_k, tile, tile_k; };   // per term; per tile of 4096 positions on 256 CUs
  static const Us us[3] = {{12, 0.72, 0.013, 0.0031}, {13, 0.55, 0.015, 0.002}, {12, 1.6, -0.00056, 0.0084}};
  const Us& u = us[kind != 0 ? 0 : adjoint ? 2 : 1];
  return u.base + u.base_k * K + (u.tile + u.tile_k * K) * (double)ntiles * 256.0 / num_cus;
}

// Fitted over 900 images and their adjoints (64 x 64 to 4096 x 4096, 8 to 4096 columns, windows of 1/64 to 2 columns'
// lengths, K = 4, 8, 12), to 20 %: the least of columns and transposed lines is then chosen but for 5 in 100.
double columns_us(const GranSplit& s, int K, int num_cus) {
  struct Us { double base, out, window, all_out, all_window; };   // a wave's run, a run of two waves per SIMD
  static const Us us[3] = {{3.6, 1.2, 0.8, 3.8, 0.72}, {3.1, 2.2, 0.81, 2.8, 0.71}, {5.6, 0.01, 1, 6.8, 1.6}};
  const Us& u = us[(K - 1) / 4];
  const double slots = 8.0 * num_cus;
  return u.base + std::hypot(u.out * s.wave_out + u.window * s.wave_window, (u.all_out * s.out + u.all_window * s.window) / slots);
}

double transposes_us(double cells) { return 19 + 4.6e-6 * cells; }

void set_split(morlet_plan_s* p, int64_t N, int64_t L, int64_t count) {
  p->gran_ng = granules_for(N);
  p->gran_nw = (2 * L + kGran - 1) / kGran;
  p->gran_split = split_granules({{p->gran_ng, p->gran_nw, count}}, p->num_cus);
}

bool build_table(morlet_plan_s* p, std::string* err) {
  if (p->gran_ng < 0) set_split(p, p->N, p->L, 1);
  p->h_tab.assign(scale_bytes(p->K, p->R), 0);
  fill_granules(p->h_tab.data() + TabLayout{p->K, p->R}.bytes(), out_kind(p), p->K, p->L, p->P_S, p->sigma, p->xi,
                p->mode, p->n0, p->cc, p->sc);
  fill_table(p->h_tab.data(), p->kind, p->K, p->R, p->L, p->P_S, p->sigma, p->xi, p->mode, p->n0, p->cc, p->sc,
             p->jac);
  (void)err;
  return true;
}

}  // namespace mk
