// Matrix exponential e^{tX} of a dense n x n operator by scaling and squaring
// with a diagonal Pade approximant (N. J. Higham, "The scaling and squaring
// method for the matrix exponential revisited", SIAM J. Matrix Anal. Appl.
// 26(4), 2005, Algorithm 2.3).  This replaces the Leja-interpolation action
// the paper uses (Sec. 3): the operator is formed once per step size and then
// applied to the low-rank factor with GEMMs.
//
//   1. ||tX||_1 (column sums on the device)  ->  degree m, scaling s
//   2. Y = tX / 2^s; even powers Y^2, Y^4, Y^6 (FP64 MFMA GEMMs)
//   3. U (odd part), V (even part) of the [m/m] numerator; denominator V - U
//   4. (V - U) F = V + U by LU with row exchanges (lu.hip)
//   5. F <- F^2, s times
//
// An exactly symmetric tX (checked entry by entry, in the pass that takes its
// norm to the host) makes every matrix above a polynomial or a rational
// function of it, so symmetric: its products then take half the work
// (gemm_sym_f64), and step 4 is F = (V - U)^-1 (V + U) with the inverse of the
// positive definite denominator (spd.hip).  Measured at n = 4096 with four
// squarings: 16.9 ms against 36.2 for the general path.  A caller that depends
// on the last bit of E (kept; see Solver::kept) takes full products and the LU
// in its kept form instead.
#include "common.h"

#include <cmath>
#include <vector>

namespace dme {

namespace {

// theta_m of Higham (2005), Table 2.3 (double precision): the largest
// ||X||_1 for which the [m/m] approximant meets the unit-roundoff backward
// error bound.
constexpr int kDegrees[5] = {3, 5, 7, 9, 13};
constexpr double kTheta[5] = {1.495585217958292e-2, 2.539398330063230e-1, 9.504178996162932e-1,
                              2.097847961257068e0, 5.371920351148152e0};

// Numerator coefficients b_j = (2m - j)! m! / ((2m)! j! (m - j)!), from the
// ratio b_{j+1} / b_j = (m - j) / ((j + 1)(2m - j)), evaluated in long double.
void pade_coeffs(int m, double* b) {
  long double c = 1.0L;
  b[0] = 1.0;
  for (int j = 0; j < m; ++j) {
    c = c * (long double)(m - j) / ((long double)(j + 1) * (long double)(2 * m - j));
    b[j + 1] = (double)c;
  }
}

}  // namespace

void expm_params(double nrm1, int* m, int* s) {
  for (int i = 0; i < 4; ++i) {
    if (nrm1 <= kTheta[i]) { *m = kDegrees[i]; *s = 0; return; }
  }
  *m = 13;
  *s = (nrm1 > 0.0) ? std::max(0, (int)std::ceil(std::log2(nrm1 / kTheta[4]))) : 0;
}

// Leading dimension of the temporaries: even, so that the products can load
// their operands 16 bytes a lane also where n is odd (n = 2025: 1.4 times as
// fast).  The padding row is carried along and never read.
int64_t expm_ld(int64_t n) { return n + (n & 1); }

size_t expm_workspace(int64_t n, int64_t count) {
  const size_t nn = (size_t)expm_ld(n) * n * sizeof(double) + 256;
  return (5 + 2 * (size_t)count) * nn + (size_t)(n + 2 * count) * sizeof(double) + 768 +
         std::max(lu_solve_workspace(n, n, count), spd_inverse_workspace(n)) +
         std::max(gemm_f64_workspace(n, n, n), gemm_sym_workspace(n, n)) + 4096;
}

// The LU of a denominator is a chain of small launches up to n of a few
// thousand, so the exponentials of a quadrature rule share one: as many as take
// at most kShared bytes (their numerators, denominators and results).  A
// solve at n = 1030 with seven nodes, all of it: 14.2 ms against 31.3.
int64_t expm_together(int64_t n, int64_t count) {
  constexpr size_t kShared = (size_t)512 << 20;
  const size_t each = 3 * (size_t)expm_ld(n) * n * sizeof(double);
  return std::max<int64_t>(1, std::min<int64_t>({count, 16, (int64_t)(kShared / std::max<size_t>(each, 1))}));
}

// E[z] = e^{t[z] X}; X, E[z] are n x n device matrices (contiguous), E[z] must
// not alias X.  m_out, s_out: of the last one.
void expm_many_f64(hipStream_t s, int64_t n, const double* X, int64_t count, const double* t, double* const* E,
                   Arena& ws, int* m_out, int* s_out, int* info_dev, bool kept) {
  if (n <= 0 || count <= 0) return;
  const int64_t ld = expm_ld(n);
  const size_t nn = (size_t)ld * n;
  double* Y = ws.get<double>(nn);
  double* Y2 = ws.get<double>(nn);
  double* Y4 = ws.get<double>(nn);
  double* Y6 = ws.get<double>(nn);
  double* T1 = ws.get<double>(nn);
  double* Us = ws.get<double>(count * nn);
  double* Vs = ws.get<double>(count * nn);
  double* colsum = ws.get<double>(n);
  double* nrm_dev = ws.get<double>(2 * count);  // the norm; whether tX is not symmetric
  const size_t mark = ws.used;

  for (int64_t z = 0; z < count; ++z) {
    copy_scaled_f64(s, X, n, Y, ld, n, n, t[z]);
    norm1_f64(s, Y, n, n, ld, colsum, nrm_dev + 2 * z);
    asymmetry_f64(s, Y, n, ld, nrm_dev + 2 * z + 1);
  }
  std::vector<double> head(2 * count, 0.0);
  DME_HIP(hipMemcpyAsync(head.data(), nrm_dev, 2 * count * sizeof(double), hipMemcpyDeviceToHost, s));
  DME_HIP(hipStreamSynchronize(s));
  struct Pending {
    int64_t z;
    int sc;
  };
  std::vector<Pending> lu;  // those whose quotient is in Us, Vs (in that order)
  bool sym = false;
  auto mm = [&](const double* P, const double* Q, double beta, double* R, int64_t ldr) {
    ws.used = mark;
    if (sym) gemm_sym_f64(s, 'N', n, n, 1.0, P, ld, Q, ld, beta, R, ldr, true, ws);
    else gemm_f64(s, 'N', 'N', n, n, n, 1.0, P, ld, Q, ld, beta, R, ldr, &ws);
  };
  // E[z] = (cur)^(2^sc), `other` is scratch
  auto square = [&](double* cur, double* other, int sc, double* Ez) {
    for (int q = 0; q < sc; ++q) {
      const bool last = q == sc - 1;
      mm(cur, cur, 0.0, last ? Ez : other, last ? n : ld);
      std::swap(cur, other);
    }
    if (sc == 0) copy_f64(s, cur, ld, Ez, n, n, n);
  };

  for (int64_t z = 0; z < count; ++z) {
    const double nrm = head[2 * z];
    sym = head[2 * z + 1] == 0.0 && !kept;
    double* U = Us + lu.size() * nn;
    double* V = Vs + lu.size() * nn;
    DME_REQUIRE(std::isfinite(nrm), DME_ENUMERIC, "expm: operator has non-finite entries");
    int m = 13, sc = 0;
    expm_params(nrm, &m, &sc);
    if (m_out) *m_out = m;
    if (s_out) *s_out = sc;
    if (count > 1) copy_scaled_f64(s, X, n, Y, ld, n, n, t[z]);
    if (sc > 0) scale_f64(s, Y, (int64_t)nn, std::ldexp(1.0, -sc));

    double b[14];
    pade_coeffs(m, b);
    mm(Y, Y, 0.0, Y2, ld);
    if (m == 13) {
      mm(Y2, Y2, 0.0, Y4, ld);
      mm(Y4, Y2, 0.0, Y6, ld);
      // U = Y (Y6 (b13 Y6 + b11 Y4 + b9 Y2) + b7 Y6 + b5 Y4 + b3 Y2 + b1 I)
      lincomb3_f64(s, n, ld, b[13], Y6, b[11], Y4, b[9], Y2, 0.0, T1);
      lincomb3_f64(s, n, ld, b[7], Y6, b[5], Y4, b[3], Y2, b[1], V);
      mm(Y6, T1, 1.0, V, ld);
      mm(Y, V, 0.0, U, ld);
      // V = Y6 (b12 Y6 + b10 Y4 + b8 Y2) + b6 Y6 + b4 Y4 + b2 Y2 + b0 I
      lincomb3_f64(s, n, ld, b[12], Y6, b[10], Y4, b[8], Y2, 0.0, T1);
      lincomb3_f64(s, n, ld, b[6], Y6, b[4], Y4, b[2], Y2, b[0], V);
      mm(Y6, T1, 1.0, V, ld);
    } else {
      // plain even powers Y^2, Y^4 = Y^2 Y^2, Y^6 = Y^4 Y^2, Y^8 = Y^6 Y^2
      const int h = m / 2;  // highest even power index: Y^{2h}
      double* P8 = T1;
      if (h >= 2) mm(Y2, Y2, 0.0, Y4, ld);
      if (h >= 3) mm(Y4, Y2, 0.0, Y6, ld);
      if (h >= 4) mm(Y6, Y2, 0.0, P8, ld);
      // odd = b1 I + b3 Y2 + b5 Y4 + b7 Y6 + b9 Y8 ; even = b0 I + b2 Y2 + ...
      const double* P[5] = {nullptr, Y2, Y4, Y6, P8};
      auto coef = [&](int j) { return (j <= m) ? b[j] : 0.0; };
      // V <- odd part first (stored in V temporarily), then U = Y * odd
      lincomb3_f64(s, n, ld, coef(3), P[1], h >= 2 ? coef(5) : 0.0, h >= 2 ? P[2] : nullptr,
                   h >= 3 ? coef(7) : 0.0, h >= 3 ? P[3] : nullptr, coef(1), V);
      if (h >= 4) lincomb3_f64(s, n, ld, 1.0, V, coef(9), P[4], 0.0, nullptr, 0.0, V);
      mm(Y, V, 0.0, U, ld);
      lincomb3_f64(s, n, ld, coef(2), P[1], h >= 2 ? coef(4) : 0.0, h >= 2 ? P[2] : nullptr,
                   h >= 3 ? coef(6) : 0.0, h >= 3 ? P[3] : nullptr, coef(0), V);
      if (h >= 4) lincomb3_f64(s, n, ld, 1.0, V, coef(8), P[4], 0.0, nullptr, 0.0, V);
    }
    // U <- V - U (denominator q_m), V <- V + U (numerator p_m); solve q F = p
    pade_pm_f64(s, U, V, (int64_t)nn);
    ws.used = mark;
    if (sym) {
      spd_inverse_f64(s, n, U, ld, Y6, ld, ws, info_dev);
      mm(Y6, V, 0.0, T1, ld);
      square(T1, V, sc, E[z]);
    } else {
      lu.push_back({z, sc});
    }
  }
  ws.used = mark;
  if (!lu.empty()) lu_solve_f64(s, n, Us, ld, Vs, ld, n, ws, info_dev, kept, (int64_t)lu.size(), (int64_t)nn, (int64_t)nn);
  sym = false;
  for (size_t i = 0; i < lu.size(); ++i) square(Vs + i * nn, T1, lu[i].sc, E[lu[i].z]);
  ws.used = mark;
}

void expm_f64(hipStream_t s, int64_t n, const double* X, double t, double* E, Arena& ws, int* m_out, int* s_out,
              int* info_dev, bool kept) {
  expm_many_f64(s, n, X, 1, &t, &E, ws, m_out, s_out, info_dev, kept);
}

}  // namespace dme
