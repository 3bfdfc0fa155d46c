// The rows of the Chebyshev-tau Helmholtz problem (D^2 - beta) f = g, n >= 2:
//   A_n a_{n-2} + B_n a_n + C_n a_{n+2} = R_n,
//   A_n = c_{n-2} beta q1, B_n = -(1 + e_n beta q2), C_n = e_{n+2} beta q3,
//   R_n = -c_{n-2} g_{n-2} q1 + e_n g_n q2 - e_{n+2} g_{n+2} q3,
// q1 = 1 / (4 n (n - 1)), q2 = 1 / (2 (n^2 - 1)), q3 = 1 / (4 n (n + 1)), c_0 = 2 (else 1),
// e_m = 1 if m <= nc - 2 else 0.
#pragma once

#include <hip/hip_runtime.h>

namespace psms {

constexpr int kTauQMax = 256;   // largest n of the table

// The coefficients of the tau rows that depend only on the index n:
// q1 = 1 / (4 n (n - 1)), q2 = 1 / (2 (n^2 - 1)), q3 = 1 / (4 n (n + 1)), n >= 2,
// evaluated at compile time (correctly rounded, as the run-time division would
// be) and read with wave-uniform addresses, so no recurrence step divides by them.
struct TauQ {
  double q[3][kTauQMax + 1];
};
constexpr TauQ make_tau_q() {
  TauQ t{};
  for (int n = 2; n <= kTauQMax; ++n) {
    const double dn = double(n);
    t.q[0][n] = 1.0 / (4.0 * dn * (dn - 1.0));
    t.q[1][n] = 1.0 / (2.0 * (dn * dn - 1.0));
    t.q[2][n] = 1.0 / (4.0 * dn * (dn + 1.0));
  }
  return t;
}
static __constant__ TauQ kTauQ = make_tau_q();

}  // namespace psms
