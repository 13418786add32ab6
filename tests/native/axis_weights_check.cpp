// Test-only C wrappers around the kernel weights of roma.h (compiled on the host
// with g++ by tests/test_axis_weights.py).
#include "roma.h"

extern "C" {
// out: w[3], dw[3], ddw[3]
void t_axis(double d, int second, double* out) { lbib::axis_weights(d, second != 0, out, out + 3, out + 6); }
// phi, phi', phi'' at one node
void t_node(double r, double* out) {
  out[0] = lbib::roma_phi(r);
  out[1] = lbib::roma_dphi(r);
  out[2] = lbib::roma_ddphi(r);
}
}
