// The event grid's FP64 integrals of the recurrence, compiled for the host.
#include "../paper_1502_04993_amd/csrc/evfun.h"

extern "C" void ev_any(int n, const double* D, const double* delta, double* F, double* H) {
  for (int k = 0; k < n; ++k) glmr_ev::interval_any(D[k], delta[k], F + k, H + k);
}

// as the kernel takes a slot
extern "C" void ev_slot(int n, const double* D, const double* delta, double* F, double* H, int* staged) {
  for (int k = 0; k < n; ++k) {
    double c[glmr_ev::EVC];
    glmr_ev::stage_pieces(delta[k], exp_f64(-delta[k]), c);
    staged[k] = glmr_ev::interval_pieces(c, (int)c[glmr_ev::EVE + 3], D[k], F + k, H + k);
    if (!staged[k]) glmr_ev::interval_any(D[k], delta[k], F + k, H + k);
  }
}

extern "C" void ev_exp(int n, const double* x, double* y) {
  for (int k = 0; k < n; ++k) y[k] = exp_f64(x[k]);
}
