// Test helper: where the sequence kernel reads when a word has no gate index to read.
#include "gst_internal.h"

// The offset of that byte in the gate set's rho, for a list whose indices lie at
// `gates` (not dereferenced), or -1 outside it.
extern "C" long pad_in_rho(const double* rho, int D, const uint8_t* gates) {
  gst::LeafLaunch a{};
  a.D = D;
  a.rho = rho;
  a.gates = gates;
  const uint8_t *p = gst::pad_index(a), *r = reinterpret_cast<const uint8_t*>(rho);
  return p >= r && p < r + D * sizeof(double) ? (long)(p - r) : -1;
}
