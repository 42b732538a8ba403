// Update pass of the two-pass convolution (mode 2; see mvd_tp_x.hip).
#include "mvd_exact_lengths.h"
#include "mvd_two_pass.h"

using namespace mvdk;

hipError_t mvd_launch_x_tp_update(const TpArgs& a, int M, int waves, size_t lds, int v, Partial* parts, int* flags,
                                  int opt) {
  switch (M) {
#define X(m, rpw, ...)                                                                                       \
  case m:                                                                                                    \
      k_xpass_tp<2, rpw, m, __VA_ARGS__><<<a.grid, 64 * waves, lds, a.stream>>>(a.jobs, a.njobs, a.tw, v,    \
                                                                                parts, flags, opt);          \
    break;
    MVD_TP_ROW(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
