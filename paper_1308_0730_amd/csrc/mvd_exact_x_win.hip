// x passes of the block-wise form (modes 0 and 2 with the window bit) with
// compile-time plans for every 5-smooth half-row length (lists in
// mvd_exact_lengths.h).
#include "mvd_ct_passes.h"
#include "mvd_exact_lengths.h"

using namespace mvdk;

#define XK(md, m, wpb, rpw, ...)                                                                               \
  k_xpass_ct<md, wpb, rpw, m, __VA_ARGS__><<<a.grid, 64 * wpb, 0, a.stream>>>(a.jobs, a.njobs, a.plans, a.tw, \
                                                                             v, parts, flags, opt)

// forward windows with the forward plans, updates with the small radices (see
// mvd_exact_x.hip)
static hipError_t launch_forward(const LaunchArgs& a, int M, int v, Partial* parts, int* flags, int opt) {
  switch (M) {
#define X(m, wpb, rpw, ...)          \
  case m:                            \
    XK(8, m, wpb, rpw, __VA_ARGS__); \
    break;
    MVD_EXACT_ROW_FWD(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t mvd_launch_x_exact_win(const LaunchArgs& a, int M, int mode, int v, Partial* parts, int* flags,
                                  int opt) {
  if (mode == 8) return launch_forward(a, M, v, parts, flags, opt);
  if (mode != 10) return hipErrorInvalidValue;
  switch (M) {
#define X(m, wpb, rpw, ...)           \
  case m:                             \
    XK(10, m, wpb, rpw, __VA_ARGS__); \
    break;
    MVD_EXACT_ROW(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
